"""The FP64 exponential of the near field's entries, seen through a Gaussian kernel
matrix evaluated in the product: one point against points whose distances
sweep the argument from 0 past the underflow, column by column."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d", [1, 2, 3])
def test_gaussian_entries_f64(d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_09707_amd import hmx as H
    n = 513
    # squared distances to the first point: 0 .. 800, dense near 0 and -745
    r2 = np.concatenate([[0.0], np.linspace(1e-12, 1.0, 128), np.linspace(1.0, 740.0, 256),
                         np.linspace(740.0, 760.0, 128)])
    pts = np.zeros((n, d))
    pts[:, 0] = np.sqrt(r2)
    P = torch.from_numpy(pts).cuda()
    # one dense leaf: eta 0, leaf >= n
    hm = H.HMatrix(P, "gaussian", 1.0, leaf_size=n, eta=0.0, compute_dtype="f64",
                   near_recompute=1)
    hs = H.HMatrix(P, "gaussian", 1.0, leaf_size=n, eta=0.0, compute_dtype="f64")
    e0 = torch.zeros(n, dtype=torch.float64, device="cuda")
    e0[0] = 1.0
    z, zs = hm.matvec(e0).cpu().numpy(), hs.matvec(e0).cpu().numpy()
    hm.close()
    hs.close()
    # the argument the kernel sees: the coordinate squared, rounded once
    want = np.exp(-(pts[:, 0] * pts[:, 0]))
    normal = want > 1e-300
    for v in (z, zs):  # evaluated in the product, and stored
        # 1 ulp of the exponential and of numpy's
        assert np.max(np.abs(v[normal] / want[normal] - 1)) <= 2 * 2.0 ** -52
        assert np.all(np.abs(v[~normal] - want[~normal]) <= 1e-300 * 2.0 ** -50)
        assert v[0] == 1.0 and v[-1] == 0.0

"""The two passes of the stored product over row tiles at the edges of their
splits: one tile and few (their columns spread over more workgroups), many,
tiles of one row vector, of ragged rows, taller than the LDS stages hold;
against the dense FP64 product."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [(60, 64, 2), (130, 64, 2), (1000, 1, 2), (1500, 7, 3), (3001, 17, 2), (4096, 64, 2),
         (9000, 100, 3), (12000, 2500, 2), (20000, 9, 2), (33000, 32, 2), (3000, 256, 2),
         (16384, 128, 2), (70000, 100, 2), (150000, 256, 2)]


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_09707_amd import hmx
    hmx.lib()
    return hmx


@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,leaf,d", CASES)
def test_product_over_tiles(H, orc, n, leaf, d, dtype, symmetric):
    """Entries and x are positive, so no sum cancels and every bound is relative
    to z itself: the ACA's tolerance times 10 (FP64, FP32 with its rounding), and
    three BF16 roundings of 2^-9 (U, V, near field) with as much again for slack."""
    eps, tol, t = {"f64": (1e-9, 1e-8, torch.float64), "f32": (1e-6, 2e-5, torch.float32),
                   "bf16": (1e-3, 1.2e-2, torch.float32)}[dtype]
    pts = synth.uniform_points(n, d, 40 + n)
    x = np.random.default_rng(n).uniform(0.5, 1.5, n)
    print("n %d leaf %d d %d %s symmetric %d" % (n, leaf, d, dtype, symmetric), flush=True)
    hm = H.HMatrix(torch.from_numpy(pts).to("cuda:0", t), "gaussian", 0.7, compute_dtype="f32" if dtype == "bf16" else dtype, storage_dtype=dtype,
                   leaf_size=leaf, eta=1.5, aca_eps=eps, max_rank=96, symmetric_far=symmetric)
    z = hm.matvec(torch.from_numpy(x).to("cuda:0", t)).double().cpu().numpy()
    rows = np.unique(np.linspace(0, n - 1, 400).astype(np.int64))
    zd = orc.dense_matvec(pts, x, "gaussian", 0.7, rows=rows)
    err = np.linalg.norm(z[rows] - zd) / np.linalg.norm(zd)
    print("  error %.2e" % err, flush=True)
    assert err <= tol
    hm.close()

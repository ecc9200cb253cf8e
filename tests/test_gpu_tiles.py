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


def test_matmat_columns_past_31_bits(H):
    """Sixteen sides on one tile of 8.4 million rows: a batch of its columns passes
    the 31-bit offsets of a buffer descriptor (a near-field block; the ACA takes no
    blocks so tall).  Every column equals the product with one vector to
    rounding: a row sums 40 terms, 1e-13 of it."""
    n1, n2, m = 8400000, 40, 16
    print("one dense block %d x %d, FP64, %d sides" % (n1, n2, m), flush=True)
    p1 = torch.from_numpy(synth.uniform_points(n1, 2, 7)).to("cuda:0")
    p2 = torch.from_numpy(synth.uniform_points(n2, 2, 8)).to("cuda:0")
    hm = H.HMatrix.rect(p1, p2, "gaussian", 4.0, compute_dtype="f64", leaf_size=1 << 24, eta=1.5)
    assert hm.stats().n_adm == 0 and hm.stats().n_dense == 1
    X = torch.from_numpy(synth.normal_vector(m * n2, 9).reshape(m, n2)).to("cuda:0")
    Z = torch.empty((m, n1), dtype=torch.float64, device="cuda:0")
    H.hmx_matmat(hm.h, X, Z)
    worst = 0.0
    for c in range(m):
        z = hm.matvec(X[c].contiguous())
        worst = max(worst, float(torch.linalg.norm(Z[c] - z) / torch.linalg.norm(z)))
    print("  worst column vs matvec: %.2e" % worst, flush=True)
    assert worst <= 1e-13
    hm.close()


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n2", [65536, 65537, 70001])
def test_source_tiles_past_short_offsets(H, orc, n2, dtype):
    """One admissible block whose source side is one tile, up to the rows that
    32-bit offsets serve and past them (64-bit addresses), against the dense
    FP64 product; bounds as in test_product_over_tiles."""
    eps, tol, t = {"f64": (1e-9, 1e-8, torch.float64), "f32": (1e-6, 2e-5, torch.float32),
                   "bf16": (1e-3, 1.2e-2, torch.float32)}[dtype]
    n1 = 200
    p1 = synth.uniform_points(n1, 2, 51)
    p2 = synth.uniform_points(n2, 2, 52)
    p2[:, 0] += 3.0  # distance >= 2 > diameter: the root block is admissible
    x = np.random.default_rng(n2).uniform(0.5, 1.5, n2)
    print("one block %d x %d %s" % (n1, n2, dtype), flush=True)
    hm = H.HMatrix.rect(torch.from_numpy(p1).to("cuda:0", t), torch.from_numpy(p2).to("cuda:0", t),
                        "gaussian", 4.0, compute_dtype="f32" if dtype == "bf16" else dtype,
                        storage_dtype=dtype, leaf_size=1 << 17, eta=1.5, aca_eps=eps, max_rank=64)
    assert hm.stats().n_adm == 1 and hm.stats().n_dense == 0
    z = hm.matvec(torch.from_numpy(x).to("cuda:0", t)).double().cpu().numpy()
    zd = orc.dense_matvec_rect(p1, p2, x, "gaussian", 4.0)
    err = np.linalg.norm(z - zd) / np.linalg.norm(zd)
    print("  error %.2e" % err, flush=True)
    assert err <= tol
    hm.close()

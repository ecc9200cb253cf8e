"""One admissible block per handle at the edges of the ACA's size classes (a
rectangular handle of two distant point sets is the single block Y1 x Y2): one
wave to many, one row to several passes, more columns than the kernels keep in
LDS, more than one wave's lanes; against the oracle and the dense product."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 1), (1, 64), (64, 64), (65, 3), (128, 127), (129, 64), (256, 256), (40, 257),
         (512, 512), (513, 40), (1024, 1023), (1025, 700), (2048, 2048), (2049, 1999),
         (4096, 4095), (4097, 513), (9000, 8193)]


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_09707_amd import hmx
    hmx.lib()
    return hmx


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


def _block(m, n, d=2):
    p1 = synth.uniform_points(m, d, 500 + m)
    p2 = synth.uniform_points(n, d, 900 + n)
    p2[:, 0] += 3.0  # distance >= 2 > diameter: the root block is admissible
    return p1, p2, synth.normal_vector(n, 17 + n)


def _product(H, p1, p2, x, kind, p0, dtype, **kw):
    t = {"f64": np.float64, "f32": np.float32}[dtype]
    hm = H.HMatrix.rect(_dev(p1.astype(t)), _dev(p2.astype(t)), kind, p0, compute_dtype=dtype,
                        leaf_size=32, eta=1.5, **kw)
    assert hm.stats().n_adm == 1 and hm.stats().n_dense == 0
    z = hm.matvec(_dev(x.astype(t))).cpu().numpy()
    r = int(hm.ranks()[0])
    hm.close()
    return z, r


@pytest.mark.parametrize("m,n", SIZES)
def test_single_block_f64(H, orc, m, n):
    """Adaptive (eps 1e-10) and fixed rank 12 against the oracle's ACA; the
    learned sizing with a target below the rank (its block continues in
    overflow storage) equals the adaptive run bit for bit."""
    p1, p2, x = _block(m, n)
    eps, kmax = 1e-10, 48
    print("block %d x %d F64" % (m, n), flush=True)
    zd = orc.dense_matvec_rect(p1, p2, x, "gaussian", 4.0)
    zo, ro, _ = orc.hmvp_rect(p1, p2, x, "gaussian", 4.0, 32, 1.5, kmax, eps, want_ranks=True)
    z, r = _product(H, p1, p2, x, "gaussian", 4.0, "f64", aca_eps=eps, max_rank=kmax)
    print("  rank %d (oracle %d), vs dense %.1e" % (r, ro[0], _rel(z, zd)), flush=True)
    # the two runs sum the norm in another order: at most the last term differs
    assert abs(r - int(ro[0])) <= 1
    assert _rel(z, zd) <= 10 * eps and _rel(z, zo) <= 10 * eps
    w = np.zeros(8961, np.float32)
    w[-1] = 3.0  # predicted rank 3: storage for 4 columns
    mlp = H.RankMLP(w)
    zl, rl = _product(H, p1, p2, x, "gaussian", 4.0, "f64", aca_eps=eps, max_rank=kmax,
                      rank_mode="learned", mlp=mlp)
    mlp.close()
    assert rl == r and np.array_equal(zl, z)
    zf, rf = _product(H, p1, p2, x, "gaussian", 4.0, "f64", max_rank=12, rank_mode="fixed")
    zfo, rfo, _ = orc.hmvp_rect(p1, p2, x, "gaussian", 4.0, 32, 1.5, 12, 0.0, fixed=True,
                                want_ranks=True)
    assert rf == rfo[0]
    # the same pivots: the errors against the dense product agree
    assert _rel(zf, zd) <= 2 * _rel(zfo, zd) + 1e-13


@pytest.mark.parametrize("m,n", SIZES)
def test_single_block_f32(H, orc, m, n):
    p1, p2, x = _block(m, n)
    kind, p0, eps = "gaussian", 4.0, 1e-4
    print("block %d x %d F32 %s" % (m, n, kind), flush=True)
    p1, p2, x = (a.astype(np.float32).astype(np.float64) for a in (p1, p2, x))
    zd = orc.dense_matvec_rect(p1, p2, x, kind, p0)
    z, r = _product(H, p1, p2, x, kind, p0, "f32", aca_eps=eps, max_rank=48)
    # the ACA's error, and FP32 rounding of sums of n terms of either sign
    scale = np.linalg.norm(orc.dense_matvec_rect(p1, p2, np.abs(x), kind, p0))
    err = np.linalg.norm(z - zd)
    print("  rank %d, error %.1e of |A| |x|" % (r, err / scale), flush=True)
    assert err <= 10 * eps * np.linalg.norm(zd) + 4e-6 * scale


@pytest.mark.parametrize("m,n", [(100, 120), (200, 256), (400, 500), (900, 1000), (1500, 1200)])
def test_single_block_many_columns(H, orc, m, n):
    """More than 64 columns with the stopping test's products (eps 0 runs to
    the exhausted residual): past the lanes of one wave."""
    p1, p2, x = _block(m, n, 3)
    print("block %d x %d, eps 0" % (m, n), flush=True)
    zd = orc.dense_matvec_rect(p1, p2, x, "matern32", 0.5)
    z, r = _product(H, p1, p2, x, "matern32", 0.5, "f64", aca_eps=0.0, max_rank=128)
    print("  rank %d, vs dense %.1e" % (r, _rel(z, zd)), flush=True)
    assert r > 64
    assert _rel(z, zd) <= 1e-10


@pytest.mark.parametrize("split_rows", [0, 1500])
@pytest.mark.parametrize("near_recompute", [0, 1])
def test_distances_that_overflow(H, near_recompute, split_rows):
    """Coordinates of 1e200: every squared distance is infinite, so no point is
    nearest to a box's centre and the first is taken (as the oracle does); the
    kernel matrix is the identity, and every low-rank block is zero.  All size
    classes, and the many-workgroup path."""
    n = 20000
    pts = synth.uniform_points(n, 2, 71) * 1e200
    x = _dev(synth.normal_vector(n, 72))
    print("N %d, coordinates to 1e200, split rows %d" % (n, split_rows), flush=True)
    hm = H.HMatrix(_dev(pts), "gaussian", 1.0, compute_dtype="f64", leaf_size=32, eta=1.5,
                   aca_eps=1e-6, max_rank=16, near_recompute=near_recompute,
                   aca_split_rows=split_rows)
    assert hm.stats().n_adm > 0
    assert torch.equal(hm.matvec(x), x)
    assert not hm.ranks().any()
    hm.close()

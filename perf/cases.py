"""The work that programs have this library do, as measurable cases.

A case is a plain dict; its ``path`` says which entry points a pass goes
through:

* ``product``    H x with a handle that the program keeps (factors and near field stored);
* ``matmat``     H X for several right-hand sides with a kept handle;
* ``build``      a new point set: build the handle, multiply once, release it;
* ``batched``    the same for many independent problems in one handle;
* ``recompute``  H x with a handle that stores no factors and no near field
                 (the method's mode without precomputation: every product runs the ACA);
* ``cg``         a kernel ridge regression solve with a budget of CG iterations;
* ``predictor``  the rank predictor: inference on a batch, and its loss and gradient.

Points are uniform in the unit square or cube, the Halton sequence, or a
32-component Gaussian mixture; vectors are standard normal.
"""
import math

import numpy as np
import torch

from paper_1708_09707_amd import hmx as H

# the paper's admissibility parameter, used throughout
ETA = 1.5


def _case(path, name=None, **kw):
    c = dict(path=path, n=4096, d=2, dist="uniform", kernel="gaussian", p0=0.01, leaf=256,
             eps=1e-5, kmax=64, compute="f32", storage="f32", symmetric=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest product in use (the FP64 parity size): launches and latency count
        _case("product", "product_4k_2d_f64", n=4096, p0=0.1, leaf=64, eps=1e-6, kmax=32,
              compute="f64", storage="f64"),
        # the headline workload's arithmetic and density (2-d, leaf 256, FP64) at the
        # largest size of which three handles fit the card
        _case("product", "product_512k_2d_f64", n=1 << 19, compute="f64", storage="f64"),
        # an ordinary 3-d product in FP32 with short, ragged row tiles (48 or 49 points)
        _case("product", "product_100k_3d_f32", n=100003, d=3, p0=0.0145, leaf=64),
        # the mixed-precision product (BF16 storage, symmetric far field) on a million points
        _case("product", "product_1m_3d_bf16", n=1 << 20, d=3, p0=0.0145, leaf=64, eps=3e-3,
              storage="bf16", symmetric=True),
        # sixteen right-hand sides at once in FP64
        _case("matmat", "matmat_128k_2d_f64_x16", n=1 << 17, compute="f64", storage="f64",
              sides=16),
        # a small new problem: build and one product, bound by launches and read-backs
        _case("build", "build_4k_2d_f64", n=4096, p0=0.1, leaf=64, eps=1e-6, kmax=32,
              compute="f64", storage="f64"),
        # the bench workload's build (2-d, leaf 256, FP32) and its first product
        _case("build", "build_1m_2d_f32", n=1 << 20),
        # a 3-d build in BF16 storage on a ragged size
        _case("build", "build_200k_3d_bf16", n=200003, d=3, p0=0.0145, leaf=64, eps=3e-3,
              storage="bf16"),
        # the paper's own workload without precomputation: Halton points, exp(-r^2),
        # leaf 2048, rank 16, FP64
        _case("recompute", "recompute_128k_2d_f64", n=1 << 17, dist="halton", p0=1.0, leaf=2048,
              eps=0.0, kmax=16, rank_mode="fixed", compute="f64", storage="f64"),
        # kernel ridge regression on a Gaussian mixture, Matern-3/2, FP64: a CG budget
        _case("cg", "cg_16k_3d_f64", n=1 << 14, d=3, dist="gmm", kernel="matern32", p0=0.1,
              leaf=64, eps=1e-8, kmax=128, compute="f64", storage="f64", symmetric=True,
              sigma2=1e-2, iters=20),
        # many small problems in one handle: build and one product
        _case("batched", "batched_32x_f32", nprob=32, lo=10.0, hi=14.0, leaf=128),
        # one training batch of the rank predictor (forward, loss and gradient)
        _case("predictor", "predictor_16k", n=16384),
    ]


def _spread(rng, lo, hi):
    """An integer, log-uniform in [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["product", "product", "build", "build", "matmat", "batched", "recompute",
                       "cg", "predictor"])
    d = rng.choice([2, 3])
    form = rng.choice(["f64", "f32", "bf16"])
    kw = dict(d=d, compute="f64" if form == "f64" else "f32", storage=form,
              symmetric=rng.random() < 0.3)
    kw["leaf"] = rng.choice([48, 64, 100, 128, 256])
    kw["kernel"] = rng.choice(["gaussian", "gaussian", "matern32"])
    kw["p0"] = round(math.exp(rng.uniform(math.log(0.005), math.log(0.1))), 4)
    if kw["kernel"] == "matern32":
        kw["p0"] = round(math.sqrt(kw["p0"]), 4)  # the length itself
    kw["eps"] = {"f64": rng.choice([1e-4, 1e-5, 1e-6]), "f32": rng.choice([1e-3, 1e-4, 1e-5]),
                 "bf16": rng.choice([1e-2, 3e-3, 1e-3])}[form]
    # sizes up to which the largest listed case costs more
    if path == "product":
        return _case(path, n=_spread(rng, 1500, 400000 if d == 2 else 100000), **kw)
    if path == "matmat":
        return _case(path, n=_spread(rng, 1500, 200000 if d == 2 else 60000),
                     sides=rng.randint(2, 24), **kw)
    if path == "build":
        return _case(path, n=_spread(rng, 1500, 400000 if d == 2 else 40000), **kw)
    if path == "batched":
        kw.update(kernel="gaussian", symmetric=False)
        lo = rng.uniform(9.0, 11.0)
        return _case(path, nprob=_spread(rng, 4, 48), lo=round(lo, 2),
                     hi=round(rng.uniform(lo, 13.0), 2), **kw)
    if path == "recompute":
        if rng.random() < 0.5:  # the paper's form
            return _case(path, n=_spread(rng, 8000, 131072), dist="halton", p0=1.0,
                         leaf=rng.choice([512, 1000, 2048]), eps=0.0,
                         kmax=rng.choice([4, 8, 12, 16]), rank_mode="fixed", compute="f64",
                         storage="f64")
        kw.update(storage=kw["compute"])
        return _case(path, n=_spread(rng, 4000, 150000 if d == 2 else 25000), **kw)
    if path == "cg":
        return _case(path, n=_spread(rng, 1500, 16384), d=3, dist="gmm", kernel="matern32",
                     p0=round(rng.uniform(0.05, 0.2), 3), leaf=rng.choice([48, 64, 128]),
                     eps=1e-8, kmax=128, compute="f64", storage="f64", symmetric=True,
                     sigma2=rng.choice([1e-2, 0.1, 1.0]), iters=rng.randint(8, 20))
    return _case(path, n=_spread(rng, 200, 65536))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + salt) % (1 << 62))


def _points(case, seed, salt=1, n=None, d=None):
    n, d = n or case["n"], d or case["d"]
    g = _gen(seed, salt)
    if case["dist"] == "halton":
        idx0 = torch.arange(n, device="cuda", dtype=torch.int64) + 1 + int(seed) % 4096
        out = torch.empty(n, d, device="cuda", dtype=torch.float64)
        for k, b in enumerate((2, 3, 5)[:d]):
            v, f, i = torch.zeros(n, device="cuda", dtype=torch.float64), 1.0 / b, idx0.clone()
            for _ in range(int(math.log(n + 4098, b)) + 2):
                v += f * (i % b)
                i = torch.div(i, b, rounding_mode="floor")
                f /= b
            out[:, k] = v
    elif case["dist"] == "gmm":
        mean = 0.1 + 0.8 * torch.rand(32, d, generator=g, device="cuda", dtype=torch.float64)
        std = 0.02 + 0.08 * torch.rand(32, generator=g, device="cuda", dtype=torch.float64)
        c = torch.randint(0, 32, (2 * n,), generator=g, device="cuda")
        p = mean[c] + std[c, None] * torch.randn(2 * n, d, generator=g, device="cuda",
                                                 dtype=torch.float64)
        out = p[((p >= 0) & (p <= 1)).all(1)][:n]
    else:
        out = torch.rand(n, d, generator=g, device="cuda", dtype=torch.float64)
    return out.to(_dtype(case)).contiguous()


def _dtype(case):
    return torch.float64 if case["compute"] == "f64" else torch.float32


def _params(case):
    p = dict(leaf_size=case["leaf"], eta=ETA, aca_eps=case["eps"], max_rank=case["kmax"],
             compute_dtype=case["compute"], storage_dtype=case["storage"],
             symmetric_far=int(case["symmetric"]), sigma2=case.get("sigma2", 0.0))
    if "rank_mode" in case:
        p["rank_mode"] = case["rank_mode"]
    if case["path"] == "recompute":
        p.update(near_recompute=1, far_recompute=1)
    return p


def _problems(case):
    """Sizes, dimensions and kernel parameters of a batch of problems (the
    case's own: the seed draws the points and the vector)."""
    g = np.random.default_rng([case["nprob"], int(1000 * case["lo"]), int(1000 * case["hi"])])
    ns = np.round(2.0 ** g.uniform(case["lo"], case["hi"], case["nprob"])).astype(int)
    ds = g.integers(2, 4, case["nprob"])
    p0 = np.exp(g.uniform(math.log(0.005), math.log(0.05), case["nprob"]))
    return [int(v) for v in ns], [int(v) for v in ds], [float(v) for v in p0]


def _predictor_inputs(case, seed):
    """Block features in the ranges that builds produce, their ranks, weights."""
    g, n = _gen(seed, 5), case["n"]

    def u(lo, hi):
        return lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)

    m = u(5, 16)
    dim = torch.randint(2, 4, (n,), generator=g, device="cuda").double()
    diam, dist, logl = torch.exp(u(-4, 1)), torch.exp(u(-3, 2)), u(-2.7, -1.3)
    X = torch.stack([m, m + u(-0.5, 0.5), diam, diam * u(0.7, 1.4), dist, diam / dist, dim, logl], 1)
    y = torch.clamp(torch.round(4 + 3 * dim * torch.log1p(diam / dist) + u(-2, 6)), 1, 64)
    X, y = X.float().contiguous(), y.float().contiguous()
    w = np.random.default_rng([int(seed), 78])
    parts = []
    for i, o in ((8, 64), (64, 64), (64, 64), (64, 1)):
        parts += [w.standard_normal(o * i) * math.sqrt(2.0 / i), 0.1 * w.standard_normal(o)]
    return X, y, np.concatenate(parts).astype(np.float32), X.mean(0), 1.0 / X.std(0)


def prepare(case, seed):
    path = case["path"]
    s = {"path": path, "case": case}
    if path == "predictor":
        X, y, w, mean, scale = _predictor_inputs(case, seed)
        mlp = H.RankMLP(w)
        mlp.set_params(mean=mean.cpu().numpy(), scale=scale.cpu().numpy())
        return dict(s, X=X, y=y, mlp=mlp)
    if path == "batched":
        ns, ds, p0 = _problems(case)
        pts = [_points(case, seed, 100 + q, ns[q], ds[q]) for q in range(len(ns))]
        x = torch.randn(sum(ns), generator=_gen(seed, 2), device="cuda", dtype=_dtype(case))
        return dict(s, points=pts, p0=p0, x=x, params=_params(case))
    pts = _points(case, seed)
    rows = (case["sides"],) if path == "matmat" else ()
    x = torch.randn(*rows, case["n"], generator=_gen(seed, 2), device="cuda", dtype=_dtype(case))
    if path == "cg":  # a smooth target with noise
        p = pts.double()
        x = (torch.sin(2 * math.pi * p[:, 0]) * p[:, 1]).to(x.dtype) + 0.01 * x
    s.update(points=pts, x=x, params=_params(case))
    if path != "build":
        s["h"] = H.HMatrix(pts, case["kernel"], case["p0"], **s["params"])
        s["z"] = torch.empty_like(x)
    return s


def run(s):
    path, case = s["path"], s["case"]
    if path in ("product", "recompute"):
        return s["h"].matvec(s["x"], s["z"])
    if path == "matmat":
        return s["h"].matmat(s["x"], s["z"])
    if path == "build":
        h = H.HMatrix(s["points"], case["kernel"], case["p0"], **s["params"])
        z = h.matvec(s["x"])
        h.close()
        return z
    if path == "batched":
        h = H.HMatrix.batched(s["points"], case["kernel"], s["p0"], **s["params"])
        z = h.matvec(s["x"])
        h.close()
        return z
    if path == "cg":
        H.hmx_cg_solve(s["h"].h, s["x"], s["z"], rel_tol=1e-6, max_iter=case["iters"],
                       raise_on_fail=False)
        return s["z"]
    pred = s["mlp"].forward(s["X"])
    loss, grad = s["mlp"].loss_grad(s["X"], s["y"], 0.9)
    return {"pred": pred, "loss": loss, "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _entries(n, d, leaf, eps):
    """Stored entries per row of a uniform problem: (near field, one factor
    side), fitted to the partitions and ranks that the library reports (N from
    2^12 to 2^20, within about 15%)."""
    tiles = 1
    while n / tiles > leaf:
        tiles *= 2
    size = n / tiles
    if d == 2:
        near = size * 34 * max(1 - 2.4 / tiles ** 0.5, 0.2)
        far = 205.0 * max(math.log2(tiles) - 4, 0)
    else:
        near = size * 180 * max(1 - 3.6 / tiles ** (1 / 3), 0.2)
        far = 2730.0 * max(math.log2(tiles) - 7.3, 0)
    digits = max(-math.log10(eps), 1.0) if eps > 0 else 5.0
    far *= (digits / 5) ** 1.45
    return min(near, n), min(far, n)


def work(case):
    path, n, d = case["path"], case["n"], case["d"]
    if path == "predictor":
        return {"bytes": n * 9 * 4 + n * 4 + 2 * 8961 * 4, "flops": 8.0 * 8832 * n}
    w, e = (8, 8) if case["compute"] == "f64" else (4, {"f32": 4, "bf16": 2}[case["storage"]])
    if path == "batched":
        parts = [(q, dd, 1) for q, dd in zip(*_problems(case)[:2])]
    else:
        parts = [(n, d, 1)]
    b = f = 0.0
    for q, dd, _ in parts:
        near, far = _entries(q, dd, case["leaf"], case["eps"])
        ev = 3 * dd + 12  # flops of a kernel evaluation
        stored = q * (near + far * (1 if case["symmetric"] else 2))
        read = q * (near + 2 * far)
        vectors = q * w * 2
        if path == "product":
            b, f = b + read * e + vectors, f + 2 * read
        elif path == "matmat":
            groups = math.ceil(case["sides"] / 16)
            b += read * e * groups + vectors * case["sides"]
            f += 2 * read * case["sides"]
        elif path == "cg":
            b += (case["iters"] + 1) * (read * e + 8 * vectors)
            f += 2 * read * (case["iters"] + 1)
        elif path == "recompute":
            b += q * dd * w + vectors
            f += q * (near + 2 * far) * (ev + 2) + q * 2 * far * 4 * 12
        else:  # build and one product: entries written once and read once
            b += stored * e + read * e + q * dd * w + vectors
            f += stored * ev + 2 * read + q * 2 * far * 4 * 12
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _dense(points, kernel, p0, X, sigma2=0.0):
    """(A + sigma2 I) X for X (n, k), A evaluated in FP64 a strip at a time."""
    P = points.double()
    P = P - P.mean(0)
    n, sq = P.shape[0], (P * P).sum(1)
    out = torch.empty_like(X)
    step = max(1, min(n, (1 << 28) // n))
    for i in range(0, n, step):
        q = P[i:i + step]
        A = torch.addmm(sq[None, :], q, P.T, alpha=-2.0).add_(sq[i:i + step, None]).clamp_(min=0)
        if kernel == "gaussian":
            A.mul_(-1.0 / p0).exp_()
        else:  # Matern-3/2
            A.sqrt_().mul_(math.sqrt(3.0) / p0)
            A = (1 + A) * torch.exp(-A)
        out[i:i + step] = A @ X
    return out + sigma2 * X


def exact(case, seed):
    path = case["path"]
    if path == "predictor":
        X, y, w, mean, scale = _predictor_inputs(case, seed)
        a, p, at, grads = (X.double() - mean.double()) * scale.double(), torch.from_numpy(w), 0, []
        p = p.double().cuda()
        for k, (i, o) in enumerate(((8, 64), (64, 64), (64, 64), (64, 1))):
            W = p[at:at + o * i].view(o, i).clone().requires_grad_()
            b = p[at + o * i:at + o * i + o].clone().requires_grad_()
            at += o * i + o
            grads += [W, b]
            a = a @ W.T + b
            a = torch.relu(a) if k < 3 else a
        e = y.double() - a[:, 0]
        loss = torch.mean(e * (0.9 - (e < 0).double()))
        g = torch.autograd.grad(loss, grads)
        return {"pred": a[:, 0].detach(), "loss": float(loss.detach()),
                "grad": torch.cat([t.reshape(-1) for t in g])}
    if path == "batched":
        ns, ds, p0 = _problems(case)
        x = torch.randn(sum(ns), generator=_gen(seed, 2), device="cuda", dtype=_dtype(case))
        out, at = [], 0
        for q in range(len(ns)):
            P = _points(case, seed, 100 + q, ns[q], ds[q])
            out.append(_dense(P, case["kernel"], p0[q], x[at:at + ns[q], None].double())[:, 0])
            at += ns[q]
        return torch.cat(out)
    if case["n"] > (1 << 19):  # more than about 20 seconds
        return None
    P = _points(case, seed)
    rows = (case["sides"],) if path == "matmat" else ()
    x = torch.randn(*rows, case["n"], generator=_gen(seed, 2), device="cuda", dtype=_dtype(case))
    if path == "matmat":
        return _dense(P, case["kernel"], case["p0"], x.double().T.contiguous()).T.contiguous()
    if path != "cg":
        return _dense(P, case["kernel"], case["p0"], x.double()[:, None])[:, 0]
    p = P.double()
    b = ((torch.sin(2 * math.pi * p[:, 0]) * p[:, 1]).to(x.dtype) + 0.01 * x).double()[:, None]
    c, r = torch.zeros_like(b), b.clone()
    q, rr = r.clone(), (r * r).sum()
    for _ in range(case["iters"]):
        Aq = _dense(P, case["kernel"], case["p0"], q, case["sigma2"])
        alpha = rr / (q * Aq).sum()
        c, r = c + alpha * q, r - alpha * Aq
        new = (r * r).sum()
        if float(new.sqrt()) <= 1e-6 * float(b.norm()):
            break
        q, rr = r + (new / rr) * q, new
    return c[:, 0]

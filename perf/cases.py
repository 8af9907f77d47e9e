"""The work that users of the library give it, as cases that can be timed and checked.

Each case names a path through the public entry points of ``paper_2202_03655_amd.hdf``, a point cloud, a kernel and the
sizes.  The clouds are the seeded synthetic shapes of ``workloads.py`` drawn with torch on the GPU, so that inputs of any
seed are made quickly; the kernels, lengthscales and tolerances are those of the repository's workloads and tests.

``prepare`` returns what a program holds before the call, ``run`` makes one pass and returns its whole outputs, ``work``
counts the bytes and operations that a pass cannot do without, and ``exact`` computes the same outputs in binary64 from
the dense kernel matrix.
"""
import math

import numpy as np
import torch

from paper_2202_03655_amd import hdf

# Point cloud + kernel + tolerance combinations.  s_k: radial functions kept per harmonic degree at the listed sizes (the
# rank depends on the data; `work` counts with these).
SETUPS = {
    "ball3_gauss": dict(cloud="ball", d=3, kernel="gaussian", l=1.0, tol=1e-6, s_k=[4, 4, 3, 2, 2, 1, 1, 1]),
    "ball3_gauss_short": dict(cloud="ball", d=3, kernel="gaussian", l=0.5, tol=1e-5,
                              s_k=[7, 6, 6, 5, 5, 4, 4, 3, 2, 2, 1, 1]),
    "normal3_matern32": dict(cloud="normal", d=3, kernel="matern32", l=10.0, tol=1e-4,
                             s_k=[7, 7, 6, 6, 5, 3, 3, 2, 2, 1, 1, 1]),
    "normal3_matern52": dict(cloud="normal", d=3, kernel="matern52", l=10.0, tol=1e-4, s_k=[3, 2, 2, 1, 1]),
    "cube4_gauss": dict(cloud="cube", d=4, kernel="gaussian", l=0.7, tol=1e-5,
                        s_k=[8, 7, 7, 6, 6, 5, 5, 4, 4, 3, 3, 2, 1, 1]),
    "cube4_gauss_long": dict(cloud="cube", d=4, kernel="gaussian", l=1.0, tol=1e-4, s_k=[5, 5, 4, 4, 3, 3, 1, 1, 1]),
    "mixture5_cauchy": dict(cloud="mixture", d=5, kernel="cauchy", l=1.0, tol=1e-4, s_k=[5, 5, 4, 4, 3, 3, 3, 2, 1, 1]),
    "mixture5_cauchy_loose": dict(cloud="mixture", d=5, kernel="cauchy", l=1.0, tol=1e-3, s_k=[5, 4, 4, 3, 2, 1, 1, 1]),
    "shell6_matern52": dict(cloud="shell", d=6, kernel="matern52", l=8.0, tol=1e-7, s_k=[3, 3, 3, 2, 2, 1, 1, 1]),
    "shell6_matern52_loose": dict(cloud="shell", d=6, kernel="matern52", l=4.0, tol=1e-5, s_k=[3, 2, 2, 2, 1, 1, 1]),
    "ball7_gauss": dict(cloud="ball", d=7, kernel="gaussian", l=1.5, tol=1e-4, s_k=[2, 2, 2, 1, 1]),
    "ball8_gauss": dict(cloud="ball", d=8, kernel="gaussian", l=1.5, tol=1e-3, s_k=[2, 2, 1, 1]),
}
# Kernel ridge regression: the housing-shaped cloud of the paper's Sec. 4.2 experiment and a mixture in d = 5.
KRR_SETUPS = {
    "housing8": dict(cloud="housing", d=8, kernel="gaussian", l=0.5, tol=1e-4, lam=0.1, sum_rank_per_point=2.8),
    "mixture5": dict(cloud="mixture", d=5, kernel="cauchy", l=1.0, tol=1e-4, lam=0.1, sum_rank_per_point=0.1),
}
DTYPES = {"f32": torch.float32, "f64": torch.float64}
KMEANS_SEED = 0x48444602


def listed():
    return [
        # one build and product of a small problem in binary64: what an interactive user or a unit of a larger program
        # calls; a chain of short kernels and host planning
        dict(name="small_step_f64", path="step", setup="ball3_gauss", n=2000, m=1, dtype="f64", rule="bound"),
        # the headline workload: factor of 1e6 points built and applied to 16 right-hand sides
        dict(name="step_1e6_f32", path="step", setup="mixture5_cauchy", n=1_000_000, m=16, dtype="f32", rule="bound"),
        # the plain binary64 path at a ragged size and few right-hand sides
        dict(name="step_ragged_f64", path="step", setup="mixture5_cauchy", n=250_007, m=5, dtype="f64", rule="bound"),
        # a block of 64 right-hand sides on a held factor: block Krylov and posterior sampling
        dict(name="product_64rhs_f32", path="product", setup="mixture5_cauchy", n=1_000_000, m=64, dtype="f32",
             noalloc=False),
        # a mid-size product in three dimensions, odd size: the repeated product of an iterative solver
        dict(name="product_1e5_f32", path="product", setup="normal3_matern32", n=100_003, m=16, dtype="f32",
             noalloc=False),
        # tolerance below binary32 (binary64 factor of binary32 data), 64 right-hand sides
        dict(name="product_tight_tol", path="product", setup="shell6_matern52", n=500_000, m=64, dtype="f32",
             noalloc=False),
        # one step of hyperparameter and inducing-point training: build, forward, gradients of l, X and V
        dict(name="train_step_f32", path="train", setup="cube4_gauss", n=200_000, m=1, dtype="f32"),
        # predictions at new points from a weight vector: general factor K(X*, X) built and applied once
        dict(name="cross_predict_f32", path="cross", setup="mixture5_cauchy", n=10_007, ny=1_000_000, m=1, dtype="f32"),
        # the product when the factor is not stored
        dict(name="matrix_free_f32", path="matrix_free", setup="mixture5_cauchy", n=1_000_000, m=16, dtype="f32"),
        # kernel ridge regression fit: k-means, block factors, preconditioner and a fixed budget of CG iterations
        dict(name="krr_fit", path="krr_fit", setup="housing8", n=13_760, k=30, its=10),
        # the KRR operator alone: what every CG iteration of a longer fit applies
        dict(name="krr_apply", path="krr_apply", setup="housing8", n=13_760, k=30),
        # exact kernel predictions of the fitted model for a test set
        dict(name="predict", path="predict", cloud="housing", d=8, kernel="gaussian", l=0.5, n=6_880, ny=13_760),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _n_max(setup, m, dtype, most):
    """Points at which the factor (8 GB) and the contraction (that of the largest listed products) are not exceeded."""
    H, S, r = _sizes(SETUPS[setup])
    wide = dtype == "f64" or SETUPS[setup]["tol"] <= 1e-6
    m16 = (m + 15) // 16 * 16
    return max(2000, int(min(most, 7e9 / ((H + S) * (8 if wide else 4)), (1.7e11 if wide else 3.4e11) / (4 * r * m16))))


def draw(rng):
    path = rng.choice(["step", "step", "product", "product", "product", "train", "cross", "matrix_free", "krr_fit",
                       "krr_apply", "predict"])
    if path in ("krr_fit", "krr_apply"):
        setup = rng.choice(sorted(KRR_SETUPS))
        # clusters of a few hundred points on average, as the paper's thirty; the mixture's are uneven
        n, mean = (_log_int(rng, 2500, 13_760), (280, 460)) if setup == "housing8" else (_log_int(rng, 2500, 5000), (200, 300))
        case = dict(path=path, setup=setup, n=n, k=max(8, min(30, n // rng.randint(*mean))))
        if path == "krr_fit":
            case["its"] = rng.randint(4, 12)
        return case
    if path == "predict":
        n = _log_int(rng, 100, 30_000)
        return dict(path=path, cloud="cube", d=rng.randint(2, 8), kernel=rng.choice(sorted(hdf.KERNELS)),
                    l=round(rng.uniform(0.3, 2.0), 3), n=n, ny=_log_int(rng, 100, min(60_000, 200_000_000 // n)))
    dtype = rng.choice(["f32", "f32", "f64"])
    if path == "train":
        setup = rng.choice(["ball3_gauss", "cube4_gauss", "cube4_gauss_long", "mixture5_cauchy_loose"])
        m = rng.choice([1, 1, 2, 3])
        return dict(path=path, setup=setup, n=_log_int(rng, 2000, _n_max(setup, 16 * m, dtype, 200_000)), m=m, dtype=dtype)
    setup = rng.choice(sorted(SETUPS))
    if path == "matrix_free":
        setup = rng.choice(["ball3_gauss_short", "normal3_matern32", "cube4_gauss_long", "mixture5_cauchy",
                            "mixture5_cauchy_loose"])
        m = rng.choice([1, 7, 16, 32])
        return dict(path=path, setup=setup, n=_log_int(rng, 20_000, _n_max(setup, m, dtype, 1_000_000)), m=m, dtype=dtype)
    if path == "cross":
        m = rng.choice([1, 1, 4, 16])
        ny = _log_int(rng, 5000, _n_max(setup, m, dtype, 1_000_000))
        return dict(path=path, setup=setup, n=_log_int(rng, 500, min(ny, 50_000)), ny=ny, m=m, dtype=dtype)
    if path == "step":
        m = rng.choice([1, 4, 16, 33])
        return dict(path=path, setup=setup, n=_log_int(rng, 1000, _n_max(setup, m, dtype, 1_000_000)), m=m, dtype=dtype,
                    rule=rng.choice(["bound", "bound", "sampled"]))
    m = _log_int(rng, 1, 256)
    noalloc = m <= 64 and rng.random() < 0.25
    return dict(path=path, setup=setup, n=_log_int(rng, 1000, _n_max(setup, m, dtype, 1_000_000)), m=m, dtype=dtype,
                noalloc=noalloc)


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed & 0x7FFFFFFF)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _directions(g, n, d):
    x = _normal(g, n, d)
    return x / x.norm(dim=1, keepdim=True)


def _points(cloud, n, d, g):
    """The shapes of workloads.py: unit ball, N(0, I), cube, shell, mixture scaled to max-norm 1, housing-like table."""
    if cloud == "ball":
        return _directions(g, n, d) * _uniform(g, n, 1) ** (1.0 / d)
    if cloud == "normal":
        return _normal(g, n, d)
    if cloud == "cube":
        return 2.0 * _uniform(g, n, d) - 1.0
    if cloud == "shell":
        return _directions(g, n, d) * (0.9 + 0.2 * _uniform(g, n, 1))
    if cloud == "mixture":
        # the ten component means belong to the workload, the points to the seed
        mu = torch.tensor(np.random.default_rng(103).normal(scale=2.0, size=(10, d)), device="cuda")
        z = torch.randint(0, 10, (n,), generator=g, device="cuda")
        x = mu[z] + 0.5 * _normal(g, n, d)
        x = x - x.mean(dim=0)
        return x / x.norm(dim=1).max()
    if cloud == "housing":
        centres = torch.tensor(np.random.default_rng(11).uniform(-1.0, 1.0, size=(6, 2)), device="cuda")
        loc = centres[torch.randint(0, 6, (n,), generator=g, device="cuda")] + 0.15 * _normal(g, n, 2)
        inc = torch.exp(1.2 + 0.45 * _normal(g, n, 1))
        age = 1.0 + 51.0 * _uniform(g, n, 1)
        rooms = torch.exp(1.6 + 0.25 * _normal(g, n, 1))
        beds = rooms * (0.15 + 0.1 * _uniform(g, n, 1))
        pop = torch.exp(7.0 + 0.7 * _normal(g, n, 1))
        occ = torch.exp(1.0 + 0.3 * _normal(g, n, 1))
        f = torch.cat([inc, age, rooms, beds, pop, occ, loc], dim=1)
        lo, hi = f.min(dim=0).values, f.max(dim=0).values
        return (f - lo) / (hi - lo)
    raise ValueError(cloud)


def _targets(x, g):
    """A smooth response of the features plus noise, as the regression experiments have."""
    y = torch.sin(3.0 * x[:, 0] + 2.0 * x[:, -1]) + x[:, 1] * x[:, 2]
    return (y + 0.05 * _normal(g, len(x))).contiguous()


def _inputs(case, seed):
    g = _gen(seed)
    path = case["path"]
    if path in ("krr_fit", "krr_apply"):
        c = KRR_SETUPS[case["setup"]]
        x = _points(c["cloud"], case["n"], c["d"], g).contiguous()
        v = _targets(x, g) if path == "krr_fit" else _normal(g, case["n"])
        return dict(c, X=x, v=v)
    if path == "predict":
        x = _points(case["cloud"], case["n"] + case["ny"], case["d"], g)
        return dict(kernel=case["kernel"], l=case["l"], X=x[:case["n"]].contiguous(), Y=x[case["n"]:].contiguous(),
                    v=_normal(g, case["ny"]))
    c = SETUPS[case["setup"]]
    dt = DTYPES[case["dtype"]]
    ny = case.get("ny", 0)
    x = _points(c["cloud"], case["n"] + ny, c["d"], g).to(dt)
    got = dict(c, X=x[:case["n"]].contiguous(), V=_normal(g, ny or case["n"], case["m"]).to(dt))
    if ny:
        got["Y"] = x[case["n"]:].contiguous()
    if path == "train":
        got["G"] = _normal(g, case["n"], case["m"]).to(dt)
    return got


# ------------------------------------------------------------------ the passes
def prepare(case, seed):
    s = _inputs(case, seed)
    s["path"] = case["path"]
    if case["path"] == "step":
        s["rule"] = case["rule"]
    elif case["path"] in ("product", "matrix_free"):
        s["factor"] = hdf.Factor(s["X"], s["kernel"], s["l"], s["tol"],
                                 storage="none" if case["path"] == "matrix_free" else "factor")
        if case.get("noalloc"):
            s["out"] = torch.empty_like(s["V"])
    elif case["path"] == "train":
        s["X"].requires_grad_(True)
        s["V"].requires_grad_(True)
        s["ell"] = torch.tensor(s["l"], dtype=s["X"].dtype, device="cuda", requires_grad=True)
    elif case["path"] == "krr_fit":
        s["k"], s["its"] = case["k"], case["its"]
    elif case["path"] == "krr_apply":
        labels, _, _ = hdf.kmeans(s["X"], case["k"])
        s["system"] = hdf.KRR(s["X"], labels, case["k"], s["kernel"], s["l"], s["tol"], s["lam"])
    return s


def run(s):
    path = s["path"]
    if path == "step":
        f = hdf.Factor(s["X"], s["kernel"], s["l"], s["tol"], rank_rule=s["rule"])
        return f.matvec(s["V"])
    if path in ("product", "matrix_free"):
        return s["factor"].matvec_noalloc(s["V"], s["out"]) if "out" in s else s["factor"].matvec(s["V"])
    if path == "train":
        f = hdf.Factor(s["X"].detach(), s["kernel"], s["l"], s["tol"])
        y = hdf.HDFMatvec.apply(s["X"], s["ell"], s["V"], f)
        dX, dl, dV = torch.autograd.grad(y, (s["X"], s["ell"], s["V"]), s["G"])
        return {"y": y.detach(), "dX": dX, "dl": dl, "dV": dV}
    if path == "cross":
        f = hdf.CrossFactor(s["X"], s["Y"], s["kernel"], s["l"], s["tol"])
        return f.matvec(s["V"])
    if path == "krr_fit":
        labels, centres, _ = hdf.kmeans(s["X"], s["k"])
        system = hdf.KRR(s["X"], labels, s["k"], s["kernel"], s["l"], s["tol"], s["lam"])
        w, _, _ = system.solve(s["v"], max_iter=s["its"], rtol=0.0)
        return {"labels": labels, "centres": centres, "w": w}
    if path == "krr_apply":
        return s["system"].apply(s["v"])
    if path == "predict":
        return hdf.kernel_matvec(s["X"], s["Y"], s["v"], s["kernel"], s["l"])
    raise ValueError(path)


# ------------------------------------------------------------------ necessary work
def _harmonics(d, k):
    return math.comb(k + d - 1, d - 1) - (math.comb(k + d - 3, d - 1) if k >= 2 else 0)


def _sizes(c):
    """Harmonics, radial functions and rank of a setup's factor."""
    H = sum(_harmonics(c["d"], k) for k in range(len(c["s_k"])))
    r = sum(_harmonics(c["d"], k) * s for k, s in enumerate(c["s_k"]))
    return H, sum(c["s_k"]), r


def work(case):
    path, n = case["path"], case["n"]
    if path == "predict":                        # per pair: the distance, the kernel (about 20), one FMA
        return dict(bytes=8.0 * (case["d"] * (n + case["ny"]) + n + case["ny"]),
                    flops=n * case["ny"] * (3.0 * case["d"] + 22))
    if path in ("krr_fit", "krr_apply"):
        c = KRR_SETUPS[case["setup"]]
        pairs = float(n) * n * (1 - 1.0 / case["k"])
        op = pairs * (3.0 * c["d"] + 22) + 4.0 * n * (n / case["k"]) * c["sum_rank_per_point"]
        if path == "krr_apply":
            return dict(bytes=8.0 * n * (c["d"] + 2), flops=op)
        b = n / case["k"]
        return dict(bytes=8.0 * n * (c["d"] + 2), flops=case["its"] * (op + 2 * n * b) + n * b * b)
    c = SETUPS[case["setup"]]
    el = 4 if case["dtype"] == "f32" else 8
    wide = 8 if c["tol"] <= 1e-6 else el
    H, S, r = _sizes(c)
    d, m = c["d"], case["m"]
    if path == "product":                        # the factor, V and the result, once each
        return dict(bytes=float(n) * ((H + S) * wide + 2 * m * el), flops=4.0 * r * n * m)
    if path == "cross":
        ny = case["ny"]
        return dict(bytes=float(el) * ((n + ny) * d + (n + ny) * m), flops=2.0 * (n + ny) * (r * m + H + 8 * S))
    if path == "train":                          # forward, dV and both gradients
        return dict(bytes=float(n) * el * (2 * d + 4 * m), flops=n * (8.0 * r * m + 4.0 * r * m * (d + 1) + 3 * H))
    return dict(bytes=float(n) * el * (d + 2 * m), flops=float(n) * (4.0 * r * m + 3 * H + 16 * S))


# ------------------------------------------------------------------ the same outputs in binary64
def _kernel(r2, kernel, l):
    """k(r) in place of the squared distances."""
    if kernel == "gaussian":
        return r2.mul_(-0.5 / (l * l)).exp_()
    if kernel == "cauchy":
        return r2.mul_(1.0 / (l * l)).add_(1.0).reciprocal_()
    z = r2.sqrt_().mul_(math.sqrt(3.0 if kernel == "matern32" else 5.0) / l)
    e = torch.exp(-z)
    return z.add_(1.0).mul_(e) if kernel == "matern32" else (z * z).div_(3.0).add_(z).add_(1.0).mul_(e)


def _slope(r2, kernel, l):
    """k'(r) / r in place of the squared distances."""
    if kernel == "gaussian":
        return r2.mul_(-0.5 / (l * l)).exp_().mul_(-1.0 / (l * l))
    if kernel == "cauchy":
        return r2.mul_(1.0 / (l * l)).add_(1.0).pow_(-2).mul_(-2.0 / (l * l))
    z = r2.sqrt_().mul_(math.sqrt(3.0 if kernel == "matern32" else 5.0) / l)
    e = torch.exp(-z)
    return e.mul_(-3.0 / (l * l)) if kernel == "matern32" else z.add_(1.0).mul_(e).mul_(-5.0 / (3.0 * l * l))


def _dist2(x, y):
    r2 = torch.addmm((y * y).sum(dim=1)[None, :], x, y.t(), alpha=-2.0)
    return r2.add_((x * x).sum(dim=1)[:, None]).clamp_(min=0.0)


def _direct_dist2(x, y):
    """Squared distances summed over the coordinate differences (no cancellation)."""
    r2 = torch.zeros(len(x), len(y), dtype=torch.float64, device=x.device)
    for j in range(x.shape[1]):
        t = x[:, j:j + 1] - y[:, j][None, :]
        r2.addcmul_(t, t)
    return r2


def _dense(x, y, v, kernel, l):
    """K(x, y) v by blocks; y is None for x itself (each pair once)."""
    b = 8192
    if y is None:
        out = torch.zeros(len(x), v.shape[1], dtype=torch.float64, device=x.device)
        for i in range(0, len(x), b):
            for j in range(i, len(x), b):
                k = _kernel(_dist2(x[i:i + b], x[j:j + b]), kernel, l)
                out[i:i + b] += k @ v[j:j + b]
                if j > i:
                    out[j:j + b] += k.t() @ v[i:i + b]
        return out
    out = torch.zeros(len(x), v.shape[1], dtype=torch.float64, device=x.device)
    for i in range(0, len(x), b):
        for j in range(0, len(y), b):
            out[i:i + b] += _kernel(_dist2(x[i:i + b], y[j:j + b]), kernel, l) @ v[j:j + b]
    return out


def _gradients(x, v, g, kernel, l):
    """dF/dX and dF/dl of F = sum_c g_c^T K v_c with the dense kernel."""
    b = 8192
    dX, dl = torch.zeros_like(x), torch.zeros((), dtype=torch.float64, device=x.device)
    for i in range(0, len(x), b):
        for j in range(0, len(x), b):
            r2 = _dist2(x[i:i + b], x[j:j + b])
            s = _slope(r2.clone(), kernel, l)
            w = g[i:i + b] @ v[j:j + b].t()
            dl -= (r2.mul_(s) * w).sum() / l
            s.mul_(w.add_(v[i:i + b] @ g[j:j + b].t()))
            dX[i:i + b] += s.sum(dim=1, keepdim=True) * x[i:i + b] - s @ x[j:j + b]
    return dX, dl


def _splitmix(state):
    m = (1 << 64) - 1
    state = (state + 0x9E3779B97F4A7C15) & m
    z = ((state ^ (state >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return state, z ^ (z >> 31)


def _lloyd(x, k, most=100):
    """Lloyd's iteration from k distinct points: (labels, centres)."""
    picked, state = [], KMEANS_SEED
    while len(picked) < k:
        state, u = _splitmix(state)
        i = (u >> 11) % len(x)
        if i not in picked:
            picked.append(i)
    c, labels = x[picked].clone(), None
    for _ in range(most):
        new = _direct_dist2(x, c).argmin(dim=1)
        if labels is not None and bool((new == labels).all()):
            break
        labels = new
        member = torch.nn.functional.one_hot(labels, k).to(torch.float64)
        count = member.sum(dim=0)
        c = torch.where(count[:, None] > 0, (member.t() @ x) / count.clamp(min=1.0)[:, None], c)
    return labels, c


def _krr_weights(x, y, labels, k, kernel, l, lam, its):
    """`its` preconditioned CG iterations from zero on lam I + K, block-diagonal preconditioner of the clusters."""
    A = _kernel(_direct_dist2(x, x), kernel, l)
    A.diagonal().add_(lam)
    blocks = []
    for c in range(k):
        at = torch.nonzero(labels == c).flatten()
        if len(at):
            blocks.append((at, torch.linalg.cholesky(A[at][:, at])))

    def solve(r):
        z = torch.empty_like(r)
        for at, L in blocks:
            z[at] = torch.cholesky_solve(r[at, None], L)[:, 0]
        return z

    w, r = torch.zeros_like(y), y.clone()
    z = solve(r)
    p, rz = z.clone(), r @ z
    for _ in range(its):
        q = A @ p
        alpha = rz / (p @ q)
        w += alpha * p
        r -= alpha * q
        z = solve(r)
        new = r @ z
        p = z + (new / rz) * p
        rz = new
    return w


def exact(case, seed):
    s = _inputs(case, seed)
    path, kernel, l = case["path"], s["kernel"], s["l"]
    if path == "predict":
        out = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        for i in range(0, case["n"], 4096):
            out[i:i + 4096] = _kernel(_direct_dist2(s["X"][i:i + 4096], s["Y"]), kernel, l) @ s["v"]
        return out
    if path == "krr_apply":
        K = _kernel(_direct_dist2(s["X"], s["X"]), kernel, l)
        return K @ s["v"] + s["lam"] * s["v"]
    if path == "krr_fit":
        labels, centres = _lloyd(s["X"], case["k"])
        w = _krr_weights(s["X"], s["v"], labels, case["k"], kernel, l, s["lam"], case["its"])
        return {"labels": None, "centres": centres, "w": w}
    x, v = s["X"].double(), s["V"].double()
    if path == "cross":
        return _dense(x, s["Y"].double(), v, kernel, l)
    if path == "train":
        g = s["G"].double()
        dX, dl = _gradients(x, v, g, kernel, l)
        return {"y": _dense(x, None, v, kernel, l), "dX": dX, "dl": dl, "dV": _dense(x, None, g, kernel, l)}
    return _dense(x, None, v, kernel, l)

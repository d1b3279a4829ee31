"""Workloads for timing the eigenvalue-count library, with their plain 64-bit references.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (the matrix on the device, the preconditioner, the probe block and the
workspace it keeps), `run` makes one call through the public entry points,
`work` says what one call cannot do without, and `exact` computes the same
outputs with plain torch in float64.

Every matrix is a grid Laplacian with a local potential (the discrete
Hamiltonians the estimator is for): uniform random, Gaussian wells, or the bare
scaled Laplacian.  `path` names the entry point:

  count      ecount.count, one interval
  slices     ecount.negcounts, `shifts` contiguous endpoints on one probe block
  batch      ecount.Batch, many problems with their own shifts
  arnoldi    ecount.count_arnoldi, an unfactored preconditioner
  block      ecount.count_block, probes in blocks of 16
  gradient   autograd.SmoothCount, forward and backward of the smoothed count
  ildl       ecount.negcounts with the factored ILDL(t) preconditioner
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1602_02306_amd import autograd as ag
from paper_1602_02306_amd import ecount as ec
from paper_1602_02306_amd import workloads as W

SMOOTH_W = 0.05


def _case(path, dims, m, k, xi=-8.0, eta=-2.0, prec="cheb", pot="wells", vec="f64", rule="gauss",
          shifts=2, max_cols=0, details=True, nprob=1, nmax=0, droptol=0.0, name=None):
    d = tuple(dims) + (1,) * (3 - len(dims))
    c = {"path": path, "ndim": len(dims), "d0": d[0], "d1": d[1], "d2": d[2], "m": m, "k": k,
         "xi": xi, "eta": eta, "prec": prec, "pot": pot, "vec": vec, "rule": rule,
         "shifts": shifts, "max_cols": max_cols, "details": details, "nprob": nprob,
         "nmax": nmax, "droptol": droptol}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: a small dense-ish spectrum count in an inner loop, where launches
        # and the latency of one wavefront count
        _case("count", (30, 30), 40, 20, 0.5, 1.5, "jacobi", "uniform", name="small_jacobi"),
        # the benchmark: one interval of a 64^3 Hamiltonian with many probes
        _case("count", (64, 64, 64), 256, 30, name="wells64"),
        # the same problem in the FP32 storage form, for half the memory
        _case("count", (64, 64, 64), 256, 30, vec="f32", name="wells64_f32"),
        # a grid too large for its basis to be kept at once: FP32 and column waves
        _case("count", (128, 128, 128), 64, 30, vec="f32", max_cols=64, name="wells128_f32_waves"),
        # spectrum slicing on a ragged box: four shifts in one run, the averaged rule
        _case("slices", (37, 29, 43), 50, 24, rule="ga", shifts=4, name="slices_ragged"),
        # a tight count (long Krylov spaces, the averaged rule), where reorthogonalization is
        # nearly everything; only the counts are asked for
        _case("count", (32, 32, 32), 32, 100, rule="ga", details=False, name="deep_krylov"),
        # a planar problem with the diagonal preconditioner: A through its CSR rows
        _case("count", (300, 300), 64, 40, 0.5, 1.5, "jacobi", "uniform", name="plane_jacobi"),
        # many uneven problems in one launch sequence, three slices each
        _case("batch", (16, 16, 16), 16, 25, shifts=4, nprob=16, nmax=40, name="batch16"),
        # an unfactored preconditioner
        _case("arnoldi", (40, 40, 40), 64, 30, prec="cheb_inv", name="arnoldi40"),
        # the block form, accurate at few steps
        _case("block", (48, 48, 48), 128, 20, name="block48"),
        # fitting a potential to a count: value and gradient
        _case("gradient", (48, 48, 48), 32, 30, name="gradient48"),
        # the incomplete factorization as a preconditioner: few steps, sequential solves
        _case("ildl", (127, 127), 50, 6, 0.0, 3000.0, "ildl", "zero", shifts=1, droptol=1e-6,
              name="laplace_ildl"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _box(rng, lo, hi):
    e = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return tuple(max(5, int(round(e * rng.uniform(0.75, 1.3)))) for _ in range(3))


# columns x rows x k^2 of the 64^3 benchmark, the largest listed case
_MOST = 64 ** 3 * 512 * 30 * 30


def draw(rng):
    while True:
        path = rng.choice(("count", "count", "count", "slices", "batch", "arnoldi", "block",
                           "gradient", "ildl"))
        m, k = _log(rng, 4, 256), rng.randint(8, 36)
        if path == "count":
            kind = rng.choice(("cheb", "cheb", "f32", "plane", "small"))
            if kind == "small":
                c = _case(path, (rng.randint(12, 50), rng.randint(12, 50)), _log(rng, 4, 128),
                          rng.randint(6, 20), 0.5, 1.5, rng.choice(("jacobi", "none")), "uniform")
            elif kind == "plane":
                c = _case(path, (_log(rng, 60, 500), _log(rng, 60, 500)), min(m, 96), k, 0.5, 1.5,
                          rng.choice(("jacobi", "none")), "uniform")
            elif kind == "f32":
                c = _case(path, _box(rng, 16, 96), m, k, vec="f32",
                          max_cols=rng.choice((0, 0, 64)))
            else:
                c = _case(path, _box(rng, 14, 72), m, k, rule=rng.choice(("gauss", "ga")),
                          max_cols=rng.choice((0, 0, 0, 96)))
        elif path == "slices":
            c = _case(path, _box(rng, 14, 48), min(m, 64), k, rule=rng.choice(("gauss", "ga")),
                      shifts=rng.randint(1, 6))
        elif path == "batch":
            c = _case(path, (12, 12, 12), rng.randint(4, 32), rng.randint(8, 25), shifts=4,
                      vec=rng.choice(("f64", "f64", "f32")), nprob=_log(rng, 2, 24),
                      nmax=rng.randint(16, 40))
        elif path == "arnoldi":
            c = _case(path, _box(rng, 12, 44), min(m, 96), k, prec="cheb_inv")
        elif path == "block":
            c = _case(path, _box(rng, 14, 56), 16 * rng.randint(1, 10), rng.randint(6, 28))
        elif path == "gradient":
            c = _case(path, _box(rng, 10, 48), rng.randint(3, 32), rng.randint(8, 30))
        else:
            c = _case(path, (rng.randint(24, 120), rng.randint(24, 96)), rng.randint(5, 100),
                      rng.randint(3, 8), 0.0, float(rng.randint(300, 2500)), "ildl", "zero",
                      shifts=1, droptol=rng.choice((1e-3, 1e-4, 1e-6)))
        if _rows_bound(c) * c["m"] * c["shifts"] * c["k"] ** 2 <= _MOST:
            return c


def _rows_bound(c):
    if c["path"] == "batch":
        return c["nprob"] * ((c["d0"] + c["nmax"]) // 2) ** 3 * 2
    return c["d0"] * c["d1"] * c["d2"]


def _dims(c):
    return (c["d0"], c["d1"], c["d2"])[:c["ndim"]]


def _potential(c, seed):
    dims = _dims(c)
    if c["pot"] == "uniform":
        return W.uniform_potential(int(np.prod(dims)), seed)
    if c["pot"] == "wells":
        return W.gaussian_wells(dims, np.random.default_rng(seed))
    return np.zeros(int(np.prod(dims)))


def _scale(c):
    # (1/h^2) on the unit square for the bare Laplacian, h = 1/(d + 1)
    return float((c["d0"] + 1) ** 2) if c["pot"] == "zero" else 1.0


def _matrix(c, V):
    A = W.laplacian_csr(_dims(c), V if c["pot"] != "zero" else None)
    A.val = A.val * _scale(c)
    return A


def _taus(c, rng):
    if c["path"] == "ildl":
        return np.array([c["eta"]])
    # shifts spread over the interval, each a little off the even spacing
    u = (np.arange(c["shifts"]) + rng.uniform(0.2, 0.8, c["shifts"])) / c["shifts"]
    return c["xi"] + (c["eta"] - c["xi"]) * u


def _batch_items(c, seed):
    # (grid, shifts, potential) of each problem; the edges are spread evenly over the range, so
    # that the size of the batch does not depend on the seed
    rng = np.random.default_rng(seed)
    out = []
    for N in np.linspace(c["d0"], c["nmax"], c["nprob"]).round():
        d = (int(N),) * 3
        taus = np.sort(rng.uniform(c["xi"], c["eta"], c["shifts"]))
        out.append((d, taus, W.gaussian_wells(d, rng)))
    return out


def _probes(c, n, seed, dtype=torch.float64):
    return W.rademacher_torch(n, c["m"], 12345 + seed, dtype=dtype)


def prepare(case, seed):
    c = case
    s = {"case": c}
    dt = torch.float32 if c["vec"] == "f32" else torch.float64
    if c["path"] == "batch":
        items = _batch_items(c, seed)
        A = W.block_diag_csr([W.laplacian_csr(d, V) for d, _, V in items])
        sizes = [int(np.prod(d)) for d, _, _ in items]
        s["batch"] = ec.Batch(ec.upload_csr(A, c["vec"]), W.cheb_invsqrt_prec(items[0][0]), sizes,
                              np.array([t for _, t, _ in items]), _probes(c, A.n, seed, dt),
                              c["k"], dims=[d for d, _, _ in items], vec=c["vec"], details=True)
        return s
    V = _potential(c, seed)
    n = V.size
    if c["path"] == "gradient":
        L = W.laplacian_csr(_dims(c))
        pos = np.nonzero(L.col_idx == np.repeat(np.arange(n), np.diff(L.row_ptr)))[0]
        s["problem"] = ag.SmoothProblem(ec.upload_csr(L), torch.from_numpy(pos).cuda(),
                                        W.make_prec("cheb", _dims(c)), _probes(c, n, seed),
                                        c["k"], SMOOTH_W)
        s["V"] = torch.from_numpy(V).cuda().requires_grad_(True)
        for e in ("xi", "eta"):
            s[e] = torch.tensor(c[e], dtype=torch.float64, device="cuda", requires_grad=True)
        return s
    A = _matrix(c, V)
    s["A"] = ec.upload_csr(A, c["vec"])
    s["V"] = _probes(c, n, seed, dt)
    s["taus"] = _taus(c, np.random.default_rng(seed))
    S = len(s["taus"]) if c["path"] in ("slices", "ildl") else 2
    if c["path"] == "ildl":
        s["prec"] = ec.ildl_precond(A, s["taus"], c["droptol"])
    else:
        s["prec"] = W.make_prec(c["prec"], _dims(c))
    if c["path"] == "arnoldi":
        need = ec.arnoldi_workspace_bytes(n, c["m"], s["prec"], c["k"])
    elif c["path"] == "block":
        need = ec.block_workspace_bytes(n, c["m"], s["prec"], c["k"])
    else:
        need = ec.workspace_bytes(n, c["m"], S, s["prec"], c["k"], c["vec"], c["rule"],
                                  max_cols=c["max_cols"])
    s["ws"] = ec.Workspace(need)
    return s


def run(state):
    s, c = state, state["case"]
    path = c["path"]
    if path == "batch":
        r = s["batch"].run()
        return {"negcounts": r.negcounts, "counts": r.counts, "variances": r.variances,
                "per_probe": r.per_probe, "k_used": r.k_used}
    if path == "gradient":
        est = ag.SmoothCount.apply(s["V"], s["xi"], s["eta"], s["problem"])
        dV, dxi, deta = torch.autograd.grad(est, (s["V"], s["xi"], s["eta"]))
        return {"estimate": est.detach(), "dV": dV, "dxi": dxi, "deta": deta}
    if path in ("slices", "ildl"):
        r = ec.negcounts(s["A"], s["prec"], s["taus"], s["V"], c["k"], c["vec"], c["rule"],
                         workspace=s["ws"], max_cols=c["max_cols"])
        out = {"negcounts": r.negcounts, "counts": r.counts, "variances": r.variances}
    else:
        if path == "arnoldi":
            r = ec.count_arnoldi(s["A"], s["prec"], c["xi"], c["eta"], s["V"], c["k"], c["vec"],
                                 workspace=s["ws"])
        elif path == "block":
            r = ec.count_block(s["A"], s["prec"], c["xi"], c["eta"], s["V"], c["k"],
                               workspace=s["ws"])
        else:
            r = ec.count(s["A"], s["prec"], c["xi"], c["eta"], s["V"], c["k"], c["vec"],
                         c["rule"], workspace=s["ws"], details=c["details"],
                         max_cols=c["max_cols"])
        out = {"estimate": r.estimate, "variance": r.variance, "neg_xi": r.neg_xi,
               "neg_eta": r.neg_eta}
    if c["details"]:
        out["per_probe"], out["k_used"] = r.per_probe, r.k_used
        if path not in ("arnoldi", "block"):
            out["alpha"], out["beta"] = r.alpha, r.beta
    return out


def _degree(c):
    return {"cheb": 4, "cheb_inv": 8}.get(c["prec"], 0)


def work(case):
    c = case
    ncol = c["m"] * (c["shifts"] if c["path"] in ("slices", "batch", "ildl") else 2)
    if c["path"] == "batch":
        edges = np.linspace(c["d0"], c["nmax"], c["nprob"]).round()
        n = float(np.sum(edges ** 3))
    else:
        n = float(c["d0"] * c["d1"] * c["d2"])
    k = c["k"]
    b = 4.0 if c["vec"] == "f32" else 8.0
    pts = 2.0 * c["ndim"] + 1.0
    # operator: one stencil or matrix row per application (2 flops a point); M twice (once in T)
    apps = {"cheb": 2 * 4, "cheb_inv": 8, "jacobi": 0, "none": 0, "ildl": 0}[c["prec"]] + 1
    op = 2.0 * pts * apps
    if c["path"] == "ildl":
        op += 2 * 2.0 * c["d1"]     # two solves with a factor about one grid line wide
    # full reorthogonalization: a dot and an update against each earlier vector
    # (twice in the Arnoldi form; 16 x 16 blocks in the block form)
    orth = {"arnoldi": 8.0, "block": 4.0 * 16}.get(c["path"], 4.0) * (k + 1) / 2.0
    flops = n * ncol * k * (op + orth)
    bytes_ = n * c["m"] * b + n * pts * (b + 4.0) + 8.0 * ncol * (2 * k + 2)
    if c["path"] == "gradient":
        flops *= 3.0
        bytes_ += 16.0 * n
    return {"bytes": bytes_, "flops": flops}


# ---------------------------------------------------------------------------
# The same outputs with plain torch in float64
# ---------------------------------------------------------------------------


def _lap(x, dims):
    """The Dirichlet Laplacian on rows ordered as the grid, any number of columns."""
    u = x.reshape(tuple(dims) + (x.shape[-1],))
    y = 2.0 * len(dims) * u
    for a, d in enumerate(dims):
        y.narrow(a, 1, d - 1).sub_(u.narrow(a, 0, d - 1))
        y.narrow(a, 0, d - 1).sub_(u.narrow(a, 1, d - 1))
    return y.reshape(x.shape)


def _cheb(x, dims, coef, lo, hi):
    """sum_j coef[j] T_j(B) x, B = (2 (L + I) - (lo + hi)) / (hi - lo)."""
    def B(u):
        return (2.0 * (_lap(u, dims) + u) - (lo + hi) * u) / (hi - lo)
    b1 = b2 = None
    for cj in list(coef[:0:-1]):
        b = cj * x
        if b1 is not None:
            b += 2.0 * B(b1)
        if b2 is not None:
            b -= b2
        b1, b2 = b, b1
    y = coef[0] * x + B(b1)
    return y - b2 if b2 is not None else y


def _coef(kind, ndim):
    lo, hi = 1.0, 1.0 + 4.0 * ndim
    f, d = ((lambda x: x ** -0.5), 4) if kind == "cheb" else ((lambda x: 1.0 / x), 8)
    th = np.pi * (np.arange(d + 1) + 0.5) / (d + 1)
    fx = f(0.5 * (lo + hi) + 0.5 * (hi - lo) * np.cos(th))
    co = np.array([2.0 / (d + 1) * np.sum(fx * np.cos(j * th)) for j in range(d + 1)])
    co[0] *= 0.5
    return [float(v) for v in co], lo, hi


def _operator(c, dims, V, tau):
    """x -> M (A - tau) M x (T (A - tau) x for the unfactored T) on columns with shifts tau."""
    V = torch.from_numpy(np.asarray(V)).cuda()
    sc = _scale(c)
    diag = 2.0 * len(dims) * sc + V
    off = diag - 2.0 * len(dims) * sc
    if c["vec"] == "f32":   # the matrix as it is given: values rounded to 32 bits
        off = diag.float().double() - 2.0 * len(dims) * sc
    off = off[:, None]

    def amul(x):
        return sc * _lap(x, dims) + (off - tau) * x

    if c["prec"] == "cheb":
        co, lo, hi = _coef("cheb", len(dims))
        return lambda x: _cheb(amul(_cheb(x, dims, co, lo, hi)), dims, co, lo, hi)
    if c["prec"] == "cheb_inv":
        co, lo, hi = _coef("cheb_inv", len(dims))
        return lambda x: _cheb(amul(x), dims, co, lo, hi)
    if c["prec"] == "jacobi":
        d = (diag[:, None] - tau).abs().rsqrt()
        return lambda x: d * amul(d * x)
    return amul


def _orth(w, Q):
    """w without its components along the columns-wise basis Q; also the components."""
    h = torch.stack([(q * w).sum(0) for q in Q])
    for q, a in zip(Q, h):
        w = w - a * q
    return w, h


def _lanczos(op, v, k):
    nu = (v * v).sum(0)
    Q = [v / nu.sqrt()]
    al, be = [], [torch.zeros_like(nu)]
    for i in range(k):
        w = op(Q[i])
        if i:
            w = w - be[i] * Q[i - 1]
        al.append((Q[i] * w).sum(0))
        w = w - al[i] * Q[i]
        for _ in range(2):
            w, _h = _orth(w, Q)
        be.append((w * w).sum(0).sqrt())
        if i + 1 < k:
            Q.append(w / be[i + 1])
    return nu, torch.stack(al), torch.stack(be)


def _jacobi_matrix(al, be, rule):
    """J_k of every column; the (2k-1)-order matrix of the averaged rule with 'ga'."""
    k = al.shape[0]
    off = be[1:k]
    if rule == "ga":
        al = torch.cat([al, al[:k - 1].flip(0)])
        off = torch.cat([off, be[k:k + 1], be[1:k - 1].flip(0)]) if k > 1 else off
    T = torch.diag_embed(al.T.contiguous())
    if off.shape[0]:
        e = off.T.contiguous()
        T = T + torch.diag_embed(e, 1) + torch.diag_embed(e, -1)
    return T


def _spread(per, S, m):
    s = per.reshape(S, m)
    d = s[1:] - s[:-1]
    var = d.var(1, unbiased=True) / m
    return s.mean(1), d.mean(1), var


def _small_eigh(T):
    return torch.linalg.eigh(T.cpu())


def exact(case, seed):
    c = case
    if c["path"] == "ildl":
        return _exact_ildl(c, seed)
    if c["path"] == "batch":
        items = _batch_items(c, seed)
        n = sum(int(np.prod(d)) for d, _, _ in items)
        probes, row, per = _probes(c, n, seed), 0, []
        for d, taus, V in items:
            nb = int(np.prod(d))
            v = probes[row:row + nb].repeat(1, c["shifts"])
            tau = torch.from_numpy(taus).cuda().repeat_interleave(c["m"])
            nu, al, be = _lanczos(_operator(c, d, V, tau), v, c["k"])
            per.append(_gauss(nu, al, be, c["rule"]))
            row += nb
        got = [_spread(p, c["shifts"], c["m"]) for p in per]
        return {"negcounts": torch.stack([g[0] for g in got]).cpu(),
                "counts": torch.stack([g[1] for g in got]).cpu(),
                "variances": torch.stack([g[2] for g in got]).cpu(),
                "per_probe": torch.stack(per), "k_used": None}
    V = _potential(c, seed)
    dims, m = _dims(c), c["m"]
    probes = _probes(c, V.size, seed)
    if c["path"] == "gradient":
        return _exact_gradient(c, V, probes)
    taus = _taus(c, np.random.default_rng(seed)) if c["path"] == "slices" else np.array([c["xi"], c["eta"]])
    S = len(taus)
    tau = torch.from_numpy(np.repeat(taus, m)).cuda()
    op = _operator(c, dims, V, tau)
    v = probes.repeat(1, S)
    alpha = beta = None
    if c["path"] == "arnoldi":
        per = _arnoldi(op, v, c["k"])
    elif c["path"] == "block":
        per = _block(op, v, c["k"])
    else:
        nu, alpha, beta = _lanczos(op, v, c["k"])
        per = _gauss(nu, alpha, beta, c["rule"])
    mean, diff, var = _spread(per, S, m)
    if c["path"] == "slices":
        out = {"negcounts": mean.cpu(), "counts": diff.cpu(), "variances": var.cpu()}
    else:
        out = {"estimate": float(diff[0]), "variance": float(var[0]) if m > 1 else math.nan,
               "neg_xi": float(mean[0]), "neg_eta": float(mean[1])}
    if c["details"]:
        out["per_probe"], out["k_used"] = per, None
        if c["path"] not in ("arnoldi", "block"):
            out["alpha"], out["beta"] = alpha, beta
    return out


def _gauss(nu, al, be, rule):
    th, Z = _small_eigh(_jacobi_matrix(al, be, rule))
    return nu * ((th < 0) * Z[:, 0, :] ** 2).sum(1).to(nu.device)


def _sign_weights(H):
    """e_1^T h(H) e_1 of every matrix, h the open left half-plane: (1 - sign(H)_11) / 2 with the
    sign by Newton's iteration, in extended precision (H is far from normal)."""
    X = H.numpy().astype(np.longdouble)
    k = X.shape[1]
    for _ in range(60):
        A = np.concatenate([X, np.broadcast_to(np.eye(k, dtype=np.longdouble), X.shape)], 2)
        logdet = np.zeros(len(X), dtype=np.longdouble)
        for i in range(k):   # Gauss-Jordan with row pivoting, all matrices at once
            p = i + np.abs(A[:, i:, i]).argmax(1)
            b = np.arange(len(A))
            A[b, p], A[b, i] = A[b, i].copy(), A[b, p].copy()
            piv = A[:, i, i].copy()
            logdet += np.log(np.abs(piv))
            A[:, i] /= piv[:, None]
            f = A[:, :, i].copy()
            f[:, i] = 0
            A -= f[:, :, None] * A[:, i:i + 1]
        mu = np.exp(-logdet / k)[:, None, None]
        Y = 0.5 * (mu * X + A[:, :, k:] / mu)
        done = np.abs(Y - X).max() <= 1e-17 * np.abs(Y).max()
        X = Y
        if done:
            break
    return torch.from_numpy((0.5 * (1 - X[:, 0, 0])).astype(np.float64))


def _arnoldi(op, v, k):
    nu = (v * v).sum(0)
    Q = [v / nu.sqrt()]
    H = torch.zeros(v.shape[1], k, k, dtype=torch.float64)
    for j in range(k):
        w, h = _orth(op(Q[j]), Q)
        w, h2 = _orth(w, Q)
        H[:, :j + 1, j] = (h + h2).T.cpu()
        nrm = (w * w).sum(0).sqrt()
        if j + 1 < k:
            H[:, j + 1, j] = nrm.cpu()
            Q.append(w / nrm)
    return nu * _sign_weights(H).to(nu.device)


def _block(op, v, k, P=16):
    n, C = v.shape
    nb = C // P

    def blocks(x):
        return x.reshape(n, nb, P).permute(1, 0, 2).contiguous()

    def flat(x):
        return x.permute(1, 0, 2).reshape(n, C)

    def qr(x):
        q, r = torch.linalg.qr(x)
        sg = torch.sign(torch.diagonal(r, dim1=1, dim2=2))
        return q * sg[:, None, :], r * sg[:, :, None]

    def tdot(a, b):   # a^T b, the right operand laid out row-major
        return torch.stack([x.T.contiguous() @ y for x, y in zip(a, b)])

    def mul(a, b):
        return torch.stack([x @ y for x, y in zip(a, b)])

    q, R0 = qr(blocks(v))
    Q = [q]
    T = torch.zeros(nb, P * k, P * k, dtype=torch.float64, device=v.device)
    for i in range(k):
        w = blocks(op(flat(Q[i])))
        h = None
        for sweep in range(2):
            for l, ql in enumerate(Q):
                g = tdot(ql, w)
                w = w - mul(ql, g)
                if l == i:
                    h = g if sweep == 0 else h + g
        a = slice(i * P, (i + 1) * P)
        T[:, a, a] = 0.5 * (h + h.transpose(1, 2))
        q, r = qr(w)
        if i + 1 < k:
            e = slice((i + 1) * P, (i + 2) * P)
            T[:, e, a] = r
            T[:, a, e] = r.transpose(1, 2)
            Q.append(q)
    th, Z = _small_eigh(T)
    Y = Z[:, :P, :].transpose(1, 2) @ R0.cpu()
    return ((th < 0)[:, :, None] * Y * Y).sum(1).reshape(C).to(v.device)


class _Apply(torch.autograd.Function):
    """y = M (A - tau) M x with its derivative in x, the potential and the shifts."""

    @staticmethod
    def forward(ctx, x, V, tau, M, lap):
        ctx.M, ctx.lap = M, lap
        ctx.save_for_backward(x, V, tau)
        t = M(x)
        return M(lap(t) + (V[:, None] - tau) * t)

    @staticmethod
    def backward(ctx, g):
        x, V, tau = ctx.saved_tensors
        a, t = ctx.M(g), ctx.M(x)
        at = a * t
        return ctx.M(ctx.lap(a) + (V[:, None] - tau) * a), at.sum(1), -at.sum(0), None, None


class _Quad(torch.autograd.Function):
    """sum_i S(theta_i) z_i(1)^2 of J_k, its gradient by divided differences."""

    @staticmethod
    def forward(ctx, al, be, w):
        th, Z = _small_eigh(_jacobi_matrix(al, be, "gauss"))
        S = 0.5 * torch.erfc(th / w)
        z = Z[:, 0, :]
        dS = -torch.exp(-(th / w) ** 2) / (w * math.sqrt(math.pi))
        dt = th[:, :, None] - th[:, None, :]
        near = dt.abs() < 1e-7 * w
        D = torch.where(near, 0.5 * (dS[:, :, None] + dS[:, None, :]),
                        (S[:, :, None] - S[:, None, :]) / torch.where(near, torch.ones_like(dt), dt))
        ctx.G = (Z @ (D * z[:, :, None] * z[:, None, :]) @ Z.transpose(1, 2)).to(al.device)
        ctx.k = al.shape[0]
        return (S * z * z).sum(1).to(al.device)

    @staticmethod
    def backward(ctx, g):
        ga = torch.diagonal(ctx.G, dim1=1, dim2=2).T * g
        gb = 2.0 * torch.diagonal(ctx.G, 1, 1, 2).T * g
        return ga, torch.cat([torch.zeros_like(gb[:1]), gb]), None


def _exact_gradient(c, V, probes):
    dims, m, k = _dims(c), c["m"], c["k"]
    co, lo, hi = _coef("cheb", len(dims))
    Vt = torch.from_numpy(V).cuda().requires_grad_(True)
    ends = [torch.tensor(c[e], dtype=torch.float64, device="cuda", requires_grad=True) for e in ("xi", "eta")]
    tau = torch.stack(ends).repeat_interleave(m)
    v = probes.repeat(1, 2)
    nu = (v * v).sum(0)
    Q, al, be = [v / nu.sqrt()], [], [torch.zeros_like(nu)]
    for i in range(k):
        w = _Apply.apply(Q[i], Vt, tau, lambda x: _cheb(x, dims, co, lo, hi), lambda x: _lap(x, dims))
        if i:
            w = w - be[i] * Q[i - 1]
        al.append((Q[i] * w).sum(0))
        w = w - al[i] * Q[i]
        for _ in range(2):
            h = torch.stack([(q * w).sum(0) for q in Q])
            w = w - sum(a * q for a, q in zip(h, Q))
        if i + 1 < k:
            be.append((w * w).sum(0).sqrt())
            Q.append(w / be[i + 1])
    s = nu * _Quad.apply(torch.stack(al), torch.stack(be), SMOOTH_W)
    est = (s[m:] - s[:m]).mean()
    dV, dxi, deta = torch.autograd.grad(est, [Vt] + ends)
    return {"estimate": est.detach(), "dV": dV, "dxi": dxi, "deta": deta}


def _exact_ildl(c, seed):
    # the factor is an input of the call; the solves with it are dense here
    A = _matrix(c, _potential(c, seed))
    tau = c["eta"]
    F = ec.ildl_factor(A, tau, c["droptol"])
    n, m = F.n, c["m"]
    L = torch.eye(n, dtype=torch.float64, device="cuda")
    rows = np.repeat(np.arange(n), np.diff(F.l_rp))
    L[torch.from_numpy(rows).cuda(), torch.from_numpy(F.l_ci.astype(np.int64)).cuda()] = torch.from_numpy(F.l_val).cuda()
    perm = torch.from_numpy(F.perm.astype(np.int64)).cuda()
    # |D|^(-1/2) block by block
    e1, eo = 1.0 / np.sqrt(np.abs(np.where(F.d_diag == 0, 1.0, F.d_diag))), np.zeros(n)
    for i in np.nonzero(F.d_off)[0]:
        b = np.array([[F.d_diag[i], F.d_off[i]], [F.d_off[i], F.d_diag[i + 1]]])
        w, z = np.linalg.eigh(b)
        r = (z / np.sqrt(np.abs(w))) @ z.T
        e1[i], e1[i + 1], eo[i] = r[0, 0], r[1, 1], r[0, 1]
    e1, eo = torch.from_numpy(e1).cuda()[:, None], torch.from_numpy(eo).cuda()[:, None]

    def E(x):
        y = e1 * x
        y[1:] += eo[:-1] * x[:-1]
        y[:-1] += eo[:-1] * x[1:]
        return y

    LT = L.T.contiguous()
    amul = _operator(dict(c, prec="none"), _dims(c), np.zeros(n), tau)

    def op(q):
        t = torch.linalg.solve_triangular(LT, E(q), upper=True, unitriangular=True)
        u = torch.empty_like(t)
        u[perm] = t
        return E(torch.linalg.solve_triangular(L, amul(u)[perm], upper=False, unitriangular=True))

    nu, al, be = _lanczos(op, _probes(c, n, seed), c["k"])
    per = _gauss(nu, al, be, c["rule"])
    return {"negcounts": per.mean().reshape(1).cpu(), "counts": torch.zeros(0), "variances": torch.zeros(0),
            "per_probe": per, "k_used": None, "alpha": al, "beta": be}

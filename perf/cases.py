"""Performance cases of the Kronecker CG library: the work that programs have it do, through KronOperator and
kron_cg_solve.

A case is one pass of one kind of work on A = sum_j K_j1 (x) K_j2 [(x) K_j3] + diag(d) + sigma2 I:

  matvec  products with a kept operator (serving, or the inner step of a caller's own iteration)
  solve   right-hand sides against a kept operator, plain CG, mixed precision or preconditioned
  step    forward and backward solve with a kept operator, gradients for every parameter (training with
          fixed structure; a batch of uneven systems, or one large sum of terms)
  fit     kron_cg_solve and its autograd backward from the factors: the operator is built anew in each pass, as
          when the factors come from hyperparameters that moved
  logdet  log determinant by probes and its gradient (the other half of Gaussian process training)
  direct  a new operator solved once by its eigendecomposition

Sizes are those of the repository's configurations, tests and benchmark and the generic ranges around them.
Solutions are asked for to relative residuals of 1e-10 and 1e-11, as where results have to hold in float64.
"""
import math

import numpy as np
import torch

from paper_2309_03060_amd import KronOperator, SystemSpec, kron_cg_solve

DEV = "cuda"


def _case(name, kind, dims, **kw):
    c = {"name": name, "kind": kind, "d1": 0, "d2": 0, "d3": 0, "terms": 1, "nrhs": 1, "diag": False, "prec": "fp32",
         "factors": "rbf", "ell": 0.2, "sigma2": 0.1, "tol": 1e-10, "precond": "none", "systems": 1}
    for k, d in enumerate(dims):
        c["d%d" % (k + 1)] = int(d)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest product: a caller's own iteration on a small grid, latency only
        _case("matvec_tiny_fp32", "matvec", (12, 10, 14), factors="wishart"),
        # an ordinary product on an odd three-mode grid (no mode a multiple of the tiles)
        _case("matvec_odd_fp32", "matvec", (97, 101, 89), nrhs=4),
        # the largest product: the benchmark's 256^3 operator with 8 right-hand sides
        _case("matvec_256_bf16x3", "matvec", (256, 256, 256), nrhs=8, prec="bf16x3", ell=0.15, sigma2=0.05),
        # one small system to the last digits: 64 x 64 points, one right-hand side
        _case("solve_64x64_fp64", "solve", (64, 64), prec="fp64", tol=1e-10),
        # the benchmark's 64^3 grid with 32 right-hand sides, mixed precision
        _case("solve_64cube_fp32", "solve", (64, 64, 64), nrhs=32, ell=0.15),
        # plain float64 CG on an odd three-mode grid
        _case("solve_odd_fp64", "solve", (91, 75, 61), nrhs=4, prec="fp64", ell=0.15),
        # preconditioned CG: two terms and a diagonal, two odd modes
        _case("solve_sum2_pcg", "solve", (150, 131), terms=2, nrhs=8, diag=True, prec="fp64", factors="wishart",
              sigma2=0.05, precond="kron_eig", tol=1e-11),
        # hyperparameter fitting: the operator is new in every pass
        _case("fit_48x40x56_fp32", "fit", (48, 40, 56), nrhs=8, ell=0.2, sigma2=0.5),
        # a batch of 128 uneven systems, 16 to 128 points a mode, forward and backward
        _case("step_uneven_batch", "step", (16, 128), systems=128),
        # sum of four 1024 x 1024 terms and a diagonal, 16 right-hand sides, forward and backward in bfloat16
        _case("step_sum4_1024_bf16", "step", (1024, 1024), terms=4, nrhs=16, diag=True, prec="bf16",
              factors="wishart", sigma2=0.0, tol=1e-11),
        # log determinant and its gradient, 16 probes
        _case("logdet_200x180", "logdet", (200, 180), nrhs=16, prec="fp64", sigma2=1.0, ell=0.1, tol=1e-10),
        # a new operator solved once by its eigendecomposition
        _case("direct_120x90x100", "direct", (120, 90, 100), nrhs=4, prec="fp64", sigma2=0.1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_dims(rng, modes, lo, hi, most):
    """Mode sizes spread over their logarithm, at most `most` unknowns."""
    while True:
        d = [_log_int(rng, lo, hi) for _ in range(modes)]
        if math.prod(d) <= most:
            return d


def draw(rng):
    kind = rng.choice(["matvec", "matvec", "matvec", "solve", "solve", "solve", "solve", "step", "fit", "logdet", "direct"])
    nrhs = _log_int(rng, 1, 16)
    if kind == "matvec":
        modes = rng.choice([2, 3, 3])
        d = _draw_dims(rng, modes, 8, 1024 if modes == 2 else 256, (1 << 25) // nrhs)
        c = _case("", kind, d, nrhs=nrhs, prec=rng.choice(["fp32", "fp32", "bf16x3", "fp64"]),
                  terms=rng.choice([1, 1, 2, 3]), diag=rng.random() < 0.3, factors="wishart")
    elif kind == "solve":
        modes = rng.choice([2, 3])
        d = _draw_dims(rng, modes, 16, 256 if modes == 2 else 112, (1 << 20) // nrhs)
        terms = rng.choice([1, 1, 2])
        if rng.random() < 0.3:
            c = _case("", kind, d, nrhs=nrhs, prec="fp64", terms=2, diag=True, factors="wishart", sigma2=0.05,
                      precond=rng.choice(["jacobi", "kron_eig"]), tol=1e-11)
        else:
            c = _case("", kind, d, nrhs=nrhs, prec=rng.choice(["fp32", "fp64"]), terms=terms,
                      diag=rng.random() < 0.3, ell=round(rng.uniform(0.12, 0.3), 3), sigma2=round(rng.uniform(0.1, 1.0), 3))
    elif kind == "step":
        c = _case("", kind, (16, _log_int(rng, 32, 128)), systems=_log_int(rng, 4, 160))
    elif kind == "fit":
        modes = rng.choice([2, 3])
        d = _draw_dims(rng, modes, 16, 200 if modes == 2 else 72, (1 << 20) // nrhs)
        c = _case("", kind, d, nrhs=nrhs, sigma2=round(rng.uniform(0.3, 1.0), 3), prec=rng.choice(["fp32", "fp64"]))
    elif kind == "logdet":
        d = _draw_dims(rng, 2, 24, 256, 1 << 16)
        c = _case("", kind, d, nrhs=_log_int(rng, 4, 32), prec="fp64", sigma2=round(rng.uniform(0.5, 2.0), 3),
                  ell=round(rng.uniform(0.1, 0.2), 3), tol=1e-10)
    else:
        modes = rng.choice([2, 3])
        d = _draw_dims(rng, modes, 16, 160, (1 << 21) // nrhs)
        c = _case("", kind, d, nrhs=nrhs, prec="fp64", sigma2=round(rng.uniform(0.1, 1.0), 3))
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------------------------------------
def _dims(case):
    return [case[k] for k in ("d1", "d2", "d3") if case[k]]


def _factor(case, gen, m, ell):
    if case["factors"] == "wishart":
        w = torch.randn(m, m, dtype=torch.float64, device=DEV, generator=gen)
        k = w @ w.T / m
        return (0.5 * (k + k.T) + 0.1 * torch.eye(m, dtype=torch.float64, device=DEV)).contiguous()
    p = torch.sort(torch.rand(m, dtype=torch.float64, device=DEV, generator=gen)).values
    d = p[:, None] - p[None, :]
    return torch.exp(-(d * d) / (2.0 * ell * ell)).contiguous()


def _systems(case, seed):
    """Every system's factors, diagonal and sigma2, then the packed right-hand sides (or probes) and loss weights."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    out = []
    if case["systems"] > 1:                       # uneven batch: modes d1..d2, each factor its own lengthscale
        sizes = np.random.default_rng(1000 * case["systems"] + case["d2"])     # the batch's sizes are the program's own
        rng = np.random.default_rng(int(seed))
        for _ in range(case["systems"]):
            dims = [int(v) for v in sizes.integers(case["d1"], case["d2"] + 1, size=2)]
            ells = rng.uniform(0.1, 0.5, size=2)
            out.append(([[_factor(case, gen, m, float(l)) for m, l in zip(dims, ells)]], None,
                        float(rng.uniform(0.1, 0.5))))
    else:
        dims = _dims(case)
        facs = [[_factor(case, gen, m, case["ell"]) for m in dims] for _ in range(case["terms"])]
        d = 0.1 + 0.9 * torch.rand(math.prod(dims), dtype=torch.float64, device=DEV, generator=gen) if case["diag"] else None
        out.append((facs, d, case["sigma2"]))
    n = sum(math.prod(int(k.shape[0]) for k in f[0]) for f, _, _ in out) * case["nrhs"]
    if case["kind"] == "logdet":
        B = torch.where(torch.rand(n, device=DEV, generator=gen) < 0.5, -1.0, 1.0).to(torch.float64)
    else:
        B = torch.randn(n, dtype=torch.float64, device=DEV, generator=gen)
    if case["kind"] == "matvec" and case["prec"] != "fp64":
        B = B.to(torch.float32)
    W = torch.randn(n, dtype=torch.float64, device=DEV, generator=gen) if case["kind"] in ("step", "fit") else None
    return out, B, W


def prepare(case, seed):
    systems, B, W = _systems(case, seed)
    state = {"case": case, "B": B, "W": W}
    specs = [SystemSpec(factors=f, sigma2=s2, diag=d) for f, d, s2 in systems]
    if case["kind"] == "fit":                      # leaves of an optimiser: the factors and the noise
        f, d, s2 = systems[0]
        state["leaves"] = [k.requires_grad_(True) for row in f for k in row]
        state["noise"] = torch.tensor(float(s2), dtype=torch.float64, device=DEV, requires_grad=True)
    elif case["kind"] == "direct":
        state["specs"] = specs
    else:
        state["op"] = KronOperator(specs, prec=case["prec"])
    return state


def run(state):
    case, B = state["case"], state["B"]
    kind, nrhs = case["kind"], case["nrhs"]
    if kind == "matvec":
        return state["op"].matvec(B, nrhs)
    kw = {"tol": case["tol"], "max_iters": 20000}
    if kind == "solve":
        return state["op"].solve(B, nrhs, precond=case["precond"], **kw)[0]
    if kind == "step":
        X, _ = state["op"].solve(B, nrhs, **kw)
        lam, dfac, ddiag, ds2, _ = state["op"].solve_backward(X, state["W"], nrhs, **kw)
        grads = torch.cat([k.reshape(-1) for s in dfac for row in s for k in row])
        return {"x": X, "db": lam, "dfactors": grads, "ddiag": [d for d in ddiag if d is not None], "dsigma2": ds2}
    if kind == "fit":
        k = len(_dims(case))
        rows = [state["leaves"][i:i + k] for i in range(0, len(state["leaves"]), k)]
        X = kron_cg_solve([SystemSpec(factors=rows, sigma2=state["noise"])], B, nrhs, prec=case["prec"], **kw)
        loss = (X * state["W"]).sum()
        return {"x": X.detach(), "grads": torch.autograd.grad(loss, state["leaves"] + [state["noise"]])}
    if kind == "logdet":
        ld, est, X, _ = state["op"].logdet(B, nrhs, tol=case["tol"], max_iters=400, want_solution=True)
        dfac, _, ds2, _ = state["op"].logdet_grad(B, nrhs, tol=case["tol"], x0=X)
        return {"logdet": ld, "est": est, "dfactors": dfac, "dsigma2": ds2}
    op = KronOperator(state["specs"], prec=case["prec"])
    X = op.eig_solve(B, nrhs)
    op.close()
    return X


# ---- the work of a pass -------------------------------------------------------------------------------------
def _mvm_flops(dims, terms, nrhs):
    return 2.0 * terms * nrhs * math.prod(dims) * sum(dims)


def _steps(case, dims):
    """CG iterations of one solve, roughly: eigenvalues above sigma2 found one after the other (RBF), or the condition
    number's bound (Wishart factors have eigenvalues of 0.1 to 4.1)."""
    digits = math.log(2.0 / case["tol"])
    if case["precond"] == "kron_eig":
        return 60
    if case["factors"] == "wishart":
        lo = 0.1 ** len(dims) * case["terms"] + case["sigma2"] + (0.1 if case["diag"] else 0.0)
        kappa = (2.0 ** len(dims) * case["terms"] + case["sigma2"] + 1.0) / lo
        return max(10, int(0.25 * math.sqrt(kappa) * digits))
    top = math.prod(min(m, m * case["ell"] * 2.5) for m in dims) / case["sigma2"]
    return max(10, int((0.1 if len(dims) == 2 else 0.25) * digits * math.sqrt(top)))


def work(case):
    """Inputs and outputs once, and the operations of the method (rough iteration counts for the solves)."""
    nrhs, terms = case["nrhs"], case["terms"]
    batch = [_dims(case)]
    if case["systems"] > 1:
        mid = (case["d1"] + case["d2"]) // 2
        batch = [[mid, mid]] * case["systems"]
    nbytes = flops = 0.0
    for dims in batch:
        n, fac, esz = math.prod(dims), 8 * terms * sum(m * m for m in dims), 8
        mvm = _mvm_flops(dims, terms, nrhs)
        grad = mvm * (len(dims) + 1) / 2.0            # one contraction per factor and the products before it
        if case["kind"] == "matvec":
            esz = 8 if case["prec"] == "fp64" else 4
            nbytes, flops = nbytes + 2 * n * nrhs * esz + fac * esz // 8, flops + mvm
        elif case["kind"] == "solve":
            nbytes, flops = nbytes + 2 * n * nrhs * 8 + fac, flops + mvm * _steps(case, dims)
        elif case["kind"] in ("step", "fit"):
            nbytes, flops = nbytes + 4 * n * nrhs * 8 + 2 * fac, flops + 2 * mvm * _steps(case, dims) + grad
        elif case["kind"] == "logdet":
            nbytes, flops = nbytes + n * nrhs * 8 + 2 * fac, flops + mvm * _steps(case, dims) + grad
        else:
            nbytes, flops = nbytes + 2 * n * nrhs * 8 + fac, flops + 2 * mvm + sum(9.0 * m ** 3 for m in dims)
    return {"bytes": nbytes, "flops": flops}


# ---- the same in plain float64 ------------------------------------------------------------------------------
def _modes(row, V, skip=None):
    """V (r, d1, .., dF) multiplied along every mode but `skip` by that mode's factor."""
    for k, K in enumerate(row):
        if k != skip:
            V = torch.movedim(torch.movedim(V, k + 1, -1).contiguous() @ K.T, -1, k + 1).contiguous()
    return V


def _product(facs, d, s2, V):
    shape = (V.shape[0],) + tuple(int(k.shape[0]) for k in facs[0])
    Y = sum(_modes(row, V.reshape(shape)).reshape(V.shape) for row in facs)
    return Y + (s2 if d is None else s2 + d) * V


def _solve(facs, d, s2, B):
    """A^{-1} B: eigenvectors of the factors for one term, else conjugate gradients restarted to rounding."""
    shape = (B.shape[0],) + tuple(int(k.shape[0]) for k in facs[0])
    if len(facs) == 1 and d is None:
        eig = [torch.linalg.eigh(k.cpu()) for k in facs[0]]
        lam = eig[0][0]
        for e in eig[1:]:
            lam = (lam[:, None] * e[0][None, :]).reshape(-1)
        Q = [e[1].to(DEV) for e in eig]
        T = _modes([q.T for q in Q], B.reshape(shape)).reshape(B.shape) / (lam.to(DEV) + s2)
        return _modes(Q, T.reshape(shape)).reshape(B.shape)
    X = torch.zeros_like(B)
    scale = B.norm(dim=1, keepdim=True)
    for _ in range(4):
        r = B - _product(facs, d, s2, X)
        p, rho, goal, x = r.clone(), (r * r).sum(1, keepdim=True), None, torch.zeros_like(B)
        goal = float((1e-13 * scale).min()) ** 2
        if float(rho.max()) <= goal:
            break
        for it in range(3000):
            q = _product(facs, d, s2, p)
            alpha = rho / (p * q).sum(1, keepdim=True)
            x, r = x + alpha * p, r - alpha * q
            new = (r * r).sum(1, keepdim=True)
            if it % 10 == 9 and float(new.max()) <= goal:
                break
            p, rho = r + (new / rho) * p, new
        X = X + x
    return X


def _gradients(facs, X, lam):
    """-sum_r lambda_r^T (dA/dtheta) x_r for every factor, the diagonal and sigma2."""
    shape = (X.shape[0],) + tuple(int(k.shape[0]) for k in facs[0])
    out = []
    for row in facs:
        for k in range(len(row)):
            Z = torch.movedim(_modes(row, X.reshape(shape), skip=k), k + 1, 0).reshape(shape[k + 1], -1).contiguous()
            L = torch.movedim(lam.reshape(shape), k + 1, 0).reshape(shape[k + 1], -1).contiguous()
            out.append(-(L @ Z.T.contiguous()))
    return out, -(lam * X).sum(0), -(lam * X).sum()


def exact(case, seed):
    systems, B, W = _systems(case, seed)
    nrhs, kind, off, parts = case["nrhs"], case["kind"], 0, []
    for facs, d, s2 in systems:
        n = math.prod(int(k.shape[0]) for k in facs[0])
        b = B[off:off + n * nrhs].view(nrhs, n).to(torch.float64)
        w = W[off:off + n * nrhs].view(nrhs, n) if W is not None else None
        off += n * nrhs
        if kind == "matvec":
            return _product(facs, d, s2, b).reshape(-1)
        x = _solve(facs, d, s2, b)
        lam = _solve(facs, d, s2, w) if w is not None else None
        parts.append((facs, d, s2, b, x, lam))
    facs, d, s2, b, x, lam = parts[0]
    if kind in ("solve", "direct"):
        return x.reshape(-1)
    if kind == "logdet":
        eig = [torch.linalg.eigh(k.cpu()) for k in facs[0]]
        spec = (eig[0][0][:, None] * eig[1][0][None, :]).reshape(-1).to(DEV) + s2
        shape = (nrhs,) + tuple(int(k.shape[0]) for k in facs[0])
        t = _modes([e[1].to(DEV).T for e in eig], b.reshape(shape)).reshape(nrhs, -1)
        est = (t * t * torch.log(spec)).sum(1)
        g, _, gs = _gradients(facs, b, x)
        return {"logdet": est.mean().reshape(1), "est": est, "dfactors": [[[-v / nrhs for v in g]]],
                "dsigma2": (-gs / nrhs).reshape(1)}
    grads = [_gradients(p[0], p[4], p[5]) for p in parts]
    if kind == "fit":
        return {"x": x.reshape(-1), "grads": tuple(grads[0][0] + [grads[0][2].reshape(())])}
    return {"x": torch.cat([p[4].reshape(-1) for p in parts]), "db": torch.cat([p[5].reshape(-1) for p in parts]),
            "dfactors": torch.cat([v.reshape(-1) for g in grads for v in g[0]]),
            "ddiag": [g[1] for g, p in zip(grads, parts) if p[1] is not None],
            "dsigma2": torch.stack([g[2] for g in grads])}

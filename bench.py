"""Benchmark: batched mixed-precision Kronecker CG on one MI355X.

Default workload (one step): 200 CG iterations, from x0 = 0, of A X = B for
the three-mode RBF Kronecker operator A = K1 (x) K2 (x) K3 + 0.05 I (256
points per mode, lengthscale 0.15, n = 16,777,216) with 8 right-hand sides
N(0, 1): low-precision CG (BF16x3 or FP32 matrix-core mode contractions,
FP64 scalars and dot accumulation) with FP64 reliable updates of the
residual, the scheme that solves this operator to a true relative residual
of 1e-6.  Inputs are resident in HBM before the timed region; the operator
is built once.  The full solve to 1e-6, mixed precision against plain FP64
CG on the GPU, runs once outside the timed region (time to solution).

Metric: RHS*iterations/s = CG iterations summed over right-hand sides
divided by the wall time of the timed steps (the FP64 residuals of the
reliable updates are inside the timed region but not counted).

Printed on one JSON line with:
  roofline      the dominant kernel's algorithmic FLOPs (or bytes) per launch
                over its average duration (HIP events on the launch stream,
                recorded around every launch inside the timed region),
                against the peak of its own arithmetic;
  cpu_baseline  the float64 oracle's CG on the same operator, timed on this
                host's cores over a bounded window of iterations;
  mixed_vs_fp64 time to 1e-6 true relative residual: mixed precision versus
                plain FP64 CG on the GPU (outside the timed region).
Other workloads: --workload c1 | c2 | c3 | c5 (see --help).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "Kron-CG RHS·iters/s + % roofline; mixed vs FP64 at 1e-6 rel residual"
HBM_PEAK_GBS = 8000.0
FP32_MFMA_PEAK_TFLOPS = 157.3

# Algorithmic HBM bytes per element of one right-hand side, per launch class
# (FP32 working vectors, 4 bytes per word):
#   slab23        : read r, p (direction formed on the fly), write T      3 words
#                   (modes 3 and 2 fused per 64 x 64 slab in LDS)
#   contract_rows : read r, p (direction formed on the fly), write T      3 words
#   contract_mid  : read T, write T'                                        2 words
#   contract_last : read T', r, p_old, write q, p_new                       5 words
#   update        : read x, r, p, q, write x, r                             6 words
# algorithmic bytes per element and RHS*iteration of each c2 launch class (FP32): slab23 reads r, p and
# writes T; contract_last reads T, p, r and writes q, p; update reads x, p, r, q and writes x, r; the
# fused persistent CG reads r, p, x and writes p, T, x (phase A), reads T, p (B), reads and writes r (C)
BYTES_PER_ELEM = {"slab23": 12, "contract_rows": 12, "contract_mid": 8, "contract_last": 20, "update": 24,
                  "cg_fused": 40}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--m", type=int, default=64, help="points per mode")
    ap.add_argument("--nrhs", type=int, default=32)
    ap.add_argument("--tol", type=float, default=1e-5)
    ap.add_argument("--cpu-iters", type=int, default=40, help="oracle CG iterations timed on the host")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-tts", action="store_true", help="skip the mixed-vs-FP64 time-to-solution runs")
    ap.add_argument("--no-autotune", dest="autotune", action="store_false",
                    help="skip the tile autotuner (cola_autotune) at operator setup")
    ap.add_argument("--workload", default="c4", choices=["c1", "c2", "c3", "c4", "c5"],
                    help="c4 (default): 256^3 x 8 RHS, windows of --window CG iterations; c2: 64^3 x 32 RHS "
                         "solved to 1e-5; c3: 256 uneven systems with backward; c5: sum of 4 1024^2 terms + diag "
                         "with backward; c1: 64^2 FP64")
    ap.add_argument("--window", type=int, default=200,
                    help="c4: CG iterations per timed step (one window of the solve, from x0 = 0)")
    ap.add_argument("--cpu-window", type=int, default=20,
                    help="c4: oracle CG iterations (one right-hand side) timed on the host")
    ap.add_argument("--no-extra", action="store_true",
                    help="c4: skip the short runs of the 64^3 x 32 and sum-of-Kronecker workloads that are "
                         "reported as extra keys")
    ap.add_argument("--prec", default=None, help="working precision for c4/c5 (fp32, bf16x3, bf16)")
    ap.add_argument("--inner-tol", type=float, default=None,
                    help="reliable-update threshold delta for c1/c4/c5 (default 0.3 on c4, 0.1 otherwise)")
    ap.add_argument("--counters", action="store_true",
                    help="short run for hardware-counter collection (c2, c4 or c5): set-up and autotuner, a "
                         "256 MiB device copy (reference for the HBM byte counters), then one solve capped "
                         "at --max-iters iterations")
    ap.add_argument("--pmc-summary", nargs="+", default=None, metavar="CSV",
                    help="summarise rocprofv3 --pmc CSV files of a --counters run of --workload (no GPU use)")
    ap.add_argument("--trace-summary", nargs=3, default=None, metavar=("PREFIX", "CMD", "TITLE"),
                    help="summarise rocprofv3 kernel-trace CSVs PREFIX_kernel_stats.csv / _kernel_trace.csv")
    ap.add_argument("--pmc-out", default=None, help="with --pmc-summary: JSON file to merge the traffic record into")
    ap.add_argument("--autograd", action="store_true",
                    help="backward runtime and peak memory: adjoint rules against unrolled autodiff (JSON)")
    ap.add_argument("--autograd-steps", type=int, nargs="+", default=[16, 32, 64, 128, 256, 512, 1024])
    ap.add_argument("--autograd-sizes", type=int, nargs="+", default=[16, 24, 32, 48, 64, 96])
    ap.add_argument("--autograd-logdet-steps", type=int, nargs="+", default=[16, 32, 64, 128, 256])
    ap.add_argument("--check-every", type=int, default=128,
                    help="CG iterations between host convergence checks (one fused launch each)")
    ap.add_argument("--max-iters", type=int, default=None,
                    help="cap on CG iterations per solve (default: the workload's own limit)")
    return ap.parse_args()


def direct_solve(op, B, nrhs, n, cg_seconds=None):
    """Kronecker-eigen direct solve (cola_eig_solve): first call (factor eigendecomposition + solve) and a
    repeat call, timed; the FP64 relative residual is formed with the library's FP64 MVM."""
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    op.eig_solve(B, nrhs)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    X = op.eig_solve(B, nrhs)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    R = (B - op.matvec(X, nrhs, prec="fp64")).view(nrhs, n)
    rel = float((R.norm(dim=1) / B.view(nrhs, n).norm(dim=1)).max())
    out = {"first_call_seconds": round(t1 - t0, 4), "solve_seconds": round(t2 - t1, 5), "relres_max": rel,
           "note": "first call includes the FP64 Jacobi eigendecomposition of every factor"}
    if cg_seconds:
        out["speedup_vs_mixed_cg_first_call"] = round(cg_seconds / (t1 - t0), 1)
    progress(f"direct eigen solve: first call {t1 - t0:.3f} s, repeat {t2 - t1:.4f} s, relres {rel:.2e}")
    return out


def slq_measure(op, factors, sigma2, n, nprobes=32, max_iters=300, tol=1e-8, seed=7):
    """Stochastic Lanczos quadrature of log det A (cola_slq_logdet) with Rademacher probes, timed; the
    closed form sum(log(eigenvalue products + sigma2)) of the single Kronecker term is the reference."""
    import numpy as np
    import torch
    import workloads as wl
    from paper_2309_03060_amd import decode_info
    Z = torch.tensor(wl.rademacher_probes(np.random.default_rng(seed), nprobes, n), device="cuda:0").reshape(-1)
    op.logdet(Z, nprobes, tol=tol, max_iters=max_iters)            # workspace allocation
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ld, est, _, info = op.logdet(Z, nprobes, tol=tol, max_iters=max_iters)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    lam = np.array([1.0])
    for f in factors:
        lam = np.kron(lam, np.linalg.eigvalsh(0.5 * (f + f.T)))
    exact = float(np.sum(np.log(lam + sigma2)))
    e = est.cpu().numpy()
    rec = decode_info(info, nprobes)
    out = {"seconds": round(dt, 4), "probes": nprobes, "lanczos_steps_max": max(r["iters"] for r in rec),
           "estimate": float(ld[0]), "closed_form": exact, "rel_error": abs(float(ld[0]) - exact) / abs(exact),
           "std_error": float(e.std(ddof=1) / np.sqrt(nprobes)),
           "note": "FP64 CG over the probes to 1e-8 (at most 300 steps); per-probe Gauss quadrature on the device"}
    progress(f"SLQ log det: {out['estimate']:.6e} vs {exact:.6e} in {dt:.3f} s")
    return out


# ---------------------------------------------------------------------------------------------
# Backward-pass memory and runtime: the adjoint rules (App. B.2) against unrolled autodiff, i.e.
# torch's autograd recording every iteration of a plain-torch CG (the comparison of App. B's figure
# on backward runtime and peak memory).  The unrolled solver below is that comparison baseline only.

def torch_kron3_mvm(K, sigma2, X):
    """(K1 (x) K2 (x) K3 + sigma2 I) X for X of shape (r, m1, m2, m3), in plain torch matmuls."""
    import torch
    r, m1, m2, m3 = X.shape
    Y = torch.matmul(X, K[2].t().contiguous())                              # mode 3
    Y = torch.matmul(K[1], Y)                                               # mode 2
    Y = torch.matmul(K[0], Y.reshape(r, m1, m2 * m3)).reshape(r, m1, m2, m3)   # mode 1
    return Y + sigma2 * X


def unrolled_cg(K, sigma2, B, iters):
    """iters steps of textbook CG (x0 = 0) on (r, m1, m2, m3) blocks, every step recorded by autograd;
    returns x and the per-step coefficients (alpha_j, beta_j) as graph tensors of shape (r,)."""
    import torch
    x = torch.zeros_like(B)
    res = B
    p = B
    rho = (res * res).sum(dim=(1, 2, 3))
    alphas, betas = [], []
    for _ in range(iters):
        q = torch_kron3_mvm(K, sigma2, p)
        alpha = rho / (p * q).sum(dim=(1, 2, 3))
        a4 = alpha[:, None, None, None]
        x = x + a4 * p
        res = res - a4 * q
        rho_new = (res * res).sum(dim=(1, 2, 3))
        beta = rho_new / rho
        p = res + beta[:, None, None, None] * p
        rho = rho_new
        alphas.append(alpha)
        betas.append(beta)
    return x, alphas, betas


def unrolled_slq_logdet(K, sigma2, Z, iters):
    """Mean over probes of ||z||^2 e1^T log(T) e1, T the Lanczos tridiagonal built from the unrolled
    CG's coefficients, its eigendecomposition by torch.linalg.eigh: all of it under autograd."""
    import torch
    _, al, be = unrolled_cg(K, sigma2, Z, iters)
    a = torch.stack(al, 1)
    b = torch.stack(be, 1)
    d = torch.cat([1.0 / a[:, :1], 1.0 / a[:, 1:] + b[:, :-1] / a[:, :-1]], 1)
    e = torch.sqrt(b[:, :-1]) / a[:, :-1]
    T = torch.diag_embed(d) + torch.diag_embed(e, 1) + torch.diag_embed(e, -1)
    lam, V = torch.linalg.eigh(T)
    est = (Z * Z).sum(dim=(1, 2, 3)) * (V[:, 0, :] ** 2 * torch.log(lam)).sum(-1)
    return est.mean()


def _rbf_factors(pts, ell):
    import torch
    out = []
    for p in pts:
        d = p[:, None] - p[None, :]
        out.append(torch.exp(-(d * d) / (2.0 * ell * ell)))
    return out


def _peak_begin():
    import torch
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    return torch.cuda.memory_allocated(), time.perf_counter()


def _peak_end(base):
    import torch
    torch.cuda.synchronize()
    return torch.cuda.max_memory_allocated() - base, time.perf_counter()


def autograd_solve_pair(pts_np, ell0, s2_0, nrhs, iters=None, tol=1e-10, max_iters=4000, seed=11,
                        run_unrolled=True):
    """One size of the solve comparison: L = <W, A^{-1} B> with A = RBF(l) (x) RBF(l) (x) RBF(l) + s2 I,
    gradients with respect to l, s2 and B.  The adjoint path is kron_cg_solve (FP64 CG to `tol`, or
    exactly `iters` steps when given); the unrolled path runs as many CG steps in plain torch.
    Peak memory is torch's allocator peak over forward + backward above what was allocated before, plus
    (adjoint path) the operator's own device buffers (cola_op_memory)."""
    import torch
    from paper_2309_03060_amd import SystemSpec, kron_cg_solve, decode_info
    dev = "cuda:0"
    m = [len(p) for p in pts_np]
    n = int(np.prod(m))
    rng = np.random.default_rng(seed)
    B0 = torch.tensor(rng.standard_normal((nrhs, n)), device=dev)
    W0 = torch.tensor(rng.standard_normal((nrhs, n)), device=dev)
    pts = [torch.tensor(p, device=dev) for p in pts_np]
    out = {"dims": m, "n": n, "nrhs": nrhs}

    def params():
        ell = torch.tensor(ell0, dtype=torch.float64, device=dev, requires_grad=True)
        s2 = torch.tensor(s2_0, dtype=torch.float64, device=dev, requires_grad=True)
        B = B0.clone().requires_grad_(True)
        return ell, s2, B

    # adjoint rules
    ell, s2, B = params()
    base, t0 = _peak_begin()
    K = _rbf_factors(pts, ell)
    opts = dict(tol=tol, max_iters=max_iters, prec="fp64", check_every=32)
    if iters is not None:
        opts.update(tol=1e-30, max_iters=iters)
    X = kron_cg_solve([SystemSpec(factors=[K], sigma2=s2)], B.reshape(-1), nrhs, **opts)
    loss = (W0.reshape(-1) * X).sum()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    loss.backward()
    peak, t2 = _peak_end(base)
    node = X.grad_fn
    rec = decode_info(node.info, nrhs)
    k = max(r["iters"] for r in rec)
    lib_peak = int(node.device_peak_bytes)
    adj = {"iters": k, "status": sorted({r["status"] for r in rec}), "forward_s": round(t1 - t0, 5), "backward_s": round(t2 - t1, 5),
           "peak_bytes": int(peak + lib_peak), "torch_peak_bytes": int(peak), "library_peak_bytes": lib_peak,
           "grad_ell": float(ell.grad), "grad_sigma2": float(s2.grad)}
    gB = B.grad.detach().clone()
    del X, loss, node, K
    out["adjoint"] = adj
    if not run_unrolled:
        return out
    # unrolled autodiff through the same number of CG steps (after two untimed steps that let the
    # BLAS library allocate its workspace, which it keeps)
    ell, s2, B = params()
    x, _, _ = unrolled_cg(_rbf_factors(pts, ell), s2, B.reshape(nrhs, *m), 2)
    x.sum().backward()
    del x
    ell, s2, B = params()
    base, t0 = _peak_begin()
    K = _rbf_factors(pts, ell)
    x, _, _ = unrolled_cg(K, s2, B.reshape(nrhs, *m), k)
    loss = (W0.reshape(nrhs, *m) * x).sum()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    loss.backward()
    peak, t2 = _peak_end(base)
    unr = {"iters": k, "forward_s": round(t1 - t0, 5), "backward_s": round(t2 - t1, 5),
           "peak_bytes": int(peak), "grad_ell": float(ell.grad), "grad_sigma2": float(s2.grad)}
    unr["grad_B_rel_diff"] = float((B.grad - gB).abs().max() / gB.abs().max())
    del x, loss, K
    out["unrolled"] = unr
    out["memory_ratio"] = round(unr["peak_bytes"] / adj["peak_bytes"], 3)
    out["backward_speedup"] = round(unr["backward_s"] / adj["backward_s"], 3)
    out["grad_rel_diff"] = {k2: abs(unr[k2] - adj[k2]) / abs(adj[k2]) for k2 in ("grad_ell", "grad_sigma2")}
    return out


def autograd_logdet_pair(pts_np, ell0, s2_0, nprobes, iters, seed=13, run_unrolled=True):
    """One size of the log det comparison, exactly `iters` Lanczos (CG) steps per probe on both paths:
    cola_slq_logdet + the Hutchinson gradient through the adjoint backward (X = G = Z), against
    autograd through the unrolled CG, the tridiagonal and its eigendecomposition."""
    import torch
    import workloads as wl
    from paper_2309_03060_amd import KronOperator, SystemSpec
    dev = "cuda:0"
    m = [len(p) for p in pts_np]
    n = int(np.prod(m))
    Z = torch.tensor(wl.rademacher_probes(np.random.default_rng(seed), nprobes, n), device=dev)
    pts = [torch.tensor(p, device=dev) for p in pts_np]
    out = {"dims": m, "n": n, "probes": nprobes, "iters": iters}
    ell = torch.tensor(ell0, dtype=torch.float64, device=dev, requires_grad=True)
    s2 = torch.tensor(s2_0, dtype=torch.float64, device=dev, requires_grad=True)
    base, t0 = _peak_begin()
    K = _rbf_factors(pts, ell)
    op = KronOperator([SystemSpec(factors=[[k.detach() for k in K]], sigma2=float(s2_0))], prec="fp64")
    ld, _, _, _ = op.logdet(Z.reshape(-1), nprobes, tol=1e-30, max_iters=iters)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    dfac, _, ds2, _ = op.logdet_grad(Z.reshape(-1), nprobes, tol=1e-30, max_iters=iters)
    torch.autograd.backward(K, dfac[0][0])
    peak, t2 = _peak_end(base)
    lib_peak = op.memory()[1]
    op.close()
    out["adjoint"] = {"forward_s": round(t1 - t0, 5), "backward_s": round(t2 - t1, 5),
                      "peak_bytes": int(peak + lib_peak), "torch_peak_bytes": int(peak),
                      "library_peak_bytes": int(lib_peak), "logdet": float(ld[0]),
                      "grad_ell": float(ell.grad), "grad_sigma2": float(ds2[0])}
    del K, dfac
    if not run_unrolled:
        return out
    ell = torch.tensor(ell0, dtype=torch.float64, device=dev, requires_grad=True)
    s2 = torch.tensor(s2_0, dtype=torch.float64, device=dev, requires_grad=True)
    unrolled_slq_logdet(_rbf_factors(pts, ell), s2, Z.reshape(nprobes, *m), 2).backward()   # library workspaces
    ell.grad = None
    s2.grad = None
    base, t0 = _peak_begin()
    K = _rbf_factors(pts, ell)
    ldu = unrolled_slq_logdet(K, s2, Z.reshape(nprobes, *m), iters)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ldu.backward()
    peak, t2 = _peak_end(base)
    out["unrolled"] = {"forward_s": round(t1 - t0, 5), "backward_s": round(t2 - t1, 5), "peak_bytes": int(peak),
                       "logdet": float(ldu.detach()), "grad_ell": float(ell.grad), "grad_sigma2": float(s2.grad)}
    del K, ldu
    out["memory_ratio"] = round(out["unrolled"]["peak_bytes"] / out["adjoint"]["peak_bytes"], 3)
    out["backward_speedup"] = round(out["unrolled"]["backward_s"] / out["adjoint"]["backward_s"], 3)
    out["grad_sigma2_rel_diff"] = abs(out["unrolled"]["grad_sigma2"] - out["adjoint"]["grad_sigma2"]) / abs(
        out["adjoint"]["grad_sigma2"])
    return out


def run_autograd_sweep(args):
    """Backward runtime and peak memory against CG steps (64^3 operator) and against problem size
    (m^3, m = 16 .. 96, solved to 1e-10) for A^{-1} b, and against steps for log det.  The unrolled
    path is skipped where its predicted memory (about 12 stored vectors per step) exceeds 96 GB."""
    import workloads as wl
    ell, s2 = 0.15, 0.05
    res = {"experiment": "autograd_memory_runtime",
           "operator": "RBF(l) (x) RBF(l) (x) RBF(l) + s2 I, l = 0.15, s2 = 0.05, gradients in l, s2, b",
           "solve_vs_steps": [], "solve_vs_size": [], "logdet_vs_steps": []}
    pts64 = wl.config2(m=64, nrhs=1).systems[0].points

    def fits(n, rows, steps):
        return 12 * 8 * n * rows * steps <= 96e9

    autograd_solve_pair(pts64, ell, s2, 1, iters=8)                     # warm-up (kernels, allocator)
    for k in args.autograd_steps:
        r = autograd_solve_pair(pts64, ell, s2, 1, iters=k, run_unrolled=fits(64 ** 3, 1, k))
        res["solve_vs_steps"].append(r)
        progress(f"autograd solve, {k} steps: adjoint {r['adjoint']['peak_bytes'] / 2**20:.1f} MiB "
                 f"{r['adjoint']['backward_s']:.4f} s; unrolled "
                 + (f"{r['unrolled']['peak_bytes'] / 2**20:.1f} MiB {r['unrolled']['backward_s']:.4f} s"
                    if "unrolled" in r else "skipped"))
    for mm in args.autograd_sizes:
        pts = wl.config2(m=mm, nrhs=1).systems[0].points
        probe = autograd_solve_pair(pts, ell, s2, 1, tol=1e-10, run_unrolled=False)
        k = probe["adjoint"]["iters"]
        r = autograd_solve_pair(pts, ell, s2, 1, tol=1e-10, run_unrolled=fits(mm ** 3, 1, k))
        res["solve_vs_size"].append(r)
        progress(f"autograd solve, {mm}^3 ({k} steps): adjoint {r['adjoint']['peak_bytes'] / 2**20:.1f} MiB; "
                 + (f"unrolled {r['unrolled']['peak_bytes'] / 2**20:.1f} MiB" if "unrolled" in r else "skipped"))
    autograd_logdet_pair(pts64, ell, s2, 8, 8)                         # warm-up of the log det path
    for k in args.autograd_logdet_steps:
        r = autograd_logdet_pair(pts64, ell, s2, 8, k, run_unrolled=fits(64 ** 3, 8, k))
        res["logdet_vs_steps"].append(r)
        progress(f"autograd log det, {k} steps: adjoint {r['adjoint']['peak_bytes'] / 2**20:.1f} MiB; "
                 + (f"unrolled {r['unrolled']['peak_bytes'] / 2**20:.1f} MiB" if "unrolled" in r else "skipped"))
    return res


def copy_bandwidth(nbytes=1 << 30, reps=10):
    """GB/s of a plain device-to-device copy (bytes read plus bytes written per second)."""
    import torch
    src = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda:0").fill_(1.0)
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        dst.copy_(src)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    del src, dst
    return 2.0 * nbytes * reps / dt / 1e9


def progress(msg):
    """One line per finished piece of work, on stderr (the JSON result stays alone on stdout)."""
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def cpu_baseline(w, iters):
    """The oracle's float64 CG (numpy) on the same operator: bounded window of iterations."""
    from oracle import cg as ocg
    from oracle import kron
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count() or 1
    s = w.systems[0]
    B = w.B[0]
    apply_A = lambda V: kron.mvm(s.factors, V, s.sigma2)
    ocg.cg(apply_A, B[:, :], tol=1e-30, max_iters=2)             # warm caches / BLAS threads
    t0 = time.perf_counter()
    res = ocg.cg(apply_A, B, tol=1e-30, max_iters=iters)
    dt = time.perf_counter() - t0
    rhs_iters = int(res.iters.sum())
    out = {"value": rhs_iters / dt, "unit": "RHS*iters/s", "cores": int(cores), "kind": "oracle",
           "sample": f"numpy float64 CG on the same operator, {B.shape[0]} RHS x {iters} iterations "
                     f"({rhs_iters} RHS*iters) in {dt:.2f} s"}
    try:                                   # the same oracle on one core, over a shorter window
        from threadpoolctl import threadpool_limits
        it1 = max(2, iters // 10)
        with threadpool_limits(limits=1):
            t0 = time.perf_counter()
            r1 = ocg.cg(apply_A, B, tol=1e-30, max_iters=it1)
            d1 = time.perf_counter() - t0
        out["single_core"] = {"value": float(r1.iters.sum()) / d1, "cores": 1,
                              "sample": f"{B.shape[0]} RHS x {it1} iterations in {d1:.2f} s"}
    except Exception as e:                 # threadpoolctl missing: report why
        out["single_core"] = {"error": str(e)[:120]}
    return out


def kernel_table(op, names):
    kern = {}
    for name in names:
        ms, cnt = op.profile_read(name)
        if cnt:
            kern[name] = {"total_ms": ms, "launches": cnt, "avg_us": 1e3 * ms / cnt}
    return kern


def solve_stats(infos, decode_info, count):
    recs = [decode_info(i, count) for i in infos]
    return (sum(r["iters"] for rec in recs for r in rec), sorted({r["status"] for rec in recs for r in rec}),
            max(r["relres"] for rec in recs for r in rec))


def timed_solves(op, B, nrhs, opts, steps, warmup, decode_info, count, backward=None):
    """warmup + timed steps of solve (and optional backward); returns (seconds, infos)."""
    import torch
    for k in range(warmup):
        X, _ = op.solve(B, nrhs, **opts)
        if backward is not None:
            op.solve_backward(X, backward, nrhs, **opts)
        torch.cuda.synchronize()
        progress(f"warmup step {k + 1}/{warmup} done")
    op.profile_enable(True)
    infos = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(steps):
        X, info = op.solve(B, nrhs, **opts)
        infos.append(info)
        if backward is not None:
            out = op.solve_backward(X, backward, nrhs, **opts)
            infos.append(out[-1])
        progress(f"timed step {k + 1}/{steps} enqueued")
    torch.cuda.synchronize()
    return time.perf_counter() - t0, infos


def run_uneven_batch(args):
    """256 uneven K1(x)K2 + s2 I systems: forward solve + adjoint backward per step."""
    import torch
    import workloads as wl
    from paper_2309_03060_amd import KronOperator, SystemSpec, decode_info
    dev = torch.device("cuda:0")
    w = wl.config3()
    specs = [SystemSpec(factors=[[torch.tensor(f, device=dev) for f in s.factors[0]]], sigma2=s.sigma2)
             for s in w.systems]
    op = KronOperator(specs, prec="fp32")
    B = torch.cat([torch.tensor(b.reshape(-1), device=dev) for b in w.B]).contiguous()
    G = torch.cat([torch.tensor(x.reshape(-1), device=dev) for x in w.W]).contiguous()
    opts = dict(tol=1e-5, max_iters=20000, prec="fp32", inner_tol=0.1, check_every=32)
    nsys = len(w.systems)
    dt, infos = timed_solves(op, B, 1, opts, args.steps, args.warmup, decode_info, nsys, backward=G)
    rhs_iters, statuses, worst = solve_stats(infos, decode_info, nsys)
    kern = kernel_table(op, ["resident"])
    op.profile_enable(False)
    # algorithmic FP32 MFMA work of the resident kernel: per item iteration 2 n (n1 + n2)
    # flops, summed over the items' iteration counts
    iters_per_sys = np.zeros(nsys)
    for info in infos:
        for k, r in enumerate(decode_info(info, nsys)):
            iters_per_sys[k] += r["iters"]
    flops = sum(it * 2.0 * s.n * (s.dims[0] + s.dims[1]) for it, s in zip(iters_per_sys, w.systems))
    roof = None
    if "resident" in kern:
        t = kern["resident"]["total_ms"] * 1e-3
        ach = flops / t / 1e12
        roof = {"kernel": "resident", "bound": "mfma", "achieved": round(ach, 3), "peak": FP32_MFMA_PEAK_TFLOPS,
                "unit": "TFLOP/s", "frac": round(ach / FP32_MFMA_PEAK_TFLOPS, 4), "traffic": None,
                "flops_per_launch": flops / kern["resident"]["launches"],
                "avg_launch_us": round(kern["resident"]["avg_us"], 1), "launches": kern["resident"]["launches"]}
    cpu = None
    if not args.no_cpu:
        from oracle import cg as ocg
        from oracle import kron
        sample = list(range(0, nsys, 16))
        t0 = time.perf_counter()
        tot = 0
        for k in sample:
            s = w.systems[k]
            res = ocg.cg(lambda V: kron.mvm(s.factors, V, s.sigma2), w.B[k], 1e-5, 20000)
            tot += int(res.iters.sum())
        dtc = time.perf_counter() - t0
        cpu = {"value": tot / dtc, "unit": "RHS*iters/s", "cores": _cores(), "kind": "oracle",
               "sample": f"numpy float64 CG to 1e-5 on {len(sample)} of the {nsys} systems "
                         f"({tot} RHS*iters in {dtc:.2f} s)"}
    op.close()
    return {"metric": METRIC, "value": round(rhs_iters / dt, 1), "unit": "RHS*iters/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(1e3 * dt / args.steps, 3),
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
            "config": {"workload": "256 independent K1(x)K2+s2 I systems, dims U{16..128}, RBF l~U[0.1,0.5], "
                                   "s2~U[0.01,0.1], 1 RHS each; forward solve to 1e-5 + adjoint backward "
                                   "(second solve + factor/sigma2 gradients) per step; FP32 resident kernel with "
                                   "FP64 reliable updates", "systems": nsys,
                       "unknowns": int(sum(s.n for s in w.systems)),
                       "rhs_iters_per_step": rhs_iters // max(1, args.steps), "statuses": statuses,
                       "worst_relres": worst, "parallelism": "single GPU"},
            "roofline": roof, "cpu_baseline": cpu}


def _cores():
    try:
        from threadpoolctl import threadpool_info
        return int(max([p.get("num_threads", 1) for p in threadpool_info()] or [1]))
    except Exception:
        return os.cpu_count() or 1


def host_info():
    """CPU model, the CPUs this process may run on, and the BLAS threads the oracle will use."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.lower().startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        avail = len(os.sched_getaffinity(0))
    except (AttributeError, OSError):
        avail = os.cpu_count() or 1
    return {"cpu_model": model, "nproc": avail, "blas_threads": _cores()}


# peak of the arithmetic each working precision's contractions run on (TFLOP/s, dense)
MFMA_PEAK_TFLOPS = {"fp32": FP32_MFMA_PEAK_TFLOPS, "bf16": 2500.0, "bf16x3": 2500.0, "fp64": 78.6}
# matrix-core products per useful one: BF16x3 forms hh, hm, mh, hl, lh and mm of the three-way splits
PRODUCTS_PER_FLOP = {"fp32": 1, "bf16": 1, "bf16x3": 6, "fp64": 1}


ENGINE_NOTE = {
    "c4": "mixed on the BF16x3 three-GEMM engine (its FP64 reliable-update residuals on the FP64 three-GEMM "
          "engine), fp64_cg on the FP64 three-GEMM engine: both sides on dense matrix-core GEMMs",
    "c5": "mixed on the BF16 two-GEMM engine (FP64 residuals on the FP64 two-GEMM engine), fp64_cg on the FP64 "
          "two-GEMM engine",
}


def class_model(cls, prec, n, dims, J, has_diag, deferral):
    """(algorithmic FLOPs, algorithmic HBM bytes) per right-hand-side iteration of one launch class of the
    low-precision MVM and CG update (FP32 working vectors: 4 bytes a word), or None for other classes.

    Three-GEMM passes (one term, three 256-wide modes): the direction pass reads r and p_old and writes p
    and its output (16 B; +8 B when it also takes x += alpha p: deferral "first", the FP32 engine); the
    middle pass reads and writes one intermediate (8 B); the last pass reads the intermediate and p and
    writes q (12 B, +4 B for a diagonal).  Deferral "split" (the BF16x3 engine, all modes 256, the
    direction in two alternating buffers): the middle and the last pass each take x += alpha p_old on
    half of x (x and p_old read, x written: +6 B per element each).  Two-GEMM passes (BF16, J terms): the pack reads r, p_old and writes p and its BF16 copy
    (14 B); mode 2 reads the BF16 copy and writes J BF16 intermediates; mode 1 reads them, p (and d) and
    writes q.  The vector update reads x, r, p, q and writes x, r (24 B; 12 B when x is left to the
    GEMM passes).  FLOPs are the mode's Table 2 contraction cost times the matrix-core products per
    useful product."""
    prod = PRODUCTS_PER_FLOP[prec]
    F = len(dims)
    if cls == "update":
        return 6.0 * n, (12.0 if deferral else 24.0) * n
    if F == 3 and J == 1 and cls.startswith("gemm_mode"):
        m = int(cls[-1])
        fl = 2.0 * n * dims[m - 1] * prod
        split = 6.0 if deferral == "split" else 0.0
        by = {3: 16.0 + (8.0 if deferral == "first" else 0.0), 2: 8.0 + split,
              1: 12.0 + (4.0 if has_diag else 0.0) + split}[m]
        return fl, by * n
    if F == 2 and cls == "gemm_pack":
        return 2.0 * n, 14.0 * n
    if F == 2 and cls == "gemm_mode2":
        return 2.0 * n * dims[1] * J * prod, (2.0 + 2.0 * J) * n
    if F == 2 and cls == "gemm_mode1":
        return 2.0 * n * dims[0] * J * prod, (2.0 * J + 8.0 + (4.0 if has_diag else 0.0)) * n
    return None


def run_single(args, name):
    """Large single-system workloads: 256^3 x 8 RHS (windows of CG iterations), the sum of 4 1024^2
    terms + diag (solve + backward per step), or the 64^2 FP64 system (one solve per step)."""
    import torch
    import workloads as wl
    from paper_2309_03060_amd import KronOperator, SystemSpec, decode_info
    dev = torch.device("cuda:0")
    window = None
    if name == "c4":
        w = wl.config4()
        prec, tol = args.prec or "bf16x3", 1e-6
        window = args.window
        label = (f"K1(x)K2(x)K3+0.05I, RBF l=0.15 on 256 U[0,1] points per mode, n=16777216, 8 RHS N(0,1); "
                 f"one step = {window} CG iterations from x0=0 ({prec} contractions, FP64 reliable updates; "
                 f"the full solve targets true relres 1e-6)")
    elif name == "c5":
        w = wl.config5()
        prec, tol, label = args.prec or "bf16", 1e-6, "sum_4 U_j(x)V_j + diag(d), Wishart 1024^2, 16 RHS, to 1e-6"
    else:
        w = wl.config1()
        prec, tol, label = "fp64", 1e-10, "K1(x)K2+0.1I RBF l=0.2, 64^2, 1 RHS, FP64 to 1e-10"
    s = w.systems[0]
    nrhs = w.B[0].shape[0]
    spec = SystemSpec(factors=[[torch.tensor(f, device=dev) for f in row] for row in s.factors], sigma2=s.sigma2,
                      diag=None if s.diag is None else torch.tensor(s.diag, device=dev))
    op = KronOperator([spec], prec="fp32" if prec == "fp64" else prec)
    B = torch.tensor(w.B[0], device=dev).reshape(-1).contiguous()
    progress(f"{name}: operator built ({prec})")
    if args.autotune:
        op.autotune(nrhs)
    full_max = args.max_iters or 60000
    # reliable-update threshold: on the 256^3 RBF operator a residual replacement every time the
    # recursive residual has fallen to 0.3 of its last true value takes 15 % fewer iterations to
    # 1e-6 than every decade (20.5k against 24.0k; 0.3 to 0.9 all give 20.0k-20.6k, 0.01 diverges)
    delta = args.inner_tol if args.inner_tol is not None else (0.3 if name == "c4" else 0.1)
    opts = dict(tol=tol, max_iters=window or full_max, prec=prec, inner_tol=delta, check_every=32)
    G = torch.tensor(w.W[0], device=dev).reshape(-1).contiguous() if (name == "c5" and w.W) else None
    dt, infos = timed_solves(op, B, nrhs, opts, args.steps, args.warmup, decode_info, nrhs, backward=G)
    rhs_iters, statuses, worst = solve_stats(infos, decode_info, nrhs)
    names = ["slab23", "contract_rows", "contract_mid", "contract_last", "gemm_pack", "gemm_mode3", "gemm_mode2",
             "gemm_mode1", "update"]
    if prec == "fp64":
        names = [k + "_fp64" for k in names] + ["small_cg64"]
    kern = kernel_table(op, names)
    resid64 = kernel_table(op, ["slab23_fp64", "contract_rows_fp64", "contract_mid_fp64", "contract_last_fp64",
                                "gemm_mode3_fp64", "gemm_mode2_fp64", "gemm_mode1_fp64"]) \
        if prec != "fp64" else {}
    op.profile_enable(False)
    n = s.n
    dims = [f.shape[0] for f in s.factors[0]]
    J = len(s.factors)
    prod = PRODUCTS_PER_FLOP[prec]
    # algorithmic FLOPs of one RHS*iteration of the working-precision MVM (Table 2 cost, per mode),
    # times the matrix-core products the working precision prescribes per useful product
    flop_rhs_it = 2.0 * n * J * sum(dims) * prod
    # where x += alpha p goes in reliable-update solves (the engine's choice for this operator and precision)
    deferral = None
    if name == "c4" and prec == "fp32":
        deferral = "first"
    elif name == "c4" and prec == "bf16x3" and all(d == 256 for d in dims):
        deferral = "split"
    models = {k: class_model(k, prec, n, dims, J, s.diag is not None, deferral) for k in kern}
    models = {k: m for k, m in models.items() if m is not None}
    per_kernel = {}
    for k, v in kern.items():
        per_kernel[k] = {"avg_us": round(v["avg_us"], 2), "launches": v["launches"],
                         "share_of_kernel_time": round(v["total_ms"] / sum(u["total_ms"] for u in kern.values()), 4)}
        if k in models:
            fl, by = models[k]
            t = v["total_ms"] * 1e-3
            per_kernel[k]["GB/s"] = round(by * rhs_iters / t / 1e9, 1)
            per_kernel[k]["TFLOP/s"] = round(fl * rhs_iters / t / 1e12, 2)
            per_kernel[k]["alg_bytes_per_elem"] = by / n
    roof = None
    if models:
        peak_tf = MFMA_PEAK_TFLOPS[prec]
        ridge = peak_tf * 1e12 / (HBM_PEAK_GBS * 1e9)          # FLOP per byte where the two bounds meet
        dom = max(models, key=lambda k: kern[k]["total_ms"])
        v = kern[dom]
        fl, by = models[dom]
        # one launch processes every active RHS once; summed over launches that is rhs_iters
        fl_launch = fl * rhs_iters / v["launches"]
        by_launch = by * rhs_iters / v["launches"]
        sec = v["avg_us"] * 1e-6
        hbm = {"achieved": round(by_launch / sec / 1e9, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
               "frac": round(by_launch / sec / 1e9 / HBM_PEAK_GBS, 4), "bytes_per_launch": round(by_launch)}
        mf = {"achieved": round(fl_launch / sec / 1e12, 2), "peak": peak_tf, "unit": "TFLOP/s",
              "frac": round(fl_launch / sec / 1e12 / peak_tf, 4), "flops_per_launch": round(fl_launch)}
        bound = "mfma" if fl / by >= ridge else "hbm"
        main, other = (mf, hbm) if bound == "mfma" else (hbm, mf)
        roof = {"kernel": dom, "bound": bound, "achieved": main["achieved"], "peak": main["peak"],
                "unit": main["unit"], "frac": main["frac"], "traffic": None,
                "arithmetic_intensity": round(fl / by, 2), "ridge": round(ridge, 1),
                "avg_launch_us": round(v["avg_us"], 2), "launches": v["launches"],
                "other_bound": other, "per_kernel": per_kernel,
                "fp64_residual_passes": {k: {"avg_us": round(u["avg_us"], 2), "launches": u["launches"]}
                                         for k, u in resid64.items()}}
        roof.update({k: main[k] for k in ("bytes_per_launch", "flops_per_launch") if k in main})
        mvm_ms = sum(u["total_ms"] for k, u in kern.items() if k.startswith("gemm") or k.startswith("contract")
                     or k.startswith("slab"))
        if mvm_ms > 0:
            agg = flop_rhs_it * rhs_iters / (mvm_ms * 1e-3) / 1e12
            roof["all_mvm_passes"] = {"achieved": round(agg, 2), "unit": "TFLOP/s", "frac": round(agg / peak_tf, 4),
                                      "note": "every MVM launch class of the working precision (operand packing "
                                              "included) against the matrix-core peak"}
        if prod > 1:
            roof["note"] = (f"{prec} issues {prod} bf16 matrix-core products per useful product (hh, hm, mh, hl, "
                            f"lh, mm of the three-way splits); FLOP figures count all of them, against the bf16 "
                            f"peak")
        roof["traffic"] = measured_traffic(name, dom, nrhs, rhs_iters, v["launches"])
    elif "small_cg64" in kern:
        # the whole FP64 solve of each (system, RHS) in one workgroup: one launch per solve
        v = kern["small_cg64"]
        flop_launch = flop_rhs_it * rhs_iters / v["launches"]
        ach = flop_launch / (v["avg_us"] * 1e-6) / 1e12
        roof = {"kernel": "small_cg64", "bound": "latency", "achieved": round(ach, 4), "peak": 78.6,
                "unit": "TFLOP/s", "frac": round(ach / 78.6, 6), "traffic": None,
                "flops_per_launch": round(flop_launch), "avg_launch_us": round(v["avg_us"], 2),
                "us_per_iteration": round(v["avg_us"] * v["launches"] * nrhs / max(rhs_iters, 1), 3),
                "per_kernel": per_kernel,
                "note": "one workgroup (one CU of 256) runs the whole solve; the chip-wide FP64 peak is "
                        "quoted for reference only: a single 4096-unknown system cannot fill the chip"}
    tts = None
    if not args.no_tts and prec != "fp64":
        res = {}
        full = dict(opts, max_iters=full_max)
        for lab, o in (("mixed", full), ("fp64_cg", dict(tol=tol, max_iters=full_max, prec="fp64",
                                                         check_every=32))):
            torch.cuda.synchronize()
            t1 = time.perf_counter()
            X, info = op.solve(B, nrhs, **o)
            torch.cuda.synchronize()
            rec = decode_info(info, nrhs)
            sec = time.perf_counter() - t1
            res[lab] = {"seconds": round(sec, 3), "iters_max": max(r["iters"] for r in rec),
                        "rhs_iters": sum(r["iters"] for r in rec),
                        "relres_max": max(r["relres"] for r in rec), "status": sorted({r["status"] for r in rec}),
                        "rhs_iters_per_s": round(sum(r["iters"] for r in rec) / sec, 1)}
            res[lab]["relres_recursive_max"] = max(r["relres_recursive"] for r in rec)
            if lab == "mixed":
                res[lab]["precision"] = prec
                res[lab]["stops_on"] = "FP64 true residual"
            else:
                res[lab]["stops_on"] = "recursive FP64 residual"
            progress(f"time-to-solution {lab}: {res[lab]['seconds']} s")
        res["speedup"] = round(res["fp64_cg"]["seconds"] / res["mixed"]["seconds"], 3)
        res["note"] = ("relres_max is the FP64 true residual of the returned x for both; "
                       "speedup = fp64_cg seconds / mixed seconds; engines: " + ENGINE_NOTE.get(name, "general passes"))
        tts = res
    direct = None
    if name in ("c4",) and not args.no_tts:
        direct = direct_solve(op, B, nrhs, n, tts["mixed"]["seconds"] if tts else None)
    op.close()
    cpu = None
    if not args.no_cpu:
        from oracle import cg as ocg
        from oracle import kron
        iters = args.cpu_window if name == "c4" else (3 if name == "c5" else 50)
        apply_A = lambda V: kron.mvm(s.factors, V, s.sigma2, s.diag)
        t0 = time.perf_counter()
        res = ocg.cg(apply_A, w.B[0][:1], tol=1e-30, max_iters=iters)
        dtc = time.perf_counter() - t0
        rate = int(res.iters.sum()) / dtc
        cpu = {"value": rate, "unit": "RHS*iters/s", "cores": _cores(), "kind": "oracle",
               "sample": f"numpy float64 CG (the oracle), 1 RHS x {iters} iterations in {dtc:.2f} s",
               "host": host_info()}
        if name == "c4":
            fp64_iters = tts["fp64_cg"]["rhs_iters"] if tts else None
            if fp64_iters:
                cpu["extrapolated_fp64_solve_hours"] = round(fp64_iters / rate / 3600.0, 2)
                cpu["extrapolation"] = ("the GPU FP64 CG's RHS*iterations to 1e-6 divided by the oracle's "
                                        "measured rate (not run)")
            try:
                from threadpoolctl import threadpool_limits
                with threadpool_limits(limits=1):
                    t0 = time.perf_counter()
                    r1 = ocg.cg(apply_A, w.B[0][:1], tol=1e-30, max_iters=2)
                    d1 = time.perf_counter() - t0
                cpu["single_core"] = {"value": float(r1.iters.sum()) / d1, "cores": 1,
                                      "sample": f"1 RHS x 2 iterations in {d1:.2f} s"}
            except Exception as e:
                cpu["single_core"] = {"error": str(e)[:120]}
        progress(f"cpu baseline: {rate:.3f} RHS*iters/s")
    extra = None
    if name == "c4" and not args.no_extra:
        extra = other_workloads(args)
    return {"metric": METRIC, "value": round(rhs_iters / dt, 1), "unit": "RHS*iters/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(1e3 * dt / args.steps, 3),
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": prec, "data": "synthetic",
            "config": {"workload": label + (" (+ adjoint backward per step)" if G is not None else ""), "n": n,
                       "nrhs": nrhs, "window_iters": window, "rhs_iters_per_step": rhs_iters // max(1, args.steps),
                       "reliable_update_delta": delta if prec != "fp64" else None,
                       "statuses": statuses, "worst_relres": worst, "parallelism": "single GPU",
                       **({"window_note": "statuses and worst_relres are those of a window of CG iterations from "
                                          "x0 = 0 (stopped by the iteration limit; the FP64 true residual can exceed "
                                          "the initial one there, CG residual norms not being monotone); the solve "
                                          "to the target is mixed_vs_fp64"} if window else {})},
            "roofline": roof, "cpu_baseline": cpu, "mixed_vs_fp64": tts, "direct_eig_solve": direct,
            "other_workloads": extra}


def other_workloads(args):
    """Short runs (2 warm-up + 5 timed steps, no time-to-solution, no CPU baseline) of the 64^3 x 32 RHS
    solve to 1e-5 and of the sum-of-Kronecker solve + backward, reported beside the main line."""
    import copy
    out = {}
    for wname in ("c2", "c5"):
        a = copy.copy(args)
        a.workload, a.steps, a.warmup, a.no_tts, a.no_cpu, a.prec, a.max_iters = wname, 5, 2, True, True, None, None
        r = run_c2(a) if wname == "c2" else run_single(a, wname)
        roof = r.get("roofline") or {}
        out[wname] = {"workload": r["config"]["workload"], "value": r["value"], "unit": r["unit"],
                      "ms_per_step": r["ms_per_step"], "dtype": r["dtype"], "steps": a.steps,
                      "worst_relres": r["config"].get("worst_relres"), "statuses": r["config"].get("statuses"),
                      "roofline": {k: roof.get(k) for k in ("kernel", "bound", "achieved", "peak", "unit", "frac",
                                                              "traffic")}}
        progress(f"extra workload {wname}: {r['value']} RHS*iters/s")
    return out


def _workload_operator(name, args, dev):
    """(workload, system, operator precision, nrhs, solve tolerance) of a single-system workload."""
    import workloads as wl
    if name == "c4":
        w = wl.config4()
        return w, w.systems[0], args.prec or "bf16x3", 8, 1e-6
    if name == "c5":
        w = wl.config5()
        return w, w.systems[0], args.prec or "bf16", 16, 1e-6
    w = wl.config2(m=args.m, nrhs=args.nrhs)
    return w, w.systems[0], "fp32", args.nrhs, args.tol


def run_counters(args):
    """Short run for rocprofv3 --pmc, in the benchmark's launch configuration.

    Order of GPU work: operator set-up and the tile autotuner, then a 256 MiB
    device-to-device copy (the reference for the HBM byte counters, and the
    marker after which dispatches belong to the solve), then one solve capped
    at --max-iters iterations (no right-hand side converges that early).
    """
    import torch
    from paper_2309_03060_amd import KronOperator, SystemSpec
    dev = torch.device("cuda:0")
    name = args.workload if args.workload in ("c4", "c5") else "c2"
    w, s, prec, nrhs, tol = _workload_operator(name, args, dev)
    spec = SystemSpec(factors=[[torch.tensor(f, device=dev) for f in row] for row in s.factors], sigma2=s.sigma2,
                      diag=None if s.diag is None else torch.tensor(s.diag, device=dev))
    op = KronOperator([spec], prec=prec)
    B = torch.tensor(w.B[0], device=dev).reshape(-1).contiguous()
    if args.autotune:
        op.autotune(nrhs)
    a = torch.ones(COPY_REF_WORDS, dtype=torch.float32, device=dev)
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    torch.mul(a, 1.0, out=b)          # elementwise kernel: 16-byte loads / stores per lane, like ours
    torch.cuda.synchronize()
    b.copy_(a)                        # runtime copy kernel: the marker that ends the set-up phase
    torch.cuda.synchronize()
    # c2: one chunk of 32 iterations, i.e. one launch of the fused persistent CG (it needs host checks)
    iters = args.max_iters or (COUNTERS_C2_ITERS if name == "c2" else 48)
    # inner_tol 1e-30: no reliable update falls due this early, so every launch has all RHS active
    _, info = op.solve(B, nrhs, tol=tol, max_iters=iters, prec=prec, inner_tol=1e-30,
                       check_every=32 if name == "c2" else 0)
    torch.cuda.synchronize()
    from paper_2309_03060_amd import decode_info
    rhs_iters = sum(r["iters"] for r in decode_info(info, nrhs))
    op.close()
    print(json.dumps({"counters_run": name, "prec": prec, "copy_bytes": 2 * COPY_REF_WORDS * 4, "max_iters": iters,
                      "rhs_iters": rhs_iters, "all_rhs_active_every_iteration": rhs_iters == iters * nrhs}))


# --- rocprofv3 counter summaries ---------------------------------------------------------------
COPY_REF_WORDS = 64 << 20            # the counters run's reference copy: 256 MiB read + 256 MiB written
PMC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic.json")
COUNTERS_C2_ITERS = 32               # c2 counters run: one fused launch of 32 iterations x 32 RHS
KERNEL_SOURCES = {                   # files each launch class is compiled from (counters go stale with them)
    "contract": ["contract.hip", "contract.h", "modepass.hip", "modepass.h", "modeslice.h", "common.h"],
    "slab23": ["slab.hip", "slab.h", "common.h"],
    "update": ["vector.hip", "vector.h", "common.h"],
    "cg_fused": ["fused.hip", "fused.h", "common.h"],
    "gemm3": ["gemm3.hip", "gemm3.h", "contract.h", "common.h"],
    "gemm2": ["gemm.hip", "gemm.h", "contract.h", "common.h"],
}
# bench launch-class name of each counter class, per workload (c2 fuses modes 2 and 3 in the slab pass,
# so its only column-layout FP32 contraction is the last mode; the fused persistent CG replaces all three)
BENCH_CLASS = {"c2": {"contract_cols_f32": "contract_last", "slab23_f32": "slab23", "update_float": "update",
                      "k_fused_cg": "cg_fused"},
               "c4": {"gemm3x3_mode3": "gemm_mode3", "gemm3x3_mode2": "gemm_mode2", "gemm3x3_mode1": "gemm_mode1",
                      "gemm3_mode3": "gemm_mode3", "gemm3_mode2": "gemm_mode2", "gemm3_mode1": "gemm_mode1",
                      "update_float": "update"},
               "c5": {"k_gemm2_pack": "gemm_pack", "k_gemm2_t": "gemm_mode2", "k_gemm2_y": "gemm_mode1",
                      "update_float": "update"}}
# RHS*iterations one dispatch of a counter class covers in the counters run (default: one iteration of
# every right-hand side)
RHS_ITERS_PER_DISPATCH = {("c2", "k_fused_cg"): COUNTERS_C2_ITERS * 32}


def source_kind(cls, workload=None):
    """KERNEL_SOURCES key of a counter or bench launch class (the bench's GEMM class names are shared by
    the three-GEMM engine of the 256^3 workload and the two-GEMM engine of the sum-of-Kronecker one)."""
    if cls.startswith("contract"):
        return "contract"
    if cls in ("k_fused_cg", "cg_fused"):
        return "cg_fused"
    if cls.startswith("gemm3"):
        return "gemm3"
    if cls.startswith("k_gemm2"):
        return "gemm2"
    if cls.startswith("gemm_"):
        return "gemm2" if workload == "c5" else "gemm3"
    return cls.split("_")[0]


def kernel_class(name):
    """Launch class of a demangled kernel name from a rocprofv3 trace."""
    import re
    m = re.search(r"k_contract<cola::Pol(\w+), \d+, \d+, (true|false)>", name)
    if m:
        return f"contract_{'rows' if m.group(2) == 'true' else 'cols'}_{m.group(1).lower()}"
    m = re.search(r"k_mode<(?:cola::)?(?:\(anonymous namespace\)::)?Mode(\w+), \d+, \d+, (true|false)", name)
    if m:
        return f"contract_{'rows' if m.group(2) == 'true' else 'cols'}_{m.group(1).lower()}"
    m = re.search(r"k_slab23<cola::Slab(\w+)[,>]", name)
    if m:
        return f"slab23_{m.group(1).lower()}"
    m = re.search(r"k_cg_update<(\w+)", name)
    if m:
        return f"update_{m.group(1)}"
    m = re.search(r"k_gemm3(x3)?<(true|false), (\d+)>", name)
    if m:                                # the direction pass, the middle pass, the pass with the epilogue
        mode = 3 if m.group(2) == "true" else (2 if m.group(3) == "0" else 1)
        return f"gemm3{m.group(1) or ''}_mode{mode}"
    m = re.search(r"cola::(?:\(anonymous namespace\)::)?(k_\w+)", name)
    return m.group(1) if m else "other"


def sources_digest(kind):
    import hashlib
    h = hashlib.sha1()
    for f in KERNEL_SOURCES[kind]:
        with open(os.path.join(ROOT, "paper_2309_03060_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def pmc_summary(csvs, workload, out_json):
    """Per launch class averages of the counters in rocprofv3 --pmc CSV files (one file per pass).

    Dispatches before the 256 MiB reference copy (operator set-up, autotuner) are dropped.  The
    byte counters are scaled so that the reference copy reads and writes exactly its size.
    Prints a markdown table; merges the traffic record of this workload into out_json.
    """
    import collections
    import csv
    per = collections.defaultdict(lambda: collections.defaultdict(list))
    dur = collections.defaultdict(list)
    ref, ref_copy = {}, {}
    for path in csvs:
        rows = list(csv.DictReader(open(path)))
        # the elementwise reference is the last multiply kernel; the runtime copy right after it
        # is the second reference and the marker
        muls = [r for r in rows if "MulFunctor" in r["Kernel_Name"]]
        if not muls:
            raise SystemExit(f"{path}: no reference copy dispatch found")
        mul_id = int(muls[-1]["Dispatch_Id"])
        ref[muls[-1]["Counter_Name"]] = float(muls[-1]["Counter_Value"])
        copies = [r for r in rows if "copyBuffer" in r["Kernel_Name"] and int(r["Dispatch_Id"]) > mul_id]
        marker = int(copies[0]["Dispatch_Id"]) if copies else mul_id
        if copies:
            ref_copy[copies[0]["Counter_Name"]] = float(copies[0]["Counter_Value"])
        for r in rows:
            if int(r["Dispatch_Id"]) <= marker:
                continue
            c = kernel_class(r["Kernel_Name"])
            per[c][r["Counter_Name"]].append(float(r["Counter_Value"]))
            if r["Counter_Name"] in ("FETCH_SIZE", "WRITE_SIZE"):
                dur[c].append((int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) * 1e-3)
    copy_kib = COPY_REF_WORDS * 4 / 1024
    scale = {k: copy_kib / v for k, v in ref.items() if k in ("FETCH_SIZE", "WRITE_SIZE") and v > 0}
    lines = [f"| class | dispatches | avg us (counter run) | " + " | ".join(
        sorted({k for d in per.values() for k in d})) + " | HBM MB/launch (scaled) |",
        "|---|---|---|" + "---|" * len({k for d in per.values() for k in d}) + "---|"]
    cols = sorted({k for d in per.values() for k in d})
    record = {}
    for c in sorted(per):
        d = per[c]
        avg = {k: sum(v) / len(v) for k, v in d.items()}
        mb = None
        if "FETCH_SIZE" in avg and "WRITE_SIZE" in avg and len(scale) == 2:
            byt = 1024 * (avg["FETCH_SIZE"] * scale["FETCH_SIZE"] + avg["WRITE_SIZE"] * scale["WRITE_SIZE"])
            mb = byt / 1e6
            bench = BENCH_CLASS.get(workload, {}).get(c)
            if bench:
                record[bench] = {"bytes_per_launch_all_rhs_active": round(byt),
                                 "fetch_kib": round(avg["FETCH_SIZE"], 1), "write_kib": round(avg["WRITE_SIZE"], 1),
                                 "sources_sha1": sources_digest(source_kind(c))}
                if (workload, c) in RHS_ITERS_PER_DISPATCH:
                    record[bench]["rhs_iters_per_dispatch"] = RHS_ITERS_PER_DISPATCH[(workload, c)]
        n = max(len(v) for v in d.values())
        du = sum(dur[c]) / len(dur[c]) if dur[c] else float("nan")
        lines.append(f"| {c} | {n} | {du:.1f} | " + " | ".join(
            f"{avg[k]:.4g}" if k in avg else "" for k in cols) + f" | {'' if mb is None else f'{mb:.1f}'} |")
    print("\n".join(lines))
    for label, d in (("elementwise copy kernel (the scale used)", ref), ("runtime copy kernel", ref_copy)):
        print(f"\n{label}, 256 MiB read + 256 MiB written: " +
              ", ".join(f"{k} {v:.1f} KiB -> scale {copy_kib / v:.3f}" for k, v in sorted(d.items())
                        if k in ("FETCH_SIZE", "WRITE_SIZE")))
    if out_json and record:
        data = json.load(open(out_json)) if os.path.exists(out_json) else {}
        data[workload] = {"scale": scale, "kernels": record}
        with open(out_json, "w") as fh:
            json.dump(data, fh, indent=1, sort_keys=True)
            fh.write("\n")


def trace_summary(prefix, cmd, title):
    """Markdown summary of a rocprofv3 --kernel-trace --stats --output-format csv run."""
    import csv
    import statistics
    stats = list(csv.DictReader(open(f"{prefix}_kernel_stats.csv")))
    per = {}
    for r in csv.DictReader(open(f"{prefix}_kernel_trace.csv")):
        per.setdefault(r["Kernel_Name"], []).append((int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) * 1e-3)
    print(f"# {title}\n\nCommand (repository root on the GPU box, `export TMPDIR=/tmp` first):\n\n    {cmd}\n")
    print("| class | kernel | calls | avg us | p50 us | p90 us | share of kernel time |")
    print("|---|---|---|---|---|---|---|")
    for r in stats[:14]:
        v = sorted(per.get(r["Name"], [0.0]))
        p90 = v[min(len(v) - 1, int(0.9 * len(v)))]
        print(f"| {kernel_class(r['Name'])} | `{r['Name'][:90]}` | {r['Calls']} | {float(r['AverageNs']) / 1e3:.2f} | "
              f"{statistics.median(v):.2f} | {p90:.2f} | {float(r['Percentage']):.2f}% |")


def measured_traffic(workload, kernel, nrhs, rhs_iters, launches):
    """HBM bytes per launch from the committed counter record, scaled to the average number of
    RHS*iterations per launch (a fused launch covers many iterations); None when there is no record or
    the kernel's sources changed since."""
    try:
        rec = json.load(open(PMC_FILE))[workload]["kernels"][kernel]
    except (OSError, KeyError, ValueError):
        return None
    if rec.get("sources_sha1") != sources_digest(source_kind(kernel, workload)):
        return None
    per_rhs_iter = rec["bytes_per_launch_all_rhs_active"] / rec.get("rhs_iters_per_dispatch", nrhs)
    return int(per_rhs_iter * rhs_iters / launches)


def main():
    args = parse()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU (right-hand sides and systems would be split across GPUs without communication); --gpus must be 1"}))
        sys.exit(2)
    if args.pmc_summary:
        pmc_summary(args.pmc_summary, args.workload, args.pmc_out)
        return
    if args.trace_summary:
        trace_summary(args.trace_summary[0], args.trace_summary[1], args.trace_summary[2])
        return
    if args.counters:
        run_counters(args)
        return
    if args.autograd:
        print(json.dumps(run_autograd_sweep(args)))
        return
    if args.workload == "c3":
        print(json.dumps(run_uneven_batch(args)))
        return
    if args.workload in ("c1", "c4", "c5"):
        print(json.dumps(run_single(args, args.workload)))
        return
    print(json.dumps(run_c2(args)))


def run_c2(args):
    """64^3 x 32 RHS: full solves to args.tol per step (fused persistent FP32 CG, FP64 reliable updates)."""
    import torch
    import workloads as wl
    from paper_2309_03060_amd import KronOperator, SystemSpec, decode_info

    dev = torch.device("cuda:0")
    w = wl.config2(m=args.m, nrhs=args.nrhs)
    s = w.systems[0]
    nrhs = args.nrhs
    n = s.n
    spec = SystemSpec(factors=[[torch.tensor(f, device=dev) for f in s.factors[0]]], sigma2=s.sigma2)
    op = KronOperator([spec], prec="fp32")
    B = torch.tensor(w.B[0], device=dev).reshape(-1).contiguous()
    if args.autotune:
        op.autotune(nrhs)
    opts = dict(tol=args.tol, max_iters=args.max_iters or 20000, prec="fp32", inner_tol=0.1,
                check_every=args.check_every,
                refine="reliable")

    for _ in range(args.warmup):
        op.solve(B, nrhs, **opts)
    torch.cuda.synchronize()

    op.profile_enable(True)
    infos = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        X, info = op.solve(B, nrhs, **opts)
        infos.append(info)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    recs = [decode_info(i, nrhs) for i in infos]
    rhs_iters = sum(r["iters"] for rec in recs for r in rec)
    statuses = sorted({r["status"] for rec in recs for r in rec})
    worst = max(r["relres"] for rec in recs for r in rec)
    value = rhs_iters / dt

    # per-kernel averages (HIP events around every launch in the timed region)
    kern = {}
    for name in BYTES_PER_ELEM:
        ms, cnt = op.profile_read(name)
        if cnt:
            kern[name] = {"total_ms": ms, "launches": cnt, "avg_us": 1e3 * ms / cnt}
    resid64 = kernel_table(op, ["slab23_fp64", "contract_last_fp64"])
    op.profile_enable(False)
    dom = max(kern, key=lambda k: kern[k]["total_ms"]) if kern else None
    roof = None
    if dom:
        # every launch of a class processes the active RHS of that iteration; the summed
        # active RHS over the region is the RHS*iterations count
        alg_bytes = BYTES_PER_ELEM[dom] * n * rhs_iters
        launches = kern[dom]["launches"]
        per_launch = alg_bytes / launches
        avg_s = kern[dom]["total_ms"] * 1e-3 / launches
        achieved = per_launch / avg_s / 1e9
        traffic = measured_traffic("c2", dom, nrhs, rhs_iters, launches) if args.m == 64 and nrhs == 32 else None
        roof = {"kernel": dom, "bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                "bytes_per_launch": int(per_launch), "avg_launch_us": round(avg_s * 1e6, 2),
                "per_kernel": {k: {"avg_us": round(v["avg_us"], 2), "launches": v["launches"],
                                   "GB/s": round(BYTES_PER_ELEM[k] * n * rhs_iters / v["launches"] /
                                                 (v["avg_us"] * 1e-6) / 1e9, 1)}
                               for k, v in kern.items()},
                "fp64_residual_passes": {k: {"avg_us": round(v["avg_us"], 2), "launches": v["launches"]}
                                         for k, v in resid64.items()}}
        copy = copy_bandwidth()
        roof["measured_copy"] = {"GB/s": round(copy, 1), "frac_of_copy": round(achieved / copy, 4),
                                 "note": "torch's device-to-device copy of 1 GiB (read + write bytes over "
                                         "time), measured after the timed region: a plain streaming rate"}

    # mixed precision vs plain FP64 at 1e-6 true relative residual
    tts = None
    if not args.no_tts:
        res = {}
        for label, o in (("mixed_fp32_reliable", dict(opts, tol=1e-6)),
                         ("mixed_fp32_restarted", dict(opts, tol=1e-6, refine="restart", inner_tol=1e-4,
                                                       max_sweeps=60)),
                         ("fp64_cg", dict(tol=1e-6, max_iters=args.max_iters or 20000, prec="fp64",
                                          check_every=args.check_every))):
            torch.cuda.synchronize()
            t1 = time.perf_counter()
            X, info = op.solve(B, nrhs, **o)
            torch.cuda.synchronize()
            t = time.perf_counter() - t1
            rec = decode_info(info, nrhs)
            res[label] = {"seconds": round(t, 4), "iters_max": max(r["iters"] for r in rec),
                          "relres_max": max(r["relres"] for r in rec),
                          "status": sorted({r["status"] for r in rec})}
            progress(f"time-to-solution {label}: {res[label]['seconds']} s")
        res["speedup"] = round(res["fp64_cg"]["seconds"] / res["mixed_fp32_reliable"]["seconds"], 3)
        # the same mixed solve on the separate-kernel path (slab23 / contract_last / update per iteration)
        op.set_engine("fused_cg", False)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        X, info = op.solve(B, nrhs, **dict(opts, tol=1e-6))
        torch.cuda.synchronize()
        rec = decode_info(info, nrhs)
        res["mixed_fp32_reliable_separate_kernels"] = {
            "seconds": round(time.perf_counter() - t1, 4), "iters_max": max(r["iters"] for r in rec),
            "relres_max": max(r["relres"] for r in rec), "status": sorted({r["status"] for r in rec})}
        op.set_engine("fused_cg", True)
        progress("time-to-solution on the separate-kernel path done")
        res["direct_eig_solve"] = direct_solve(op, B, nrhs, n, res["mixed_fp32_reliable"]["seconds"])
        res["slq_logdet"] = slq_measure(op, s.factors[0], s.sigma2, n)
        res["speedup_same_kernels"] = round(res["fp64_cg"]["seconds"] /
                                            res["mixed_fp32_reliable_separate_kernels"]["seconds"], 3)
        res["note"] = ("relres_max is the FP64 true residual of the returned x for every solve; "
                       "speedup = fp64_cg seconds / mixed_fp32_reliable seconds, where the mixed solve runs on "
                       "the persistent fused FP32 engine and fp64_cg on the separate FP64 kernels (slab, "
                       "contraction, update); speedup_same_kernels compares fp64_cg with the mixed solve on "
                       "the same separate kernels in FP32")
        tts = res

    cpu = None
    if not args.no_cpu:
        cpu = cpu_baseline(w, args.cpu_iters)

    out = {
        "metric": METRIC, "value": round(value, 1), "unit": "RHS*iters/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(1e3 * dt / args.steps, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"K1(x)K2(x)K3+0.01I, RBF l=0.15 on {args.m} U[0,1] points per mode, "
                               f"n={n}, {nrhs} RHS N(0,1), FP32 inner CG + FP64 refinement to true relres "
                               f"{args.tol:g}", "n": n, "nrhs": nrhs, "factor_dim": args.m,
                   "rhs_iters_per_step": rhs_iters // max(1, args.steps), "statuses": statuses,
                   "mixed_scheme": "FP32 CG with FP64 reliable updates (delta 0.1)",
                   "worst_relres": worst, "parallelism": "single GPU"},
        "roofline": roof, "cpu_baseline": cpu, "mixed_vs_fp64": tts,
    }
    op.close()
    return out




if __name__ == "__main__":
    main()

"""Benchmark of the retrieved-matvec hot path on one MI355X.

Headline workload: the batched 1-bit workload, 384 codebooks (128 each at
32 x 32, 48 x 48 and 64 x 64 units; Bernoulli, 4 x 4 checkerboard and stripe
families) x 4 incidence angles (theta 0/20/40/60 deg in the phi = 0 plane) =
1,536 right-hand sides sharing one global matrix stored for 64 x 64.  A step
is one whole batched solve: plane-wave excitation of every right-hand side,
right block-Jacobi GMRES(20) on complex64 block spectra to 1e-3 inside an
outer FP64 refinement (complex128 residual) to 1e-6, and the bistatic RCS of
every right-hand side on a 1-degree phi = 0 cut.  A right-hand side counts
toward `value` only if its RCS is within 1e-4 (relative L2 over the cut) of
the RCS of the FP64 reference solution of the same system (refined to 1e-10,
solved once before the timed steps); every right-hand side is checked.

Secondary legs (keys of the same JSON line): the 2-bit 32 x 32 compressed
solve (ACA far factors, block ILU), the plain complex128 1-bit 6 x 6 case,
the 128 x 128 x 16 large case, the differentiation workload, and the
preconditioner study.  `--c2-compressed` runs the batched workload on its
compressed split-BF16 store instead (a separate, long run with progress
lines; not part of the default line).
"""
from __future__ import annotations

import os


def _cpu_share() -> int:
    """Host threads for the CPU baseline: the affinity set, capped by the
    thread count the environment grants (OMP_NUM_THREADS) when it is set."""
    n = len(os.sched_getaffinity(0))
    env = os.environ.get("OMP_NUM_THREADS", "")
    if env.isdigit() and int(env) > 0:
        n = min(n, int(env))
    return max(1, n)


CORES = _cpu_share()
for _v in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS"):
    os.environ[_v] = str(CORES)

import argparse  # noqa: E402
import json  # noqa: E402
import sys  # noqa: E402
import time  # noqa: E402

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
PEAK_FP32_TFLOPS = 157.3  # MI355X FP32 vector / matrix peak
RCS_TARGET = 1e-4
PRECOND_NAMES = {0: "unpreconditioned", 1: "block-Jacobi", 2: "block-ILU(0) r={r}"}

# HBM bytes of one call, from rocprofv3 FETCH_SIZE and WRITE_SIZE runs scaled
# by the same counters on a plain device copy of known size (profiles/); valid
# for the kernels as they were when taken.
PROFILED_TRAFFIC = {
    # 2-bit 32x32 compressed matvec (convert + far_near + reduce) at 48 groups
    "c1_matvec": {"bytes": 358.9e6, "groups": 48},
    # frequency product of the 1,536-RHS spectral matvec (spec_product_stream_kernel,
    # which serves shape 6 on wide batches: 8 frequencies x 80 rows x 64 RHS)
    "c2_product": {"bytes": 40.14e9, "shape": 6},
}


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=3)
    p.add_argument("--warmup", type=int, default=1)
    p.add_argument("--no-legs", action="store_true", help="headline only")
    p.add_argument("--no-cpu-baseline", action="store_true")
    p.add_argument("--no-sweep", action="store_true", help="skip the preconditioner study")
    p.add_argument("--n-per-size", type=int, default=128, help="codebooks per array size of the batched workload")
    p.add_argument("--c2-compressed", action="store_true",
                   help="run the batched workload on its compressed split-BF16 store (long; progress lines)")
    p.add_argument("--matvec-only", action="store_true",
                   help="time only the batched spectral matvec (W warmup calls, the first tunes; K timed): the "
                        "command profiler summaries are taken on")
    p.add_argument("--only", default="",
                   help="comma-separated secondary legs to run alone (no headline, no CPU baseline), e.g. "
                        "c1_2bit_32x32,large_128x128: the commands profiler summaries of those legs are taken on")
    p.add_argument("--c1-precond", type=int, default=2,
                   help="2-bit 32x32 leg: 0 none, 1 block-Jacobi, 2 near-field block ILU(0)")
    return p.parse_args()


def rcs_errors(sig, ref):
    """Relative L2 error of each right-hand side's RCS cut ([B][n_dir] arrays)."""
    import numpy as np
    return np.linalg.norm(sig - ref, axis=1) / np.maximum(np.linalg.norm(ref, axis=1), 1e-300)


def spectral_cost(n, D, B):
    """Algorithmic bytes and flops of one spectral matvec (complex64 spectra):
    bytes = the spectra read once (the compact vectors are small beside them);
    flops of the per-frequency products (8 n^2 per frequency per RHS) and of
    the forward and inverse 2-D transforms (2 G lines of 5 G log2 G each per
    grid, real flops of a radix-2 count, whether the transform runs fused or
    as row and column passes)."""
    import math
    G = 1
    while G < 2 * D + 1:
        G *= 2
    G2 = G * G
    byt = n * n * G2 * 8
    flops = 8.0 * n * n * G2 * B + 4 * 5.0 * G2 * math.log2(G) * n * B
    return byt, flops, G


def product_cost(n, D, B):
    """Algorithmic flops and HBM bytes of one frequency product over the batch
    (complex64 spectra): 8 n^2 flops per frequency per RHS; the transformed
    input grids read once, the output grids written once, the spectra read
    once."""
    G = 1
    while G < 2 * D + 1:
        G *= 2
    G2 = G * G
    return 8.0 * n * n * G2 * B, (2 * B * n * G2 + n * n * G2) * 8


def timed_product(r3m, ctx, store, batch, x, reps):
    """Seconds per r3m_spectral_product call (the frequency product alone, one
    kernel launch) on the grids of a matvec of x, HIP events on the stream the
    call launches on (torch's current stream)."""
    import torch
    y = torch.zeros_like(x)
    work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C64), dtype=torch.uint8, device=x.device)
    r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C64, x, y, work)
    r3m.r3m_spectral_product(ctx, store, batch, work)  # warm
    s = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(s)
    for _ in range(reps):
        r3m.r3m_spectral_product(ctx, store, batch, work)
    e1.record(s)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / 1e3 / reps


def timed_matvec(r3m, ctx, store, batch, x, vt, reps):
    """Seconds per r3m_retrieved_matvec call (retrieval index reused), HIP
    events on the stream the call launches on."""
    import torch
    y = torch.zeros_like(x)
    work = torch.empty(max(r3m.matvec_work_bytes(ctx, store, batch, vt), 16), dtype=torch.uint8, device=x.device)
    r3m.r3m_retrieved_matvec(ctx, store, batch, vt, x, y, work)
    s = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(s)
    for _ in range(reps):
        r3m.r3m_retrieved_matvec(ctx, store, batch, vt, x, y, work, index_ready=True)
    e1.record(s)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / 1e3 / reps


# ------------------------------------------------------- batched (headline)

def c2_setup(ctx, args):
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_1BIT, batched_1bit
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    w = batched_1bit(args.n_per_size)
    unit = macro_unit(SIDES_1BIT)
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    batch = r3m.Batch.from_codebooks(w.codebooks, w.sizes, dev, repeat=len(w.angles_deg))
    t0 = time.perf_counter()
    dense = pipeline.fill_blocks(ctx, geom, 63, r3m.C128, dev)
    torch.cuda.synchronize()
    t_fill = time.perf_counter() - t0
    t0 = time.perf_counter()
    s64 = pipeline.spectral_store(ctx, geom, 64, 2, r3m.C64, dev, dense_c128=dense)
    s128 = pipeline.spectral_store(ctx, geom, 64, 2, r3m.C128, dev, dense_c128=dense)
    torch.cuda.synchronize()
    t_spec = time.perf_counter() - t0
    inc = [[np.deg2rad(a), 0.0, 1.0] for _ in w.codebooks for a in w.angles_deg]
    sizes = np.array([L for L in w.sizes for _ in w.angles_deg])
    return {"w": w, "unit": unit, "geom": geom, "batch": batch, "dense": dense, "s64": s64, "s128": s128,
            "inc": inc, "dirs": cb.phi0_cut(1.0), "sizes": sizes, "N": batch.total_units * unit.n_a,
            "setup_s": {"fill_c128_all_blocks": t_fill, "spectra_c64_c128": t_spec}}


def c2_solve(ctx, S, store, store64, tol, refine_tol, work, b, x, sig):
    """One batched solve: excitation, refined GMRES, RCS (all on the device)."""
    from paper_2112_05082_amd import r3m
    from workloads.configs import BATCHED_SOLVE as P
    r3m.r3m_plane_wave_rhs(ctx, S["geom"], S["batch"], S["inc"], b)
    _, rep = r3m.r3m_gmres_solve(ctx, store, store64, S["batch"], b, x, tol, P["restart"], P["max_iter"], work,
                                 refine_tol=refine_tol, max_refine=P["max_refine"],
                                 precond=r3m.PRECOND_BLOCK_JACOBI, allow_not_converged=True)
    r3m.r3m_rcs(ctx, S["geom"], S["batch"], x, S["dirs"], 1.0, sig)
    return rep


def headline_c2(ctx, args):
    import numpy as np
    import torch
    from paper_2112_05082_amd import r3m
    from workloads.configs import BATCHED_SOLVE as P
    dev = "cuda:0"
    S = c2_setup(ctx, args)
    batch, N = S["batch"], S["N"]
    B = batch.B
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    x = torch.zeros_like(b)
    sig = torch.zeros((B, len(S["dirs"])), dtype=torch.float64, device=dev)
    work = torch.empty(r3m.gmres_work_bytes(ctx, S["s64"], batch, P["restart"], S["s128"]), dtype=torch.uint8,
                       device=dev)
    # FP64 reference: the same system refined to 1e-10
    t0 = time.perf_counter()
    rep_ref = c2_solve(ctx, S, S["s64"], S["s128"], P["inner_tol"], P["ref_refine_tol"], work, b, x, sig)
    torch.cuda.synchronize()
    t_ref = time.perf_counter() - t0
    sig_ref = sig.cpu().numpy()
    ref_ok = all(r[3] for r in rep_ref)
    for _ in range(args.warmup):
        c2_solve(ctx, S, S["s64"], S["s128"], P["inner_tol"], P["refine_tol"], work, b, x, sig)
    torch.cuda.synchronize()
    errs, reps = [], []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        reps.append(c2_solve(ctx, S, S["s64"], S["s128"], P["inner_tol"], P["refine_tol"], work, b, x, sig))
        errs.append(rcs_errors(sig.cpu().numpy(), sig_ref))  # read-back of sigma: part of the step
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    ok = sum(int((e <= RCS_TARGET).sum()) for e in errs)
    err_all = np.concatenate(errs)
    rep = reps[-1]
    # the dominant kernel of a step: the frequency product over the whole batch
    # (one launch; timed alone), and the whole spectral matvec around it
    xm = b.to(torch.complex64)
    del work
    torch.cuda.empty_cache()
    mv = timed_matvec(r3m, ctx, S["s64"], batch, xm, r3m.C64, 5)
    pr = timed_product(r3m, ctx, S["s64"], batch, xm, 10)
    byt, flops, G = spectral_cost(S["s64"].n, 63, B)
    pflops, pbytes = product_cost(S["s64"].n, 63, B)
    del xm
    torch.cuda.empty_cache()
    iters = np.array([r[0] for r in rep])
    by_size = {int(L): {"rhs": int((S["sizes"] == L).sum()),
                        "max_rcs_err": float(err_all.reshape(args.steps, B)[:, S["sizes"] == L].max()),
                        "inner_iters_mean": float(iters[S["sizes"] == L].mean()),
                        "inner_iters_max": int(iters[S["sizes"] == L].max())}
               for L in (32, 48, 64)}
    plan = r3m.decode_plan(r3m.matvec_plan(ctx, S["s64"], batch))
    tr = PROFILED_TRAFFIC["c2_product"]
    traffic = tr["bytes"] if tr and plan.get("shape") == tr["shape"] else None
    out = {
        "value": ok / dt,
        "ms_per_step": dt / args.steps * 1e3,
        "rcs_rel_err_max": float(err_all.max()),
        "rcs_rel_err_median": float(np.median(err_all)),
        "rhs_checked": int(err_all.size),
        "rhs_within_target": ok,
        "codebooks_per_s": len(S["w"].codebooks) * args.steps / dt,
        "converged": all(r[3] for r in rep), "max_rel_residual": max(r[2] for r in rep),
        "inner_iters_max": int(iters.max()), "refine_steps_max": max(r[1] for r in rep),
        "by_size": by_size,
        "reference": {"refine_tol": P["ref_refine_tol"], "solve_s": t_ref, "converged": ref_ok,
                      "max_rel_residual": max(r[2] for r in rep_ref)},
        "roofline": {"bound": "mfma", "achieved": pflops / pr / 1e12, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s",
                     "frac": pflops / pr / 1e12 / PEAK_FP32_TFLOPS,
                     "traffic": traffic, "plan": plan,
                     "kernel": "spec_product_stream_kernel: the per-frequency product of the spectral matvec over "
                               "the 1,536-RHS batch (FP32 matrix cores), one launch timed alone",
                     "kernel_ms": pr * 1e3, "algorithmic_flops_per_launch": pflops,
                     "algorithmic_bytes_per_launch": pbytes, "hbm_gbs_algorithmic": pbytes / pr / 1e9,
                     "grid": [G, G],
                     "matvec": {"ms": mv * 1e3, "tflops_algorithmic": flops / mv / 1e12,
                                "kernels": "fused forward transform + frequency product + fused inverse transform",
                                "algorithmic_flops": flops, "spectra_bytes": byt}},
        "setup_s": S["setup_s"],
        "_S": S,
        "_rep": rep,
    }
    return out


def matvec_only(ctx, args):
    """The batched workload's spectral matvec alone: a seeded complex64 vector,
    W untimed calls (the first one runs the autotuner), K timed calls."""
    import torch
    from paper_2112_05082_amd import r3m
    from workloads import codebooks as cb
    S = c2_setup(ctx, args)
    batch = S["batch"]
    x = torch.from_numpy(cb.random_complex(S["N"], 5)).to("cuda:0").to(torch.complex64)
    y = torch.zeros_like(x)
    work = torch.empty(r3m.matvec_work_bytes(ctx, S["s64"], batch, r3m.C64), dtype=torch.uint8, device="cuda:0")
    for _ in range(max(1, args.warmup)):
        r3m.r3m_retrieved_matvec(ctx, S["s64"], batch, r3m.C64, x, y, work)
    torch.cuda.synchronize()
    mv = timed_matvec(r3m, ctx, S["s64"], batch, x, r3m.C64, args.steps)
    del work
    pr = timed_product(r3m, ctx, S["s64"], batch, x, args.steps)
    byt, flops, G = spectral_cost(S["s64"].n, 63, batch.B)
    pflops, pbytes = product_cost(S["s64"].n, 63, batch.B)
    # a plain device copy of known size: the reference for the HBM counters
    src = torch.ones(256 << 20, dtype=torch.uint8, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    return {"matvec_ms": mv * 1e3, "product_ms": pr * 1e3, "product_tflops": pflops / pr / 1e12,
            "rhs": batch.B, "grid": [G, G], "steps": args.steps,
            "plan": r3m.decode_plan(r3m.matvec_plan(ctx, S["s64"], batch)),
            "algorithmic_flops_per_call": flops, "product_flops": pflops, "product_bytes": pbytes,
            "calibration_copy_bytes": 256 << 20}


def c2_compressed(ctx, args):
    """The batched workload on its configured store: dense complex64 near
    blocks and split-BF16 ACA far factors (tol 1e-4, rank <= 12).  FP64
    refinement driven from here (residual with the complex128 spectral store,
    correction solves of at most 40 GMRES(20) iterations on the compressed
    store), so that a progress line is printed after every correction."""
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads.configs import BATCHED_SOLVE as P
    dev = "cuda:0"
    S = c2_setup(ctx, args)
    batch, N, B = S["batch"], S["N"], S["batch"].B
    t0 = time.perf_counter()
    comp = pipeline.compressed_store(ctx, S["geom"], 64, 2, r3m.C64, r3m.BF16X2, 1e-4, 12, dev,
                                     dense_c128=S["dense"])
    torch.cuda.synchronize()
    t_aca = time.perf_counter() - t0
    print(f"[c2-compressed] store ready: mean rank {comp.ranks.mean():.2f}, ACA {t_aca:.1f} s", file=sys.stderr,
          flush=True)
    sig = torch.zeros((B, len(S["dirs"])), dtype=torch.float64, device=dev)
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    x = torch.zeros_like(b)
    work = torch.empty(r3m.gmres_work_bytes(ctx, S["s64"], batch, P["restart"], S["s128"]), dtype=torch.uint8,
                       device=dev)
    c2_solve(ctx, S, S["s64"], S["s128"], P["inner_tol"], P["ref_refine_tol"], work, b, x, sig)
    sig_ref = sig.cpu().numpy()
    del work
    torch.cuda.empty_cache()
    mv = timed_matvec(r3m, ctx, comp, batch, b.to(torch.complex64), r3m.C64, 1)
    print(f"[c2-compressed] compressed matvec {mv * 1e3:.1f} ms", file=sys.stderr, flush=True)
    w_in = torch.empty(r3m.gmres_work_bytes(ctx, comp, batch, P["restart"]), dtype=torch.uint8, device=dev)
    w_mv = torch.empty(r3m.matvec_work_bytes(ctx, S["s128"], batch, r3m.C128), dtype=torch.uint8, device=dev)
    r3m.r3m_plane_wave_rhs(ctx, S["geom"], batch, S["inc"], b)
    x = torch.zeros_like(b)
    r = b.clone()
    d = torch.zeros_like(b)
    zx = torch.zeros_like(b)
    spans = [(int(batch.unit_off[i]) * 40, int(batch.unit_off[i] + batch.L[i, 0] * batch.L[i, 1]) * 40)
             for i in range(B)]
    bn = np.array([float(torch.linalg.vector_norm(b[a:e])) for a, e in spans])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    total_it = np.zeros(B, dtype=np.int64)
    for step in range(200):
        _, rep = r3m.r3m_gmres_solve(ctx, comp, None, batch, r, d, P["inner_tol"], P["restart"], 40, w_in,
                                     precond=r3m.PRECOND_BLOCK_JACOBI, allow_not_converged=True)
        total_it += np.array([q[0] for q in rep])
        x += d
        r3m.r3m_retrieved_matvec(ctx, S["s128"], batch, r3m.C128, x, zx, w_mv)
        torch.sub(b, zx, out=r)
        rel = np.array([float(torch.linalg.vector_norm(r[a:e])) for a, e in spans]) / bn
        print(f"[c2-compressed] correction {step + 1}: max residual {rel.max():.2e}, "
              f"inner iterations so far max {total_it.max()}, {time.perf_counter() - t0:.1f} s", file=sys.stderr,
              flush=True)
        if rel.max() <= P["refine_tol"]:
            break
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    r3m.r3m_rcs(ctx, S["geom"], batch, x, S["dirs"], 1.0, sig)
    err = rcs_errors(sig.cpu().numpy(), sig_ref)
    return {"workload": "batched 1-bit 1,536 RHS on the compressed store: dense c64 near (|d| <= 2), split-BF16 "
                        "ACA far factors (tol 1e-4, rank <= 12), inner block-Jacobi GMRES(20) to 1e-3 (at most 40 "
                        "iterations per correction), FP64 refinement residual on complex128 spectra to 1e-6",
            "solve_s": dt, "solves_per_s": int((err <= RCS_TARGET).sum()) / dt, "rcs_rel_err_max": float(err.max()),
            "max_rel_residual": float(rel.max()), "corrections": step + 1, "inner_iters_max": int(total_it.max()),
            "matvec_ms": mv * 1e3, "mean_far_rank": float(comp.ranks.mean()), "aca_s": t_aca}


# ------------------------------------------------------------ secondary legs

def algorithmic(store, L, n_a):
    """Algorithmic bytes and flops of one retrieved matvec (active-only work).

    bytes: near blocks + far factors at their actual ranks (storage precision)
           + x read once + y written once (complex128 vectors) + state bytes;
    flops: 8 n_a^2 per near unit pair + 16 r(d) n_a per far unit pair.
    """
    import numpy as np
    D = store.Dx
    nr = store.near_radius
    es = 8 if store.near_dtype == 1 else 16
    n = store.n
    n_near = (2 * min(nr, D) + 1) ** 2
    byt = n_near * n * n * es
    flops = 0.0
    fi = 0
    for dy in range(-D, D + 1):
        for dx in range(-D, D + 1):
            pairs = (L - abs(dx)) * (L - abs(dy))
            if max(abs(dx), abs(dy)) <= nr:
                flops += 8.0 * n_a * n_a * pairs
            else:
                r = int(store.ranks[fi])
                fi += 1
                byt += 2 * n * r * es
                flops += 16.0 * r * n_a * pairs
    byt += 2 * L * L * n_a * 16 + L * L
    return float(byt), float(flops), float(np.mean(store.ranks)) if store.ranks is not None else 0.0


def c1_leg(ctx, args):
    """2-bit 32x32 units, one uniform codebook (seed 1), normal incidence:
    compressed store (dense c64 near |d| <= 2, ACA c64 far at tol 1e-4),
    near-field block ILU(0) radius 1, GMRES(60) to 5e-5, 360-direction RCS,
    checked against the plain FP64 GPU path (all 3,969 blocks dense
    complex128) solved to 1e-10; speedup over that plain path solved to the
    same 5e-5 (both warm)."""
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_2BIT, TWOBIT_SOLVE as P
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    L = 32
    unit = macro_unit(SIDES_2BIT)
    n_a = unit.n_a
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    batch = r3m.Batch.from_codebooks([cb.uniform(L, 4, 1)], [L], dev)
    N = L * L * n_a
    dirs = cb.phi0_cut(1.0)
    dense = pipeline.fill_blocks(ctx, geom, L - 1, r3m.C128, dev)
    store = pipeline.compressed_store(ctx, geom, L, 2, r3m.C64, r3m.C64, 1e-4, 40, dev, dense_c128=dense)
    plain = r3m.Store(unit.n, 4, L - 1, L - 1, L - 1, r3m.C128, dense)
    pc = args.c1_precond
    bufs = {}

    def solve(st, tol):
        if id(st) not in bufs:
            bufs[id(st)] = (torch.zeros(N, dtype=torch.complex128, device=dev),
                            torch.empty(r3m.gmres_work_bytes(ctx, st, batch, P["restart"], precond=pc,
                                                             ilu_radius=P["ilu_radius"]),
                                        dtype=torch.uint8, device=dev))
        b, work = bufs[id(st)]
        r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]], b)
        x = torch.empty_like(b)
        _, rep = r3m.r3m_gmres_solve(ctx, st, None, batch, b, x, tol, P["restart"], P["max_iter"], work,
                                     allow_not_converged=True, precond=pc, ilu_radius=P["ilu_radius"])
        sig = torch.empty(len(dirs), dtype=torch.float64, device=dev)
        r3m.r3m_rcs(ctx, geom, batch, x, dirs, 1.0, sig)
        return x, sig, rep

    _, sig_ref, rep_ref = solve(plain, 1e-10)
    sig_ref = sig_ref.cpu().numpy()

    def timed(st, tol, reps):
        solve(st, tol)  # warm: graphs, factors, tuning
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        outs = [solve(st, tol) for _ in range(reps)]
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / reps, outs

    t_mixed, outs = timed(store, P["tol"], 10)
    errs = [float(np.linalg.norm(o[1].cpu().numpy() - sig_ref) / np.linalg.norm(sig_ref)) for o in outs]
    t_plain, outs_p = timed(plain, P["tol"], 2)
    err_plain = float(np.linalg.norm(outs_p[-1][1].cpu().numpy() - sig_ref) / np.linalg.norm(sig_ref))
    mv = timed_matvec(r3m, ctx, store, batch, outs[-1][0], r3m.C128, 50)
    mvp = timed_matvec(r3m, ctx, plain, batch, outs[-1][0], r3m.C128, 10)
    byt, flops, mean_rank = algorithmic(store, L, n_a)
    groups = r3m.matvec_groups(ctx, store, batch)
    tr = PROFILED_TRAFFIC["c1_matvec"]
    traffic = tr["bytes"] if tr and groups == tr["groups"] else None
    del bufs
    return {"workload": f"2-bit DCM 32x32, near c64 |d|<=2 dense, far ACA tol 1e-4 c64, "
                        f"{PRECOND_NAMES.get(pc, '?').format(r=P['ilu_radius'])} GMRES({P['restart']}) "
                        f"tol {P['tol']:g}, 360-direction RCS",
            "solves_per_s": sum(e <= RCS_TARGET for e in errs) / (t_mixed * len(errs)),
            "rcs_rel_err": max(errs), "gmres_iters": outs[-1][2][0][0],
            "plain_fp64_same_tol": {"solve_s": t_plain, "iters": outs_p[-1][2][0][0], "rcs_rel_err": err_plain,
                                    "matvec_ms": mvp * 1e3},
            "speedup_vs_plain_fp64_same_tol": t_plain / t_mixed,
            "reference_iters_1e-10": rep_ref[0][0],
            "matvec_ms": mv * 1e3, "matvec_gbps": byt / mv / 1e9, "matvec_tflops": flops / mv / 1e12,
            "roofline": {"bound": "alu", "achieved": flops / mv / 1e12, "peak": PEAK_FP32_TFLOPS,
                         "unit": "TFLOP/s", "frac": flops / mv / 1e12 / PEAK_FP32_TFLOPS, "traffic": traffic,
                         "displacement_groups": groups, "algorithmic_flops_per_launch": flops,
                         "algorithmic_bytes_per_launch": byt},
            "mean_far_rank": mean_rank, "max_aca_err": float(store.rel_err.max())}


def c0_leg(ctx, args):
    """Plain 1-bit 6x6, complex128, all 121 blocks dense: GMRES to 1e-8 and
    the RCS against the oracle's dense-LU solution; the matvec timed over 1000
    replays of a captured HIP graph, warm and with the 256 MB Infinity Cache
    flushed (a 1 GiB device write) before each of 100 replays."""
    import numpy as np
    import torch
    from oracle import efie, excitation, farfield, solve as osolve
    from oracle.constants import wavenumber
    from paper_2112_05082_amd import pipeline, r3m
    from workloads.configs import FREQ_HZ, plain_6x6
    dev = "cuda:0"
    w = plain_6x6()
    unit = w.unit()
    L = w.L
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    store = pipeline.dense_store(ctx, geom, L, r3m.C128, dev)
    batch = r3m.Batch.from_codebooks(w.codebooks, [L], dev)
    N = L * L * unit.n_a
    from workloads import codebooks as cb
    dirs = cb.phi0_cut(1.0)
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    x = torch.zeros_like(b)
    work = torch.empty(r3m.gmres_work_bytes(ctx, store, batch, 100), dtype=torch.uint8, device=dev)
    sig = torch.zeros(len(dirs), dtype=torch.float64, device=dev)

    def one():
        r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]], b)
        _, rep = r3m.r3m_gmres_solve(ctx, store, None, batch, b, x, w.gmres_tol, 100, 1000, work)
        r3m.r3m_rcs(ctx, geom, batch, x, dirs, 1.0, sig)
        return rep

    one()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(10):
        rep = one()
    torch.cuda.synchronize()
    t_solve = (time.perf_counter() - t0) / 10
    k = wavenumber(FREQ_HZ)
    Zk = efie.direct_system(unit, w.codebooks[0], L, k, extract=1)
    mesh, _ = efie.active_array_mesh(unit, w.codebooks[0], L)
    sref = farfield.rcs(mesh, osolve.lu_solve(Zk, excitation.plane_wave(mesh, k)), k, dirs)
    err = float(np.linalg.norm(sig.cpu().numpy() - sref) / np.linalg.norm(sref))
    # graph-replayed matvecs
    y = torch.zeros_like(b)
    mw = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C128), dtype=torch.uint8, device=dev)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(3):  # tunes the launch shape and builds the retrieval index before capture
            r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C128, x, y, mw, stream=s.cuda_stream)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C128, x, y, mw, stream=s.cuda_stream, index_ready=True)
        y_eager = y.clone()
        g.replay()
        s.synchronize()
        assert torch.equal(y, y_eager), "graph replay differs from the eager matvec"
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(s)
        for _ in range(1000):
            g.replay()
        e1.record(s)
        e1.synchronize()
        warm_us = e0.elapsed_time(e1) / 1000 * 1e3
        flush = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
        tot = 0.0
        for _ in range(100):
            flush.fill_(1)
            e0.record(s)
            g.replay()
            e1.record(s)
            e1.synchronize()
            tot += e0.elapsed_time(e1)
        flushed_us = tot / 100 * 1e3
    del flush
    byt = 121 * 80 * 80 * 16 + 2 * N * 16
    return {"workload": "plain 1-bit 6x6, complex128, all 121 blocks dense, GMRES(100) to 1e-8, 360-direction RCS",
            "solve_ms": t_solve * 1e3, "solves_per_s": 1.0 / t_solve, "gmres_iters": rep[0][0],
            "rcs_rel_err_vs_oracle_lu": err,
            "matvec_us_graph_warm": warm_us, "matvec_us_graph_flushed": flushed_us,
            "matvec_gbps_flushed": byt / (flushed_us * 1e-6) / 1e9, "algorithmic_bytes": byt}


def spectral_32x32_leg(ctx, args):
    """The 2-bit 32x32 workload through the FFT form of the matvec
    (complex64 block spectra: the dense operator, no compression)."""
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_2BIT, TWOBIT_SOLVE as P
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    L = 32
    unit = macro_unit(SIDES_2BIT)
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    batch = r3m.Batch.from_codebooks([cb.uniform(L, 4, 1)], [L], dev)
    dirs = cb.phi0_cut(1.0)
    N = L * L * unit.n_a
    spec = pipeline.spectral_store(ctx, geom, L, 2, r3m.C64, dev)
    spec128 = pipeline.spectral_store(ctx, geom, L, 2, r3m.C128, dev)
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    pc = args.c1_precond
    work = torch.empty(r3m.gmres_work_bytes(ctx, spec128, batch, P["restart"], precond=pc,
                                            ilu_radius=P["ilu_radius"]), dtype=torch.uint8, device=dev)

    def solve(st, tol):
        r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]], b)
        x = torch.empty_like(b)
        _, rep = r3m.r3m_gmres_solve(ctx, st, None, batch, b, x, tol, P["restart"], P["max_iter"], work,
                                     allow_not_converged=True, precond=pc, ilu_radius=P["ilu_radius"])
        sig = torch.empty(len(dirs), dtype=torch.float64, device=dev)
        r3m.r3m_rcs(ctx, geom, batch, x, dirs, 1.0, sig)
        return x, sig, rep

    _, sig_ref, _ = solve(spec128, 1e-10)
    sig_ref = sig_ref.cpu().numpy()
    solve(spec, P["tol"])
    torch.cuda.synchronize()
    reps = 5
    t0 = time.perf_counter()
    outs = [solve(spec, P["tol"]) for _ in range(reps)]
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    err = max(float(np.linalg.norm(o[1].cpu().numpy() - sig_ref) / np.linalg.norm(sig_ref)) for o in outs)
    mv = timed_matvec(r3m, ctx, spec, batch, outs[-1][0], r3m.C128, 20)
    byt, flops, G = spectral_cost(spec.n, L - 1, 1)
    return {"solves_per_s": reps / dt, "rcs_rel_err_vs_fp64_spectra": err, "gmres_iters": outs[-1][2][0][0],
            "matvec_ms": mv * 1e3, "matvec_gbps": byt / mv / 1e9, "matvec_tflops": flops / mv / 1e12,
            "grid": [G, G], "spectra_bytes": byt}


def large_leg(ctx, args):
    """1-bit 128x128 units x 16 Bernoulli codebooks, normal incidence: inner
    GMRES on complex64 block spectra, FP64 refinement residual on complex128
    spectra of the same blocks, to 1e-5 (the large workload)."""
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads.configs import FREQ_HZ, SIDES_1BIT, large_128x128
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    w = large_128x128(16)
    unit = macro_unit(SIDES_1BIT)
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    batch = r3m.Batch.from_codebooks(w.codebooks, w.sizes, dev)
    dense = pipeline.fill_blocks(ctx, geom, 127, r3m.C128, dev)
    s64 = pipeline.spectral_store(ctx, geom, 128, 2, r3m.C64, dev, dense_c128=dense)
    s128 = pipeline.spectral_store(ctx, geom, 128, 2, r3m.C128, dev, dense_c128=dense)
    del dense
    torch.cuda.empty_cache()
    N = batch.total_units * unit.n_a
    g = torch.Generator(device=dev).manual_seed(5)
    xr = torch.complex(torch.randn(N, generator=g, device=dev), torch.randn(N, generator=g, device=dev))
    mv64 = timed_matvec(r3m, ctx, s64, batch, xr.to(torch.complex64), r3m.C64, 10)
    del xr
    torch.cuda.empty_cache()
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]] * batch.B, b)
    x = torch.zeros_like(b)
    restart = 30
    work = torch.empty(r3m.gmres_work_bytes(ctx, s64, batch, restart, s128), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    # block-Jacobi: per-codebook ILU factors of 16 x 128 x 128 units would hold 30 GB
    _, rep = r3m.r3m_gmres_solve(ctx, s64, s128, batch, b, x, 1e-3, restart, 3000, work,
                                 refine_tol=w.refine_tol, max_refine=20, precond=r3m.PRECOND_BLOCK_JACOBI,
                                 allow_not_converged=True)
    torch.cuda.synchronize()
    t_solve = time.perf_counter() - t0
    byt, flops, G = spectral_cost(80, 127, batch.B)
    return {"workload": "1-bit 128x128 units x 16 Bernoulli codebooks, normal incidence, block spectra "
                        "(complex64 inner GMRES(30) to 1e-3, complex128 refinement residual to 1e-5)",
            "rhs": batch.B, "matvec_ms_c64": mv64 * 1e3, "matvec_tflops_c64": flops / mv64 / 1e12,
            "solve_s": t_solve, "solves_per_s": batch.B / t_solve,
            "converged": all(r[3] for r in rep), "max_rel_residual": max(r[2] for r in rep),
            "inner_iters_max": max(r[0] for r in rep), "refine_steps_max": max(r[1] for r in rep)}


def relaxed_leg(ctx, args):
    """The differentiation workload: 2-bit 32x32 relaxed codebook (softmax of
    N(0,1) logits, seed 3), J = mean RCS over 16 directions in a 30-degree
    cone; one forward (relaxed solve + objective) and one backward (adjoint
    solve with the transposed operator + gradient) on complex128 spectra,
    block ILU(0) of the blended near field (radius 1), GMRES(60) to 1e-8."""
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from paper_2112_05082_amd.relaxed import RelaxedRcs
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_2BIT
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    L = 32
    unit = macro_unit(SIDES_2BIT)
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    pc = r3m.PRECOND_BLOCK_ILU
    store = pipeline.spectral_store(ctx, geom, L, 1, r3m.C128, dev)
    batch = r3m.Batch.from_codebooks([np.zeros(L * L, np.uint8)], [L], dev)
    obj = RelaxedRcs(ctx, geom, store, batch, [[0.0, 0.0, 1.0]], cb.cone16(30.0), tol=1e-8, precond=pc)
    logits = torch.from_numpy(np.random.default_rng(3).standard_normal((L * L, 4))).to(dev)
    for _ in range(2):
        lg = logits.clone().requires_grad_(True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        J = obj(torch.softmax(lg, dim=1))
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        it_f = obj.last_reports[0][0]
        J.sum().backward()
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        it_b = obj.last_reports[0][0]
    return {"workload": "2-bit 32x32 relaxed codebook (softmax of N(0,1) logits, seed 3), J = mean RCS over "
                        "16 directions in a 30-degree cone, complex128 spectra, block-ILU(0) r=1 GMRES(60) to 1e-8",
            "J": J.item(), "forward_s": t1 - t0, "backward_s": t2 - t1, "forward_iters": it_f,
            "adjoint_iters": it_b, "grad_norm": float(lg.grad.norm().item()), "gradients_per_s": 1.0 / (t2 - t0)}


def sweep_leg(ctx, args):
    """Preconditioner study in the manner of the paper's iteration histogram
    over 90 random codebooks: GMRES(60) iterations to 1e-5 for 1-bit 16x16
    Bernoulli(p) codebooks, p = 0.1 .. 0.9, 10 seeds each, normal incidence, on
    the complex128 dense store, without preconditioner, with block-Jacobi and
    with the near-field block ILU(0) of radius 1 and 2."""
    import numpy as np
    import torch
    from paper_2112_05082_amd import pipeline, r3m
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_1BIT
    from workloads.mesh import macro_unit
    dev = "cuda:0"
    L, seeds = 16, 10
    unit = macro_unit(SIDES_1BIT)
    geom = r3m.UnitGeom.from_macro(unit, FREQ_HZ, 1)
    store = pipeline.dense_store(ctx, geom, L, r3m.C128, dev)
    cases = [("none", r3m.PRECOND_NONE, 1), ("block_jacobi", r3m.PRECOND_BLOCK_JACOBI, 1),
             ("block_ilu_r1", r3m.PRECOND_BLOCK_ILU, 1), ("block_ilu_r2", r3m.PRECOND_BLOCK_ILU, 2)]
    ps = [round(0.1 * k, 1) for k in range(1, 10)]
    iters = {name: np.zeros((len(ps), seeds), dtype=np.int64) for name, _, _ in cases}
    secs = {name: 0.0 for name, _, _ in cases}
    b = torch.zeros(L * L * unit.n_a, dtype=torch.complex128, device=dev)
    works = {name: torch.empty(r3m.gmres_work_bytes(ctx, store, r3m.Batch.from_codebooks(
        [cb.bernoulli(L, 0)], [L], dev), 60, precond=pc, ilu_radius=rad), dtype=torch.uint8, device=dev)
        for name, pc, rad in cases}
    for ip, p in enumerate(ps):
        for sd in range(seeds):
            batch = r3m.Batch.from_codebooks([cb.bernoulli(L, 100 * ip + sd, p)], [L], dev)
            r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]], b)
            for name, pc, rad in cases:
                x = torch.zeros_like(b)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                _, rep = r3m.r3m_gmres_solve(ctx, store, None, batch, b, x, 1e-5, 60, 4000, works[name],
                                             precond=pc, ilu_radius=rad, allow_not_converged=True)
                torch.cuda.synchronize()
                secs[name] += time.perf_counter() - t0
                iters[name][ip, sd] = rep[0][0] if rep[0][3] else -rep[0][0]
    del works
    return {"workload": "1-bit 16x16 Bernoulli(p) codebooks, p = 0.1..0.9 x 10 seeds (seed 100 i + s), "
                        "complex128 dense store, GMRES(60) to 1e-5 (negative: not converged within 4000)",
            "p": ps, "mean_iters": {k: v.mean(axis=1).round(1).tolist() for k, v in iters.items()},
            "max_iters": {k: v.max(axis=1).tolist() for k, v in iters.items()},
            "all_converged": bool(all((v > 0).all() for v in iters.values())),
            "total_solve_s": secs}


# ------------------------------------------------------------- CPU baseline

def _oracle_matvec_worker(args):
    """One process: the oracle's FP64 block retrieved matvec of the 8x8 sample
    (one warm-up, then the median of five)."""
    import numpy as np
    blocks, D, off, states, L, seed = args
    from oracle import retrieval
    from workloads import codebooks as cb
    x = cb.random_complex(L * L * int(off[1]), seed)
    retrieval.retrieved_matvec(blocks, D, D, off, states, L, x)
    ts = []
    for _ in range(5):
        t = time.perf_counter()
        retrieval.retrieved_matvec(blocks, D, D, off, states, L, x)
        ts.append(time.perf_counter() - t)
    return float(np.median(ts))


def cpu_baseline(head):
    """The oracle on the host cores (CORES threads; OMP/OpenBLAS/MKL pinned
    to it), real EFIE blocks from the oracle's own fill:
      - a bounded sample of the batched workload: the oracle's block-Toeplitz
        retrieved matvec (FP64) of 1-bit 8x8 Bernoulli codebooks, one per
        worker process, one warm-up then the median of five; extrapolated to
        the batched solve by unit-pair count (L^4 against 8^4) and by the
        matvecs each right-hand side took in the timed GPU solve;
      - the plain 1-bit 6x6 case in full: dense LU of the direct active-only
        system (one warm-up, median of five)."""
    import multiprocessing as mp

    import numpy as np
    from oracle import efie, solve as osolve
    from oracle.constants import wavenumber
    from workloads import codebooks as cb
    from workloads.configs import FREQ_HZ, SIDES_1BIT
    from workloads.mesh import macro_unit
    k = wavenumber(FREQ_HZ)
    unit = macro_unit(SIDES_1BIT)
    Ls = 8
    t0 = time.perf_counter()
    blocks = efie.displacement_blocks(unit, Ls - 1, Ls - 1, k, extract=1)
    t_fill = time.perf_counter() - t0
    off = np.arange(0, unit.n + 1, unit.n_a)
    jobs = [(blocks, Ls - 1, off, cb.bernoulli(Ls, 7000 + i), Ls, i) for i in range(CORES)]
    with mp.get_context("fork").Pool(CORES) as pool:
        per = pool.map(_oracle_matvec_worker, jobs)
    t_mv = float(np.median(per))  # seconds per 8x8 matvec on one core
    # extrapolation to the batched solve
    rep, sizes = head["_rep"], head["_S"]["sizes"]
    work_s = 0.0
    for r, L in zip(rep, sizes):
        matvecs = r[0] + r[1] + 1  # inner iterations + refinement residuals + final check
        work_s += t_mv * (L / Ls) ** 4 * matvecs
    solves_per_s = len(sizes) / (work_s / CORES)
    # the plain 6x6 case in full
    st = cb.bernoulli(6, 0)
    Zk = efie.direct_system(unit, st, 6, k, extract=1)
    from oracle import excitation
    mesh, _ = efie.active_array_mesh(unit, st, 6)
    U = excitation.plane_wave(mesh, k)
    osolve.lu_solve(Zk, U)
    ts = []
    for _ in range(5):
        t = time.perf_counter()
        osolve.lu_solve(Zk, U)
        ts.append(time.perf_counter() - t)
    return {"value": float(solves_per_s), "unit": "codebook solves/s", "cores": CORES, "kind": "oracle",
            "sample": (f"oracle FP64 block-Toeplitz retrieved matvec of 1-bit 8x8 codebooks with real EFIE blocks "
                       f"(oracle fill {t_fill:.1f} s, untimed), {CORES} worker processes, median "
                       f"{t_mv * 1e3:.1f} ms per matvec per core; EXTRAPOLATED to the 1,536-RHS batched solve by "
                       f"unit-pair count (L^4 / 8^4) x the matvecs each RHS took on the GPU"),
            "matvec_8x8_s": t_mv, "extrapolated_batch_s": float(work_s / CORES),
            "plain_6x6_dense_lu": {"solve_s": float(np.median(ts)), "solves_per_s": 1.0 / float(np.median(ts)),
                                   "unknowns": int(Zk.shape[0]), "measured": "in full"}}


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; --gpus must be 1"}))
        sys.exit(2)
    import torch

    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    legs = {"c1_2bit_32x32": c1_leg, "c0_plain_6x6": c0_leg, "spectral_32x32": spectral_32x32_leg,
            "large_128x128": large_leg, "relaxed_32x32": relaxed_leg, "precond_sweep_16x16": sweep_leg}
    if args.only:
        out = {}
        for name in args.only.split(","):
            t0 = time.perf_counter()
            out[name] = legs[name](ctx, args)
            out[name]["leg_s"] = time.perf_counter() - t0
            print(f"[bench] {name} done in {out[name]['leg_s']:.1f} s", file=sys.stderr, flush=True)
        # a plain device copy of known size: the reference for the HBM counters
        src = torch.ones(256 << 20, dtype=torch.uint8, device="cuda:0")
        torch.empty_like(src).copy_(src)
        torch.cuda.synchronize()
        ctx.close()
        print(json.dumps(out), flush=True)
        return
    if args.matvec_only:
        out = matvec_only(ctx, args)
        ctx.close()
        print(json.dumps({"matvec_only": out}), flush=True)
        return
    if args.c2_compressed:
        out = c2_compressed(ctx, args)
        ctx.close()
        print(json.dumps({"c2_compressed": out}), flush=True)
        return
    head = headline_c2(ctx, args)
    out = {
        "metric": "retrieved complex matvec GB/s (% HBM peak) + codebook solves/s at 1e-4 RCS err",
        "value": head["value"],
        "unit": "codebook solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 (c64 spectra and inner Krylov basis, f32 products) / f64 Krylov arithmetic and refinement residual",
        "data": "synthetic (seeded 1-bit codebooks: Bernoulli, checkerboard, stripes; PEC patch units)",
        "config": {"workload": f"batched 1-bit {3 * args.n_per_size} codebooks (32x32/48x48/64x64) x 4 angles = "
                               f"{12 * args.n_per_size} RHS, one global matrix for 64x64 as complex64 block spectra, "
                               "block-Jacobi GMRES(20) to 1e-3 with FP64 refinement (complex128 spectra) to 1e-6, "
                               "360-direction RCS per RHS; a solve counts if its RCS is within 1e-4 of the FP64 "
                               "reference (refined to 1e-10)",
                   "rhs": 12 * args.n_per_size},
        "roofline": head["roofline"],
    }
    out["batched_1536"] = {k: v for k, v in head.items() if not k.startswith("_") and k != "roofline"}
    torch.cuda.empty_cache()
    if not args.no_legs:
        legs = [("c1_2bit_32x32", c1_leg), ("c0_plain_6x6", c0_leg), ("spectral_32x32", spectral_32x32_leg),
                ("large_128x128", large_leg), ("relaxed_32x32", relaxed_leg)]
        if not args.no_sweep:
            legs.append(("precond_sweep_16x16", sweep_leg))
        for name, fn in legs:
            t0 = time.perf_counter()
            out[name] = fn(ctx, args)
            out[name]["leg_s"] = time.perf_counter() - t0
            torch.cuda.empty_cache()
            print(f"[bench] {name} done in {out[name]['leg_s']:.1f} s", file=sys.stderr, flush=True)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(head)
    ctx.close()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()

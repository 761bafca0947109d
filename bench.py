"""Benchmark: EnKF analysis steps/sec of the CGD-EnKF HIP path on one MI355X.

Workload (default): the Lorenz-96 twin experiment with n=4096, F=8, every
2nd variable observed (m=2048), N=64, R=0.5 I, forecast spread N(0,1),
5 RK4 steps of dt=0.05 between analyses, stochastic EnKF, FP32 block CG to a
relative residual of 1e-6.  The cycles are driven by the GPU analyses
(untimed, with host forecasts); every cycle's inputs stay resident in HBM,
then W warm-up and K timed analyses replay them back to back.  One step is
one whole analysis (gather, block CG, ensemble update).

Workload `batched`: 256 independent Lorenz-96 filters of uneven size
(n = 4 U{256..8192}, m = n/4 random observed variables, N in {16, 32, 64},
R = I), FP32 block CG to 1e-6, solved by one batched call (three launches: the
gather, one CG workgroup per member of every filter, the update) captured in
a HIP graph; one step is one graph replay (256 analyses).

Modes of the single analysis (`--mode`): `full` (Algorithm 1, the default),
`reduced` (Algorithm 2 with CG on the N x N system), `senkf` (the sEnKF of
Appendix A; on the twin workload its own cycles diverge, so the CGD-EnKF
drives them and the sEnKF is timed on the same inputs) and `gain` (the
explicit-gain form of Figure 2, one CG per column of K^T).  Workload `ex1b`:
Example 1b's first analysis at m = p = 4000, N = 50, FP64, tol 1e-12.

Prints one JSON line.  `value` is analyses/s over the K timed steps.

`--copy-calibration` first runs a plain device copy of a known size, the
reference that scales rocprofv3's FETCH_SIZE / WRITE_SIZE counters to bytes,
so that one counter run covers both the copy and the solver.
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

METRIC = "EnKF analysis steps/sec at rel. residual 1e-6; CG iters & time learned vs plain"
HBM_PEAK_GBS = 8000.0
FP32_MFMA_PEAK_TFLOPS = 157.3  # MI355X dense FP32 matrix peak
FP64_MFMA_PEAK_TFLOPS = 78.6  # MI355X dense FP64 matrix peak
BF16_MFMA_PEAK_TFLOPS = 2500.0  # MI355X dense BF16 matrix peak (no sparsity)

# HBM traffic per launch of the column solver on the Lorenz-96 twin workload,
# from rocprofv3 --pmc FETCH_SIZE and WRITE_SIZE (KiB per dispatch, scaled by
# a plain 1 GiB copy measured in the same run: FETCH_SIZE x 2.0, WRITE_SIZE
# x 1.0), valid only for the kernel sources it was measured on.
_COL_SOURCES = ["paper_2606_19224_amd/csrc/cg_columns.hip", "paper_2606_19224_amd/csrc/exchange.h",
                "paper_2606_19224_amd/csrc/mfma_util.h", "paper_2606_19224_amd/csrc/update_tile.h",
                "paper_2606_19224_amd/csrc/internal.h"]
_TILE_SOURCES = ["paper_2606_19224_amd/csrc/cg_tile.hip", "paper_2606_19224_amd/csrc/exchange.h",
                 "paper_2606_19224_amd/csrc/mfma_util.h", "paper_2606_19224_amd/csrc/internal.h"]
_KT_SOURCES = ["paper_2606_19224_amd/csrc/gain_cg.hip", "paper_2606_19224_amd/csrc/modes.h",
               "paper_2606_19224_amd/csrc/mfma_util.h", "paper_2606_19224_amd/csrc/internal.h"]
_BM_SOURCES = ["paper_2606_19224_amd/csrc/cg_batched.hip", "paper_2606_19224_amd/csrc/mfma_util.h",
               "paper_2606_19224_amd/csrc/internal.h"]
# rocprofv3 FETCH_SIZE / WRITE_SIZE per dispatch (KiB, mean over the run's
# dispatches of the kernel) and the scale factors a plain 1 GiB copy gives in
# the same runs; valid only for the sources they were taken on.
MEASURED_TRAFFIC = {
    "k_cg_split": {
        "workload": "l96-twin", "sources": _COL_SOURCES, "sha256_16": "d622da2685420c65",
        "fetch_kib_raw": 6378.1, "fetch_scale": 2.0, "write_kib_raw": 6297.0, "write_scale": 1.0,
    },
    "k_cg_tile": {
        "workload": "adv-diff", "sources": _TILE_SOURCES, "sha256_16": "5cfba8b2e2f544f5",
        "fetch_kib_raw": 580223.6, "fetch_scale": 2.0, "write_kib_raw": 1232412.7,
        "write_scale": 1.0,
    },
    "k_cg_tilemx": {
        "workload": "adv-diff", "sources": _TILE_SOURCES, "sha256_16": "5cfba8b2e2f544f5",
        "fetch_kib_raw": 941428.7, "fetch_scale": 2.0, "write_kib_raw": 1685711.9,
        "write_scale": 1.0,
    },
    "k_cg_tilesplit": {
        "workload": "adv-diff", "sources": _TILE_SOURCES, "sha256_16": "5cfba8b2e2f544f5",
        "fetch_kib_raw": 619080.5, "fetch_scale": 2.0, "write_kib_raw": 1243155.9,
        "write_scale": 1.0,
    },
    "k_bm_solve": {  # 256 filters
        "sources": _BM_SOURCES, "sha256_16": "6937ab435f991660",
        "fetch_kib_raw": 1925472.7, "fetch_scale": 2.0, "write_kib_raw": 2672372.8,
        "write_scale": 1.0,
    },
    "k_kt_cg": {
        "workload": "l96-twin", "sources": _KT_SOURCES, "sha256_16": "3de1ede2fed59586",
        "fetch_kib_raw": 859114.1, "fetch_scale": 2.0, "write_kib_raw": 1706404.6,
        "write_scale": 1.0,
    },
}


def measured_traffic(kernel: str, workload: str = "batched"):
    """Bytes per launch from the committed counter runs of `kernel` on
    `workload`, or None when the kernel's sources changed since (or none were
    taken)."""
    import hashlib
    rec = MEASURED_TRAFFIC.get(kernel)
    if rec is None or rec.get("workload", "batched") != workload:
        return None
    h = hashlib.sha256()
    for f in rec["sources"]:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    if h.hexdigest()[:16] != rec["sha256_16"]:
        return None
    return 1024.0 * (rec["fetch_kib_raw"] * rec["fetch_scale"] + rec["write_kib_raw"] * rec["write_scale"])


def cg_bytes(m, N, k, it, b_x=4, b_s=4, b_v=4) -> float:
    """Algorithmic HBM bytes of one solve launch (gather + `it` CG iterations
    + the final S^T Z), the streaming model of the unfused iteration:
    gather reads k*m*N X values, idx/w, eps, writes S and D; each iteration
    reads S twice and moves 8 m x N vectors; the finish reads S and Z."""
    gather = k * m * N * b_x + 8 * m * k + m * N * b_x + 2 * m * N * b_v
    return gather + it * (2 * m * N * b_s + 8 * m * N * b_v) + (m * N * b_s + m * N * b_v)


def cg_flops(m, N, k, it) -> float:
    return 2 * m * k * N + it * (4 * m * N * N + 12 * m * N) + 2 * m * N * N


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--prec", default=None, choices=["fp32", "fp64", "mixed", "bf16split"],
                    help="mixed: BF16 copy of S for the inner CG, FP32 data, FP64 outer residual")
    ap.add_argument("--mode", default="full", choices=["full", "reduced", "senkf", "gain"])
    ap.add_argument("--cpu-seconds", type=float, default=30.0,
                    help="budget of the oracle CPU-baseline sample (0 disables it)")
    ap.add_argument("--grid", type=int, default=0)
    ap.add_argument("--rows-per-block", type=int, default=0)
    ap.add_argument("--solver", type=int, default=0, help="0 auto, 1 streaming, 2 resident, 3 columns, 4 split, 5 row-block x member-group")
    ap.add_argument("--workload", default="l96-twin",
                    choices=["l96-twin", "adv-diff", "batched", "warmstart", "l96-small",
                             "ex1b"],
                    help="adv-diff: the 2-D advection-diffusion analysis (n=65536, m=16384, "
                         "N=128, k=4), one input replayed")
    ap.add_argument("--cooperative", action="store_true",
                    help="launch the per-member solvers cooperatively (no start-up census)")
    ap.add_argument("--precond", default="none", choices=["none", "diag_r"],
                    help="diag_r: CG preconditioned by diag(R) (the L^-1 scaling of Algorithm 2)")
    ap.add_argument("--epochs", type=int, default=10, help="warm-start training epochs")
    ap.add_argument("--train-cycles", type=int, default=100, help="cycles per training seed")
    ap.add_argument("--count", type=int, default=256, help="filters in the batched workload")
    ap.add_argument("--phase-trace", action="store_true",
                    help="row-block x member-group solvers: add the per-step phase durations of "
                         "one traced analysis (its trace variant) to the line")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run a plain copy of known size first (HBM counter calibration)")
    return ap.parse_args()


COPY_BYTES = 1 << 30


def copy_calibration():
    """A plain copy of COPY_BYTES (reads and writes that many bytes once) for
    scaling the HBM counters: 3 copies, then one JSON line."""
    import torch
    src = torch.ones(COPY_BYTES // 4, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes": COPY_BYTES, "copies": 3}), file=sys.stderr, flush=True)
    del src, dst
    torch.cuda.empty_cache()


def _blas_info():
    try:
        from threadpoolctl import threadpool_info
        info = [d for d in threadpool_info() if d.get("user_api") == "blas"]
        if info:
            return info[0].get("internal_api", "?"), max(d.get("num_threads", 1) for d in info)
    except Exception:
        pass
    return "?", os.cpu_count() or 1


def _timed_runs(fn, runs, budget_s):
    """`runs` timed runs of fn(count) -> analyses done, each run repeating fn
    until budget_s / runs has passed; returns the per-run rates (analyses/s)."""
    rates = []
    for _ in range(runs):
        done, t0 = 0.0, time.perf_counter()
        while True:
            done += fn(done)
            if time.perf_counter() - t0 >= budget_s / runs:
                break
        rates.append(done / (time.perf_counter() - t0))
    return rates


def cpu_baseline(problems, tol, budget_s, precond="none", columns=None, mode="full",
                 gpu_out=None):
    """The FP64 oracle on a bounded sample of the same workload, timed on the
    host cores: the matrix-free textbook CG (PCG with M = diag(r) when the GPU
    path is preconditioned) with the same stop rule on all BLAS threads (the
    reported value), the same on one thread, and the Cholesky solve of the
    formed innovation matrix.  Each leg is the median of 3 runs.  With
    `columns`, a CG run solves only that many members of an analysis and its
    rate is scaled to whole analyses (members / N per analysis).  With
    `gpu_out` (the GPU's X_a of the first input, FP64 numpy), the record
    also carries its relative Frobenius error against the oracle's direct
    solve of that input."""
    import oracle
    from threadpoolctl import threadpool_limits
    blas, threads = _blas_info()
    solver = "pcg_free" if precond == "diag_r" else "cg_free"
    if mode == "reduced":
        solver = "reduced cg"
    if mode == "senkf":
        solver = "senkf"

    def cg_leg(done):
        p = problems[int(done) % len(problems)]
        if mode == "senkf":     # Appendix A's diagonal form: no system is solved
            oracle.senkf(p.Xf, p.idx, p.w, p.y, p.r, p.eps)
            return 1.0
        if mode == "gain":      # Figure 2: `columns` of the n columns of K^T, scaled
            S = oracle.obs_anomalies(p.idx, p.w, p.Xf)
            Psi = oracle.innovation_matrix(S, p.r)
            B = oracle.cross_covariance(oracle.state_anomalies(p.Xf), S).T
            for i in range(columns):
                oracle.textbook_cg(oracle.matvec_dense(Psi), B[:, i], tol, p.maxit)
            return columns / p.Xf.shape[0]
        if mode == "reduced":   # Algorithm 2, the N x N system by textbook CG from W = 0
            oracle.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg", tol=tol,
                                maxit=p.maxit)
            return 1.0
        if columns is None:
            oracle.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver=solver, tol=tol,
                                 maxit=p.maxit)
            return 1.0
        S = oracle.obs_anomalies(p.idx, p.w, p.Xf)
        D = oracle.innovations(p.idx, p.w, p.Xf, p.y, p.eps)[:, :columns]
        mv = oracle.matvec_free(S, p.r)
        if solver == "pcg_free":
            Z, _, _ = oracle.solve_pcg_columns(mv, 1.0 / p.r, D, tol, p.maxit)
        else:
            Z, _, _ = oracle.solve_cg_columns(mv, D, tol, p.maxit)
        # these members' columns of the update X_a = X_f + A (S^T Z)/(N-1)
        A = oracle.state_anomalies(p.Xf)
        _ = p.Xf[:, :columns] + A @ (S.T @ Z) / (p.Xf.shape[1] - 1)
        return columns / p.Xf.shape[1]

    direct = {}

    def chol_leg(done):
        i = int(done) % len(problems)
        p = problems[i]
        if mode == "reduced":
            res = oracle.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="direct")
        elif mode == "senkf":   # the sEnKF's own result; the timing is the exact EnKF's
            res = oracle.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cholesky")
            if i == 0 and "Xa" not in direct:
                direct["Xa"] = oracle.senkf(p.Xf, p.idx, p.w, p.y, p.r, p.eps)
        else:
            res = oracle.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cholesky")
        if i == 0 and "Xa" not in direct:
            direct["Xa"] = res["Xa"]
        return 1.0

    if mode in ("reduced", "senkf"):
        columns = None   # a reduced or sEnKF analysis is cheap enough to time whole
    if mode == "gain":
        columns = columns or 8
    legs = 3 if columns is None else 2  # config-scale samples skip the 1-thread CG leg
    share = budget_s / (legs + 1)
    cg = _timed_runs(cg_leg, 3, share * 2)
    one = None
    if columns is None:
        with threadpool_limits(limits=1):
            one = _timed_runs(cg_leg, 3, share)
    chol = _timed_runs(chol_leg, 3 if columns is None else 1, share)
    what = (f"{columns} of {problems[0].Xf.shape[0]} columns of K^T per analysis, scaled to "
            f"whole analyses" if mode == "gain" else
            f"{columns} of {problems[0].Xf.shape[1]} members per analysis, scaled to whole "
            f"analyses" if columns else f"whole analyses of the {len(problems)} distinct inputs, "
                                        f"taken in order and repeated")
    rec = {"value": float(np.median(cg)), "unit": "analyses/s", "cores": int(threads),
           "kind": "oracle",
           "sample": f"{what}; " + (
               "FP64 sEnKF, Appendix A's diagonal form (oracle.senkf)" if mode == "senkf" else
               "FP64 textbook CG per column of K^T on the formed Psi_z (Figure 2, the steps "
               "of oracle.enkf_gain_cg)" if mode == "gain" else
               "FP64 Algorithm 2 with textbook CG on the N x N system "
               "(oracle.enkf_reduced solver='cg')" if mode == "reduced" else
               f"FP64 textbook matrix-free {'P' if solver == 'pcg_free' else ''}CG "
               f"(oracle.enkf_analysis solver='{solver}')") +
               f", median of 3 runs of {share * 2 / 3:.1f} s each",
           "cpu_count": os.cpu_count(), "blas": blas, "runs": [round(x, 4) for x in cg],
           "cholesky": {"value": float(np.median(chol)), "unit": "analyses/s",
                        "cores": int(threads), "runs": [round(x, 4) for x in chol],
                        "what": ("Algorithm 2 with the N x N system by Cholesky"
                                 if mode == "reduced" else
                                 "the exact EnKF for comparison: formed innovation matrix, "
                                 "scipy cho_factor/cho_solve" if mode == "senkf" else
                                 "formed innovation matrix, scipy cho_factor/cho_solve")}}
    if one is not None:
        rec["single_thread"] = {"value": float(np.median(one)), "unit": "analyses/s", "cores": 1,
                                "runs": [round(x, 4) for x in one]}
    if gpu_out is not None and "Xa" in direct:
        ref = direct["Xa"]
        rec["gpu_rel_err_Xa"] = {
            "value": float(np.linalg.norm(gpu_out - ref) / np.linalg.norm(ref)),
            "against": ("the oracle's sEnKF (FP64) on the first input: rounding only"
                        if mode == "senkf" else
                        "the oracle's " + ("Algorithm 2 with a Cholesky solve" if mode == "reduced"
                                           else "Cholesky solve of the formed innovation matrix")
                        + " (FP64) on the first input; CG stops at rel. residual 1e-6, so this "
                          "is the stop rule's error plus rounding")}
    return rec


def main():
    args = parse()
    if args.prec is None:  # the n=40 and Example 1b analyses in FP64, the others in FP32
        args.prec = "fp64" if args.workload in ("l96-small", "ex1b") else "fp32"
    if args.gpus != 1:
        print(f"bench.py measures one GPU; --gpus {args.gpus} is not supported (the analysis "
              f"is sized for one GPU's share, and runs on several GPUs are not part of it)",
              file=sys.stderr)
        sys.exit(2)
    if args.copy_calibration:
        copy_calibration()
    if args.workload == "batched":
        bench_batched(args)
        return
    if args.workload == "warmstart":
        bench_warmstart(args)
        return
    bench_single(args)


L96_WORKLOAD = ("Lorenz-96 twin experiment n=4096 F=8, every 2nd variable observed (m=2048), "
                "N=64, R=0.5I, spread N(0,1), 5 RK4 steps dt=0.05 between analyses, stochastic "
                "EnKF, block CG to rel. residual 1e-6")
SMALL_WORKLOAD = ("Lorenz-96 n=40 F=8, truth after 1000 RK4 steps dt=0.05, N=20 members = truth + "
                  "N(0,1), every 2nd variable observed (m=20), R=I, stochastic EnKF, CG to rel. "
                  "residual 1e-10; one input replayed")
EX1B_WORKLOAD = ("Example 1b's first analysis: m=p=4000, truth and initial members N(0, I), N=50, "
                 "H=F=I, R=I, Q=0.1I (model noise added to each member), stochastic EnKF, CG to "
                 "rel. residual 1e-12; one input replayed")
ADV_WORKLOAD = ("2-D advection-diffusion 256x256 (n=65536): truth and N=128 members unit-variance "
                "Gaussian random fields (length scale 8 cells) advanced 20 upwind steps; m=16384 "
                "random-cell observations with bilinear weights (k=4); diag R ~ U[0.5, 2]; "
                "stochastic EnKF; block CG to rel. residual 1e-6; one input replayed")


def solver_roofline(info, args, m, N, k, n, it_max):
    """Algorithmic bytes and flops of the timed solver launch, its name, and
    what limits it (from the profiles: the roofline is the streaming model's
    HBM bound, the limiter is what the counters and phase timings show)."""
    b_x = 8 if args.prec == "fp64" else 4
    b_s = 2 if args.prec == "mixed" else b_x
    bytes_alg = np.array([cg_bytes(m, N, k, int(i), b_x, b_s, b_x) for i in it_max])
    flops_alg = np.array([cg_flops(m, N, k, int(i)) for i in it_max])
    tname = 'double' if args.prec == 'fp64' else 'float'
    mfma = False
    # the gather as a launch of its own ahead of the timed one, which reads S and D back
    gath = k * m * N * b_x + 8 * m * k + m * N * b_x + 2 * m * N * b_x
    wide64 = args.prec == "fp64" and N > 64  # these solvers' FP64 forms past N = 64
    if wide64 and info["solver"] == "k_cg_columns":
        bytes_alg = bytes_alg - gath + m * N * (b_s + b_x)
        kernel = (f"k_cg_columns_wide<double> (CG and S^T Z; the update is a launch of its own), "
                  f"{info['workgroups']} workgroups, one per member")
        limiter = "each member's pass over S through its CU's path to L2"
    elif wide64 and info["solver"] == "k_cg_tile":
        bytes_alg = bytes_alg - gath + m * N * (b_s + b_x)
        kernel = (f"k_cg_tile64 (CG and S^T Z, both S-products on the 16x16x4 FP64 MFMA, S "
                  f"resident in LDS), {info['workgroups']} workgroups: groups of 16 members x "
                  f"blocks of {info['rows_per_block']} rows")
        limiter = ("the per-iteration reduce-scatter/all-gather of each member group's S^T r, "
                   "two 64-bit words a double")
        mfma = True
    elif info["solver"] in ("k_cg_columns", "k_cg_split"):
        # the gather is a launch of its own ahead of the timed solver launch: the solver
        # reads S and D back instead, and also applies the update (reads X_f, writes X_a)
        bytes_alg = bytes_alg - gath + m * N * (b_s + b_x) + 2.0 * n * N * b_x
        # few rows: one wave per member (two rows a lane where NP values of S fit 256 bytes)
        np_ = 16 if N <= 16 else 32 if N <= 32 else 64
        if info["solver"] == "k_cg_columns" and args.prec in ("fp32", "fp64") and N <= 64 \
                and m <= (64 if np_ * b_x > 256 else 128):
            kernel = (f"k_cg_columns_small<{tname}> (CG + S^T Z + ensemble update in one launch), "
                      f"{info['workgroups']} workgroups, one wave per member")
            limiter = ("one wave's serial chain of short products, sums, a square root and two "
                       "divisions per step")
        elif info["solver"] == "k_cg_columns":
            kernel = (f"k_cg_columns<{tname}> (CG + S^T Z + ensemble update in one launch), "
                      f"{info['workgroups']} workgroups, one per member")
            limiter = ("per-row VALU issue and latency of one workgroup per member (S^T p and "
                       "S g are per-member products on the VALU; the update runs on the MFMA)")
        else:
            kernel = (f"k_cg_split<{tname}> (CG + S^T Z + ensemble update in one launch), "
                      f"{info['workgroups']} workgroups, {info['workgroups'] // N} per "
                      f"member, {info['rows_per_block']} rows of S each in LDS")
            limiter = ("per-iteration exchange latency between a member's workgroups and VALU "
                       "issue of the row pass: S stays in LDS, so HBM traffic is a fraction of "
                       "the streaming model; S^T p and S g are per-member products on the VALU, "
                       "not the MFMA (k_cg_resident is the MFMA variant)")
    elif info["solver"] == "k_cg_tile":
        kernel = (f"k_cg_tile<float> (gather + CG loop + S^T Z, both S-products on the 16x16x4 "
                  f"MFMA, S resident in LDS), {info['workgroups']} workgroups: groups of 32 "
                  f"members x blocks of {info['rows_per_block']} rows")
        limiter = ("the FP32 MFMA products (two S-products per iteration) plus the per-iteration "
                   "reduce-scatter/all-gather of each member group's S^T r")
        mfma = True
    elif info["solver"] == "k_cg_tilemx":
        kernel = (f"k_cg_tilemx<float> (gather + refinement loop + S^T Z: inner CG on a BF16 "
                  f"copy of S in LDS, 16x16x32 BF16 MFMA; outer residual and S^T Z on the "
                  f"16x16x4 FP64 MFMA from the FP32 S), {info['workgroups']} workgroups: "
                  f"groups of 32 members x blocks of {info['rows_per_block']} rows")
        limiter = ("the per-step reduce-scatter/all-gather of each member group's S^T r; the "
                   "BF16 products take a small part of each step")
        mfma = True
    elif info["solver"] == "k_cg_tilesplit":
        kernel = (f"k_cg_tilesplit = k_cg_tilemx<float, split-BF16> (gather + CG loop + S^T Z: "
                  f"each S-product as five 16x16x32 BF16 MFMA products, S in LDS as two BF16 "
                  f"parts and the vector in three; final S^T Z and true residual on the FP64 "
                  f"MFMA from the FP32 S), {info['workgroups']} workgroups: groups of 32 "
                  f"members x blocks of {info['rows_per_block']} rows")
        limiter = ("the per-step reduce-scatter/all-gather of each member group's S^T r; the "
                   "five BF16 products per S-product take a small part of each step")
        mfma = True
    elif info["solver"] == "k_cg_resident":
        kernel = (f"k_cg_resident<{tname}> (gather + CG loop + S^T Z, both S-products on the "
                  f"16x16x4 MFMA), {info['workgroups']} workgroups of "
                  f"{info['rows_per_block']} rows")
        limiter = "exchange of the per-workgroup Gram partials every iteration"
        mfma = True
    else:
        kernel = (f"{info['solver']}<{tname}> (gather + CG loop + S^T Z), "
                  f"{info['workgroups']} workgroups of {info['rows_per_block']} rows")
        limiter = "grid-wide barriers and streamed row blocks"
    return bytes_alg, flops_alg, kernel, limiter, mfma


def tile_phase_trace(kname, Xf, idx, w, y, r, eps, tol, maxit, prec, precond):
    """Median phase durations (us) of the row-block x member-group solvers'
    steps 1-8, from one traced analysis (cgd_tuning.trace: workgroup 0's
    timestamps of the 100 MHz real-time counter, taken by the trace variant
    of the kernel), and for the mixed kernel each outer step's two halves."""
    import torch

    from paper_2606_19224_amd import binding

    tr = torch.zeros(256, dtype=torch.int64, device=Xf.device)
    ws = None
    for _ in range(3):
        tr.zero_()
        o = binding.analysis(Xf, idx, w, y, r, eps, tol=tol, maxit=maxit, prec=prec,
                             precond=precond, stats=False, solver=5, trace=tr, workspace=ws)
        ws = o["workspace"]
    torch.cuda.synchronize()
    t = tr.cpu().numpy().astype(np.int64)
    us = lambda a, b: (a - b) / 100.0
    names = (["decide", "Q_and_update", "gram", "publish", "owner_step", "all_gather"]
             if kname in ("k_cg_tilemx", "k_cg_tilesplit") else
             ["decide", "Q", "update_and_gram", "publish", "owner_step", "all_gather"])
    rows = []
    for kit in range(1, 9):
        b, nb = 128 + 12 * kit, 128 + 12 * (kit + 1)
        s = t[b:b + 6]
        if s.min() == 0 or t[nb] == 0:
            continue
        rows.append([us(s[1], s[0]), us(s[2], s[1]), us(s[3], s[2]), us(s[5], s[3]), us(s[4], s[5]),
                     us(t[nb], s[4])])
    out = {"kernel": kname, "steps": "1-8 (those without an outer step)"}
    if rows:
        med = np.median(np.array(rows), axis=0)
        out.update({k: round(float(v), 2) for k, v in zip(names, med)})
        out["step_total"] = round(float(med.sum()), 2)
    out["loop_total"] = round(us(t[250], t[0]), 1)
    if kname in ("k_cg_tilemx", "k_cg_tilesplit"):
        outer = []
        for no in range(12):
            s = t[20 + 8 * no: 28 + 8 * no]
            if s[0]:
                outer.append({"at_step": int(s[7]), "W": round(us(s[3], s[0]), 2),
                              "residual_and_exchange": round(us(s[6], s[3]), 2)})
        out["outer_steps"] = outer
    return out


def bench_single(args):
    """One analysis per step on the Lorenz-96 twin experiment (the default:
    cycles driven by the GPU analyses, untimed, then replayed) or on the 2-D
    advection-diffusion input (one input replayed)."""
    import torch

    import workloads as W
    from paper_2606_19224_amd import binding

    dev = torch.device("cuda:0")
    dt = torch.float64 if args.prec == "fp64" else torch.float32
    K, Wm = args.steps, args.warmup
    adv = args.workload == "adv-diff"
    small = args.workload == "l96-small"
    ex1b = args.workload == "ex1b"
    replay = adv or small or ex1b  # one input replayed
    tol = 1e-10 if small else 1e-12 if ex1b else 1e-6
    t = lambda a, d=dt: torch.as_tensor(np.ascontiguousarray(a), dtype=d, device=dev)
    inputs, problems, gen_out, gen_iters = [], [], [], []
    t0 = time.perf_counter()
    if replay:
        p = W.config3() if adv else W.example1b(m=4000, N=50) if ex1b else W.config1()
        n, m, N, k = p.Xf.shape[0], p.m, p.N, p.idx.shape[1]
        idx_d, w_d, r_d = t(p.idx, torch.int32), t(p.w), t(p.r)
    else:
        cyc = W.L96Cycler(tol=1e-6, maxit=1000)
        n, m, N, k = cyc.n, cyc.idx.shape[0], cyc.N, 1
        idx_d, w_d, r_d = t(cyc.idx, torch.int32), t(cyc.w), t(cyc.r)
    precond = None if args.precond == "none" else args.precond
    plan = binding.Plan(n, m, N, k, prec=args.prec, reduced=args.mode == "reduced", tol=tol,
                        maxit=2000 if adv else 1000, device=dev, grid=args.grid,
                        solver=args.solver, rows_per_block=args.rows_per_block, precond=precond,
                        cooperative=args.cooperative, senkf=args.mode == "senkf",
                        gain=args.mode == "gain")
    out = torch.empty((n, N), dtype=dt, device=dev)
    # The sEnKF's gains, all from the same X_f, overshoot on the twin experiment and its
    # own cycles diverge within a few analyses: there the CGD-EnKF analysis drives the
    # trajectory and the sEnKF is timed on the same inputs.
    driver = (binding.Plan(n, m, N, k, prec=args.prec, tol=tol, maxit=1000, device=dev)
              if args.mode == "senkf" and not replay else None)

    def gpu_analysis(p):
        Xf, y, eps = t(p.Xf), t(p.y), t(p.eps)
        plan.check(Xf, idx_d, w_d, y, r_d, eps, out)
        plan(Xf, idx_d, w_d, y, r_d, eps, out)
        inputs.append((Xf, y, eps))
        problems.append(p)
        gen_out.append(out.clone())
        gen_iters.append(plan.iters.clone())
        if driver is not None:
            nxt = torch.empty_like(out)
            driver(Xf, idx_d, w_d, y, r_d, eps, nxt)
            return nxt.double().cpu().numpy()
        return out.double().cpu().numpy()

    if replay:
        gpu_analysis(p)
        inputs, problems = inputs * (K + Wm), problems * (K + Wm)
        gen_out, gen_iters = gen_out * (K + Wm), gen_iters * (K + Wm)
        what = f"generated the {'advection-diffusion' if adv else 'n=40 Lorenz-96'} input"
    else:
        for _ in range(K + Wm):
            cyc.step(gpu_analysis)
        what = f"generated {K + Wm} GPU-driven cycles"
    torch.cuda.synchronize()
    print(f"{what} in {time.perf_counter() - t0:.1f} s", file=sys.stderr, flush=True)

    outs = [torch.empty((n, N), dtype=dt, device=dev) for _ in range(K)]
    events = [binding.EventPair() for _ in range(K)]
    for i in range(Wm):
        Xf, y, eps = inputs[K + i]
        plan(Xf, idx_d, w_d, y, r_d, eps, outs[0])
    torch.cuda.synchronize()
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    start.record()
    for i in range(K):
        Xf, y, eps = inputs[i]
        plan(Xf, idx_d, w_d, y, r_d, eps, outs[i], events=events[i])
    stop.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    ms_total = start.elapsed_time(stop)
    per_launch_ms = np.array([e.elapsed_ms() for e in events])
    it_np = torch.stack(gen_iters[:K]).cpu().numpy()
    it_max = it_np.max(axis=1)
    repeatable = all(torch.equal(outs[i], gen_out[i]) for i in range(K))
    # the true relative residual of the last timed input (FP64-accumulated, in the norm of
    # the stop rule), from one more call with statistics
    Xf, y, eps = inputs[K - 1]
    relres_max = None   # the sEnKF solves no system; the gain form reports none
    if args.mode not in ("senkf", "gain"):
        chk = binding.analysis(Xf, idx_d, w_d, y, r_d, eps, tol=tol, maxit=plan.maxit,
                               prec=args.prec, reduced=args.mode == "reduced", precond=precond,
                               solver=args.solver, rows_per_block=args.rows_per_block)
        relres_max = chk["stats"]["relres_max"]

    value = K / (ms_total / 1e3)
    b_x = 8 if args.prec == "fp64" else 4
    mfma = False
    if args.mode == "full":
        info = plan.solver_info()
        bytes_alg, flops_alg, kernel, limiter, mfma = solver_roofline(info, args, m, N, k, n,
                                                                      it_max)
    elif args.mode == "gain":
        # the explicit-gain form: per CG step S read once (both products in one pass)
        # and the n columns' z, r, p each read and written once; then K^T D over the rows
        bytes_alg = np.array([float(b_x) * (int(i) * (m * N + 6 * m * n) + 2 * m * N
                                            + n * N * 2) for i in it_max])
        flops_alg = np.array([4.0 * m * N * n * (int(i) + 1) + 2.0 * m * n * N for i in it_max])
        kernel = ("k_kt_cg (explicit-gain CG: one workgroup per 16 columns of K^T, one row "
                  "pass per step with both S-products on the MFMA, vectors in HBM)")
        limiter = "HBM: the n columns' z, r, p are read and written once per step"
        mfma = True
    elif args.mode == "senkf":
        # one pass over m (gather of H X_f rows, centring, the row scaling, the N x N
        # product Zhat^T diag(...)^{-1} (Y - Z) on the MFMA), then X_f + A W
        bytes_alg = np.full(K, float(k * m * N * b_x + 8 * m * k + 2 * m * b_x + m * N * b_x
                                     + 2 * n * N * b_x))
        flops_alg = np.full(K, float(2 * m * k * N + 2 * m * N * N + 2 * n * N * N))
        kernel = ("sEnKF analysis, all launches (gather + N x N product on the MFMA + "
                  "X_f + A W on the MFMA)")
        limiter = "HBM: the gathered rows of X_f, then X_f read and X_a written once"
        mfma = True
    else:
        # reduced: one pass over m forming the N x 2N matrix (gather, centring, scaling, the
        # product), the N x N CG (2 N^3 flops per step over all columns), then X_a = X_f W;
        # the events bracket all of its launches
        bytes_alg = np.full(K, float(k * m * N * b_x + 8 * m * k + 2 * m * b_x + m * N * b_x
                                     + 2 * n * N * b_x))
        flops_alg = np.array([float(2 * m * k * N + 4 * m * N * N + 2 * n * N * N
                                    + 2 * int(i) * N ** 3) for i in it_max])
        kernel = ("reduced analysis, all launches (gather + N x 2N product on the MFMA + "
                  "N x N CG, one wavefront per column + X_f W on the MFMA)")
        limiter = "launch and synchronisation latency of the small N x N stages"
        mfma = True
    achieved = bytes_alg.sum() / (per_launch_ms.sum() / 1e3) / 1e9
    tflops = flops_alg.sum() / (per_launch_ms.sum() / 1e3) / 1e12
    kname = kernel.split("<")[0].split(" ")[0]
    traffic = None
    if (args.mode == "full" and precond is None and (args.prec == "fp32" or
                                                      kname in ("k_cg_tilemx", "k_cg_tilesplit"))
            or args.mode == "gain" and args.prec == "fp32"):
        traffic = measured_traffic(kname, "adv-diff" if adv else "ex1b" if ex1b else "l96-twin")
    # S resident on chip with both S-products on the MFMA: the FP32 MFMA peak
    # bounds the kernel (its HBM traffic is the exchange, not S); otherwise the
    # streaming model's bytes against HBM
    # (the mixed kernel's contraction is BF16: its peak is the dense BF16 one)
    mfma_bound = kname in ("k_cg_tile", "k_cg_tile64", "k_cg_tilemx", "k_cg_tilesplit")
    mpeak = (BF16_MFMA_PEAK_TFLOPS if kname in ("k_cg_tilemx", "k_cg_tilesplit") else
             FP64_MFMA_PEAK_TFLOPS if kname == "k_cg_tile64" else FP32_MFMA_PEAK_TFLOPS)
    roof = {
        "bound": "mfma" if mfma_bound else "hbm",
        "kernel": kernel,
        "achieved": round(tflops if mfma_bound else achieved, 4 if mfma_bound else 2),
        "peak": mpeak if mfma_bound else HBM_PEAK_GBS,
        "unit": "TFLOP/s" if mfma_bound else "GB/s",
        "frac": round(tflops / mpeak if mfma_bound else achieved / HBM_PEAK_GBS, 5),
        "traffic": traffic,
        "streaming_model_GBps": round(achieved, 2),
        "avg_launch_us": round(per_launch_ms.mean() * 1e3, 2),
        "alg_bytes_per_launch": float(bytes_alg.mean()),
        "alg_flops_per_launch": float(flops_alg.mean()),
        "achieved_tflops": round(flops_alg.sum() / (per_launch_ms.sum() / 1e3) / 1e12, 4),
        "limiter": limiter,
        "mfma_s_products": mfma,
    }
    if traffic:
        roof["measured_hbm_GBps"] = round(traffic / (per_launch_ms.mean() / 1e3) / 1e9, 2)
    rec = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "analyses/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": Wm,
        "ms_per_step": round(ms_total / K, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp32": "f32", "fp64": "f64", "mixed": "bf16+f32 (f64 outer residual)",
                  "bf16split": "split-bf16 (S in 2 parts, vectors in 3)+f32"}[args.prec],
        "data": "synthetic",
        "config": {
            "workload": (ADV_WORKLOAD if adv else SMALL_WORKLOAD if small else
                         EX1B_WORKLOAD if ex1b else L96_WORKLOAD),
            "tol": tol,
            "mode": args.mode, "prec": args.prec, "precond": args.precond,
            "launch": "cooperative" if args.cooperative else "plain + start-up census",
            "n": n, "m": m,
            "N": N, "k": k, "inputs_replayed": K,
            **({"cycles_driven_by": "the CGD-EnKF analysis (the sEnKF's own cycles diverge)"}
               if driver is not None else {}),
        },
        "cg_iters": {"max": int(it_np.max()), "mean_of_max": float(it_max.mean()),
                     "min": int(it_np.min())},
        "true_relres_max": relres_max,
        "roofline": roof,
        "wall_s_timed": round(wall, 4),
        "bitwise_repeatable": bool(repeatable),
    }
    if args.phase_trace and kname in ("k_cg_tile", "k_cg_tilemx", "k_cg_tilesplit"):
        Xf, y, eps = inputs[0]
        rec["phase_trace_us"] = tile_phase_trace(kname, Xf, idx_d, w_d, y, r_d, eps, tol,
                                                 plan.maxit, args.prec, precond)
    if args.cpu_seconds > 0:
        uniq = problems[:1] if replay else problems
        rec["cpu_baseline"] = cpu_baseline(uniq, tol, args.cpu_seconds, args.precond,
                                           columns=4 if adv else None, mode=args.mode,
                                           gpu_out=gen_out[0].double().cpu().numpy())
    print(json.dumps(rec), flush=True)


def batched_solve_bytes(p, it, members) -> float:
    """Bytes one problem of the batched CG launch moves through its workgroups
    (L2 serves most of them), FP32.  Groups of four members: a first pass over S
    and r, then `it` steps, each reading S once per group and r, p and diag(R), and
    writing r and p.  One member a workgroup: S, r, p and diag(R) per member."""
    m, N = p.m, p.N
    if members == 4:
        groups = (N + 3) // 4
        return 4.0 * groups * m * ((it + 1) * (N + 1) + 4 * (4 * it + 1))
    return 4.0 * N * m * ((it + 1) * (N + 1) + 4 * it + 1)


def batched_solve_flops(p, it) -> float:
    """Operations of one problem's solve: S^T d, then two S-products and the vector
    updates a step for every member."""
    m, N = p.m, p.N
    return 2.0 * m * N * N + it * (4.0 * m * N * N + 12.0 * m * N)


def bench_batched(args):
    import torch

    import workloads as W
    from paper_2606_19224_amd import binding

    dev = torch.device("cuda:0")
    K, Wm = args.steps, args.warmup
    t0 = time.perf_counter()
    probs = W.config4(count=args.count)
    print(f"generated {len(probs)} filters in {time.perf_counter() - t0:.1f} s", file=sys.stderr,
          flush=True)
    t = lambda a, d=torch.float32: torch.as_tensor(np.ascontiguousarray(a), dtype=d, device=dev)
    dev_probs = [{"Xf": t(p.Xf), "idx": t(p.idx, torch.int32), "w": t(p.w), "y": t(p.y),
                  "r": t(p.r), "eps": t(p.eps)} for p in probs]
    # rows per gather / update entry from the autotuned table (defaults where it has none)
    from paper_2606_19224_amd import autotune
    table = autotune.load_table()
    b = binding.Batch(dev_probs, prec="fp32", tiles="auto")
    status, stats = b.run(tol=1e-6, maxit=1000, stats=True)
    torch.cuda.synchronize()
    eager = [o.clone() for o in b.outs]
    it_max = np.array([s["iters_max"] for s in stats])
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        b.run(tol=1e-6, maxit=1000, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for _ in range(Wm):
        g.replay()
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(K)]
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for i in range(K):
        evs[i][0].record()
        g.replay()
        evs[i][1].record()
    stop.record()
    torch.cuda.synchronize()
    ms_total = start.elapsed_time(stop)
    per_ms = np.array([a.elapsed_time(c) for a, c in evs])
    repeatable = all(torch.equal(x, y) for x, y in zip(eager, b.outs))
    # the CG launch alone (the dominant kernel), bracketed by the library's
    # profiling events on the launch stream, over as many eager runs
    kev = [binding.EventPair() for _ in range(K)]
    for i in range(K):
        b.run(tol=1e-6, maxit=1000, events=kev[i])
    torch.cuda.synchronize()
    solve_ms = np.array([e.elapsed_ms() for e in kev])
    nprob = len(probs)
    value = K * nprob / (ms_total / 1e3)
    members = int(b.plan.members)
    bytes_alg = sum(batched_solve_bytes(p, int(i), members) for p, i in zip(probs, it_max))
    flops_alg = sum(batched_solve_flops(p, int(i)) for p, i in zip(probs, it_max))
    tflops = flops_alg / (solve_ms.mean() / 1e3) / 1e12
    kernel = ("k_bm_solve (one workgroup per four members of every filter, both S-products on "
              "the 4x4x1 MFMA); the step also runs k_bm_gather and k_bcol_update" if members == 4
              else "k_bcol_solve<float> (one workgroup per member of every filter, S-products on "
              "the VALU); the step also runs k_bcol_gather and k_bcol_update")
    traffic = measured_traffic("k_bm_solve") if members == 4 and args.count == 256 else None
    # the measured HBM bytes where there are any, else the operations (the vector ALUs
    # have the matrix cores' FP32 rate); the larger share of its peak bounds the launch
    gbs = traffic / (solve_ms.mean() / 1e3) / 1e9 if traffic else 0.0
    if gbs / HBM_PEAK_GBS > tflops / FP32_MFMA_PEAK_TFLOPS:
        bound = {"bound": "hbm", "achieved": round(gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                 "frac": round(gbs / HBM_PEAK_GBS, 5)}
    else:
        bound = {"bound": "mfma", "achieved": round(tflops, 4), "peak": FP32_MFMA_PEAK_TFLOPS,
                 "unit": "TFLOP/s", "frac": round(tflops / FP32_MFMA_PEAK_TFLOPS, 5)}
    rec = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "analyses/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": Wm,
        "ms_per_step": round(ms_total / K, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": f"{nprob} independent Lorenz-96 filters, n = 4*U{{256..8192}}, m = n/4 "
                        "random observed variables, N in {16,32,64}, R=I, stochastic EnKF, FP32 "
                        "CG to rel. residual 1e-6 per member, gather + CG + update launches "
                        "captured once as a HIP graph; one step = one replay",
            "filters": nprob, "sum_n": int(sum(p.n for p in probs)),
            "sum_m": int(sum(p.m for p in probs)),
            "tiles": ("autotuned table " + os.path.relpath(autotune.table_path(), ROOT)
                      if table else "library defaults (no tuned table)"),
            "tile_choices": sorted({f"{g}/{u}" for g, u in b.tiles}),
        },
        "cg_iters": {"max": int(it_max.max()), "mean_of_max": float(it_max.mean()),
                     "min_of_max": int(it_max.min())},
        "roofline": {
            **bound,
            "kernel": kernel,
            "traffic": traffic,
            "avg_launch_us": round(solve_ms.mean() * 1e3, 2),
            "alg_flops_per_launch": float(flops_alg),
            "achieved_tflops": round(tflops, 4),
            "bytes_through_workgroups_per_launch": float(bytes_alg),
            "limiter": ("r and p of every member through HBM, S from L2, and each wave's tile in "
                        "series: load, first product, vector updates, second product"),
            "graph_replay_avg_us": round(per_ms.mean() * 1e3, 2),
        },
        "graph_replays_bitwise_equal_eager": bool(repeatable),
        "status": int(status),
    }
    if args.cpu_seconds > 0:
        # the filters in order, each one whole analysis of that filter
        rec["cpu_baseline"] = cpu_baseline(probs, 1e-6, args.cpu_seconds,
                                           gpu_out=b.outs[0].double().cpu().numpy())
    print(json.dumps(rec), flush=True)


def bench_warmstart(args):
    """Learned warm start on the Lorenz-96 twin experiment: pairs from cycles
    with seeds 1-4 (the first 20000 of 25600), training on the GPU, then K
    held-out analyses (seed 5) timed for the zero start, the learned start
    (network inference included) and the Jacobi start."""
    import torch

    import workloads as W
    from paper_2606_19224_amd import binding
    from paper_2606_19224_amd import warmstart as WS

    dev = torch.device("cuda:0")
    t = lambda a, d=torch.float32: torch.as_tensor(np.ascontiguousarray(a), dtype=d, device=dev)
    net = binding.WarmStartNet(seed=0)
    col = WS.PairCollector(net)
    t0 = time.perf_counter()
    idx_d = w_d = r_d = None
    for seed in (1, 2, 3, 4):
        cyc = W.L96Cycler(seed=seed)
        if idx_d is None:
            idx_d, w_d, r_d = t(cyc.idx, torch.int32), t(cyc.w), t(cyc.r)

        def analyse(p):
            out = col.add(t(p.Xf), idx_d, w_d, t(p.y), r_d, t(p.eps))
            return out["Xa"].double().cpu().numpy()

        for _ in range(args.train_cycles):
            cyc.step(analyse)
    feat, target = col.tensors(count=20000)
    torch.cuda.synchronize()
    t_pairs = time.perf_counter() - t0
    print(f"generated {feat.shape[0]} pairs in {t_pairs:.1f} s", file=sys.stderr, flush=True)
    t0 = time.perf_counter()
    hist = WS.train(net, feat, target, epochs=args.epochs, batch=64, lr=1e-3)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    print(f"trained {args.epochs} epochs in {t_train:.1f} s, losses {hist}", file=sys.stderr,
          flush=True)
    del feat, target, col

    # held-out cycles (seed 5), driven by zero-start analyses
    K, Wm = args.steps, args.warmup
    cyc = W.L96Cycler(seed=5)
    n, m, N, k = cyc.n, cyc.idx.shape[0], cyc.N, 1
    inputs = []

    def drive(p):
        Xf, y, eps = t(p.Xf), t(p.y), t(p.eps)
        out = binding.analysis(Xf, idx_d, w_d, y, r_d, eps, tol=1e-6, maxit=1000, prec="fp32",
                               stats=False)
        inputs.append((Xf, y, eps))
        return out["Xa"].double().cpu().numpy()

    for _ in range(K + Wm):
        cyc.step(drive)
    plan0 = binding.Plan(n, m, N, k, prec="fp32", tol=1e-6, maxit=1000, device=dev)
    planw = binding.Plan(n, m, N, k, prec="fp32", tol=1e-6, maxit=1000, device=dev,
                         fallback_on_stall=True)
    out = torch.empty((n, N), dtype=torch.float32, device=dev)
    z0 = torch.empty((m, N), dtype=torch.float32, device=dev)

    def run(kind, X):
        Xf, y, eps = X
        if kind == "zero":
            plan0(Xf, idx_d, w_d, y, r_d, eps, out)
            return plan0.iters
        if kind == "learned":
            net.predict_z0(Xf, idx_d, w_d, y, r_d, eps, out=z0)
        else:
            f, s = net.features(Xf, idx_d, w_d, y, r_d, eps)
            WS.jacobi_z0(net, f, s, out=z0)
        planw(Xf, idx_d, w_d, y, r_d, eps, out, z0=z0)
        return planw.iters

    res = {}
    for kind in ("zero", "learned", "jacobi"):
        for i in range(Wm):
            run(kind, inputs[K + i])
        torch.cuda.synchronize()
        its = []
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for i in range(K):
            its.append(run(kind, inputs[i]).clone())
        stop.record()
        torch.cuda.synchronize()
        ms = start.elapsed_time(stop)
        it = torch.stack(its).cpu().numpy()
        res[kind] = {"analyses_per_s": round(K / (ms / 1e3), 3), "ms_per_step": round(ms / K, 5),
                     "iters_mean": round(float(it.mean()), 3),
                     "iters_max_mean": round(float(it.max(axis=1).mean()), 3)}
    # the network inference alone (rows pass + fused network), HIP events around each call
    ev0, ev1 = binding.HipEvent(), binding.HipEvent()
    inf_ms = []
    for i in range(K):
        Xf, y, eps = inputs[i]
        ev0.record()
        net.predict_z0(Xf, idx_d, w_d, y, r_d, eps, out=z0)
        ev1.record()
        inf_ms.append(binding.HipEvent.elapsed_ms(ev0.ev, ev1.ev))
    inf_s = float(np.mean(inf_ms)) / 1e3
    # useful flops of the four layers: 2 * C_in * C_out * 5 taps per position and member
    net_flops = 2.0 * 5 * (3 * 64 + 64 * 64 + 64 * 64 + 64 * 1) * m * N
    # stall fallbacks of the learned start (one extra pass with statistics)
    nfb = 0
    for i in range(K):
        Xf, y, eps = inputs[i]
        net.predict_z0(Xf, idx_d, w_d, y, r_d, eps, out=z0)
        st = binding.analysis(Xf, idx_d, w_d, y, r_d, eps, tol=1e-6, maxit=1000, prec="fp32",
                              z0=z0, fallback_on_stall=True)["stats"]
        nfb += st["n_fallbacks"]
    rec = {
        "metric": METRIC,
        "value": res["learned"]["analyses_per_s"],
        "unit": "analyses/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": Wm,
        "ms_per_step": res["learned"]["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": "learned warm start on the Lorenz-96 twin experiment n=4096 F=8, m=2048, "
                        "N=64, R=0.5I: 4-layer conv1d net (kernel 5, 64 channels, BF16 MFMA) "
                        "trained on the GPU on 20000 (innovation, converged z) pairs from seeds "
                        "1-4, evaluated on held-out seed-5 cycles; value = analyses/s with the "
                        "learned start, network inference included",
            "train_pairs": 20000, "epochs": args.epochs,
        },
        "zero_start": res["zero"],
        "learned_start": res["learned"],
        "jacobi_start": res["jacobi"],
        "learned_fallback_rate": round(nfb / (K * N), 4),
        "roofline": {
            "bound": "mfma",
            "kernel": "warm-start inference per analysis: k_feat_rows2 + k_infer<128> (fused "
                      "4-layer network, BF16 16x16x32 MFMA, FP32 accumulation)",
            "achieved": round(net_flops / inf_s / 1e12, 2),
            "peak": 2500.0,
            "unit": "TFLOP/s",
            "frac": round(net_flops / inf_s / 1e12 / 2500.0, 5),
            "traffic": None,
            "avg_launch_us": round(inf_s * 1e6, 2),
            "alg_flops_per_launch": net_flops,
        },
        "training": {"pairs_s": round(t_pairs, 2), "train_s": round(t_train, 2),
                     "loss_first_epoch": hist[0], "loss_last_epoch": hist[-1]},
    }
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()

"""Benchmark: A + A^H throughput and FISTA time-to-accuracy on one MI355X.

One step = one FISTA iteration of the whole hot path on the 32 x 32 C-scan
workload (per-position bins): forward operator with the residual epilogue,
adjoint operator, fused soft-threshold / momentum update and the FP64
reductions of the objective, residual and stopping statistics.  The reported
value is the A + A^H throughput in algorithmic GFLOP/s (8 flops per complex
multiply-accumulate of the windowed direct sum, selected bins only), with the
inputs resident in HBM.

Prints ONE JSON line.  Extra fields: the dominant kernel's roofline, the FP64
oracle timed on host cores ("cpu_baseline", with a structured FP64 baseline of
one BLAS complex GEMM per lateral offset beside it), the FISTA time to a
relative error of 1e-2, and per-kernel timings.

    python bench.py [--steps K] [--warmup W] [--gpus 1]
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

METRIC = "A+A^H GFLOP/s & FISTA time to 1e-2 rel error: FP32 plain vs BF16/learned"
PEAK_FP32_MFMA = 157.3e12
PEAK_BF16_MFMA = 2.5e15
PEAK_HBM = 8e12
# VALU issue model of the phasor path: one wave64 instruction per SIMD every 4
# cycles (256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz = 39.3e12 lane slots/s), and a
# (term, bin) pair needs at least 9 instructions: the phase product, a convert,
# a scale, sin, cos and 4 FMAs (the counters show the transcendentals taking no
# more issue slots than the others)
PHASOR_SLOTS_PER_TERM = 9
PEAK_PHASOR_TERMS = 256 * 4 * 16 * 2.4e9 / PHASOR_SLOTS_PER_TERM

# HBM bytes per launch of the dominant kernels, from two rocprofv3 counter runs
# (FETCH_SIZE, then WRITE_SIZE, each scaled by what the same counter reads for a
# 256 MiB device copy), keyed by workload, kernel and tiling (split partials
# are part of the traffic).  Each entry holds the SHA-256 prefix of the kernel
# source it was measured on; a changed source or another tiling reports null.
TRAFFIC = {
    # 32 x 32 C-scan, FP32 union-GEMM, shipped tiling (profiles/cscan32_fp32_gemm.md)
    "cscan32/gemm/forward/fs12-zs8-nw4-np4-zc16": {"bytes": 82.529e6, "sha": "99b98f25ae46cafa"},
    "cscan32/gemm/adjoint/as32-np4-kc8-nw4": {"bytes": 79.707e6, "sha": "99b98f25ae46cafa"},
    # 64 x 64 C-scan (profiles/cscan64_fp32_gemm.md)
    "cscan64/gemm/forward/fs6-zs8-nw4-np4-zc16": {"bytes": 219.210e6, "sha": "99b98f25ae46cafa"},
    "cscan64/gemm/adjoint/as16-np4-kc16-nw4": {"bytes": 277.596e6, "sha": "99b98f25ae46cafa"},
    # transform-domain contraction (profiles/cscan32_fp32_transform.md, cscan64_fp32_transform.md):
    # the table once plus the transform rows in and out
    "cscan32/transform/forward/fs1-zs1-nw1-np0-zc0": {"bytes": 82.259e6, "sha": "59811daac8b9428b"},
    "cscan32/transform/adjoint/as1-np0-kc0-nw0": {"bytes": 91.067e6, "sha": "59811daac8b9428b"},
    "cscan64/transform/forward/fs1-zs1-nw1-np0-zc0": {"bytes": 484.323e6, "sha": "59811daac8b9428b"},
    "cscan64/transform/adjoint/as1-np0-kc0-nw0": {"bytes": 530.794e6, "sha": "59811daac8b9428b"},
    # the same with the BF16 table (profiles/cscan32_bf16_transform.md, cscan64_bf16_transform.md)
    "cscan32/transform-bf16/adjoint/as1-np0-kc0-nw0": {"bytes": 50.911e6, "sha": "59811daac8b9428b"},
    "cscan32/transform-bf16/forward/fs1-zs1-nw1-np0-zc0": {"bytes": 46.163e6, "sha": "59811daac8b9428b"},
    "cscan64/transform-bf16/adjoint/as1-np0-kc0-nw0": {"bytes": 278.595e6, "sha": "59811daac8b9428b"},
    "cscan64/transform-bf16/forward/fs1-zs1-nw1-np0-zc0": {"bytes": 258.679e6, "sha": "59811daac8b9428b"},
    # BF16 GEMMs with phasor tables (profiles/cscan32_bf16_gemm.md, cscan64_bf16_gemm.md):
    # mostly re-reads of the table tiles, one per workgroup and offset (the
    # tables, 170 MB at 32 x 32, sit in the last-level cache); the 32 x 32
    # forward is two launches (full bin tiles, then the short last one)
    "cscan32/gemm-bf16/forward/fs12-zs8-wr1": {"bytes": 285.967e6, "sha": "6a80aa6837cf854b"},
    "cscan32/gemm-bf16/adjoint/as12-wr1-nz2": {"bytes": 803.656e6, "sha": "6a80aa6837cf854b"},
    "cscan64/gemm-bf16/forward/fs2-zs8-wr1": {"bytes": 509.592e6, "sha": "6a80aa6837cf854b"},
    "cscan64/gemm-bf16/adjoint/as3-wr1-nz2": {"bytes": 681.340e6, "sha": "6a80aa6837cf854b"},
}
TRAFFIC_SRC = {"gemm": "paper_2012_04534_amd/csrc/gemm_f32.hip",
               "transform": "paper_2012_04534_amd/csrc/fft.hip",
               "transform-bf16": "paper_2012_04534_amd/csrc/fft.hip",
               "gemm-bf16": "paper_2012_04534_amd/csrc/gemm_bf16.hip",
               "phasor": "paper_2012_04534_amd/csrc/phasor.hip"}


def source_sha(rel):
    import hashlib
    with open(os.path.join(ROOT, rel), "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def tiling_key(info, direction):
    if info["dtype"] == 1 and info["algo"] == 1:   # BF16 GEMM: d_y and depth splits, wave rows
        return ("as%d-wr%d-nz%d" % (info["adj_split"], info["adj_rows"], info["adj_tile"]) if direction == "adjoint"
                else "fs%d-zs%d-wr%d" % (info["fwd_split"], info["fwd_zsplit"], info["fwd_rows"]))
    if direction == "adjoint":
        return "as%d-np%d-kc%d-nw%d" % (info["adj_split"], info["adj_tile"], info["adj_chunk"], info["adj_waves"])
    return "fs%d-zs%d-nw%d-np%d-zc%d" % (info["fwd_split"], info["fwd_zsplit"], info["fwd_waves"],
                                         info["fwd_tile"], info["fwd_chunk"])


def traffic_bytes(workload, algo_name, direction, info):
    e = TRAFFIC.get("%s/%s/%s/%s" % (workload, algo_name, direction, tiling_key(info, direction)))
    if e is None or source_sha(TRAFFIC_SRC[algo_name]) != e["sha"]:
        return None
    return int(e["bytes"])


def window_terms(g, bins, per_pos):
    """Algorithmic complex MACs of one apply (voxels inside each window x bins)."""
    nx, ny = g["nx"], g["ny"]
    wx = nx - 1 if g["win_x"] < 0 else min(g["win_x"], nx - 1)
    wy = ny - 1 if g["win_y"] < 0 else min(g["win_y"], ny - 1)
    cy = np.array([min(p + wy, ny - 1) - max(p - wy, 0) + 1 for p in range(ny)])
    cx = np.array([min(p + wx, nx - 1) - max(p - wx, 0) + 1 for p in range(nx)])
    return int(cy.sum()) * int(cx.sum()) * bins.shape[-1] * g["nz"]


def mirror_share(g):
    """Offset classes (|d_x|, |d_y|) over window voxels: the FP32 GEMMs add the
    voxels at mirrored offsets first and form one product for them."""
    def axis(n, win):
        w = n - 1 if win < 0 else min(win, n - 1)
        p = np.arange(n)
        voxels = np.minimum(p + w, n - 1) - np.maximum(p - w, 0) + 1
        return np.minimum(w, np.maximum(p, n - 1 - p)).sum() + n, voxels.sum()
    (fx, vx), (fy, vy) = axis(g["nx"], g["win_x"]), axis(g["ny"], g["win_y"])
    return float(fx * fy) / float(vx * vy)


def table_bytes(g, info, entry):
    """The transform contraction's stored table: (ly/2+1)(lx/2+1) entries, with both
    axes alike (where it is symmetric in them) one of each pair, by nz depths and the
    union's bins padded to even, `entry` bytes each."""
    nox, noy = [(g["n" + a] + info["win_" + a]) // 2 + 1 for a in "xy"]
    alike = g["nx"] == g["ny"] and info["win_x"] == info["win_y"] and g["dx"] == g["dy"]
    entries = nox * (nox + 1) // 2 if alike else nox * noy
    return entries * g["nz"] * (info["union_size"] + info["union_size"] % 2) * entry


def operator_outputs(ufss, W, g, w, bins, dev, tcfg):
    """A x and A^H y of every operator form at the full workload, for the
    inputs the CPU leg samples (x = CN seed 5, y = CN seed 6), on the host."""
    import torch
    x = torch.from_numpy(W.cn((g["ny"], g["nx"], g["nz"]), 5).astype(np.complex64)).to(dev)
    y = torch.from_numpy(W.cn((g["ny"], g["nx"], w["m"]), 6).astype(np.complex64)).to(dev)
    forms = [("gemm_f32", ufss.F32, ufss.ALGO_GEMM), ("gemm_bf16", ufss.BF16, ufss.ALGO_GEMM),
             ("transform_f32", ufss.F32, ufss.ALGO_FFT), ("transform_bf16", ufss.BF16, ufss.ALGO_FFT)]
    if w["per_position"]:
        forms.append(("phasor_f32", ufss.F32, ufss.ALGO_PHASOR))
    out = {}
    for name, dt, algo in forms:
        p = ufss.Plan(g, w["m"], w["per_position"], bins, dtype=dt, algo=algo)
        if algo == ufss.ALGO_GEMM:
            autotune(ufss, p, tcfg)
        yo = torch.empty_like(y)
        xo = torch.empty_like(x)
        ufss.ufss_forward(p, x, yo)
        ufss.ufss_adjoint(p, y, xo)
        out[name] = (yo.cpu().numpy(), xo.cpu().numpy())
        p.close()
    return out


def cpu_baseline(w, bins, seconds=12.0, gpu_outputs=None):
    """Time the FP64 oracle on a bounded sample of the same workload; the
    sampled rows and columns also give each GPU operator form's error against
    the oracle (max |gpu - oracle| / max |oracle| over the sample)."""
    from oracle import operator as O
    from paper_2012_04534_amd import workloads as W
    try:
        from threadpoolctl import threadpool_limits
        limit = threadpool_limits(limits=1)
    except Exception:  # pragma: no cover
        limit = None
    g = w["geom"]
    x = W.cn((g["ny"], g["nx"], g["nz"]), 5)
    y = W.cn((g["ny"], g["nx"], w["m"]), 6)
    rng = np.random.default_rng(0)
    wx = g["nx"] - 1 if g["win_x"] < 0 else g["win_x"]
    wy = g["ny"] - 1 if g["win_y"] < 0 else g["win_y"]
    cmac, n_fwd, n_adj = 0, 0, 0
    gerr = {k: [0.0, 0.0, 0.0, 0.0] for k in (gpu_outputs or {})}   # fwd num, den, adj num, den
    t_gpu_cmp = 0.0
    t0 = time.perf_counter()
    while time.perf_counter() - t0 - t_gpu_cmp < seconds:
        py, px = int(rng.integers(g["ny"])), int(rng.integers(g["nx"]))
        row = O.apply_A_at(g, bins, x, py, px)
        tc = time.perf_counter()
        for k, (yg, _) in (gpu_outputs or {}).items():
            gerr[k][0] = max(gerr[k][0], float(np.abs(yg[py, px] - row).max()))
            gerr[k][1] = max(gerr[k][1], float(np.abs(row).max()))
        t_gpu_cmp += time.perf_counter() - tc
        nvx = min(px + wx, g["nx"] - 1) - max(px - wx, 0) + 1
        nvy = min(py + wy, g["ny"] - 1) - max(py - wy, 0) + 1
        cmac += nvx * nvy * g["nz"] * w["m"]
        n_fwd += 1
        vy, vx = int(rng.integers(g["ny"])), int(rng.integers(g["nx"]))
        col = O.apply_AH_at(g, bins, y, vy, vx)
        tc = time.perf_counter()
        for k, (_, xg) in (gpu_outputs or {}).items():
            gerr[k][2] = max(gerr[k][2], float(np.abs(xg[vy, vx] - col).max()))
            gerr[k][3] = max(gerr[k][3], float(np.abs(col).max()))
        t_gpu_cmp += time.perf_counter() - tc
        npx = min(vx + wx, g["nx"] - 1) - max(vx - wx, 0) + 1
        npy = min(vy + wy, g["ny"] - 1) - max(vy - wy, 0) + 1
        cmac += npx * npy * g["nz"] * w["m"]
        n_adj += 1
    dt = time.perf_counter() - t0 - t_gpu_cmp
    if limit is not None:
        limit.unregister()
    host = {"affinity_cpus": len(os.sched_getaffinity(0))}
    try:
        with open("/proc/cpuinfo") as f:
            host["cpu_model"] = next(ln.split(":", 1)[1].strip() for ln in f if ln.startswith("model name"))
    except (OSError, StopIteration):
        pass
    try:
        cfg = np.show_config(mode="dicts")
        host["blas"] = cfg["Build Dependencies"]["blas"]["name"]
    except Exception:  # pragma: no cover
        pass
    return {
        "value": round(8.0 * cmac / dt / 1e9, 4), "unit": "GFLOP/s", "cores": 1,
        "kind": "oracle", "host": host,
        "sample": "%d rows of A x (one scan position each) and %d columns of A^H y (one voxel "
                  "column each) at the full 32x32 C-scan geometry, FP64 numpy direct sum, "
                  "1 BLAS thread, %.1f s" % (n_fwd, n_adj, dt),
        "gpu_operator_error_vs_oracle": {
            k: {"forward": v[0] / v[1], "adjoint": v[2] / v[3]} for k, v in gerr.items() if v[1] > 0},
    }


def window_offsets(g):
    """Lateral offsets d = p - v inside the aperture window, (d_y, d_x) pairs."""
    wx = g["nx"] - 1 if g["win_x"] < 0 else min(g["win_x"], g["nx"] - 1)
    wy = g["ny"] - 1 if g["win_y"] < 0 else min(g["win_y"], g["ny"] - 1)
    return [(dy, dx) for dy in range(-wy, wy + 1) for dx in range(-wx, wx + 1)]


def structured_plan(g, bins, offsets):
    """Tables of the structured CPU baseline: for each offset d the phasors
    P_d[z][k] = g(d, z) exp(-j 2 pi f_k (tau(d, z) - t0)) over the union of the
    selected bins (FP64), H_k on that union and each selection's union index."""
    from oracle import geometry as G
    bins = np.asarray(bins)
    ub = np.unique(bins)
    f = G.bin_freq(g, ub)
    z = G.depth(g, np.arange(g["nz"]))
    t0 = G.t0(g)
    tabs = {}
    for dy, dx in offsets:
        ddx, ddy = dx * g["dx"], dy * g["dy"]
        delay = G.tau(g, ddx, ddy, z) - t0
        tabs[(dy, dx)] = np.exp(-2j * math.pi * np.outer(delay, f)) * G.directivity(g, ddx, ddy, z)[:, None]
    return ub, G.pulse_spectrum(g, ub), tabs, np.searchsorted(ub, bins)


def _shift_ranges(n_y, n_x, dy, dx):
    return max(0, dy), min(n_y, n_y + dy), max(0, dx), min(n_x, n_x + dx)


def structured_forward(plan, x, offsets):
    """y = A x as one BLAS GEMM per lateral offset (positions p = v + d):
    Y[p][k] += sum_z x[p - d][z] P_d[z][k], then selection and H_k."""
    ub, H, tabs, sel = plan
    n_y, n_x, n_z = x.shape
    Y = np.zeros((n_y, n_x, len(ub)), complex)
    for dy, dx in offsets:
        y0, y1, x0, x1 = _shift_ranges(n_y, n_x, dy, dx)
        if y0 >= y1 or x0 >= x1:
            continue
        xs = x[y0 - dy:y1 - dy, x0 - dx:x1 - dx, :].reshape(-1, n_z)
        Y[y0:y1, x0:x1, :] += (xs @ tabs[(dy, dx)]).reshape(y1 - y0, x1 - x0, -1)
    if sel.ndim == 1:
        return Y[:, :, sel] * H[sel]
    return np.take_along_axis(Y, sel, axis=2) * H[sel]


def structured_adjoint(plan, y, offsets, n_z):
    """x = A^H y as one BLAS GEMM per lateral offset (voxels v = p - d):
    x[v][z] += sum_k conj(P_d[z][k]) (H r)[v + d][k]."""
    ub, H, tabs, sel = plan
    n_y, n_x, _ = y.shape
    R = np.zeros((n_y, n_x, len(ub)), complex)
    if sel.ndim == 1:
        R[:, :, sel] = y * H[sel]
    else:
        np.put_along_axis(R, sel, y * H[sel], axis=2)
    X = np.zeros((n_y, n_x, n_z), complex)
    for dy, dx in offsets:
        y0, y1, x0, x1 = _shift_ranges(n_y, n_x, dy, dx)
        if y0 >= y1 or x0 >= x1:
            continue
        rs = R[y0:y1, x0:x1, :].reshape(-1, len(ub))
        X[y0 - dy:y1 - dy, x0 - dx:x1 - dx, :] += np.conj(np.conj(rs) @ tabs[(dy, dx)].T).reshape(
            y1 - y0, x1 - x0, n_z)
    return X


def _offset_terms(g, m, offsets):
    """Algorithmic complex MACs of the given offsets (in-grid positions x N_z x M)."""
    t = 0
    for dy, dx in offsets:
        t += max(0, g["ny"] - abs(dy)) * max(0, g["nx"] - abs(dx))
    return t * g["nz"] * m


def structured_rate(g, bins, m, offsets, threads):
    """FP64 A + A^H rate of the structured baseline over the given offsets."""
    from threadpoolctl import threadpool_limits
    from paper_2012_04534_amd import workloads as W
    with threadpool_limits(limits=threads):
        t0 = time.perf_counter()
        plan = structured_plan(g, bins, offsets)
        t_plan = time.perf_counter() - t0
        x = W.cn((g["ny"], g["nx"], g["nz"]), 5)
        y = W.cn((g["ny"], g["nx"], m), 6)
        t0 = time.perf_counter()
        structured_forward(plan, x, offsets)
        structured_adjoint(plan, y, offsets, g["nz"])
        dt = time.perf_counter() - t0
    cmac = 2 * _offset_terms(g, m, offsets)
    return {"value": round(8.0 * cmac / dt / 1e9, 3), "unit": "GFLOP/s", "cores": threads,
            "apply_s": round(dt, 3), "plan_s": round(t_plan, 3), "offsets": len(offsets)}


def cpu_structured(w, bins):
    """The structured FP64 CPU baseline: A and A^H as one complex GEMM per
    lateral offset (numpy / BLAS), phasor tables built once per plan; on all
    host cores of this process (at most 16) at the full 32 x 32 C-scan, on one
    core over every 16th offset, and on all cores over 48 offsets of the 64 x 64
    C-scan (shared bins, window +-16)."""
    from paper_2012_04534_amd import workloads as W
    threads = max(1, min(16, len(os.sched_getaffinity(0))))
    g = w["geom"]
    offs = window_offsets(g)
    out = structured_rate(g, bins, w["m"], offs, threads)
    out["kind"] = "structured FP64 CPU baseline (one BLAS complex GEMM per lateral offset)"
    out["sample"] = "one A and one A^H at the full 32x32 C-scan (all %d offsets)" % len(offs)
    one = structured_rate(g, bins, w["m"], offs[::16], 1)
    one["sample"] = "one A and one A^H over every 16th offset of the 32x32 C-scan"
    out["single_core"] = one
    from oracle import select as S
    w3 = W.workload("cscan64")
    g3 = w3["geom"]
    b3 = S.select_freqs(g3, w3["m"], w3["per_position"], w3["seed"])
    o3 = window_offsets(g3)
    o3 = o3[::max(1, len(o3) // 48)][:48]
    c3 = structured_rate(g3, b3, w3["m"], o3, threads)
    c3["sample"] = "one A and one A^H over 48 of the %d offsets of the 64x64 C-scan" % len(window_offsets(g3))
    out["cscan64_sample"] = c3
    # FISTA at this rate: K iterations of one A and one A^H each (extrapolated)
    out["fista_%d_extrapolated_s" % w["iters"]] = round(w["iters"] * out["apply_s"], 2)
    return out


def cpu_oracle_fista_bscan(gpu=None):
    """The plain oracle's FISTA (200 iterations, dense FP64 A, one core) on the
    32-position B-scan workload, with L from its eigenvalues and the lambda rule;
    with the GPU's run (its iterate, L and lambda) also the oracle's FISTA at the
    GPU's L and lambda and the GPU iterate's error against it."""
    from threadpoolctl import threadpool_limits
    from oracle import operator as O
    from oracle import select as S
    from oracle import solver as V
    from paper_2012_04534_amd import workloads as W
    w = W.workload("bscan32")
    g = w["geom"]
    bins = S.select_freqs(g, w["m"], w["per_position"], w["seed"])
    y = W.cn((g["ny"], g["nx"], w["m"]), 7).reshape(-1)
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        A = O.dense_A(g, bins)
        L = V.lipschitz_dense(A)
        t_setup = time.perf_counter() - t0
        lam = V.lambda_rule(lambda v: A.conj().T @ v, y, w["mu"])
        t0 = time.perf_counter()
        V.fista(lambda v: A @ v, lambda v: A.conj().T @ v, y, lam, L, w["iters"])
        dt = time.perf_counter() - t0
        out = {"iters": w["iters"], "solve_s": round(dt, 3), "setup_s": round(t_setup, 3), "cores": 1,
               "sample": "the 32-position B-scan workload in full: dense FP64 A (%d x %d), numpy, "
                         "one BLAS thread" % A.shape}
        if gpu is not None:
            xg, Lg, lamg = gpu
            a, _ = V.fista(lambda v: A @ v, lambda v: A.conj().T @ v, y, lamg, Lg, w["iters"])
            out["gpu_fista_iterate_error_vs_oracle"] = float(np.linalg.norm(xg - a) / np.linalg.norm(a))
            out["gpu_L_over_1.01_eigvalsh"] = float(Lg / (1.01 * L))
    return out


WEIGHTS = os.path.join(ROOT, "paper_2012_04534_amd", "weights", "unrolled_cscan32_s16c8.bin")
# Tilings the autotuner chose on MI355X for the workloads timed here (read-only;
# --retune times the candidates again, --tune-cache uses another file).
SHIPPED_TUNING = os.path.join(ROOT, "paper_2012_04534_amd", "tuning_gfx950.json")


def autotune(ufss, plan, cfg):
    """Tiling from the cache of `cfg` (path, read, write), else by timing."""
    path, read, write = cfg
    return ufss.ufss_autotune(plan, path, read, write)


LEVELS = [0.3, 0.1, 0.03, 0.01]


def level_iters(err, levels=LEVELS):
    """First iteration (1-based) whose error is at or below each level (None: not reached)."""
    out = []
    for lev in levels:
        hit = np.flatnonzero(np.asarray(err) <= lev)
        out.append(int(hit[0]) + 1 if hit.size else None)
    return out


def timed_fista(ufss, plan, y, lam, L, k, x, a_ref=None, x0=None):
    """Wall time of ONE FISTA run of k iterations (from zero, or from x0) with
    its per-iteration FP64 statistics (and the error against a_ref), GPU
    synchronised on both sides; returns (seconds, stats)."""
    import torch
    if x0 is None:
        x.zero_()
    else:
        x.copy_(x0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    st = ufss.ufss_fista(plan, y, lam, L, k, x, a_ref=a_ref)
    torch.cuda.synchronize()
    return time.perf_counter() - t0, st


def levels_wall_time(ufss, plan, y, lam, L, x, a_ref, iters):
    """Wall time to each level: one timed run of exactly the iterations that
    level needs (its statistics included), per level reached."""
    out = []
    for k in iters:
        out.append(None if k is None else round(timed_fista(ufss, plan, y, lam, L, k, x, a_ref)[0], 5))
    return out


def time_to_accuracy(ufss, W, plan, g, w, bins, y, lam, L, t_l, dev, tcfg, timed_levels=None):
    """Time to relative errors 0.3 ... 1e-2 against the plain FP32 FISTA
    iterate at the workload's K (FISTA-K on the GEMM operator), for plain FP32
    and BF16 FISTA on the GEMM and on the transform operator.  Every time is
    the wall time of one run (statistics included) of the iterations the level
    needs (``timed_levels``: indices of the levels timed, default all); the
    ratios compare precisions on the same operator, at 1e-2."""
    import torch
    K = w["iters"]
    timed_levels = range(len(LEVELS)) if timed_levels is None else timed_levels
    own = None
    if plan.info()["dtype"] != ufss.F32:      # the reference and the FP32 rows need an FP32 plan
        own = plan = ufss.Plan(g, w["m"], w["per_position"], bins, dtype=ufss.F32)
        autotune(ufss, plan, tcfg)
    a_ref = torch.zeros((g["ny"], g["nx"], g["nz"]), dtype=torch.complex64, device=dev)
    ufss.ufss_fista(plan, y, lam, L, K, a_ref)
    out = {"reference": "plain FP32 FISTA iterate after %d iterations (GEMM operator)" % K,
           "timing": "wall time of one run (per-iteration statistics and error included) of the "
                     "iterations each level needs",
           "lipschitz_s": round(t_l, 4), "L": L, "lambda": lam, "levels": LEVELS}
    x = torch.zeros_like(a_ref)
    for tag, dt, algo in (("fp32", ufss.F32, None), ("fp32_transform", ufss.F32, ufss.ALGO_FFT),
                          ("bf16", ufss.BF16, ufss.ALGO_GEMM), ("bf16_transform", ufss.BF16, ufss.ALGO_FFT)):
        p = plan
        if algo is not None:
            p = ufss.Plan(g, w["m"], w["per_position"], bins, dtype=dt, algo=algo)
            if algo == ufss.ALGO_GEMM:
                autotune(ufss, p, tcfg)
        timed_fista(ufss, p, y, lam, L, 3, x, a_ref)            # warm-up
        t_all, st = timed_fista(ufss, p, y, lam, L, K, x, a_ref)
        iters = level_iters(st["err_ref"])
        it_t = [k if j in timed_levels else None for j, k in enumerate(iters)]
        out[tag] = {"s_per_iter_full_run": round(t_all / K, 6), "iters_to_level": iters,
                    "time_to_level_s": levels_wall_time(ufss, p, y, lam, L, x, a_ref, it_t),
                    "err_at_K": float(st["err_ref"][-1])}
        if p is not plan:
            p.close()
    # like for like: BF16 against FP32 on the same operator, at the 1e-2 level
    def ratio(a, b):
        ta, tb = out[a]["time_to_level_s"][-1], out[b]["time_to_level_s"][-1]
        return None if ta is None or tb is None else round(ta / tb, 2)
    out["bf16_speedup_same_operator"] = {"gemm": ratio("fp32", "bf16"),
                                         "transform": ratio("fp32_transform", "bf16_transform")}
    out["transform_vs_gemm_fp32"] = ratio("fp32", "fp32_transform")
    if own is not None:
        own.close()
    return out


def measured_problem(ufss, W, w, bins, dev, tcfg):
    """The workload's scene and noisy measurements y = A x + n (FP32 GEMM plan),
    L by power iteration on the transform plan (the same operator, cheaper) and
    lambda by the mu rule."""
    import torch
    g = w["geom"]
    plan = ufss.Plan(g, w["m"], w["per_position"], bins, dtype=ufss.F32, algo=ufss.ALGO_GEMM)
    autotune(ufss, plan, tcfg)
    x_true = W.scene(g, w["n_scat"], amp=w["amp"], seed=w["seed"], back_wall=w["back_wall"])
    xt = torch.from_numpy(x_true.astype(np.complex64)).to(dev)
    y0 = torch.empty((g["ny"], g["nx"], w["m"]), dtype=torch.complex64, device=dev)
    ufss.ufss_forward(plan, xt, y0)
    sig = W.noise_sigma(float((y0.abs() ** 2).sum().item()), y0.numel(), w["snr_db"])
    y = (y0 + sig * torch.from_numpy(W.cn(tuple(y0.shape), w["seed"] + 1).astype(np.complex64)).to(dev)).contiguous()
    pt = ufss.Plan(g, w["m"], w["per_position"], bins, algo=ufss.ALGO_FFT)
    t_l = time.perf_counter()
    L = ufss.ufss_lipschitz(pt, max_iters=200, rtol=1e-6, margin=0.01, seed=4)
    t_l = time.perf_counter() - t_l
    pt.close()
    x = torch.zeros_like(xt)
    lam = ufss.ufss_fista(plan, y, ufss.lambda_from_mu(w["mu"]), L, 1, x)["lambda"]
    return plan, y, L, lam, t_l


def learned_block(ufss, W, g, w, bins, L_gemm, dev, tcfg, n_scenes=8):
    """The learned unrolled solver against its judge (config of the learned
    solver: FISTA-200 on the same operator), on held-out evaluation scenes,
    with the residual fallback rule: per operator (transform, GEMM) the mean
    network time, its error, the fallbacks, and plain FP32 FISTA's wall time to
    the same error levels on the same scenes and operator."""
    import torch
    from paper_2012_04534_amd import learned as LN
    if not os.path.exists(WEIGHTS):
        return None
    out = {"checkpoint": os.path.relpath(WEIGHTS, ROOT), "reference": "plain FP32 FISTA-200 on the same operator",
           "eval_scenes": n_scenes, "eval_set": "held-out seeds 2005/0..%d" % (n_scenes - 1)}
    for name, algo in (("transform", ufss.ALGO_FFT), ("gemm", ufss.ALGO_GEMM)):
        plan = ufss.Plan(g, w["m"], w["per_position"], bins, algo=algo)
        if algo == ufss.ALGO_GEMM:
            autotune(ufss, plan, tcfg)
        L = L_gemm
        data = LN.make_dataset(plan, g, n_scenes, LN.EVAL_SEED, 200, L, mu=w["mu"], back_wall=w["back_wall"],
                               dev=dev)
        net = ufss.Net(plan, stages=16, channels=8, L=L, mu=w["mu"])
        ufss.ufss_unrolled_load(net, WEIGHTS)
        x = torch.zeros_like(data[0][1])
        ufss.ufss_unrolled_forward(net, data[0][0], x)         # warm-up
        r = LN.evaluate(net, plan, data, L, w["mu"])
        f_iters, f_time = [], []
        for yy, tgt, _ in data:
            lam = -w["mu"]
            timed_fista(ufss, plan, yy, lam, L, 3, x, tgt)
            _, st = timed_fista(ufss, plan, yy, lam, L, 200, x, tgt)
            it = level_iters(st["err_ref"])
            f_iters.append(it)
            f_time.append(levels_wall_time(ufss, plan, yy, lam, L, x, tgt, it))
        mean_or_none = lambda v: None if any(q is None for q in v) else float(np.mean(v))
        fista_t = [mean_or_none([row[j] for row in f_time]) for j in range(len(LEVELS))]
        t_net = float(r["time_s"].mean())
        err = float(r["err"].mean())
        reached = [lev for lev in LEVELS if err <= lev]
        row = {"net_time_s_mean": round(t_net, 5), "err_mean": err, "err_max": float(r["err"].max()),
               "fallbacks": int(r["fallback"].sum()), "fallback_time_s": float(r["t_fallback"].sum()),
               "fista_iters_to_level": [mean_or_none([row[j] for row in f_iters]) for j in range(len(LEVELS))],
               "fista_time_to_level_s": fista_t,
               "net_levels_reached": reached}
        # plain FISTA time to the finest level the network reaches, over the network's time
        if reached:
            j = LEVELS.index(reached[-1])
            row["speedup_at_finest_level_reached"] = (None if fista_t[j] is None else
                                                      round(fista_t[j] / t_net, 2))
        row["time_to_1e-2_s"] = round(t_net, 5) if err <= 1e-2 else None
        out[name] = row
        net.close()
        del data
        plan.close()
    return out


def cscan64_rates(ufss, W, dev, ev_time, tcfg):
    """A + A^H rates of the 64 x 64 precision-study workload, FP32 and BF16."""
    import torch
    w = W.workload("cscan64")
    g = w["geom"]
    bins, _ = ufss.ufss_select_freqs(g, w["m"], False, w["seed"])
    cm = window_terms(g, bins, False)
    x = torch.from_numpy(W.cn((g["ny"], g["nx"], g["nz"]), 1).astype(np.complex64)).to(dev)
    y = torch.empty((g["ny"], g["nx"], w["m"]), dtype=torch.complex64, device=dev)
    out = {"cmac_per_apply": cm}
    xo = torch.empty_like(x)          # adjoint output (the inputs stay fixed)
    for tag, dt, peak in (("fp32", ufss.F32, PEAK_FP32_MFMA), ("bf16", ufss.BF16, PEAK_BF16_MFMA)):
        p = ufss.Plan(g, w["m"], False, bins, dtype=dt)
        autotune(ufss, p, tcfg)
        tf = ev_time(lambda: ufss.ufss_forward(p, x, y), 3)
        ta = ev_time(lambda: ufss.ufss_adjoint(p, y, xo), 3)
        tfl = 16.0 * cm / ((tf + ta) * 1e-3)
        out[tag] = {"forward_ms": round(tf, 3), "adjoint_ms": round(ta, 3),
                    "a_plus_ah_tflops": round(tfl / 1e12, 2), "frac_of_mfma_peak": round(tfl / peak, 4)}
        if dt == ufss.F32:          # as the roofline's needed_frac
            out[tag]["needed_frac"] = round(tfl * 0.75 * mirror_share(g) / peak, 4)
        p.close()
    out["fp32_transform"] = transform_rates(ufss, g, w["m"], False, bins, x, y, xo, ev_time, cm)
    return out


def transform_rates(ufss, g, m, per_pos, bins, x, y, xo, ev_time, cm):
    """The transform-domain operator (UFSS_ALGO_FFT) on the same problem: apply
    times, the direct-sum-equivalent rate (the same algorithmic count as the
    GEMM rows, so the two compare as times) and its contraction kernels against
    HBM: each streams its table once."""
    p = ufss.Plan(g, m, per_pos, bins, algo=ufss.ALGO_FFT)
    tf = ev_time(lambda: ufss.ufss_forward(p, x, y), 3)
    ta = ev_time(lambda: ufss.ufss_adjoint(p, y, xo), 3)
    cf = ufss.ufss_time_kernel(p, 0, 20)
    ca = ufss.ufss_time_kernel(p, 1, 20)
    info = p.info()
    lx, ly = g["nx"] + info["win_x"], g["ny"] + info["win_y"]
    tab = table_bytes(g, info, 8)
    p.close()
    return {"forward_ms": round(tf, 4), "adjoint_ms": round(ta, 4),
            "direct_sum_equivalent_tflops": round(16.0 * cm / ((tf + ta) * 1e-3) / 1e12, 1),
            "transform_size": [ly, lx], "table_bytes": tab,
            "contraction_ms": [round(cf, 4), round(ca, 4)],
            "contraction_gbs": [round(tab / (cf * 1e-3) / 1e9, 1), round(tab / (ca * 1e-3) / 1e9, 1)],
            "contraction_frac_of_hbm": [round(tab / (cf * 1e-3) / PEAK_HBM, 3),
                                        round(tab / (ca * 1e-3) / PEAK_HBM, 3)]}


def batch_rate(ufss, W, dev, tcfg, iters=100):
    """The 64 uneven scans (FP32, tilings from the autotuner cache or a quick
    search) as one persistent batch: setup (plans, tilings, L), creation
    (lambdas, descriptors, capture and instantiation of the K-iteration graph)
    and the replay of K iterations are timed separately; beside them, the same
    scans one after another with single-scan FISTA."""
    import torch
    specs = W.batch_workload()
    plans, ys, xs, Ls, cm = [], [], [], [], 0
    path, read, write = tcfg
    t0 = time.perf_counter()
    for s in specs:
        g = s["geom"]
        _, band = ufss.ufss_select_freqs(g, 1, False, 0)
        m = min(s["m"], band)
        bins, _ = ufss.ufss_select_freqs(g, m, s["per_position"], s["seed"])
        p = ufss.Plan(g, m, s["per_position"], bins, algo=ufss.ALGO_GEMM)
        ufss.ufss_autotune(p, path, use_cache=read, write_cache=write, quick=True)
        xt = torch.from_numpy(W.scene(g, s["n_scat"], amp=s["amp"], seed=s["seed"]).astype(np.complex64)).to(dev)
        y = torch.empty((g["ny"], g["nx"], m), dtype=torch.complex64, device=dev)
        ufss.ufss_forward(p, xt, y)
        Ls.append(ufss.ufss_lipschitz(p, max_iters=30, rtol=1e-3, margin=0.05))
        plans.append(p)
        ys.append(y)
        xs.append(torch.zeros((g["ny"], g["nx"], g["nz"]), dtype=torch.complex64, device=dev))
        cm += window_terms(g, bins, s["per_position"])
    torch.cuda.synchronize()
    setup = time.perf_counter() - t0
    t0 = time.perf_counter()
    b = ufss.Batch(plans, ys, xs, [-0.1] * len(plans), Ls, iters)
    torch.cuda.synchronize()
    t_create = time.perf_counter() - t0
    b.run()                                            # first replay (warm)
    reps = []
    for _ in range(3):
        for x in xs:
            x.zero_()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, lams = b.run()
        torch.cuda.synchronize()
        reps.append(time.perf_counter() - t0)
    dt = float(np.median(reps))
    b.close()
    # the same scans one at a time (single-scan FISTA, 5 iterations each)
    k1 = 5
    t_seq = 0.0
    for p, y, x, L, lam in zip(plans, ys, xs, Ls, lams):
        x.zero_()
        ufss.ufss_fista(p, y, lam, L, 1, x)
        x.zero_()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ufss.ufss_fista(p, y, lam, L, k1, x)
        torch.cuda.synchronize()
        t_seq += time.perf_counter() - t0
    for p in plans:
        p.close()
    return {"scans": len(specs), "iters": iters, "setup_s": round(setup, 2),
            "create_capture_instantiate_s": round(t_create, 3),
            "replay_s": round(dt, 4), "replay_ms_per_iter": round(dt / iters * 1e3, 4),
            "cmac_per_apply": cm,
            "a_plus_ah_tflops_replay": round(16.0 * cm * iters / dt / 1e12, 2),
            "sequential_single_scan_ms_per_iter": round(t_seq / k1 * 1e3, 4)}


def gpu_clocks():
    """Current GPU clocks (not locked on the box), read once with rocm-smi in a
    child process; a failure is reported, never raised.  Skipped under a
    profiler, whose preloaded library would also load into the child."""
    import subprocess
    if any(k.startswith("ROCPROF") for k in os.environ):
        return {"unavailable": "under rocprofv3"}
    try:
        r = subprocess.run(["rocm-smi", "--showclocks", "--json"], capture_output=True, text=True,
                           timeout=10)
        data = json.loads(r.stdout)
        card = next(iter(data.values()))
        return {k: v for k, v in card.items() if "clock" in k.lower() or "clk" in k.lower()}
    except Exception as e:  # noqa: BLE001 - reporting only
        return {"unavailable": type(e).__name__}


def bscan_fista(ufss, W, dev):
    """FISTA on the 32-position B-scan workload (shared bins, K = 200), the
    configuration the oracle's own FISTA is timed on: plan, L and solve times."""
    import torch
    w = W.workload("bscan32")
    g = w["geom"]
    t0 = time.perf_counter()
    bins, _ = ufss.ufss_select_freqs(g, w["m"], w["per_position"], w["seed"])
    plan = ufss.Plan(g, w["m"], w["per_position"], bins)
    L = ufss.ufss_lipschitz(plan, margin=0.01)
    torch.cuda.synchronize()
    setup = time.perf_counter() - t0
    y = torch.from_numpy(W.cn((g["ny"], g["nx"], w["m"]), 7).astype(np.complex64)).to(dev)
    x = torch.zeros((g["ny"], g["nx"], g["nz"]), dtype=torch.complex64, device=dev)
    ufss.ufss_fista(plan, y, ufss.lambda_from_mu(w["mu"]), L, 5, x)
    x.zero_()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    st = ufss.ufss_fista(plan, y, ufss.lambda_from_mu(w["mu"]), L, w["iters"], x)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    plan.close()
    return {"iters": w["iters"], "solve_s": round(dt, 4), "plan_and_L_s": round(setup, 3),
            "_iterate": (x.cpu().numpy().reshape(-1), L, st["lambda"])}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="cscan32")
    ap.add_argument("--algo", default="auto", choices=["auto", "fft"],
                    help="auto: the windowed GEMM (or, if faster, the phasor path); fft: time "
                         "the transform-domain operator instead (FP32)")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--quick", action="store_true", help="skip time-to-accuracy and extras")
    ap.add_argument("--dtype", default="f32", choices=["f32", "bf16"],
                    help="operator precision of the timed FISTA steps (default f32, the headline)")
    ap.add_argument("--tune-cache", default=None,
                    help="autotuner cache file (read and written) instead of the shipped one")
    ap.add_argument("--retune", action="store_true", help="time the tiling candidates again")
    ap.add_argument("--calib-copy-mb", type=int, default=0,
                    help="also run a plain device copy of this size (counter calibration)")
    args = ap.parse_args()
    # autotuner cache: (path, read, write)
    if args.tune_cache:
        tcfg = (args.tune_cache, True, True)
    elif args.retune or not os.path.exists(SHIPPED_TUNING):
        tcfg = (None, False, False)
    else:
        tcfg = (SHIPPED_TUNING, True, False)
    if args.gpus != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path "
              "(its sharding is a design only); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2012_04534_amd import ufss
    from paper_2012_04534_amd import workloads as W

    dev = torch.device("cuda:0")
    w = W.workload(args.workload)
    g = w["geom"]
    m, per_pos = w["m"], w["per_position"]
    bins, _ = ufss.ufss_select_freqs(g, m, per_pos, w["seed"])
    cmac = window_terms(g, bins, per_pos)
    flop_pair = 16.0 * cmac           # A + A^H

    def ev_time(fn, reps):
        fn()
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    shape_x = (g["ny"], g["nx"], g["nz"])
    shape_y = (g["ny"], g["nx"], m)
    extras = {"algos": {}}
    # pick the operator algorithm by measurement (FP32)
    bf16 = args.dtype == "bf16"
    pdt = ufss.BF16 if bf16 else ufss.F32
    # the phasor algorithm is FP32 only
    algos = [ufss.ALGO_GEMM, ufss.ALGO_PHASOR] if (per_pos and not bf16) else [ufss.ALGO_GEMM]
    if args.algo == "fft":
        algos = [ufss.ALGO_FFT]
    xr = torch.from_numpy(W.cn(shape_x, 1).astype(np.complex64)).to(dev)
    yr = torch.empty(shape_y, dtype=torch.complex64, device=dev)
    xo = torch.empty_like(xr)
    best = None
    tuned = {}
    for algo in algos:
        plan = ufss.Plan(g, m, per_pos, bins, algo=algo, dtype=pdt)
        if algo == ufss.ALGO_GEMM:
            tuned = dict(zip(("fwd_split", "adj_split"), autotune(ufss, plan, tcfg)))
        tf = ev_time(lambda: ufss.ufss_forward(plan, xr, yr), 5)
        ta = ev_time(lambda: ufss.ufss_adjoint(plan, yr, xo), 5)
        name = {ufss.ALGO_GEMM: "gemm-bf16" if bf16 else "gemm", ufss.ALGO_PHASOR: "phasor",
                ufss.ALGO_FFT: "transform-bf16" if bf16 else "transform"}[algo]
        extras["algos"][name] = {"forward_ms": round(tf, 4), "adjoint_ms": round(ta, 4),
                                 "a_plus_ah_gflops": round(flop_pair / ((tf + ta) * 1e-3) / 1e9, 1)}
        if best is None or tf + ta < best[1]:
            best = (algo, tf + ta, name)
        plan.close()
    algo, _, algo_name = best
    if not bf16 and algo != ufss.ALGO_FFT:
        # the transform-domain operator on the same problem, reported beside the
        # windowed GEMM (which stays the timed path)
        extras["transform"] = transform_rates(ufss, g, m, per_pos, bins, xr, yr, xo, ev_time, cmac)
    torch.cuda.synchronize()
    t_plan = time.perf_counter()
    plan = ufss.Plan(g, m, per_pos, bins, algo=algo, dtype=pdt)
    torch.cuda.synchronize()
    t_plan = time.perf_counter() - t_plan
    extras["plan_build_s"] = round(t_plan, 4)
    if algo == ufss.ALGO_GEMM:
        autotune(ufss, plan, tcfg)
        extras["autotuned"] = tuned
        extras["tuning"] = ("shipped cache" if tcfg[0] == SHIPPED_TUNING else
                            "cache " + tcfg[0] if tcfg[0] else "timed")

    # synthetic scene and measurements: y = A x + n at the workload's SNR
    x_true = W.scene(g, w["n_scat"], amp=w["amp"], seed=w["seed"], back_wall=w["back_wall"])
    xt = torch.from_numpy(x_true.astype(np.complex64)).to(dev)
    y0 = torch.empty(shape_y, dtype=torch.complex64, device=dev)
    ufss.ufss_forward(plan, xt, y0)
    torch.cuda.synchronize()
    sig = W.noise_sigma(float((y0.abs() ** 2).sum().item()), y0.numel(), w["snr_db"])
    y = (y0 + sig * torch.from_numpy(W.cn(shape_y, w["seed"] + 1).astype(np.complex64)).to(dev)).contiguous()

    t_l = time.perf_counter()
    L = ufss.ufss_lipschitz(plan, max_iters=200, rtol=1e-6, margin=0.01, seed=4)
    t_l = time.perf_counter() - t_l
    x = torch.zeros(shape_x, dtype=torch.complex64, device=dev)
    st = ufss.ufss_fista(plan, y, ufss.lambda_from_mu(w["mu"]), L, 1, x)
    lam = st["lambda"]

    # warmup, then exactly K timed FISTA iterations
    x.zero_()
    ufss.ufss_fista(plan, y, lam, L, max(args.warmup, 1), x)
    x.zero_()
    # the core kernels of the timed steps are bracketed by HIP events on their
    # launch stream (the library's kernel timing mode)
    ufss.ufss_plan_kernel_timing(plan, True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ufss.ufss_fista(plan, y, lam, L, args.steps, x)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ufss.ufss_plan_kernel_timing(plan, False)
    ms_step = (t1 - t0) * 1e3 / args.steps
    value = flop_pair / (ms_step * 1e-3) / 1e9

    # dominant kernel: average launch duration over the timed steps
    k_f, k_a, n_f, n_a = ufss.ufss_plan_kernel_times(plan)
    extras["kernel_launches_timed"] = {"forward": n_f, "adjoint": n_a}
    dom, k_ms = ("adjoint", k_a) if k_a >= k_f else ("forward", k_f)
    if algo == ufss.ALGO_FFT:
        # the contraction streams its table of complex entries (8 bytes, 4 in
        # BF16) once per launch: bound by HBM
        tab = table_bytes(g, plan.info(), 4 if bf16 else 8)
        roof = {"bound": "hbm", "achieved": round(tab / (k_ms * 1e-3) / 1e9, 1),
                "peak": PEAK_HBM / 1e9, "unit": "GB/s"}
    elif algo == ufss.ALGO_PHASOR:
        # per (term, bin): one complex MAC (8 algorithmic flops) on the VALU plus
        # the phase it needs; peak from the issue model above
        roof = {"bound": "alu", "achieved": round(8.0 * cmac / (k_ms * 1e-3) / 1e12, 3),
                "peak": round(PEAK_PHASOR_TERMS * 8.0 / 1e12, 2), "unit": "TFLOP/s",
                "peak_basis": "VALU issue: %d lane slots per term" % PHASOR_SLOTS_PER_TERM}
    else:
        roof = {"bound": "mfma", "achieved": round(8.0 * cmac / (k_ms * 1e-3) / 1e12, 3),
                "peak": (PEAK_BF16_MFMA if bf16 else PEAK_FP32_MFMA) / 1e12, "unit": "TFLOP/s"}
        if not bf16:
            # `achieved` counts the windowed sum; of its products the kernels form
            # one per class of mirrored offsets, each in Gauss's three real products,
            # so `frac` can pass 1: the share of the peak spent on products that
            # the kernels need (no padding, no union bins) is `needed_frac`
            roof["needed_frac"] = round(roof["achieved"] * 0.75 * mirror_share(g) / roof["peak"], 4)
    roof["frac"] = round(roof["achieved"] / roof["peak"], 4)
    pinfo = plan.info()
    roof["traffic"] = traffic_bytes(args.workload, algo_name, dom, pinfo) \
        if algo_name in TRAFFIC_SRC else None
    roof["tiling"] = tiling_key(pinfo, dom)
    roof["kernel"] = "%s %s core (%.4f ms per launch)" % (algo_name, dom, k_ms)
    extras["kernel_ms"] = {"forward_core": round(k_f, 4), "adjoint_core": round(k_a, 4)}

    result = {
        "metric": METRIC, "value": round(value, 2), "unit": "GFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_step, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": args.dtype,
        "data": "synthetic",
        "config": {"workload": "%s: %dx%d scan positions, %dx%dx%d voxels, N_t=%d, M=%d %s bins, "
                               "%s window, %d scatterers%s, %g dB SNR, FISTA mu=%g" % (
                                   args.workload, g["nx"], g["ny"], g["nx"], g["ny"], g["nz"], g["nt"], m,
                                   "per-position" if per_pos else "shared",
                                   "full" if g["win_x"] < 0 else "+-%d" % g["win_x"], w["n_scat"],
                                   " + back wall" if w["back_wall"] is not None else "",
                                   w["snr_db"], w["mu"]),
                   "operator_algo": algo_name, "cmac_per_apply": cmac},
        "roofline": roof,
    }

    if not args.quick:
        result["fista"] = time_to_accuracy(ufss, W, plan, g, w, bins, y, lam, L, t_l, dev, tcfg)
        result["fista"]["learned"] = learned_block(ufss, W, g, w, bins, L, dev, tcfg)
        extras["cscan64"] = cscan64_rates(ufss, W, dev, ev_time, tcfg)
        # the precision study's own workload: BF16 against FP32 on the 64 x 64
        # C-scan, time to the 1e-2 level only (its FP32 iterations take 26 ms)
        w64 = W.workload("cscan64")
        b64, _ = ufss.ufss_select_freqs(w64["geom"], w64["m"], w64["per_position"], w64["seed"])
        p64, y64, L64, lam64, tl64 = measured_problem(ufss, W, w64, b64, dev, tcfg)
        result["fista_cscan64"] = time_to_accuracy(ufss, W, p64, w64["geom"], w64, b64, y64, lam64, L64,
                                                   tl64, dev, tcfg, timed_levels=[len(LEVELS) - 1])
        p64.close()
        del y64
        extras["batch64"] = batch_rate(ufss, W, dev, tcfg)
        extras["bscan32_fista"] = bscan_fista(ufss, W, dev)

    gpu_outputs = None if args.no_cpu else operator_outputs(ufss, W, g, w, bins, dev, tcfg)
    extras["gpu_clocks"] = gpu_clocks()
    result["extras"] = extras
    plan.close()

    if args.calib_copy_mb > 0:
        n = args.calib_copy_mb * (1 << 20) // 4
        a = torch.ones(n, dtype=torch.float32, device=dev)
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        result["extras"]["calib_copy_bytes_each_way"] = n * 4

    if not args.no_cpu:
        result["cpu_baseline"] = cpu_baseline(w, bins, gpu_outputs=gpu_outputs)
        result["cpu_baseline"]["structured"] = cpu_structured(w, bins)
        bs = extras.get("bscan32_fista", {}).get("_iterate")
        result["cpu_baseline"]["bscan32_oracle_fista"] = cpu_oracle_fista_bscan(bs)
    extras.get("bscan32_fista", {}).pop("_iterate", None)
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()

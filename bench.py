#!/usr/bin/env python3
"""Benchmark of Sparse Reference Attention (Avatar V) on one MI355X.

One step = one sra_forward + one sra_backward (the whole hot path: schedule upload,
forward, delta, dK/dV, dQ) over the 720p workload with every input already resident in
HBM: 1 sample, generation 21x45x80 = 75,600 tokens, reference 21x45x80 = 75,600 tokens,
40 heads, head_dim 128, bf16, one reference latent frame per self-attention group.

Prints ONE JSON line. value = useful TFLOP/s of the step: only visible query-key pairs
count, 4*d FLOP per pair forward and 10*d backward. Also reported: % of the bf16 dense
MFMA peak, ms per layer forward/backward, the roofline of the dominant kernel (timed with
hipEvents on its launch stream inside the library), forward and backward time against
reference length at the 480p sweep shape, the 480p layer and the varlen packed batch (also
with the temporal window and with reference token masks) per call, the tiny workload as
achieved bytes per second, and the CPU oracle on a bounded sample.
"""
from __future__ import annotations

import argparse
import csv
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0  # MI355X dense bf16 MFMA (published)
PEAK_HBM_GBS = 8000.0
METRIC = "SRA useful TFLOP/s + % bf16 MFMA peak; ms/layer vs reference length"
CSRC = os.path.join(ROOT, "paper_2606_13872_amd", "csrc")
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_720p.json")
KERNEL_SYMBOLS = {"forward": "sra_fwd_kernel", "dkdv": "sra_dkv_kernel", "dq": "sra_dq_kernel",
                  "delta": "sra_delta_kernel"}
KERNEL_SOURCES = {"forward": ["sra_fwd.hip"], "dkdv": ["sra_grad.hip", "sra_dkv.h"], "dq": ["sra_grad.hip", "sra_dq.h"],
                  "delta": ["sra_bwd.hip"]}
# schedule.cpp sets the launch order of the work items, which decides how often a tile is
# fetched again from HBM
COMMON_SOURCES = ["sra_config.h", "sra_device.h", "sra_tiles.h", "sra_kernels.h", "schedule.cpp"]
COPY_KERNEL = "neg_kernel"  # calibration: torch.neg over a float32 buffer reads and writes it once


def _args():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="720p",
                    help="720p (default), varlen, 480p, tiny, ...; <name>@h<N> is that layer with N heads "
                         "(one GPU's share when heads are split across GPUs)")
    ap.add_argument("--sweep-reps", type=int, default=2, help="forward calls per sweep point (0 = skip)")
    ap.add_argument("--cpu-rows", type=int, default=4096, help="gen rows in the CPU-oracle sample (0 = skip)")
    ap.add_argument("--tiny-reps", type=int, default=200, help="calls per pass of the tiny workload (0 = skip)")
    ap.add_argument("--other-reps", type=int, default=2,
                    help="timed calls per pass of the 480p and varlen workloads (0 = skip)")
    ap.add_argument("--gen-only-reps", type=int, default=None,
                    help="forward calls timed with the reference as context only (default: --steps; 0 = skip)")
    ap.add_argument("--copy-mib", type=int, default=0,
                    help="run one plain copy kernel (torch.neg, fp32) over this many MiB first: the "
                         "calibration for the HBM byte counters")
    ap.add_argument("--pmc-summary", nargs=2, metavar=("FETCH_CSV", "WRITE_CSV"),
                    help="no GPU: turn two rocprofv3 --pmc counter files (FETCH_SIZE, WRITE_SIZE) of a "
                         "--copy-mib run into per-launch HBM bytes per kernel, written to --traffic-out")
    ap.add_argument("--traffic-out", default=TRAFFIC_FILE)
    return ap.parse_args()


def _kernel_source_hash(kernel):
    """Hash of the sources a kernel is built from: stored traffic is only used while it matches."""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel] + COMMON_SOURCES:
        h.update(f.encode())
        with open(os.path.join(CSRC, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _counter_per_dispatch(path, counter):
    """{short kernel name: (mean counter value per dispatch, dispatches)} from a rocprofv3 csv."""
    tot, disp = {}, {}
    with open(path, newline="") as fh:
        for r in csv.DictReader(fh):
            if r["Counter_Name"] != counter:
                continue
            name = r["Kernel_Name"]
            key = next((k for k, sym in KERNEL_SYMBOLS.items() if sym in name), None)
            if key is None and COPY_KERNEL in name:
                key = "copy"
            if key is None:
                continue
            tot[key] = tot.get(key, 0.0) + float(r["Counter_Value"])
            disp.setdefault(key, set()).add(r["Dispatch_Id"])
    return {k: (tot[k] / len(disp[k]), len(disp[k])) for k in tot}


def _pmc_summary(fetch_csv, write_csv, copy_mib, workload_name, out_path):
    """Per-launch HBM bytes of each kernel: FETCH_SIZE and WRITE_SIZE (KiB per dispatch), each
    scaled so that the copy of known size reads and writes exactly its buffer (torch runs a copy
    of 2 GiB and more as several dispatches: their sum counts)."""
    fetch = _counter_per_dispatch(fetch_csv, "FETCH_SIZE")
    write = _counter_per_dispatch(write_csv, "WRITE_SIZE")
    if "copy" not in fetch or "copy" not in write:
        raise SystemExit("the counter files hold no copy-kernel dispatch: profile a --copy-mib run")
    known_kib = copy_mib * 1024.0
    fs, ws = known_kib / (fetch["copy"][0] * fetch["copy"][1]), known_kib / (write["copy"][0] * write["copy"][1])
    kernels = {}
    for k in KERNEL_SYMBOLS:
        if k in fetch and k in write:
            kernels[k] = {"symbol": KERNEL_SYMBOLS[k], "source_hash": _kernel_source_hash(k),
                          "fetch_bytes": round(fetch[k][0] * fs * 1024), "write_bytes": round(write[k][0] * ws * 1024),
                          "fetch_kib_raw": fetch[k][0], "write_kib_raw": write[k][0], "dispatches": fetch[k][1]}
    data = {"workload": workload_name,
            "calibration": {"kernel": f"{COPY_KERNEL} over {copy_mib} MiB of float32",
                            "fetch_kib_raw": fetch["copy"][0], "write_kib_raw": write["copy"][0],
                            "fetch_scale": fs, "write_scale": ws},
            "kernels": kernels}
    with open(out_path, "w") as fh:
        json.dump(data, fh, indent=1)
    print(json.dumps(data, indent=1))


def _stored_traffic(kernel, workload_name):
    """HBM bytes per launch of `kernel` from the counter runs, or None if absent or stale."""
    try:
        with open(TRAFFIC_FILE) as fh:
            data = json.load(fh)
    except (OSError, ValueError):
        return None
    k = data.get("kernels", {}).get(kernel)
    if data.get("workload") != workload_name or not k or k.get("source_hash") != _kernel_source_hash(kernel):
        return None
    return int(k["fetch_bytes"]) + int(k["write_bytes"])


def _workload_config(w):
    s = w.samples
    return {
        "workload": f"{w.name}: {len(s)} sample(s), gen "
                    + ",".join(f"{g.gen_frames}x{g.gen_h}x{g.gen_w}" for g in s)
                    + ", ref " + ",".join(f"{g.ref_frames}x{g.ref_h}x{g.ref_w}" for g in s)
                    + f", H={w.heads}, d={w.head_dim}, group=1 frame, forward+backward",
        "batch": len(s),
        "heads": w.heads,
        "head_dim": w.head_dim,
        "gen_tokens": sum(g.n_gen for g in s),
        "ref_tokens": sum(g.n_ref for g in s),
        "parallelism": "single GPU",
    }


def _fit(xs, ys):
    """Least-squares line ys ~ icpt + slope * xs, with R^2."""
    n = len(xs)
    mx, my = sum(xs) / n, sum(ys) / n
    sxx = sum((x - mx) ** 2 for x in xs)
    slope = sum((x - mx) * (y - my) for x, y in zip(xs, ys)) / sxx
    icpt = my - slope * mx
    ss_res = sum((y - (icpt + slope * x)) ** 2 for x, y in zip(xs, ys))
    ss_tot = sum((y - my) ** 2 for y in ys)
    return {"slope_ms_per_1k_tokens": round(slope * 1000, 5), "intercept_ms": round(icpt, 4),
            "r2": round(1 - ss_res / ss_tot, 6) if ss_tot > 0 else 1.0}


def _sweep(sra, torch, reps):
    from sra_inputs import SWEEP_POINTS, make_inputs, workload

    def timed(fn):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    rs, ms, ms_b, pairs = [], [], [], []
    for n in SWEEP_POINTS:
        w = workload(f"sweep_{n}")
        x = make_inputs(w.samples, w.heads, w.head_dim, w.seed, w.rms_norm_qk, device="cuda", grads=True)
        args = [x[k] for k in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")]
        o = sra.forward(*args, w.samples)
        out = {"o_gen": o[0], "o_ref": o[1], "lse_gen": o[2], "lse_ref": o[3]}
        g = sra.backward(*args, *o, x["do_gen"], x["do_ref"], w.samples)
        torch.cuda.synchronize()
        ms.append(timed(lambda: sra.forward(*args, w.samples, out=out)))
        ms_b.append(timed(lambda: sra.backward(*args, *o, x["do_gen"], x["do_ref"], w.samples, out=g)))
        rs.append(sum(s.n_ref for s in w.samples))
        gp, rp = sra.pair_counts(w.samples, w.heads, w.head_dim)
        pairs.append(gp + rp)
        del x, out, args, o, g
        torch.cuda.empty_cache()
        print(f"[bench] sweep R={rs[-1]} fwd {ms[-1]:.2f} ms bwd {ms_b[-1]:.2f} ms", file=sys.stderr, flush=True)
    return {
        "shape": "480p sweep: gen 21x30x52, ref n x 30x52 frames, H=40, d=128, forward and backward",
        "ref_tokens": rs,
        "ms_fwd": [round(m, 3) for m in ms],
        "ms_bwd": [round(m, 3) for m in ms_b],
        "visible_pairs_per_head": pairs,
        "fit_ms_vs_ref_tokens": _fit(rs, ms),
        "fit_bwd_ms_vs_ref_tokens": _fit(rs, ms_b),
        "ms_ratio_last_first": round(ms[-1] / ms[0], 3),
        "bwd_ms_ratio_last_first": round(ms_b[-1] / ms_b[0], 3),
        "pairs_ratio_last_first": round(pairs[-1] / pairs[0], 3),
    }


def _other_workloads(sra, torch, reps):
    """The other full-size workloads, one forward and one backward call each: the 480p layer,
    the varlen packed batch, and that batch with the refiner's temporal window and with
    reference token masks. ms per call and useful TFLOP/s (visible pairs only)."""
    from sra_inputs import make_inputs, workload

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    res = {}
    for name in ("480p", "varlen", "varlen_window", "varlen_tokens"):
        w = workload(name)
        H, d = w.heads, w.head_dim
        x = make_inputs(w.samples, H, d, w.seed, w.rms_norm_qk, device="cuda", grads=True)
        args = [x[k] for k in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")]
        o = sra.forward(*args, w.samples)
        out = {"o_gen": o[0], "o_ref": o[1], "lse_gen": o[2], "lse_ref": o[3]}
        g = sra.backward(*args, *o, x["do_gen"], x["do_ref"], w.samples)
        ms_f = timed(lambda: sra.forward(*args, w.samples, out=out))
        ms_b = timed(lambda: sra.backward(*args, *o, x["do_gen"], x["do_ref"], w.samples, out=g))
        ff, bf = sra.useful_flops(w.samples, H, d)
        cfg = _workload_config(w)
        res[name] = {"workload": cfg["workload"].replace(", group=1 frame, forward+backward", ""),
                     "gen_tokens": cfg["gen_tokens"], "ref_tokens": cfg["ref_tokens"],
                     "visible_pairs": ff // (4 * d),
                     "ms_fwd": round(ms_f, 3), "ms_bwd": round(ms_b, 3),
                     "fwd_tflops": round(ff / (ms_f * 1e-3) / 1e12, 2),
                     "bwd_tflops": round(bf / (ms_b * 1e-3) / 1e12, 2),
                     "pct_bf16_peak": round(100 * (ff + bf) / ((ms_f + ms_b) * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 2)}
        del x, out, args, o, g
        torch.cuda.empty_cache()
        print(f"[bench] {name} fwd {ms_f:.2f} ms bwd {ms_b:.2f} ms", file=sys.stderr, flush=True)
    return res


def _cpu_info():
    """Host CPU model and the cores this process may use."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:  # pragma: no cover
        usable = os.cpu_count() or 1
    return model, os.cpu_count() or 1, usable


def _cpu_baseline(x_gpu, w, gen_rows, torch, layer_pairs):
    """The oracle as it stands, timed on the host cores on bounded samples of the workload.

    Legs (float32 unless stated, head 0):
      fwd   forward_rows of gen_rows gen + gen_rows ref query rows of the layer (each row's
            full key set), and the same rows in float64 beside it;
      dq    dq_rows of gen_rows / 2 gen + gen_rows / 2 ref rows of the layer (S, P, O for D,
            dP and dQ of each row, 8 d FLOP per visible pair);
      slice the oracle's full forward and backward (explicit mask over all rows) on a slice of
            the layer with the same per-frame shape: its first generation latent frame and its
            first reference latent frame, plus dkv_keys (the sampled dK/dV entry point) on 64
            of its keys;
      tiny  the full forward and backward of the tiny workload.
    Seconds per layer are extrapolated from the rates, by visible pairs: the forward from the
    fwd leg (rows of the real layer), the backward from the slice's full backward. value is the
    step's useful FLOP (4 d forward + 10 d backward per pair) over those extrapolated seconds.
    """
    import numpy as np

    import oracle
    from sra_inputs import SampleGeom, make_inputs, to_numpy64, workload

    try:
        from threadpoolctl import threadpool_info
        blas_threads = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    except Exception:  # pragma: no cover
        blas_threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    threads = max(blas_threads, torch.get_num_threads())
    model, ncpu, usable = _cpu_info()
    d = w.head_dim
    g = w.samples[0]
    G, R, F = g.n_gen, g.n_ref, g.ref_h * g.ref_w
    names = ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref", "do_gen", "do_ref")
    xh = {k: x_gpu[k][:, 0:1].float().cpu().numpy() for k in names if k in x_gpu}
    rng = np.random.default_rng(0)
    rows_g = np.sort(rng.choice(G, size=min(gen_rows, G), replace=False))
    rows_r = G + np.sort(rng.choice(R, size=min(gen_rows, R), replace=False)) if R else np.zeros(0, int)
    rows = np.concatenate([rows_g, rows_r])

    def pairs_of(n_gen_rows, n_ref_rows):
        return n_gen_rows * (G + R) + n_ref_rows * F * g.group_frames

    def timed_rows(fn, rr, dtype):
        t = time.perf_counter()
        for b0 in range(0, rr.size, 128):
            fn(xh, w.samples, 0, 0, rr[b0:b0 + 128], dtype=dtype)
        return time.perf_counter() - t

    legs = {}
    # forward rows of the real layer, fp32 (the oracle's precision) and fp64
    t32 = timed_rows(oracle.forward_rows, rows, np.float32)
    p_f = pairs_of(rows_g.size, rows_r.size)
    legs["fwd"] = {"rows": int(rows.size), "visible_pairs": int(p_f), "s": round(t32, 2),
                   "tflops": round(4 * d * p_f / t32 / 1e12, 6), "dtype": "float32"}
    half = rows_g.size // 2
    sub64 = np.concatenate([rows_g[:half // 2], rows_r[:half // 2]])
    t64 = timed_rows(oracle.forward_rows, sub64, np.float64)
    p64 = pairs_of(half // 2, min(half // 2, rows_r.size))
    legs["fwd_float64"] = {"rows": int(sub64.size), "visible_pairs": int(p64), "s": round(t64, 2),
                           "tflops": round(4 * d * p64 / t64 / 1e12, 6), "dtype": "float64"}
    # dQ rows of the real layer (fp32): 8 d FLOP executed per visible pair
    subq = np.concatenate([rows_g[:half], rows_r[:half]])
    tq = timed_rows(oracle.dq_rows, subq, np.float32)
    pq = pairs_of(min(half, rows_g.size), min(half, rows_r.size))
    legs["dq"] = {"rows": int(subq.size), "visible_pairs": int(pq), "s": round(tq, 2),
                  "executed_tflops": round(8 * d * pq / tq / 1e12, 6), "dtype": "float32"}
    # slice of the layer: one gen frame and one ref frame, full forward + backward and dkv_keys
    sl = [SampleGeom(1, g.gen_h, g.gen_w, 1, g.ref_h, g.ref_w)]
    Gs, Rs = sl[0].n_gen, sl[0].n_ref
    xs = {k: v[:(Gs if k.endswith("gen") else Rs)].astype(np.float32) for k, v in xh.items()}
    gp_s, rp_s = oracle.pair_counts(sl)
    t = time.perf_counter()
    oracle.sra_forward(xs, sl, dtype=np.float32)
    tf_s = time.perf_counter() - t
    t = time.perf_counter()
    oracle.sra_backward(xs, sl, dtype=np.float32)
    tb_s = time.perf_counter() - t  # includes the forward it recomputes
    keys = np.sort(rng.choice(Gs + Rs, size=64, replace=False))
    t = time.perf_counter()
    oracle.dkv_keys(xs, sl, 0, 0, keys, dtype=np.float32)
    tk_s = time.perf_counter() - t
    ps = gp_s + rp_s
    legs["slice"] = {"geometry": f"gen 1x{g.gen_h}x{g.gen_w}, ref 1x{g.ref_h}x{g.ref_w}, 1 head",
                     "visible_pairs": int(ps), "fwd_s": round(tf_s, 2), "bwd_s": round(tb_s, 2),
                     "fwd_tflops": round(4 * d * ps / tf_s / 1e12, 6),
                     "bwd_tflops": round(10 * d * ps / tb_s / 1e12, 6),
                     "dkv_keys_64_s": round(tk_s, 2), "dtype": "float32"}
    # the tiny workload, full forward and backward (fp32)
    tw = workload("tiny")
    xt = {k: to_numpy64(v).astype(np.float32)
          for k, v in make_inputs(tw.samples, tw.heads, tw.head_dim, tw.seed, tw.rms_norm_qk).items()}
    gt, rt = oracle.pair_counts(tw.samples)
    t = time.perf_counter()
    for _ in range(10):
        oracle.sra_forward(xt, tw.samples, dtype=np.float32)
    tft = (time.perf_counter() - t) / 10
    t = time.perf_counter()
    for _ in range(10):
        oracle.sra_backward(xt, tw.samples, dtype=np.float32)
    tbt = (time.perf_counter() - t) / 10
    pt = (gt + rt) * tw.heads
    legs["tiny"] = {"fwd_ms": round(tft * 1e3, 3), "bwd_ms": round(tbt * 1e3, 3),
                    "fwd_tflops": round(4 * tw.head_dim * pt / tft / 1e12, 6),
                    "bwd_tflops": round(10 * tw.head_dim * pt / tbt / 1e12, 6), "dtype": "float32"}
    # per-layer extrapolation (all heads and samples), by visible pairs
    fwd_rate = 4 * d * p_f / t32
    bwd_rate = 10 * d * ps / tb_s
    s_fwd = 4 * d * layer_pairs / fwd_rate
    s_bwd = 10 * d * layer_pairs / bwd_rate
    work = t32 + t64 + tq + tf_s + tb_s + tk_s + 10 * (tft + tbt)
    return {
        "value": round(14 * d * layer_pairs / (s_fwd + s_bwd) / 1e12, 6),
        "unit": "TFLOP/s",
        "cores": threads,
        "kind": "oracle",
        "sample": (f"oracle in float32 on head 0 of sample 0 of the {w.name} layer: forward rows ({rows.size} rows), dQ rows "
                   f"({subq.size} rows), and the full forward + backward of a one-gen-frame, one-ref-frame slice; "
                   f"step rate = useful FLOP over the seconds per layer extrapolated from them ({work:.1f} s of "
                   f"CPU work in all)"),
        "cpu_model": model, "nproc": ncpu, "usable_cores": usable,
        "blas_threads": blas_threads, "torch_threads": torch.get_num_threads(),
        "seconds_per_layer_extrapolated": {"fwd": round(s_fwd, 1), "bwd": round(s_bwd, 1),
                                           "step": round(s_fwd + s_bwd, 1)},
        "legs": legs,
    }


def _gen_only(sra, torch, ins, fo, w, H, d, reps, line):
    """Forward with the reference as cached context only (gen rows alone), timed."""
    go_out = {"o_gen": fo["o_gen"], "lse_gen": fo["lse_gen"], "workspace": fo["workspace"]}
    sra.forward(ins[0], ins[1], ins[2], None, ins[4], ins[5], w.samples, out=go_out, gen_queries_only=True)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        sra.forward(ins[0], ins[1], ins[2], None, ins[4], ins[5], w.samples, out=go_out, gen_queries_only=True)
    e1.record()
    torch.cuda.synchronize()
    go_ms = e0.elapsed_time(e1) / reps
    go_pairs, _ = sra.pair_counts(w.samples, H, d, flags=sra.FLAG_GEN_QUERIES_ONLY)
    line["gen_queries_only_fwd"] = {"ms": round(go_ms, 3),
                                    "tflops": round(4 * d * go_pairs * H / (go_ms * 1e-3) / 1e12, 2)}
    print(f"[bench] gen-only forward {go_ms:.2f} ms", file=sys.stderr, flush=True)


def _tiny(sra, torch, reps):
    """The tiny workload (1 head, d = 64, 128 gen + 256 ref tokens): launch- and latency-bound,
    so it is reported as achieved bytes per second (algorithmic bytes / time), per call (wall
    time between events, launches included) and per kernel time; the host's own time per call
    (Python binding, C entry point and launches, without waiting for the GPU) is given beside
    them."""
    from sra_inputs import make_inputs, workload

    w = workload("tiny")
    H, d = w.heads, w.head_dim
    x = make_inputs(w.samples, H, d, w.seed, w.rms_norm_qk, device="cuda", grads=True)
    ins = [x[k] for k in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")]
    o = sra.forward(*ins, w.samples)
    fo = {"o_gen": o[0], "o_ref": o[1], "lse_gen": o[2], "lse_ref": o[3]}
    g = sra.backward(*ins, *o, x["do_gen"], x["do_ref"], w.samples)
    torch.cuda.synchronize()
    T = sum(s.n_gen + s.n_ref for s in w.samples)
    fwd_bytes = T * H * (4 * d * 2 + 4)       # q, k, v read, o written (bf16); lse written
    bwd_bytes = T * H * (8 * d * 2 + 4)       # q, k, v, o, do read, dq, dk, dv written; lse read

    fo["workspace"] = torch.empty(sra.Problem(w.samples, H, d).workspace_size(False), dtype=torch.uint8,
                                  device="cuda")
    g["workspace"] = torch.empty(sra.Problem(w.samples, H, d).workspace_size(True), dtype=torch.uint8,
                                 device="cuda")

    def run(fn):
        # wall time per call without the timing events, then the kernels' own time with them
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        t = time.perf_counter()
        for _ in range(reps):
            fn()
        host = (time.perf_counter() - t) * 1e3 / reps
        e1.record()
        torch.cuda.synchronize()
        sra.kernel_timing_enable(True)
        for _ in range(reps):
            fn()
        kt = sra.kernel_timing()
        sra.kernel_timing_enable(False)
        return e0.elapsed_time(e1) / reps, sum(v[0] for v in kt.values()) / reps, host

    f_call, f_kern, f_host = run(lambda: sra.forward(*ins, w.samples, out=fo))
    # the allocation-free entry point: its schedule stays resident between calls with the same
    # geometry, so a repeated call copies nothing from the host
    fn = {k: v for k, v in fo.items() if k != "workspace"}
    sra.forward_noalloc(*ins, w.samples, out=fn)  # the first call on a device loads its static array
    torch.cuda.synchronize()
    n_call, n_kern, n_host = run(lambda: sra.forward_noalloc(*ins, w.samples, out=fn))
    b_call, b_kern, b_host = run(lambda: sra.backward(*ins, *o, x["do_gen"], x["do_ref"], w.samples, out=g))
    print(f"[bench] tiny fwd {f_call * 1e3:.1f} us/call, bwd {b_call * 1e3:.1f} us/call", file=sys.stderr, flush=True)
    return {"workload": "tiny: gen 2x8x8, ref 4x8x8, H=1, d=64", "bound": "launch/latency",
            "fwd_bytes": fwd_bytes, "bwd_bytes": bwd_bytes,
            "fwd_us_per_call": round(f_call * 1e3, 2), "fwd_us_kernels": round(f_kern * 1e3, 2),
            "fwd_gbps_call": round(fwd_bytes / (f_call * 1e-3) / 1e9, 3),
            "fwd_gbps_kernels": round(fwd_bytes / (f_kern * 1e-3) / 1e9, 3),
            "fwd_us_host": round(f_host * 1e3, 2), "bwd_us_host": round(b_host * 1e3, 2),
            "fwd_noalloc_us_per_call": round(n_call * 1e3, 2), "fwd_noalloc_us_host": round(n_host * 1e3, 2),
            "fwd_noalloc_gbps_call": round(fwd_bytes / (n_call * 1e-3) / 1e9, 3),
            "bwd_us_per_call": round(b_call * 1e3, 2), "bwd_us_kernels": round(b_kern * 1e3, 2),
            "bwd_gbps_call": round(bwd_bytes / (b_call * 1e-3) / 1e9, 3),
            "bwd_gbps_kernels": round(bwd_bytes / (b_kern * 1e-3) / 1e9, 3)}


def main():
    args = _args()
    if args.pmc_summary:
        _pmc_summary(args.pmc_summary[0], args.pmc_summary[1], args.copy_mib, args.workload, args.traffic_out)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on exactly one GPU; the library has no multi-GPU "
                                   "path (heads would shard across GPUs with no collective inside the kernels)"}))
        sys.exit(2)
    import torch

    from paper_2606_13872_amd import sra
    from sra_inputs import make_inputs, workload

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        sys.exit(1)
    w = workload(args.workload)
    dev = torch.device("cuda:0")
    H, d = w.heads, w.head_dim
    print(f"[bench] inputs {w.name}", file=sys.stderr, flush=True)
    x = make_inputs(w.samples, H, d, w.seed, w.rms_norm_qk, device=dev)  # with dO
    ins = [x[k] for k in ("q_gen", "k_gen", "v_gen", "q_ref", "k_ref", "v_ref")]
    G, R = ins[0].shape[0], ins[3].shape[0]
    bf = dict(dtype=torch.bfloat16, device=dev)
    fo = {"o_gen": torch.empty((G, H, d), **bf), "o_ref": torch.empty((R, H, d), **bf),
          "lse_gen": torch.empty((H, G), dtype=torch.float32, device=dev),
          "lse_ref": torch.empty((H, R), dtype=torch.float32, device=dev)}
    bo = {n: torch.empty(((G if n.endswith("gen") else R), H, d), **bf)
          for n in ("dq_gen", "dk_gen", "dv_gen", "dq_ref", "dk_ref", "dv_ref")}
    p = sra.Problem(w.samples, H, d)
    fo["workspace"] = torch.empty(p.workspace_size(False), dtype=torch.uint8, device=dev)
    bo["workspace"] = torch.empty(p.workspace_size(True), dtype=torch.uint8, device=dev)

    if args.copy_mib > 0:
        src = torch.ones(args.copy_mib * 262144, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.neg(src, out=dst)
        torch.cuda.synchronize()
        del src, dst

    def step():
        sra.forward(*ins, w.samples, out=fo)
        sra.backward(*ins, fo["o_gen"], fo["o_ref"], fo["lse_gen"], fo["lse_ref"], x["do_gen"], x["do_ref"],
                     w.samples, out=bo)

    for i in range(args.warmup):
        step()
        torch.cuda.synchronize()
        print(f"[bench] warmup {i + 1}/{args.warmup}", file=sys.stderr, flush=True)
    sra.kernel_timing_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        step()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kt = sra.kernel_timing()
    sra.kernel_timing_enable(False)
    ms_step = wall * 1e3 / args.steps
    print(f"[bench] timed {args.steps} steps: {ms_step:.2f} ms/step", file=sys.stderr, flush=True)

    fwd_flops, bwd_flops = sra.useful_flops(w.samples, H, d)
    pairs = fwd_flops // (4 * d)
    value = (fwd_flops + bwd_flops) / (ms_step * 1e-3) / 1e12
    avg = {k: (v[0] / v[1] if v[1] else 0.0) for k, v in kt.items()}
    ms_fwd = avg["forward"] * (kt["forward"][1] / args.steps) if kt["forward"][1] else 0.0
    ms_bwd = sum(kt[k][0] for k in ("delta", "dkdv", "dq", "fill")) / args.steps
    # algorithmic FLOP per launch of each matrix kernel (per visible pair and head)
    kernel_flops = {"forward": 4 * d * pairs, "dkdv": 8 * d * pairs, "dq": 6 * d * pairs}
    dom = max(kernel_flops, key=lambda k: kt[k][0])
    achieved = kernel_flops[dom] / (avg[dom] * 1e-3) / 1e12
    roofline = {"kernel": {"forward": "sra_fwd_kernel", "dkdv": "sra_dkv_kernel", "dq": "sra_dq_kernel"}[dom],
                "bound": "mfma", "achieved": round(achieved, 2), "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                "frac": round(achieved / PEAK_BF16_TFLOPS, 4), "traffic": _stored_traffic(dom, w.name),
                "traffic_unit": "HBM bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
                "avg_launch_ms": round(avg[dom], 3),
                "per_kernel_ms": {k: round(avg[k], 3) for k in avg if kt[k][1]}}
    line = {
        "metric": METRIC, "value": round(value, 2), "unit": "TFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_step, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
        "data": "synthetic", "config": _workload_config(w),
        "pct_bf16_peak": round(100 * value / PEAK_BF16_TFLOPS, 2),
        "ms_fwd": round(ms_fwd, 3), "ms_bwd": round(ms_bwd, 3),
        "fwd_tflops": round(fwd_flops / (ms_fwd * 1e-3) / 1e12, 2) if ms_fwd else None,
        "bwd_tflops": round(bwd_flops / (ms_bwd * 1e-3) / 1e12, 2) if ms_bwd else None,
        "roofline": roofline,
    }
    # reference as cached context only (the denoising-step path): gen rows alone
    go_reps = args.steps if args.gen_only_reps is None else args.gen_only_reps
    if go_reps > 0:
        _gen_only(sra, torch, ins, fo, w, H, d, go_reps, line)
    if args.cpu_rows > 0:
        print("[bench] cpu oracle sample", file=sys.stderr, flush=True)
        line["cpu_baseline"] = _cpu_baseline(x, w, args.cpu_rows, torch, pairs)
    del x, ins, fo, bo
    torch.cuda.empty_cache()
    if args.sweep_reps > 0:
        line["sweep"] = _sweep(sra, torch, args.sweep_reps)
    if args.other_reps > 0:
        line["other_workloads"] = _other_workloads(sra, torch, args.other_reps)
    if args.tiny_reps > 0:
        line["tiny"] = _tiny(sra, torch, args.tiny_reps)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()

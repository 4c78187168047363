#!/usr/bin/env python3
"""Benchmark of the cluster-driven KV-cache hot path on one MI355X.

A timed "step" is one autoregressive decode step of the workload: for every
layer, mosaic_decode_step -- mosaic_retrieve (mean query, scores, top-k, page
list) followed by mosaic_attend (split-KV attention over the retrieved pages +
combine) -- the layers chained on one stream in order, as a decoder issues them.
The stream is ingested beforehand through mosaic_ingest_frame (timed separately:
frames/s, with its own roofline figure), and the multi-token question is
prefilled once.  All inputs are resident in HBM before any timed region starts.

Prints ONE JSON line.  The headline numbers are those of the full streaming stack
(config 2 of the benchmark definition: 28 layers, 4096 frames, ~15 GB of KV
streamed from HBM, per-layer calls); `extra` holds the same stack with all layers
in one call, the single-layer config 1, the 8-stream question prefill (config 4),
the host-offload tier (config 3, measured in a process of its own) and the
extensions.

`roofline` refers to the split-KV attention kernel (the dominant kernel):
algorithmic bytes = K and V of the retrieved tokens read once, divided by that
kernel's mean duration, measured with a HIP start/stop event pair attached to
every launch on the library's stream (the kernel's own begin/end timestamps).
`roofline.traffic` is read from the rocprofv3 counter summary under profiles/.
`cpu_baseline` is the fp64 CPU oracle timed on this host on a bounded sample of
the same workload (whole streams of a few units; one thread and all cores).
"""
from __future__ import annotations

import argparse
import json
import os
import subprocess
import sys
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0      # MI355X HBM3E, published
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "attend_kernels_hbm_traffic_pmc.txt")


def measured_traffic_bytes(workload, calls, kernel):
    """HBM bytes per launch of an attention kernel as the hardware counters saw them (FETCH_SIZE +
    WRITE_SIZE from two rocprofv3 --pmc runs, each scaled by the same counter read on a plain copy of
    known size): the `traffic_bytes <workload> <calls> <kernel> <bytes>` lines of the committed
    summary.  Raises if the summary has no line for the key: a changed kernel or workload must be
    measured again, not reported with old bytes."""
    with open(TRAFFIC_FILE) as fh:
        for line in fh:
            w = line.split()
            if len(w) == 5 and w[0] == "traffic_bytes" and (w[1], w[2], w[3]) == (workload, calls, kernel):
                return int(w[4])
    raise KeyError(f"{TRAFFIC_FILE} has no traffic_bytes line for {workload} {calls} {kernel}")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=64)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="cfg2", choices=["cfg0", "cfg1", "cfg2", "cfg3", "cfg4", "maintainer", "prefetch", "nested"])
    ap.add_argument("--layers", type=int, default=0, help="override the layer count")
    ap.add_argument("--frames", type=int, default=0, help="override the frame count")
    ap.add_argument("--all-layers-call", action="store_true",
                    help="one retrieve/attend call for all layers instead of per-layer calls")
    ap.add_argument("--two-calls", action="store_true",
                    help="per-layer decode steps as mosaic_retrieve + mosaic_attend instead of mosaic_decode_step")
    ap.add_argument("--no-extra", action="store_true",
                    help="skip the legs reported under `extra`")
    ap.add_argument("--extra-steps", type=int, default=32)
    ap.add_argument("--cpu-seconds", type=float, default=8.0, help="budget of each timed decode part of the oracle leg")
    ap.add_argument("--cpu-units", type=int, default=0, help="units the oracle leg samples (0 = one per host thread, at most 8)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one plain 256 MiB device copy (counter calibration for rocprofv3 --pmc)")
    ap.add_argument("--aug-window", type=int, default=0, help="retrieval augmentation: local window in frames")
    ap.add_argument("--aug-reps", action="store_true", help="retrieval augmentation: global representatives")
    ap.add_argument("--check-units", type=int, default=2,
                    help="units spot-checked against the oracle before timing (0 = none)")
    return ap.parse_args()


def n_tok_all(m, L):
    """Selected token count of every unit (one small D2H per layer)."""
    H = m.cfg.n_kv_heads
    out = []
    buf = np.empty(H, dtype=np.int32)
    for l in range(L):
        rc = m._L.mosaic_get_selection(m._h, l, None, None, None, None, 0, buf.ctypes.data)
        if rc != 0:
            m._check(rc)
        out.extend(buf.tolist())
    return out


def run_leg(wl, *, steps, warmup, all_layers, check_units, cpu_seconds, calibrate=False, aug=None,
            two_calls=False, cpu_units=0, traffic_lookup=True, ingest_without_recluster=False):
    """aug = (window_frames, global_reps) switches the retrieval augmentation of Sec. V-C on.
    Per-layer decode steps go through mosaic_decode_step (selection and attention in one kernel
    where the library supports it) unless two_calls asks for mosaic_retrieve + mosaic_attend."""
    import torch
    from paper_2604_10060_amd import binding, inputs

    dev = "cuda:0"
    L, Hq, D, T, F = wl.n_layers, wl.n_q_heads, wl.head_dim, wl.tokens_per_frame, wl.n_frames
    esz = 4 if wl.kv_dtype == "fp32" else 2
    one_call = not all_layers and not two_calls
    mode = "all_layers" if all_layers else ("per_layer_decode_step" if one_call else "per_layer")

    # ---- synthetic stream, generated on the device ---------------------------------
    t0 = time.time()
    st = inputs.SceneStream(wl, device=dev)
    shape = (F, L, wl.n_kv_heads, T, D)
    K_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    V_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    for f in range(F):
        K_all[f], V_all[f] = st.frame(f)
    torch.cuda.synchronize()
    log(f"[bench] {wl.name}/{mode}: {F} frames generated in {time.time() - t0:.1f}s "
        f"({2 * K_all.numel() * esz / 1e9:.2f} GB KV)")

    if calibrate:
        a = torch.empty(256 << 20, dtype=torch.uint8, device=dev).fill_(1)
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        lib_ = binding.load_library()   # k_calibration_copy: reads 256 MiB, writes 256 MiB
        assert lib_.mosaic_calibration_copy(b.data_ptr(), a.data_ptr(), a.numel(),
                                            torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        del a, b

    aug_cfg = dict(aug_window_frames=aug[0], aug_global_reps=int(aug[1])) if aug else {}
    # (batched ingest calls run their assignment chain beside the next call's page stores)
    m = binding.Mosaic(binding.config_for(wl, ingest_overlap=1, **aug_cfg), device=dev)
    frame_bytes = L * wl.n_kv_heads * T * D * esz
    kp, vp = K_all.data_ptr(), V_all.data_ptr()
    lib, h = m._L, m._h

    def ingest(batch):
        m.reset()
        torch.cuda.synchronize()
        t = time.perf_counter()
        f = 0
        while f < F:
            nb = min(batch, F - f)
            rc = lib.mosaic_ingest_frame(h, kp + f * frame_bytes, vp + f * frame_bytes, nb)
            if rc != 0:
                m._check(rc)
            f += nb
        torch.cuda.synchronize()
        return F / (time.perf_counter() - t)

    ingest(16)                              # warm-up pass
    fps_b16 = ingest(16)
    fps_b1 = ingest(1)                      # the stream the queries run against
    log(f"[bench] ingest: {fps_b1:.0f} frames/s (1 frame per call), {fps_b16:.0f} frames/s (16 per call)")

    # ---- questions ------------------------------------------------------------------
    q_question = st.question(st.draw_scene(), wl.question_tokens, 0).contiguous()
    n_q = warmup + steps
    q_dec = torch.stack([st.question(st.draw_scene(), 1, 1 + i) for i in range(n_q)])  # [n][L][1][Hq][D]
    out = torch.empty((L, 1, Hq, D), dtype=wl.torch_dtype, device=dev)
    lse = torch.empty((L, 1, Hq), dtype=torch.float32, device=dev)
    layer_q_bytes = Hq * D * esz
    torch.cuda.synchronize()

    # ---- parity spot check in the timed launch configuration ------------------------
    checked = None
    if check_units > 0:
        from tests import harness
        from oracle import mosaic_oracle as orc
        rng = np.random.Generator(np.random.PCG64(7))
        all_units = [(l, hh) for l in range(L) for hh in range(wl.n_kv_heads)]
        pick = [all_units[i] for i in rng.choice(len(all_units), min(check_units, len(all_units)),
                                                 replace=False)]
        t0 = time.time()
        oracles = {}
        A = m.assignments()
        for (l, hh) in pick:
            o = orc.OracleUnit(wl.n_clusters, D, T, F, wl.warmup_frames, wl.lloyd_iters, wl.recluster_every)
            Ku = inputs.unit_pages(K_all, l, hh)
            for f in range(F):
                o.ingest(Ku[f])
            u = l * wl.n_kv_heads + hh
            assert np.array_equal(A[u], o.assignments()), f"unit {(l, hh)}: assignments differ from the oracle"
            oracles[(l, hh)] = o
        rep = harness.Report()
        lm = "all" if all_layers else ("fused" if one_call else "per_layer")
        if aug:
            harness.query_augmented_with_parity(m, wl, q_question, oracles, K_all, V_all, rep, aug[0], aug[1])
            harness.query_augmented_with_parity(m, wl, q_dec[0], oracles, K_all, V_all, rep, aug[0], aug[1])
        else:
            harness.query_with_parity(m, wl, q_question, oracles, K_all, V_all, rep, lm)
            harness.query_with_parity(m, wl, q_dec[0], oracles, K_all, V_all, rep, lm)
        checked = {"units": [list(p) for p in pick], "max_out_err": rep.max_out_err,
                   "max_lse_err": rep.max_lse_err, "topk_near_ties": rep.topk_near_ties}
        log(f"[bench] parity spot check on units {pick}: out err {rep.max_out_err:.2e} "
            f"({time.time() - t0:.1f}s)")

    # ---- question prefill (once, timed) ---------------------------------------------
    oq = torch.empty_like(q_question)
    lq = torch.empty(q_question.shape[:-1], dtype=torch.float32, device=dev)

    def run_question():
        if all_layers:
            m.retrieve(-1, q_question); m.attend(-1, q_question, oq, lq)
        else:
            for l in range(L):
                m.retrieve(l, q_question[l]); m.attend(l, q_question[l], oq[l], lq[l])
    run_question()
    torch.cuda.synchronize()
    t = time.perf_counter()
    run_question()
    torch.cuda.synchronize()
    question_ms = (time.perf_counter() - t) * 1e3

    # ---- decode steps ---------------------------------------------------------------
    qbase = q_dec.data_ptr()
    step_q_bytes = L * layer_q_bytes
    op, lp = out.data_ptr(), lse.data_ptr()
    out_layer, lse_layer = Hq * D * esz, Hq * 4

    def retrieve_step(i):
        qp = qbase + i * step_q_bytes
        if all_layers:
            m.retrieve_raw(-1, qp, 1)
        else:
            for l in range(L):
                m.retrieve_raw(l, qp + l * layer_q_bytes, 1)

    def step(i):
        qp = qbase + i * step_q_bytes
        if all_layers:
            m.retrieve_raw(-1, qp, 1)
            m.attend_raw(-1, qp, 1, op, lp)
        elif one_call:
            for l in range(L):
                m.decode_step_raw(l, qp + l * layer_q_bytes, 1, op + l * out_layer, lp + l * lse_layer)
        else:
            for l in range(L):
                m.retrieve_raw(l, qp + l * layer_q_bytes, 1)
                m.attend_raw(l, qp + l * layer_q_bytes, 1, op + l * out_layer, lp + l * lse_layer)

    for i in range(warmup):
        step(i)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for i in range(warmup, n_q):
        step(i)
    torch.cuda.synchronize()
    us_per_step = (time.perf_counter() - t) / steps * 1e6

    # per-step latencies of the same steps: one event between consecutive steps on the
    # library's stream (the binding runs on torch's current stream), read after the pass
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    for j, i in enumerate(range(warmup, n_q)):
        evs[j].record()
        step(i)
    evs[steps].record()
    torch.cuda.synchronize()
    per_step = np.array([evs[j].elapsed_time(evs[j + 1]) * 1e3 for j in range(steps)])

    # a plain streaming kernel on the same box (256 MiB read + 256 MiB written) as the
    # achievable-bandwidth reference next to the published peak
    ca = torch.empty(256 << 20, dtype=torch.uint8, device=dev).fill_(1)
    cb = torch.empty_like(ca)
    cs = torch.cuda.current_stream().cuda_stream
    lib.mosaic_calibration_copy(cb.data_ptr(), ca.data_ptr(), ca.numel(), cs)
    c0, c1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    c0.record()
    for _ in range(4):
        lib.mosaic_calibration_copy(cb.data_ptr(), ca.data_ptr(), ca.numel(), cs)
    c1.record()
    torch.cuda.synchronize()
    stream_gbps = 4 * 2 * ca.numel() / (c0.elapsed_time(c1) * 1e-3) / 1e9
    del ca, cb

    # kernel-only time of the attention kernel: HIP start/stop events attached to each launch
    m.profile_enable(True)
    for i in range(warmup, n_q):
        step(i)
    kern_ms, launches = m.profile_read()
    m.profile_enable(False)
    # algorithmic bytes: K and V of the retrieved tokens, read once
    tok_total = 0
    for i in range(warmup, n_q):
        retrieve_step(i)
        tok_total += sum(n_tok_all(m, L))
    bytes_total = tok_total * 2 * D * esz
    bytes_per_launch = bytes_total / max(launches, 1)
    kern_us = kern_ms * 1e3 / max(launches, 1)
    achieved = bytes_per_launch / (kern_us * 1e-6) / 1e9
    step_gbps = (bytes_total / steps) / (us_per_step * 1e-6) / 1e9
    stats = m.stats()
    kernel = ("k_attend_decode_mfma" if stats.attend_impl == binding.ATTEND_MFMA else "k_attend_fp32")
    if one_call and stats.last_decode_fused:       # selection and attention ran as one kernel
        kernel = "k_decode_fused"

    # ---- ingest against its roofline ------------------------------------------------
    # Algorithmic bytes per frame: the K and V pages read once and written once into the store
    # (the key summary is formed from the same read) plus the fp64 summary row per unit.
    U = L * wl.n_kv_heads
    ingest_bytes = 4 * U * T * D * esz + U * D * 8
    ingest_rf = {"bytes_per_frame": ingest_bytes,
              "frames_per_s": round(fps_b1, 1), "frames_per_s_batch16": round(fps_b16, 1), "ingest_overlap": 1,
              "hbm_frac": round(fps_b1 * ingest_bytes / 1e9 / HBM_PEAK_GBPS, 4),
              "hbm_frac_batch16": round(fps_b16 * ingest_bytes / 1e9 / HBM_PEAK_GBPS, 4),
              "recluster_every": wl.recluster_every}
    m.close()
    m = None
    if ingest_without_recluster and wl.recluster_every > 0:
        torch.cuda.empty_cache()
        m = binding.Mosaic(binding.config_for(wl, recluster_every=0, ingest_overlap=1), device=dev)   # (ingest() below sees this context)
        lib, h = m._L, m._h
        ingest(16)
        nr16, nr1 = ingest(16), ingest(1)
        ingest_nr = {"frames_per_s_without_reclustering": round(nr1, 1),
                     "frames_per_s_batch16_without_reclustering": round(nr16, 1),
                     "hbm_frac_without_reclustering": round(nr1 * ingest_bytes / 1e9 / HBM_PEAK_GBPS, 4),
                     "hbm_frac_batch16_without_reclustering": round(nr16 * ingest_bytes / 1e9 / HBM_PEAK_GBPS, 4)}
        m.close()
        m = None
    else:
        ingest_nr = {}

    cpu = None
    if cpu_seconds > 0:
        cpu = cpu_baseline(wl, K_all, V_all, q_dec[warmup:], cpu_seconds, cpu_units)

    del K_all, V_all
    torch.cuda.empty_cache()
    traffic = measured_traffic_bytes(wl.name, mode, kernel) if traffic_lookup else None
    return {
        "us_per_step": us_per_step,
        "config": {"workload": wl.name, "layers": L, "q_heads": Hq, "kv_heads": wl.n_kv_heads,
                   "head_dim": D, "frames": F, "tokens_per_frame": T, "clusters": wl.n_clusters,
                   "top_k": wl.top_k, "calls": mode, "kv_splits": stats.last_n_splits},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBPS,
                     "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBPS, 4),
                     "traffic": traffic,
                     "kernel": kernel, "kernel_us": round(kern_us, 3),
                     "launches": int(launches), "bytes_per_launch": round(bytes_per_launch)},
        "cpu_baseline": cpu,
        "step_us_median": round(float(np.median(per_step)), 3),
        "step_us_p95": round(float(np.percentile(per_step, 95)), 3),
        "step_hbm_gbps": round(step_gbps, 1),
        "step_hbm_frac": round(step_gbps / HBM_PEAK_GBPS, 4),
        "stream_kernel_gbps": round(stream_gbps, 1),
        "frac_of_stream_kernel": round(achieved / stream_gbps, 4),
        "ingest_frames_per_s": round(fps_b1, 1),
        "ingest_frames_per_s_batch16": round(fps_b16, 1),
        "ingest_roofline": {"bound": "hbm", "peak": HBM_PEAK_GBPS, "unit": "GB/s", **ingest_rf, **ingest_nr},
        "question_tokens": wl.question_tokens,
        "question_ms": round(question_ms, 4),
        "parity_spot_check": checked,
    }


def run_prefill_leg(n_streams=8, check=True):
    """Config 4: `n_streams` independent video streams, each with its own context
    on its own HIP stream; one 256-token question chunk per stream is prefilled
    against the retrieved KV (the MFMA path).  Reports the MFMA roofline of
    k_attend_prefill_mfma and the aggregate question latency."""
    import torch
    from paper_2604_10060_amd import binding, inputs
    dev = "cuda:0"
    ctxs = []
    for sid in range(n_streams):
        wl = inputs.cfg4_stream(sid)
        st = inputs.SceneStream(wl, device=dev)
        K, V = st.frames(0, wl.n_frames)
        stream = torch.cuda.Stream(device=dev)
        with torch.cuda.stream(stream):
            m = binding.Mosaic(binding.config_for(wl), device=dev, stream=stream)
            for f in range(0, wl.n_frames, 64):
                m.ingest_frame(K[f:f + 64], V[f:f + 64])
            q = st.question(st.draw_scene(), wl.question_tokens, 0)[0].contiguous()
            out = torch.empty_like(q)
            lse = torch.empty(q.shape[:-1], dtype=torch.float32, device=dev)
        ctxs.append((wl, st, K, V, m, q, out, lse, stream))
    torch.cuda.synchronize()
    wl0 = ctxs[0][0]
    Tq, Hq, D, G = wl0.question_tokens, wl0.n_q_heads, wl0.head_dim, wl0.group

    def issue():
        for (wl, st, K, V, m, q, out, lse, stream) in ctxs:
            m.retrieve_raw(0, q.data_ptr(), Tq)
            m.attend_raw(0, q.data_ptr(), Tq, out.data_ptr(), lse.data_ptr())
    issue()
    torch.cuda.synchronize()
    reps = 5
    t = time.perf_counter()
    for _ in range(reps):
        issue()
    torch.cuda.synchronize()
    wall_us = (time.perf_counter() - t) / reps * 1e6
    # kernel time and flops of the prefill attention kernel, one stream at a time
    kern_us_total, flops_total, tok_total = 0.0, 0.0, 0
    for (wl, st, K, V, m, q, out, lse, stream) in ctxs:
        m.profile_enable(True)
        for _ in range(reps):
            m.retrieve_raw(0, q.data_ptr(), Tq)
            m.attend_raw(0, q.data_ptr(), Tq, out.data_ptr(), lse.data_ptr())
        ms, n = m.profile_read()
        m.profile_enable(False)
        ntok = sum(n_tok_all(m, 1))                     # retrieved tokens, all KV heads
        kern_us_total += ms * 1e3 / n
        flops_total += 4.0 * Tq * G * ntok * D          # QK^T and PV, all query heads
        tok_total += ntok
    checked = None
    if check:
        from tests import harness
        from oracle import mosaic_oracle as orc
        wl, st, K, V, m, q, out, lse, stream = ctxs[5]   # a low-coherence stream
        o = orc.OracleUnit(wl.n_clusters, D, wl.tokens_per_frame, wl.n_frames, wl.warmup_frames,
                           wl.lloyd_iters, wl.recluster_every)
        Ku = inputs.unit_pages(K, 0, 1)
        for f in range(wl.n_frames):
            o.ingest(Ku[f])
        rep = harness.Report()
        with torch.cuda.stream(stream):
            harness.query_with_parity(m, wl, q[None], {(0, 1): o}, K, V, rep)
        checked = {"stream": 5, "unit": [0, 1], "max_out_err": rep.max_out_err, "max_lse_err": rep.max_lse_err}
    tflops = flops_total / (kern_us_total * 1e-6) / 1e12
    for c in ctxs:
        c[4].close()
    del ctxs
    torch.cuda.empty_cache()
    return {"config": {"workload": "cfg4_prefill_stream x%d" % n_streams, "question_tokens": Tq,
                       "frames": wl0.n_frames, "clusters": wl0.n_clusters, "top_k": wl0.top_k},
            "question_us_all_streams_concurrent": round(wall_us, 1),
            "roofline": {"bound": "mfma", "achieved": round(tflops, 1), "peak": 2500.0, "unit": "TFLOP/s",
                         "frac": round(tflops / 2500.0, 4), "traffic": None,
                         "kernel": "k_attend_prefill_mfma",
                         "kernel_us": round(kern_us_total / n_streams, 2),
                         "flop_per_launch": round(flops_total / n_streams)},
            "retrieved_tokens_per_stream": tok_total // n_streams,
            "parity_spot_check": checked}


def run_maintainer_leg(layers=4, query_every=64, decode=64, check=True):
    """Self-adaptive maintainer (Sec. VI) on the config-2 stream recipe (geometric scenes, 5 %
    outlier tokens), `layers` of its 28 layers: 32 initial clusters in a table of 256, thresholds
    tau_min 4 / tau_max 16 / N0 32 (squared distance; within-scene spread of this recipe is 0.4-2,
    two merged scenes ~64).  Eager mode splits every invalid cluster at once; deferred mode follows
    Alg. 1 with a decode query every `query_every` frames (its selection is the resident set).
    Reports ingest rates, split counts of both modes (the paper's Sec. VIII figure is the
    reduction of split operations by deferral) and the decode step on the resulting clustering."""
    import torch
    from paper_2604_10060_amd import binding, inputs
    dev = "cuda:0"
    wl = inputs.CONFIGS[2].scaled(name="cfg2_recipe_maintained", n_layers=layers, n_clusters=256, top_k=16,
                                  recluster_every=0)
    mt = dict(mode=1, c_init=32, tau_min=4.0, tau_max=16.0, n0=32.0, split_iters=4, buf_max=256)
    L, Hq, D, T, F, H = wl.n_layers, wl.n_q_heads, wl.head_dim, wl.tokens_per_frame, wl.n_frames, wl.n_kv_heads
    st = inputs.SceneStream(wl, device=dev)
    shape = (F, L, H, T, D)
    K_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    V_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    for f in range(F):
        K_all[f], V_all[f] = st.frame(f)
    n_q = F // query_every + decode + 8
    q_dec = torch.stack([st.question(st.draw_scene(), 1, 1 + i) for i in range(n_q)])   # [n][L][1][Hq][D]
    out = torch.empty((L, 1, Hq, D), dtype=wl.torch_dtype, device=dev)
    lse = torch.empty((L, 1, Hq), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    lq = Hq * D * 2

    def step(m, i):
        qp = q_dec.data_ptr() + i * L * lq
        for l in range(L):
            m.retrieve_raw(l, qp + l * lq, 1)
            m.attend_raw(l, qp + l * lq, 1, out.data_ptr() + l * lq, lse.data_ptr() + l * Hq * 4)

    res = {}
    for name, mode in (("eager", binding.MAINT_EAGER), ("deferred", binding.MAINT_DEFERRED)):
        m = binding.Mosaic(binding.config_for(wl, warmup_frames=0, maint_mode=mode, init_clusters=mt["c_init"],
                                              split_iters=mt["split_iters"], buffer_max=mt["buf_max"],
                                              tau_min=mt["tau_min"], tau_max=mt["tau_max"], tau_n0=mt["n0"]),
                           device=dev)
        fps = {}
        for batch in (16, 1):
            m.reset()
            torch.cuda.synchronize()
            t = time.perf_counter()
            f, qi = 0, 0
            while f < F:
                nb = min(batch, F - f)
                m.ingest_frame(K_all[f:f + nb], V_all[f:f + nb])
                f += nb
                if mode == binding.MAINT_DEFERRED and f % query_every == 0 and f >= 2 * mt["c_init"]:
                    step(m, qi); qi += 1
            torch.cuda.synchronize()
            fps[batch] = F / (time.perf_counter() - t)
        s = m.stats()
        slots = m.maintainer()["n_slots"]
        _, sizes = m.centroids()
        for i in range(8):
            step(m, F // query_every + i)
        torch.cuda.synchronize()
        t = time.perf_counter()
        for i in range(decode):
            step(m, F // query_every + 8 + i)
        torch.cuda.synchronize()
        step_us = (time.perf_counter() - t) / decode * 1e6
        res[name] = {"ingest_frames_per_s": round(fps[1], 1), "ingest_frames_per_s_batch16": round(fps[16], 1),
                     "splits_immediate": int(s.splits_immediate), "splits_deferred": int(s.splits_deferred),
                     "deferred_inserts": int(s.deferred_inserts), "forced_absorbs": int(s.forced_absorbs),
                     "clusters_per_unit_mean": round(float(slots.mean()), 1),
                     "largest_cluster_frames": int(sizes.max()),
                     "decode_step_us": round(step_us, 2)}
        if check and mode == binding.MAINT_EAGER:
            from oracle import mosaic_oracle as orc
            l0, h0 = layers - 1, 1
            o = orc.OracleUnit(wl.n_clusters, D, T, F, 0, wl.lloyd_iters, 0, maintainer=mt)
            Ku = inputs.unit_pages(K_all, l0, h0)
            for f in range(F):
                o.ingest(Ku[f])
            u = l0 * H + h0
            same = bool(np.array_equal(m.assignments()[u], o.assignments())) and int(slots[u]) == o.n_slots
            assert same, "maintainer leg: assignments differ from the oracle"
            res[name]["parity_spot_check"] = {"unit": [l0, h0], "assignments_equal": same,
                                              "oracle_counters": o.counters()}
        m.close()
        del m
    e, d = res["eager"], res["deferred"]
    tot_e = e["splits_immediate"] + e["splits_deferred"]
    tot_d = d["splits_immediate"] + d["splits_deferred"]
    del K_all, V_all
    torch.cuda.empty_cache()
    return {"config": {"workload": wl.name, "layers": layers, "frames": F, "tokens_per_frame": T,
                       "cluster_table": wl.n_clusters, "init_clusters": mt["c_init"], "top_k": wl.top_k,
                       "tau_min": mt["tau_min"], "tau_max": mt["tau_max"], "tau_n0": mt["n0"],
                       "buffer_max": mt["buf_max"], "query_every_frames_deferred": query_every},
            "eager": e, "deferred": d,
            "split_operations_eager": tot_e, "split_operations_deferred": tot_d,
            "split_reduction_by_deferral": round(1.0 - tot_d / tot_e, 4) if tot_e else None}


def run_nested_leg(layers=4, steps=64, n_quality=24, check=True):
    """Nested visual-semantic hierarchy and two-stage retrieval (Sec. V-B, V-C) on the config-2 stream
    recipe, `layers` of its 28 layers, 512 clusters per unit and top-16 retrieval, against the flat
    index on the same stream: 16 visual partitions of 32 cluster ids, the 4 best partitions kept by
    the first stage (128 instead of 512 candidates); 1024-wide synthetic visual embeddings from 16
    appearance classes whose scenes share half of their key centre.  Reports ingest rates, the time of a retrieve call and of a decode step,
    candidates scored, and -- reported, never gated -- how many of the frames of the scene a
    question is about each index retrieves."""
    import torch
    from paper_2604_10060_amd import binding, inputs
    dev = "cuda:0"
    P, top_p = 16, 4
    wl = inputs.CONFIGS[2].scaled(name="cfg2_recipe_nested", n_layers=layers, n_clusters=512, top_k=16,
                                  recluster_every=0, visual_dim=1024, n_visual=16, visual_key_corr=0.5)
    L, Hq, D, T, F, H = wl.n_layers, wl.n_q_heads, wl.head_dim, wl.tokens_per_frame, wl.n_frames, wl.n_kv_heads
    st = inputs.SceneStream(wl, device=dev)
    shape = (F, L, H, T, D)
    K_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    V_all = torch.empty(shape, dtype=wl.torch_dtype, device=dev)
    for f in range(F):
        K_all[f], V_all[f] = st.frame(f)
    E_all = st.embeddings(0, F).contiguous()
    n_q = steps + 8 + n_quality
    scenes = [st.draw_scene() for _ in range(n_q)]
    q_dec = torch.stack([st.question(scenes[i], 1, 1 + i) for i in range(n_q)])   # [n][L][1][Hq][D]
    out = torch.empty((L, 1, Hq, D), dtype=wl.torch_dtype, device=dev)
    lse = torch.empty((L, 1, Hq), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    lq = Hq * D * 2

    def step(m, i, attend=True):
        qp = q_dec.data_ptr() + i * L * lq
        for l in range(L):
            m.retrieve_raw(l, qp + l * lq, 1)
            if attend:
                m.attend_raw(l, qp + l * lq, 1, out.data_ptr() + l * lq, lse.data_ptr() + l * Hq * 4)

    res = {}
    for name in ("flat", "nested"):
        nested = name == "nested"
        kw = dict(n_partitions=P, visual_dim=wl.visual_dim, top_partitions=top_p) if nested else {}
        m = binding.Mosaic(binding.config_for(wl, **kw), device=dev)
        fps = {}
        for batch in (16, 1):
            m.reset()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for f in range(0, F, batch):
                nb = min(batch, F - f)
                if nested:
                    m.ingest_frame_visual(K_all[f:f + nb], V_all[f:f + nb], E_all[f:f + nb])
                else:
                    m.ingest_frame(K_all[f:f + nb], V_all[f:f + nb])
            torch.cuda.synchronize()
            fps[batch] = F / (time.perf_counter() - t)
        times = {}
        for what, attend in (("retrieve_call_us", False), ("decode_step_us", True)):
            for i in range(8):
                step(m, i, attend)
            torch.cuda.synchronize()
            t = time.perf_counter()
            for i in range(steps):
                step(m, 8 + i, attend)
            torch.cuda.synchronize()
            times[what] = (time.perf_counter() - t) / steps * 1e6 / (1 if attend else L)
        # what the selection looks like (reported, not gated)
        cand, hit, toks = [], [], []
        for i in range(n_quality):
            qi = steps + 8 + i
            step(m, qi, attend=False)
            want = np.flatnonzero(st.scene_of_frame == scenes[qi])
            for l in range(L):
                ids, n_ids, scores, tk = m.selection(l)
                for h in range(H):
                    cand.append(int(np.isfinite(scores[h]).sum()))
                    got = np.unique(tk[h] // T)
                    hit.append(len(np.intersect1d(got, want)) / max(len(want), 1))
                    toks.append(len(tk[h]))
        _, sizes = m.centroids()
        res[name] = {"ingest_frames_per_s": round(fps[1], 1), "ingest_frames_per_s_batch16": round(fps[16], 1),
                     "retrieve_call_us": round(times["retrieve_call_us"], 2),
                     "decode_step_us": round(times["decode_step_us"], 2),
                     "candidates_scored_mean": round(float(np.mean(cand)), 1),
                     "non_empty_clusters_mean": round(float((sizes > 0).sum(axis=1).mean()), 1),
                     "question_scene_frames_retrieved_mean": round(float(np.mean(hit)), 4),
                     "retrieved_tokens_mean": round(float(np.mean(toks)), 1)}
        if check and nested:
            from oracle import mosaic_oracle as orc
            l0, h0 = layers - 1, 1
            u = l0 * H + h0
            E64 = E_all.cpu().numpy().astype(np.float64)
            vis = orc.OracleUnit(P, wl.visual_dim, 1, F, wl.warmup, wl.lloyd_iters)
            o = orc.OracleUnit(wl.n_clusters, D, T, F, wl.warmup, wl.lloyd_iters, 0, 0, nested=P)
            Ku = inputs.unit_pages(K_all, l0, h0)
            part = np.full(F, -1, dtype=np.int32)
            for f in range(F):
                vis.ingest(E64[f][None, :])
                if vis.ready:
                    part[: f + 1] = vis.assignments()
                o.ingest_nested(Ku[f], part)
            same_p = bool(np.array_equal(m.partitions()["frame_to_partition"], vis.assignments()))
            same_a = bool(np.array_equal(m.assignments()[u], o.assignments()))
            qi = steps + 8 + n_quality - 1
            ids, n_ids, _, _ = m.selection(l0)
            want = o.retrieve_nested(q_dec[qi, l0].float().cpu().numpy().astype(np.float64), h0, wl.group,
                                     top_p, wl.top_k)
            same_s = bool(np.array_equal(ids[h0, : n_ids[h0]], want["ids"]))
            assert same_p and same_a and same_s, "nested leg: partitions, assignments or selection differ from the oracle"
            res[name]["parity_spot_check"] = {"unit": [l0, h0], "partitions_equal": same_p,
                                              "assignments_equal": same_a, "selection_equal": same_s}
        m.close()
        del m
    del K_all, V_all
    torch.cuda.empty_cache()
    return {"config": {"workload": wl.name, "layers": layers, "frames": F, "tokens_per_frame": T,
                       "clusters": wl.n_clusters, "top_k": wl.top_k, "partitions": P, "top_partitions": top_p,
                       "visual_dim": wl.visual_dim, "appearance_classes": wl.n_visual,
                       "visual_key_corr": wl.visual_key_corr},
            "flat": res["flat"], "nested": res["nested"]}


def run_prefetch_leg(layers=3, steps=96, rhos=(0.95, 0.7)):
    """Overlap-aware cross-layer prefetch (Sec. VII-B) on the config-3 host tier, `layers` of its 28
    layers, with adjacent layers' states correlated by rho (the stream generator's stand-in for the
    similarity that residual connections give real models).  Per decode step and layer l:
      sequential   retrieve(l, q_l); attend(l)                      -- every fetch is on the critical path
      proxy        retrieve(l, q_l); prefetch(l+1, q_l); attend(l)  -- the paper's scheme
      lookahead    retrieve(l+1, q_{l+1}) before attend(l)          -- needs q_{l+1} early: an upper bound
    4 topics, steps/4 consecutive steps each.  Reports step latencies and how much of what the
    retrievals needed had been prefetched."""
    import torch
    from paper_2604_10060_amd import binding, inputs
    dev = "cuda:0"
    out_all = {}
    for rho in rhos:
        wl = inputs.CONFIGS[3].scaled(n_layers=layers, layer_corr=rho)
        L, Hq, D, T, F = wl.n_layers, wl.n_q_heads, wl.head_dim, wl.tokens_per_frame, wl.n_frames
        st = inputs.SceneStream(wl, device=dev)
        topics = [st.draw_scene() for _ in range(4)]
        per_topic = steps // 4
        qs = torch.stack([st.question(topics[i // per_topic], 1, 1 + i) for i in range(steps)])   # [n][L][1][Hq][D]
        out = torch.empty((L, 1, Hq, D), dtype=wl.torch_dtype, device=dev)
        lse = torch.empty((L, 1, Hq), dtype=torch.float32, device=dev)
        lq = Hq * D * 2
        res = {}
        for mode in ("sequential", "proxy", "proxy_top8", "lookahead"):
            m = binding.Mosaic(binding.config_for(wl, tier=binding.TIER_HOST, slab_frames=16, cache_fraction=0.10,
                                                  cache_pages_per_unit=F,
                                                  prefetch_top_k=8 if mode == "proxy_top8" else 0), device=dev)
            for f0 in range(0, F, 256):
                K, V = st.frames(f0, min(F, f0 + 256))
                for b in range(0, K.shape[0], 64):
                    m.ingest_frame(K[b:b + 64], V[b:b + 64])
            torch.cuda.synchronize()

            def step(i):
                qp = qs.data_ptr() + i * L * lq
                op, lp = out.data_ptr(), lse.data_ptr()
                if mode == "lookahead":
                    m.retrieve_raw(0, qp, 1)
                for l in range(L):
                    if mode == "lookahead":
                        if l + 1 < L:
                            m.retrieve_raw(l + 1, qp + (l + 1) * lq, 1)
                    else:
                        m.retrieve_raw(l, qp + l * lq, 1)
                        if mode.startswith("proxy") and l + 1 < L:
                            m.prefetch_raw(l + 1, qp + l * lq, 1)
                    m.attend_raw(l, qp + l * lq, 1, op + l * lq, lp + l * Hq * 4)

            lat = []
            for i in range(steps):
                torch.cuda.synchronize()
                t = time.perf_counter()
                step(i)
                torch.cuda.synchronize()
                lat.append((time.perf_counter() - t) * 1e6)
            s = m.stats()
            lat = np.array(lat)
            cold = lat[::per_topic]
            warm = np.delete(lat, np.arange(0, steps, per_topic))
            res[mode] = {"step_us_warm_median": round(float(np.median(warm)), 1),
                         "step_us_warm_mean": round(float(warm.mean()), 1),
                         "step_us_topic_switch_mean": round(float(cold.mean()), 1),
                         "cache_hits": int(s.cache_hits), "cache_misses": int(s.cache_misses),
                         "prefetch_fetched": int(s.prefetch_fetched), "prefetch_useful": int(s.prefetch_useful),
                         "h2d_gb": round(s.h2d_bytes / 1e9, 2)}
            m.close()
            del m
            torch.cuda.empty_cache()
        q_ = res["sequential"]
        for name in ("proxy", "proxy_top8"):
            p = res[name]
            # of the clusters the retrievals needed from the host, the share that had arrived by prefetch
            p["share_of_fetches_prefetched"] = round(p["prefetch_useful"] / max(p["prefetch_useful"] + p["cache_misses"], 1), 4)
            p["prefetch_precision"] = round(p["prefetch_useful"] / max(p["prefetch_fetched"], 1), 4)
            p["warm_step_change_vs_sequential"] = round(p["step_us_warm_mean"] / q_["step_us_warm_mean"] - 1.0, 4)
            p["topic_switch_change_vs_sequential"] = round(p["step_us_topic_switch_mean"] / q_["step_us_topic_switch_mean"] - 1.0, 4)
        out_all["rho_%.2f" % rho] = res
    return {"config": {"workload": "cfg3_host_offload", "layers": layers, "layers_of_full_config": 28,
                       "frames": 16384, "tokens_per_frame": 196, "clusters": 512, "top_k": 32,
                       "slab_frames": 16, "cache_fraction": 0.10, "decode_steps": steps}, **out_all}


def host_layers_that_fit(wl_full, cfg_kw, reserve=0.35, cap_bytes=64 << 30):
    """As many of the configuration's layers as pinned host memory allows: the largest layer count whose
    pinned arena is at most (1 - reserve) of MemAvailable and of cap_bytes.  The cap is what these boxes
    have been seen to grant: hipHostMalloc of 64 GiB succeeds and works, 96 GiB is refused, and a run
    that asked for more than 64 GiB ended in a segmentation fault, so nothing larger is ever requested."""
    from paper_2604_10060_amd import binding
    avail = None
    with open("/proc/meminfo") as fh:
        info = {l.split(":")[0]: int(l.split()[1]) * 1024 for l in fh if ":" in l}
    avail = info.get("MemAvailable", info.get("MemTotal", 0))
    budget = min(int(avail * (1.0 - reserve)), cap_bytes)
    best = 1
    for layers in range(1, wl_full.n_layers + 1):
        _, hbytes = binding.workspace_sizes(binding.config_for(wl_full.scaled(n_layers=layers), **cfg_kw))
        if hbytes <= budget:
            best = layers
    return best, {"MemTotal_GB": round(info.get("MemTotal", 0) / 1e9, 1), "MemAvailable_GB": round(avail / 1e9, 1),
                  "pinned_budget_GB": round(budget / 1e9, 1)}


HOST_MAINT = dict(mode=1, c_init=64, tau_min=1.0, tau_max=4.0, n0=32.0, split_iters=4, buf_max=0)


def run_host_leg(layers=0, steps=128, check=True):
    """Config 3 (host-offload tier): clusters live in pinned host memory in slabs of 8 frames, the GPU
    cluster cache holds at most 10 % of the stream's pages and 10 % of the cluster table (LRU), the fetch
    for layer l+1 is issued before attention of layer l.  The self-adaptive maintainer (Sec. VI) keeps the
    clusters small enough for that cache: 64 initial clusters in the table of 512, thresholds tau_min 1 /
    tau_max 4 / N0 32 (a fixed number of clusters without splitting degenerates on this stream: single
    clusters of > 1400 frames, top-32 selections of half the stream).  As many of the 28 layers as the box
    grants pinned memory for (the per-layer shape is kept).  4 question topics, steps/4 consecutive decode
    steps each (a topic switch means cold misses).  A selection that does not fit the cache is counted
    (`steps_refused_by_cache_capacity`), not hidden."""
    import torch
    from paper_2604_10060_amd import binding, inputs
    dev = "cuda:0"
    base = inputs.CONFIGS[3]
    F0 = base.n_frames
    mt = HOST_MAINT
    host_kw = dict(tier=binding.TIER_HOST, slab_frames=8, cache_fraction=0.10, cache_pages_per_unit=F0 // 10,
                   warmup_frames=0, maint_mode=mt["mode"], init_clusters=mt["c_init"], split_iters=mt["split_iters"],
                   tau_min=mt["tau_min"], tau_max=mt["tau_max"], tau_n0=mt["n0"])
    mem = None
    m = None
    if layers <= 0:
        # as many layers as pinned memory allows: bounded by MemAvailable and by what hipHostMalloc
        # grants on these boxes (far below the free host memory)
        layers, mem = host_layers_that_fit(base, host_kw)
    wl = base.scaled(n_layers=layers)
    L, Hq, D, T, F, H = wl.n_layers, wl.n_q_heads, wl.head_dim, wl.tokens_per_frame, wl.n_frames, wl.n_kv_heads
    log(f"[bench] {wl.name}: {layers} of 28 layers ({mem})")
    # measured pinned host-to-device rate of this machine: one 1 GiB copy
    src = torch.empty(1 << 30, dtype=torch.uint8, pin_memory=True)
    dst = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    dst.copy_(src, non_blocking=True)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(); dst.copy_(src, non_blocking=True); e1.record()
    torch.cuda.synchronize()
    pcie_gbps = (1 << 30) / (e0.elapsed_time(e1) * 1e-3) / 1e9
    del src, dst
    st = inputs.SceneStream(wl, device=dev)
    if m is None:
        m = binding.Mosaic(binding.config_for(wl, **host_kw), device=dev)
    dbytes, hbytes = binding.workspace_sizes(binding.config_for(wl, **host_kw))
    cu = (layers - 1, 2)                             # unit checked against the oracle
    keepK, keepV = [], []
    t0 = time.perf_counter()
    gen_s = 0.0
    for f0 in range(0, F, 256):
        tg = time.perf_counter()
        K, V = st.frames(f0, min(F, f0 + 256))
        torch.cuda.synchronize()
        gen_s += time.perf_counter() - tg
        if check:
            keepK.append(K[:, cu[0], cu[1]].cpu()); keepV.append(V[:, cu[0], cu[1]].cpu())
        for b in range(0, K.shape[0], 64):
            m.ingest_frame(K[b:b + 64], V[b:b + 64])
    torch.cuda.synchronize()
    ingest_fps = F / (time.perf_counter() - t0 - gen_s)
    log(f"[bench] {wl.name} x{layers} layers: host-tier ingest {ingest_fps:.0f} frames/s, "
        f"pinned H2D {pcie_gbps:.1f} GB/s")
    _, sizes = m.centroids()
    s_ing = m.stats()
    log(f"[bench] cluster sizes (frames): max {sizes.max()}, mean {sizes[sizes > 0].mean():.1f}, "
        f"clusters in use {float((sizes > 0).sum()) / sizes.shape[0]:.0f} of {wl.n_clusters} per unit, "
        f"{s_ing.splits_immediate} splits")
    topics = [st.draw_scene() for _ in range(4)]
    per_topic = steps // 4
    qs = torch.stack([st.question(topics[i // per_topic], 1, 1 + i) for i in range(steps)])   # [n][L][1][Hq][D]
    out = torch.empty((L, 1, Hq, D), dtype=wl.torch_dtype, device=dev)
    lse = torch.empty((L, 1, Hq), dtype=torch.float32, device=dev)
    esz = 2
    lq = Hq * D * esz
    m.profile_enable(True)                           # times the copy stream's fetches

    def step(i):
        qp = qs.data_ptr() + i * L * lq
        m.retrieve_raw(0, qp, 1)
        for l in range(L):
            if l + 1 < L:
                m.retrieve_raw(l + 1, qp + (l + 1) * lq, 1)
            m.attend_raw(l, qp + l * lq, 1, out.data_ptr() + l * lq, lse.data_ptr() + l * Hq * 4)

    lat, refused_steps = [], 0
    for i in range(steps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        try:
            step(i)
        except binding.MosaicError as ex:
            if ex.code != binding.ECAPACITY:
                raise
            refused_steps += 1
            log(f"[bench] step {i}: {ex}")
        torch.cuda.synchronize()
        lat.append((time.perf_counter() - t) * 1e6)
    # the attention kernel on warm steps (everything selected is in the GPU cluster cache)
    att_us = att_bytes = 0.0
    if refused_steps == 0:
        for i in range(2):                       # the last step again: after it its whole selection is cached
            step(steps - 1)
        torch.cuda.synchronize()
        m.profile_read()
        for i in range(8):                       # ... so these launches run without a fetch kernel beside them
            step(steps - 1)
        att_ms, att_n = m.profile_read()
        warm_tokens = int(sum(n_tok_all(m, L)))          # selection of the last step issued, all layers
        att_us = att_ms * 1e3 / max(att_n, 1)
        att_bytes = warm_tokens / L * 2 * D * esz
    s = m.stats()
    lat = np.array(lat)
    cold = lat[::per_topic]
    warm = np.delete(lat, np.arange(0, steps, per_topic))
    h2d_gbps = s.h2d_bytes / (s.h2d_busy_ms * 1e-3) / 1e9 if s.h2d_busy_ms > 0 else 0.0
    checked = None
    if check and refused_steps == 0:
        from oracle import mosaic_oracle as orc
        Ku = torch.cat(keepK).float().numpy().astype(np.float64)
        Vu = torch.cat(keepV).float().numpy().astype(np.float64)
        o = orc.OracleUnit(wl.n_clusters, D, T, F, 0, wl.lloyd_iters, 0, maintainer=mt)
        for f in range(F):
            o.ingest(Ku[f])
        u = cu[0] * H + cu[1]
        assert np.array_equal(m.assignments()[u], o.assignments()), "host tier: assignments differ from the oracle"
        q_last = qs[steps - 1]
        step(steps - 1)
        torch.cuda.synchronize()
        ids, n_ids, sc, toks = m.selection(cu[0])
        qh = q_last[cu[0]].float().cpu().numpy().astype(np.float64)
        ids_o, sc_o, tok_o, gap = o.retrieve(qh, cu[1], wl.group, wl.top_k)
        assert np.array_equal(ids[cu[1], : n_ids[cu[1]]], ids_o) and np.array_equal(toks[cu[1]], tok_o)
        want, _ = orc.attend(qh, Ku.reshape(-1, D), Vu.reshape(-1, D), tok_o, cu[1], wl.group)
        got = out[cu[0], :, cu[1] * wl.group:(cu[1] + 1) * wl.group].float().cpu().numpy()
        err = float(np.abs(got - want).max())
        assert err <= 2e-2, f"host tier attention err {err}"
        checked = {"unit": list(cu), "assignments_equal": True, "oracle_counters": o.counters(), "max_out_err": err}
    m.close()
    del m
    torch.cuda.empty_cache()
    # Alg. 1 in full on the same stream (deferred splits; a decode query every 64 frames makes its
    # selection resident): how many split operations deferral saves.  The cache holds the whole stream
    # here so that no selection is refused while clusters wait for their split.
    deferred = None
    try:
        kw = dict(host_kw)
        kw.update(maint_mode=binding.MAINT_DEFERRED, buffer_max=512, cache_pages_per_unit=F0)
        md = binding.Mosaic(binding.config_for(wl, **kw), device=dev)
        qi = 0
        for f0 in range(0, F, 256):
            K, V = st.frames(f0, min(F, f0 + 256))
            for b in range(0, K.shape[0], 64):
                md.ingest_frame(K[b:b + 64], V[b:b + 64])
                if f0 + b + 64 >= 2 * mt["c_init"]:
                    qq = st.question(st.draw_scene(), 1, 5000 + qi); qi += 1
                    for l in range(L):
                        md.retrieve(l, qq[l].contiguous())
        torch.cuda.synchronize()
        sd = md.stats()
        _, dsizes = md.centroids()
        deferred = {"splits_immediate": int(sd.splits_immediate), "splits_deferred": int(sd.splits_deferred),
                    "deferred_inserts": int(sd.deferred_inserts), "forced_absorbs": int(sd.forced_absorbs),
                    "largest_cluster_frames": int(dsizes.max()), "buffer_max": 512, "query_every_frames": 64}
        md.close()
        del md
    except Exception as ex:                          # noqa: BLE001
        deferred = {"error": str(ex)[:300]}
    torch.cuda.empty_cache()
    tot_e = int(s_ing.splits_immediate + s_ing.splits_deferred)
    out_d = {"config": {"workload": wl.name, "layers": layers, "layers_of_full_config": 28,
                        "frames": F, "tokens_per_frame": T, "cluster_table": wl.n_clusters, "top_k": wl.top_k,
                        "slab_frames": 8, "cache_fraction_of_clusters": 0.10, "cache_pages_per_unit": F0 // 10,
                        "cache_fraction_of_pages": 0.10, "maintainer": mt,
                        "pinned_host_GB": round(hbytes / 1e9, 1), "device_arena_GB": round(dbytes / 1e9, 1),
                        "host_memory": mem},
             "decode_step_us_warm_median": round(float(np.median(warm)), 1),
             "decode_step_us_topic_switch_mean": round(float(cold.mean()), 1),
             "steps_refused_by_cache_capacity": refused_steps,
             "ingest_frames_per_s": round(ingest_fps, 1),
             "clusters": {"in_use_per_unit_mean": round(float((sizes > 0).sum()) / sizes.shape[0], 1),
                          "largest_frames": int(sizes.max()), "splits_eager": tot_e,
                          "forced_absorbs": int(s_ing.forced_absorbs), "deferred_mode": deferred},
             "roofline": {"bound": "pcie", "achieved": round(h2d_gbps, 2), "peak": round(pcie_gbps, 2),
                          "unit": "GB/s", "frac": round(h2d_gbps / pcie_gbps, 4) if pcie_gbps else None,
                          "peak_kind": "measured: one 1 GiB pinned hipMemcpyAsync on this box",
                          "bytes": int(s.h2d_bytes), "copies": int(s.h2d_copies),
                          "busy_ms": round(s.h2d_busy_ms, 3)},
             "cache": {"hits": int(s.cache_hits), "misses": int(s.cache_misses)},
             "attention_warm": {"kernel": "k_attend_decode_mfma", "kernel_us": round(att_us, 1),
                                "bytes_per_launch": int(att_bytes),
                                "hbm_gbps": round(att_bytes / (att_us * 1e-6) / 1e9, 1) if att_us else None,
                                "frac_of_8TBps": round(att_bytes / (att_us * 1e-6) / 8e12, 4) if att_us else None},
             "parity_spot_check": checked}
    if deferred and "error" not in deferred and tot_e:
        tot_d = deferred["splits_immediate"] + deferred["splits_deferred"]
        out_d["clusters"]["split_reduction_by_deferral"] = round(1.0 - tot_d / tot_e, 4)
    return out_d


def cpu_baseline(wl, K_all, V_all, q_steps, budget_s, n_units=0):
    """The oracle as it stands, on this host, on a bounded sample of the same workload: the WHOLE
    stream of a few (layer, KV head) units (units are independent, so a unit is a fair sample of
    the job) -- (i) on one thread, (ii) on all host threads, one unit per thread (the C code
    releases the GIL) -- for Frame Encoding (frames/s) and for decode steps (retrieve + attend).
    Unit times are scaled to the whole job (all L * Hkv units)."""
    from oracle import mosaic_oracle as orc
    from paper_2604_10060_amd import inputs
    L, H, G, D, T, F = wl.n_layers, wl.n_kv_heads, wl.group, wl.head_dim, wl.tokens_per_frame, wl.n_frames
    units = [(l, h) for l in range(L) for h in range(H)]
    nproc = os.cpu_count() or 1
    try:
        nproc = min(nproc, len(os.sched_getaffinity(0)))
    except AttributeError:
        pass
    threads = max(1, min(nproc, 16))
    n_s = min(len(units), n_units if n_units > 0 else min(threads, 8))
    sample = [units[i] for i in np.linspace(0, len(units) - 1, n_s).astype(int)]
    threads = min(threads, n_s)
    log(f"[bench] oracle: nproc {nproc}, {threads} threads, {n_s} of {len(units)} units sampled")
    pages = {lh: (inputs.unit_pages(K_all, *lh), inputs.unit_pages(V_all, *lh)) for lh in sample}

    def ingest_unit(lh):
        o = orc.OracleUnit(wl.n_clusters, D, T, F, wl.warmup_frames, wl.lloyd_iters, wl.recluster_every)
        Ku = pages[lh][0]
        for f in range(F):
            o.ingest(Ku[f])
        return o

    # (i) one thread: one unit's whole stream
    t = time.perf_counter()
    first = ingest_unit(sample[0])
    t_one = time.perf_counter() - t
    # (ii) all threads: one unit per thread, all sampled units
    t = time.perf_counter()
    with ThreadPoolExecutor(threads) as ex:
        oracles = list(ex.map(ingest_unit, sample))
    t_all = time.perf_counter() - t
    state = {lh: (o, pages[lh][0].reshape(-1, D), pages[lh][1].reshape(-1, D)) for lh, o in zip(sample, oracles)}
    del first
    fps_one = F / (t_one * len(units))                       # whole job on one thread
    fps_all = F / (t_all * len(units) / n_s)                 # whole job, n_s units at a time
    log(f"[bench] oracle ingest: one unit stream {t_one:.1f}s on one thread; {n_s} streams {t_all:.1f}s on {threads} threads "
        f"-> whole job {fps_one:.1f} / {fps_all:.1f} frames/s")
    q_h = q_steps.float().cpu().numpy().astype(np.float64)        # [n][L][1][Hq][D]

    def one(lh, i):
        l, h = lh
        o, Ku, Vu = state[lh]
        ids, sc, tok, gap = o.retrieve(q_h[i, l], h, G, wl.top_k)
        orc.attend(q_h[i, l], Ku, Vu, tok, h, G)

    def timed(parallel):
        done, t0 = 0, time.perf_counter()
        with ThreadPoolExecutor(threads) as ex:
            while done < len(q_h) and (time.perf_counter() - t0) < budget_s:
                if parallel:
                    list(ex.map(lambda lh: one(lh, done), sample))
                else:
                    for lh in sample:
                        one(lh, done)
                done += 1
        return (time.perf_counter() - t0) / max(done, 1) * 1e6 * (len(units) / n_s), done

    us_one, n_one = timed(False)
    us_all, n_all = timed(True)
    return {"value": round(us_all, 1), "unit": "us", "cores": threads, "kind": "oracle",
            "sample": f"decode steps (retrieve + attend) on the whole streams of {n_s} of {len(units)} units, times "
                      f"scaled to all units: {n_all} steps on {threads} threads, {n_one} steps on one thread",
            "nproc": nproc,
            "value_one_thread": round(us_one, 1),
            "ingest_frames_per_s": round(fps_all, 2), "ingest_frames_per_s_one_thread": round(fps_one, 2),
            "ingest_sample": f"whole stream ({F} frames, re-clustering every {wl.recluster_every}) of {n_s} units on "
                             f"{threads} threads ({t_all:.1f} s) and of one unit on one thread ({t_one:.1f} s), "
                             f"scaled to all {len(units)} units"}


def host_leg_in_its_own_process(layers):
    """Config 3 needs tens of GB of pinned host memory next to an 18 GB cluster cache: it runs in a
    process of its own (started before this process touches the GPU) so that no other leg's
    allocations stand beside it.  Returns the leg's JSON (or an error record)."""
    cmd = [sys.executable, os.path.abspath(__file__), "--workload", "cfg3"] + (["--layers", str(layers)] if layers else [])
    try:
        p = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
        sys.stderr.write(p.stderr[-4000:])
        lines = [l for l in p.stdout.splitlines() if l.startswith("{")]
        if p.returncode != 0 or not lines:
            return {"error": f"cfg3 process ended with {p.returncode}: {p.stderr[-300:]}"}
        return json.loads(lines[-1])
    except Exception as ex:                          # noqa: BLE001
        return {"error": repr(ex)[:300]}


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py: this build runs on exactly one GPU (units are independent; "
              "no collective path exists); --gpus must be 1", file=sys.stderr)
        sys.exit(2)
    from paper_2604_10060_amd import inputs

    if args.workload == "cfg4":
        print(json.dumps(run_prefill_leg(check=args.check_units > 0)))
        return
    if args.workload == "prefetch":
        print(json.dumps(run_prefetch_leg(layers=args.layers or 3)))
        return
    if args.workload == "maintainer":
        print(json.dumps(run_maintainer_leg(layers=args.layers or 4, check=args.check_units > 0)))
        return
    if args.workload == "nested":
        print(json.dumps(run_nested_leg(layers=args.layers or 4, check=args.check_units > 0)))
        return
    if args.workload == "cfg3":
        print(json.dumps(run_host_leg(layers=args.layers, check=args.check_units > 0)))
        return
    wl = inputs.CONFIGS[int(args.workload[-1])]
    modified = bool(args.layers or args.frames)
    if args.layers:
        wl = wl.scaled(n_layers=args.layers)
    if args.frames:
        wl = wl.scaled(n_frames=args.frames)
    headline = args.workload == "cfg2" and not modified and not args.all_layers_call
    with_extra = headline and not args.no_extra
    extra = {} if with_extra else None
    if with_extra:          # first, while this process has not touched the GPU yet
        extra["cfg3_host_offload"] = host_leg_in_its_own_process(0)
    aug = (args.aug_window, args.aug_reps) if (args.aug_window or args.aug_reps) else None
    main_leg = run_leg(wl, steps=args.steps, warmup=args.warmup, all_layers=args.all_layers_call,
                       check_units=args.check_units,
                       cpu_seconds=0 if args.no_cpu_baseline else args.cpu_seconds, cpu_units=args.cpu_units,
                       calibrate=args.calibrate_copy, aug=aug, two_calls=args.two_calls,
                       traffic_lookup=not modified and aug is None, ingest_without_recluster=True)
    if with_extra:
        def keep(leg, *more):
            out = {"decode_step_us": round(leg["us_per_step"], 2), "config": leg["config"],
                   "step_us_median": leg["step_us_median"], "step_us_p95": leg["step_us_p95"],
                   "roofline": leg["roofline"], "step_hbm_gbps": leg["step_hbm_gbps"],
                   "step_hbm_frac": leg["step_hbm_frac"], "parity_spot_check": leg["parity_spot_check"]}
            out.update({k: leg[k] for k in more})
            return out
        # every leg in its own try block: none of them takes the headline line down
        try:
            leg = run_leg(inputs.CONFIGS[2], steps=args.steps, warmup=args.warmup, all_layers=True, check_units=1,
                          cpu_seconds=0)
            extra["cfg2_all_layers"] = keep(leg, "stream_kernel_gbps", "frac_of_stream_kernel", "question_ms")
        except Exception as ex:                      # noqa: BLE001
            extra["cfg2_all_layers"] = {"error": repr(ex)[:300]}
        for name, two in (("cfg1_decode_step", False), ("cfg1_retrieve_then_attend", True)):
            try:
                leg = run_leg(inputs.CONFIGS[1], steps=256, warmup=10, all_layers=False, check_units=1,
                              cpu_seconds=0, two_calls=two)
                extra[name] = keep(leg, "ingest_roofline", "question_ms")
            except Exception as ex:                  # noqa: BLE001
                extra[name] = {"error": repr(ex)[:300]}
        try:
            extra["cfg4_prefill_8_streams"] = run_prefill_leg()
        except Exception as ex:                      # noqa: BLE001
            extra["cfg4_prefill_8_streams"] = {"error": repr(ex)[:300]}
        try:
            leg = run_leg(inputs.CONFIGS[1], steps=256, warmup=10, all_layers=False,
                          check_units=1, cpu_seconds=0, aug=(16, True), traffic_lookup=False)
            extra["next2_augmentation_cfg1"] = {
                "augmentation": {"window_frames": 16, "global_reps": True},
                "decode_step_us": round(leg["us_per_step"], 2), "step_us_median": leg["step_us_median"],
                "step_us_p95": leg["step_us_p95"], "roofline": leg["roofline"],
                "question_ms": leg["question_ms"], "parity_spot_check": leg["parity_spot_check"]}
        except Exception as ex:                      # noqa: BLE001
            extra["next2_augmentation_cfg1"] = {"error": repr(ex)[:300]}
        try:
            extra["next1_maintainer"] = run_maintainer_leg()
        except Exception as ex:                      # noqa: BLE001
            extra["next1_maintainer"] = {"error": repr(ex)[:300]}
        try:
            extra["next4_nested_index"] = run_nested_leg()
        except Exception as ex:                      # noqa: BLE001
            extra["next4_nested_index"] = {"error": repr(ex)[:300]}
        try:
            import torch
            torch.cuda.empty_cache()
            extra["next3_cross_layer_prefetch"] = run_prefetch_leg(layers=2, steps=64, rhos=(0.95,))
        except Exception as ex:                      # noqa: BLE001
            extra["next3_cross_layer_prefetch"] = {"error": repr(ex)[:300]}
    us = main_leg.pop("us_per_step")
    result = {
        "metric": "decode_step_retrieve_attend_latency_us",
        "value": round(us, 3),
        "unit": "us",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(us / 1e3, 6),
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": wl.kv_dtype,
        "data": "synthetic",
    }
    result.update(main_leg)
    result["extra"] = extra
    print(json.dumps(result))


if __name__ == "__main__":
    main()

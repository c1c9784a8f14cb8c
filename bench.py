"""Benchmark of the radiance-cache hot path on one MI355X.

A step is one 1920x1080 frame of the cache: encode 2,073,600 synthetic query
records and run inference on them (one fused kernel), encode 65,536 training
records, shuffle them with the LCG and take four Adam steps on disjoint
batches of 16,384 records (Sec. 3.3 and 3.5 of the paper), all on one stream.  Inputs
are resident in HBM before the timed region.  The default form is FP32: FP32
weights, activations and sums, with the layer products on the FP32 matrix cores
(v_mfma_f32_16x16x4_f32; plain FP32 FMAs would cap at half that rate, since
packed FP32 is not used).  The FP16 and BF16 matrix-core forms run the same
frame and are reported under "forms", and so is the plain FP32 form with no
matrix instructions at all (fp32_valu, vector ALUs: the baseline the
matrix-core forms are compared with).  Prints one JSON line.

Each form first runs frames back to back for --settle-s seconds (the GPU's
clocks rise over the first tens of milliseconds of sustained load), then W
untimed warm-up frames, then K timed frames back to back between two device
synchronisations; per-component times come from events recorded in every timed
frame and read afterwards.

    python bench.py [--steps K] [--warmup W] [--settle-s S] [--form fp32|fp16|bf16]
                    [--no-forms] [--no-cpu-baseline] [--serve-requests R]
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

import synthdata as sd  # noqa: E402

METRIC = "MLP queries/s + train samples/s (64-wide, 5 hidden); p50/p99 serve latency"
N_QUERIES = 1920 * 1080
N_TRAIN_BATCHES = 4
TRAIN_BATCH = 16384
WIDTH, N_HIDDEN = 64, 5
FLOP_PER_QUERY = 2 * sd.n_params(WIDTH, N_HIDDEN)                 # 41,344
FLOP_PER_TRAIN_SAMPLE = 2 * (sd.n_params() + (sd.n_params() - 64 * 64) + sd.n_params())  # 115,840
# fp32_valu: plain FP32 FMAs on the vector ALUs without packed FP32, 256 CUs x 4 SIMDs x 16 lanes x 2 FLOP x 2.4 GHz
PEAK_TFLOPS = {"fp32": 157.3, "fp16": 2500.0, "bf16": 2500.0, "fp32_valu": 78.6}
BOUND = {"fp32": "mfma", "fp16": "mfma", "bf16": "mfma", "fp32_valu": "alu"}
QUERY_KERNEL = {"fp32": "k_fwd_raw_fp32", "fp16": "k_fwd_raw_mfma_fixed", "bf16": "k_fwd_raw_mfma_fixed",
                "fp32_valu": "k_fwd_raw_fp32_valu"}
MLP_KERNEL = {"fp32": "k_fwd_fp32", "fp16": "k_fwd_mfma_fixed", "bf16": "k_fwd_mfma_fixed", "fp32_valu": "k_fwd_fp32_valu"}
# The frame's training records go to the training kernels raw (encoded there,
# nrc_train_frame_raw) in every form.
RAW_TRAIN = {"fp32": True, "fp16": True, "bf16": True, "fp32_valu": True}
HBM_PEAK_GBS = 8000.0


def log(*a):
    print(*a, file=sys.stderr, flush=True)


KERNEL_SOURCES = {"k_fwd_raw_mfma_fixed": ["mlp_mfma.hip", "mfma_ops.h", "encode_impl.h", "nrc_internal.h"],
                  "k_fwd_raw_fp32": ["mlp_fp32.hip", "encode_impl.h", "nrc_internal.h"],
                  "k_fwd_raw_fp32_valu": ["mlp_fp32_valu.hip", "encode_impl.h", "nrc_internal.h"]}


def measured_traffic(kernel: str, form: str):
    """HBM bytes per launch from the rocprofv3 FETCH_SIZE / WRITE_SIZE summary in
    profiles/, scaled by the copy-kernel calibration recorded there; None when
    there is none or the kernel's sources changed since it was taken."""
    import glob
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES.get(kernel, []):
        with open(os.path.join(ROOT, "paper_2106_12372_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    digest = h.hexdigest()
    for path in glob.glob(os.path.join(ROOT, "profiles", "*.md")):
        with open(path) as fh:
            for line in fh:
                if not line.startswith("traffic:"):
                    continue
                kv = dict(tok.split("=", 1) for tok in line.split()[1:])
                if kv.get("kernel") == kernel and kv.get("form") == form and kv.get("src_sha256") == digest:
                    return float(kv["bytes_per_launch"])
    return None


def settle(step, seconds: float) -> int:
    """Runs frames back to back for `seconds` of wall time before the warm-up
    steps.  Under sustained load the GPU's clocks rise over the first tens of
    milliseconds (the fused query kernel goes from about 100 to under 80 us in
    FP16); a renderer calling the cache every frame runs at the settled rate,
    which is what the timed steps measure.  Returns the frames run."""
    import torch
    n, t0 = 0, time.perf_counter()
    while time.perf_counter() - t0 < seconds:
        for _ in range(10):
            step(None)
        torch.cuda.synchronize()
        n += 10
    return n


def frame_bench(form: str, steps: int, warmup: int, settle_s: float):
    import torch
    from paper_2106_12372_amd import nrc as N

    dev = torch.device("cuda", 0)
    cfg = N.make_config(width=WIDTH, n_hidden=N_HIDDEN, precision=form)
    cache = N.Cache(cfg, device=dev)
    cache.set_weights(sd.glorot_weights(WIDTH, N_HIDDEN))
    raw_q = torch.from_numpy(sd.raw_records(N_QUERIES, sd.SEED_QUERIES)).to(dev)
    raw_r_np = sd.raw_records(N_TRAIN_BATCHES * TRAIN_BATCH, sd.SEED_RECORDS)
    raw_r = torch.from_numpy(raw_r_np).to(dev)
    y = torch.from_numpy(sd.targets(raw_r_np)).to(dev)
    enc_q = torch.empty((N_QUERIES, 64), dtype=cache.enc_dtype, device=dev)
    enc_r = torch.empty((N_TRAIN_BATCHES * TRAIN_BATCH, 64), dtype=cache.enc_dtype, device=dev)
    rgb = torch.empty((N_QUERIES, 3), dtype=torch.float32, device=dev)
    n_rec = N_TRAIN_BATCHES * TRAIN_BATCH
    frame_scratch = N._aligned_bytes(N.nrc_frame_scratch_bytes(cfg, n_rec, N_TRAIN_BATCHES, TRAIN_BATCH), dev)
    stream = torch.cuda.current_stream(dev)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    frame_no = [0]
    last = {}

    def step(evs):
        if evs is not None:
            evs[0].record(stream)
        N.nrc_forward_raw(cache, raw_q, rgb=rgb)           # encode + inference, one kernel
        if evs is not None:
            evs[1].record(stream)
        # LCG shuffle, then 4 steps on disjoint batches, a new shuffle each frame
        if RAW_TRAIN[form]:
            # the training kernels encode the gathered raw records themselves
            last["loss"], last["skipped"] = N.nrc_train_frame_raw(cache, raw_r, y, steps=N_TRAIN_BATCHES,
                                                                  batch=TRAIN_BATCH, seed=frame_no[0],
                                                                  scratch=frame_scratch)
        else:
            N.nrc_encode(cache, raw_r, enc=enc_r)
            if evs is not None:
                evs[2].record(stream)
            last["loss"], last["skipped"] = N.nrc_train_frame(cache, enc_r, y, steps=N_TRAIN_BATCHES,
                                                              batch=TRAIN_BATCH, seed=frame_no[0],
                                                              scratch=frame_scratch)
        frame_no[0] += 1
        if evs is not None:
            evs[3].record(stream)

    settled = settle(step, settle_s)
    for _ in range(warmup):
        step(None)
    # The timed steps run back to back with nothing else on the stream; the
    # components are timed in a second pass with events between them (an event
    # between two kernels costs the stream a few microseconds).
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(steps):
        step(None)
    t_enq = time.perf_counter() - t0
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms = elapsed * 1e3 / steps
    evs = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(steps)]
    for k in range(steps):
        step(evs[k])
    torch.cuda.synchronize()
    if RAW_TRAIN[form]:
        # no record-encoding launch: the frame's training part runs from the
        # second event to the last
        comp = np.mean([[e[0].elapsed_time(e[1]), 0.0, e[1].elapsed_time(e[3])] for e in evs], axis=0)
    else:
        comp = np.mean([[e[i].elapsed_time(e[i + 1]) for i in range(3)] for e in evs], axis=0)

    # The same queries through the two-kernel path (encode to HBM, then inference).
    uevs = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(steps)]
    for e in uevs:
        e[0].record(stream)
        N.nrc_encode(cache, raw_q, enc=enc_q)
        e[1].record(stream)
        N.nrc_forward(cache, enc_q, rgb=rgb)
        e[2].record(stream)
    torch.cuda.synchronize()
    ue = np.mean([[e[0].elapsed_time(e[1]), e[1].elapsed_time(e[2])] for e in uevs], axis=0)

    t_q = comp[0] * 1e-3
    achieved = N_QUERIES * FLOP_PER_QUERY / t_q / 1e12
    enc_bytes = 2 if form in ("fp16", "bf16") else 4
    t_fwd = ue[1] * 1e-3
    out = {
        "form": form,
        "ms_per_step": ms,
        "queries_per_s": N_QUERIES / (ms * 1e-3),
        "train_samples_per_s": N_TRAIN_BATCHES * TRAIN_BATCH / (ms * 1e-3),
        # encode_records is 0 where the training kernels encode the raw records
        # (no launch of its own)
        "components_ms": {"query_pass_fused": comp[0], "encode_records": comp[1],
                          "shuffle_and_train_4_steps": comp[2]},
        "unfused_ms": {"encode_queries": ue[0], "forward": ue[1]},
        "query_pass_queries_per_s": N_QUERIES / t_q,
        "mlp_only_queries_per_s": N_QUERIES / t_fwd,
        "train_only_samples_per_s": N_TRAIN_BATCHES * TRAIN_BATCH / (comp[2] * 1e-3),
        "roofline": {
            "kernel": QUERY_KERNEL[form],
            "bound": BOUND[form],
            "achieved": achieved,
            "peak": PEAK_TFLOPS[form],
            "unit": "TFLOP/s",
            "frac": achieved / PEAK_TFLOPS[form],
            "traffic": measured_traffic(QUERY_KERNEL[form], form),
            "traffic_unit": "bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
            "flop_per_query": FLOP_PER_QUERY,
            "queries_per_launch": N_QUERIES,
            "avg_launch_ms": comp[0],
            "hbm_gbs_algorithmic": N_QUERIES * (56 + 12) / t_q / 1e9,
        },
        "mlp_only_roofline": {
            "kernel": MLP_KERNEL[form],
            "bound": BOUND[form],
            "achieved": N_QUERIES * FLOP_PER_QUERY / t_fwd / 1e12,
            "peak": PEAK_TFLOPS[form],
            "unit": "TFLOP/s",
            "frac": N_QUERIES * FLOP_PER_QUERY / t_fwd / 1e12 / PEAK_TFLOPS[form],
            "avg_launch_ms": ue[1],
            "hbm_gbs_algorithmic": N_QUERIES * (64 * enc_bytes + 12) / t_fwd / 1e9,
        },
        "final_loss": float(last["loss"][-1].item()),
        "skipped_steps": int(last["skipped"].sum().item()),
    }
    frame_flop = N_QUERIES * FLOP_PER_QUERY + N_TRAIN_BATCHES * TRAIN_BATCH * FLOP_PER_TRAIN_SAMPLE
    out["frame_tflops"] = frame_flop / (ms * 1e-3) / 1e12
    # the whole frame (query pass, record encoding, shuffle, four steps)
    # against the matrix-core peak of the form's arithmetic
    out["frame_roofline"] = {"flop_per_frame": frame_flop, "achieved": out["frame_tflops"],
                             "peak": PEAK_TFLOPS[form], "unit": "TFLOP/s",
                             "frac": out["frame_tflops"] / PEAK_TFLOPS[form]}
    out["settle_frames"] = settled
    out["host_enqueue_ms_per_step"] = t_enq * 1e3 / steps
    out["query_pass_by_preset_ms"] = preset_bench(form, raw_q, rgb, steps)
    return out


def preset_bench(form: str, raw_q, rgb, steps: int):
    """The fused query pass under each encoding preset: config (sin and cos of 6
    octaves), paper (12 sines, quartic one-blobs), paper-tri (12 triangle waves,
    the cheap primitive of Sec. 5) and paper-gauss (Gaussian one-blobs, the
    kernel the quartic replaces); average kernel time in ms."""
    import torch
    from paper_2106_12372_amd import nrc as N

    stream = torch.cuda.current_stream(raw_q.device)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    out = {}
    for name, preset in (("config", N.NRC_PRESET_CONFIG), ("paper", N.NRC_PRESET_PAPER),
                         ("paper_tri", N.NRC_PRESET_PAPER_TRI), ("paper_gauss", N.NRC_PRESET_PAPER_GAUSS)):
        cache = N.Cache(N.make_config(width=WIDTH, n_hidden=N_HIDDEN, precision=form, enc_preset=preset),
                        device=raw_q.device)
        cache.set_weights(sd.glorot_weights(WIDTH, N_HIDDEN))
        # creating the cache idles the GPU: settle the clocks again first
        t0 = time.perf_counter()
        while time.perf_counter() - t0 < 0.2:
            for _ in range(20):
                N.nrc_forward_raw(cache, raw_q, rgb=rgb)
            torch.cuda.synchronize()
        evs = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(steps + 2)]
        for e in evs:
            e[0].record(stream)
            N.nrc_forward_raw(cache, raw_q, rgb=rgb)
            e[1].record(stream)
        torch.cuda.synchronize()
        t = sum(e[0].elapsed_time(e[1]) for e in evs[2:])
        out[name] = t / steps
    return out


def serve_bench(form: str, n_requests: int, serial: bool, loads=(0.8,), capacity_rps=None,
                arena: int = 64 << 30):
    """Serving form: 8 resident caches, a Poisson stream mixing inference requests
    (log-uniform 1k..2M queries) and 16,384-record training steps 60:40, admission
    against a device arena (64 GB by default).  First the closed-loop capacity
    (every request submitted at once), then an open-loop run at each of `loads`
    x capacity with Poisson arrivals; latency is submit -> completion observed
    by the server.  `serial` serves one request at a time on one stream."""
    import torch
    from paper_2106_12372_amd import nrc as N

    dev = torch.device("cuda", 0)
    n_caches = 8
    cfg = N.make_config(width=WIDTH, n_hidden=N_HIDDEN, precision=form)
    trace = sd.serve_trace(n_requests, n_caches=n_caches, seed=sd.SEED_SERVE)
    enc_cache = N.Cache(cfg, device=dev)
    enc_pool = N.nrc_encode(enc_cache, torch.from_numpy(sd.raw_records(2_000_000, sd.SEED_QUERIES)).to(dev))
    train_enc, train_tgt = [], []
    for c in range(n_caches):
        raw = sd.raw_records(TRAIN_BATCH, 1000 + c)
        train_enc.append(N.nrc_encode(enc_cache, torch.from_numpy(raw).to(dev)))
        train_tgt.append(torch.from_numpy(sd.targets(raw)).to(dev))
    rgb_out = [torch.empty((2_000_000, 3), dtype=torch.float32, device=dev) for _ in range(n_caches)]
    torch.cuda.synchronize()
    srv = N.Server(n_caches, cfg, arena_bytes=arena, n_streams=1 if serial else 4,
                   max_inflight=1 if serial else 64, device=dev)
    for c in range(n_caches):
        srv.set_weights(c, sd.glorot_weights(WIDTH, N_HIDDEN, seed=100 + c))

    def submit(r):
        c = r["cache"]
        if r["kind"] == "infer":
            n = min(r["n"], 2_000_000)
            return srv.submit_infer(c, enc_pool[:n], rgb_out[c][:n])
        return srv.submit_train(c, train_enc[c], train_tgt[c])

    def collect(tickets):
        res = []
        for t in tickets:
            r = srv.poll(t)
            while r is None:
                r = srv.poll(t)
            res.append(r)
        return res

    n_q = sum(min(r["n"], 2_000_000) for r in trace if r["kind"] == "infer")
    n_s = sum(r["n"] for r in trace if r["kind"] == "train")
    # warm-up, then closed-loop capacity
    collect([submit(r) for r in trace[:50]])
    t0 = time.perf_counter()
    res = collect([submit(r) for r in trace])
    makespan = max(x["t_done"] for x in res) - min(x["t_submit"] for x in res)
    cap_rps = len(trace) / makespan
    # open loop at load x capacity (of the reference server when given)
    gaps = np.diff([0.0] + [r["t_arrive"] for r in trace])
    runs = []
    for load in loads:
        rate = load * (capacity_rps if capacity_rps else cap_rps)
        arrivals = np.cumsum(gaps / gaps.mean() / rate)
        tickets = []
        t0 = time.perf_counter()
        for k, r in enumerate(trace):
            while time.perf_counter() - t0 < arrivals[k]:
                pass
            tickets.append(submit(r))
        res = collect(tickets)
        lat = np.array([x["t_done"] - x["t_submit"] for x in res]) * 1e3
        lat_inf = np.array([x["t_done"] - x["t_submit"] for x, r in zip(res, trace) if r["kind"] == "infer"]) * 1e3
        lat_tr = np.array([x["t_done"] - x["t_submit"] for x, r in zip(res, trace) if r["kind"] == "train"]) * 1e3
        span = max(x["t_done"] for x in res) - min(x["t_submit"] for x in res)
        runs.append({
            "load": load, "offered_requests_per_s": rate,
            "p50_ms": float(np.percentile(lat, 50)), "p99_ms": float(np.percentile(lat, 99)),
            "p50_infer_ms": float(np.percentile(lat_inf, 50)), "p99_infer_ms": float(np.percentile(lat_inf, 99)),
            "p50_train_ms": float(np.percentile(lat_tr, 50)), "p99_train_ms": float(np.percentile(lat_tr, 99)),
            "queries_per_s": n_q / span, "train_samples_per_s": n_s / span,
            "failed": int(sum(1 for x in res if x["status"] != 0)),
        })
    srv.close()
    out = {
        "form": form, "serial": serial, "requests": len(trace), "caches": n_caches,
        "arena_gb": arena / 2 ** 30,
        "capacity": {"requests_per_s": cap_rps, "queries_per_s": n_q / makespan,
                     "train_samples_per_s": n_s / makespan, "makespan_ms": makespan * 1e3},
        "open_loop": runs,
    }
    main_run = runs[min(range(len(runs)), key=lambda i: abs(runs[i]["load"] - 0.8))]
    out.update({k: main_run[k] for k in ("offered_requests_per_s", "p50_ms", "p99_ms", "failed")})
    return out


def cpu_baseline():
    """The FP64 oracle on the host cores: one full frame (encode + inference of
    2,073,600 queries, encode of 65,536 records, shuffle, four training steps)."""
    from oracle import nrc_oracle as O
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:  # pragma: no cover
        threads = len(os.sched_getaffinity(0))
    raw_q = sd.raw_records(N_QUERIES, sd.SEED_QUERIES)
    raw_r = sd.raw_records(N_TRAIN_BATCHES * TRAIN_BATCH, sd.SEED_RECORDS)
    y = sd.targets(raw_r).astype(np.float64)
    st = O.CacheState(sd.glorot_weights(WIDTH, N_HIDDEN))
    # whole frames until at least 10 s of host work (at most 3 frames)
    frames, t0 = 0, time.perf_counter()
    while frames < 3 and (frames == 0 or time.perf_counter() - t0 < 10.0):
        q_enc = O.encode(raw_q)
        r_enc = O.encode(raw_r)
        O.frame_shuffled(st, q_enc, r_enc, y, N_TRAIN_BATCHES, TRAIN_BATCH, frames)
        frames += 1
    t = (time.perf_counter() - t0) / frames
    out = {"value": N_QUERIES / t, "unit": "queries/s", "cores": int(threads), "kind": "oracle",
           "sample": f"{frames} full frame{'s' if frames > 1 else ''} (mean time per frame): FP64 NumPy "
                     "encode + inference of "
                     "2,073,600 queries, encode of 65,536 records, LCG shuffle, four 16,384-record "
                     "training steps",
           "seconds": t, "frames": frames, "train_samples_per_s": N_TRAIN_BATCHES * TRAIN_BATCH / t}
    out["single_thread"] = cpu_baseline_single_thread(raw_q, raw_r, y, st)
    return out


def cpu_baseline_single_thread(raw_q, raw_r, y, st):
    """The same oracle on one host thread, on a sample of the frame: encode +
    inference of the first 131,072 queries (1/16 of the frame) and one
    16,384-record training step, scaled to a whole frame (16 x the query sample
    plus four steps)."""
    from oracle import nrc_oracle as O
    from threadpoolctl import threadpool_limits
    nq = 131072
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        O.predict(st, O.encode(raw_q[:nq]))
        tq = time.perf_counter() - t0
        st1 = O.CacheState(st.w.copy())
        t0 = time.perf_counter()
        O.train_step(st1, O.encode(raw_r[:TRAIN_BATCH]), y[:TRAIN_BATCH])
        ts = time.perf_counter() - t0
    t = tq * (N_QUERIES / nq) + N_TRAIN_BATCHES * ts
    return {"value": N_QUERIES / t, "unit": "queries/s", "cores": 1, "kind": "oracle",
            "sample": "one thread: encode + inference of 131,072 queries and one 16,384-record training "
                      "step, scaled to a frame (16 x queries + 4 x step)",
            "seconds_per_frame": t, "query_sample_s": tq, "train_step_s": ts}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--settle-s", type=float, default=0.5,
                    help="seconds of back-to-back frames before the warm-up steps (clocks settle)")
    ap.add_argument("--form", default="fp32", choices=["fp32", "fp16", "bf16", "fp32_valu"])
    ap.add_argument("--no-forms", action="store_true", help="skip the other precision forms")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--calib-copy", action="store_true",
                    help="also run a plain 256 MiB device copy (reference for HBM byte counters)")
    ap.add_argument("--serve-requests", type=int, default=2000,
                    help="requests in the serving trace (0 skips the serving run)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU; --gpus {args.gpus} is not supported (the cache is a "
              "single-GPU workload; see the sharding notes in the design document)", file=sys.stderr)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    torch.cuda.set_device(0)

    if args.calib_copy:
        src = torch.ones(64 << 20, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    log(f"frame bench: form {args.form}, {args.settle_s} s settle, {args.warmup} warmup + "
        f"{args.steps} timed steps")
    main_res = frame_bench(args.form, args.steps, args.warmup, args.settle_s)
    forms = {}
    if not args.no_forms:
        for f in ("fp32", "fp16", "bf16", "fp32_valu"):
            if f == args.form:
                continue
            log(f"frame bench: form {f}")
            forms[f] = frame_bench(f, args.steps, args.warmup, args.settle_s)
    serve = None
    if args.serve_requests > 0:
        log(f"serving: 8 caches, fp16, {args.serve_requests} requests")
        mix = serve_bench("fp16", args.serve_requests, serial=False, loads=(0.5, 0.8, 0.95))
        log("serving: 8 caches, fp16, 512 MB arena (admission by memory binds)")
        small = serve_bench("fp16", args.serve_requests, serial=False, loads=(0.8,), arena=512 << 20)
        log("serving: serial plain fp32 (vector ALUs), same trace and offered load")
        ser = serve_bench("fp32_valu", args.serve_requests, serial=True, loads=(0.8,),
                          capacity_rps=mix["capacity"]["requests_per_s"])
        serve = {"continuous_fp16": mix, "continuous_fp16_512mb_arena": small, "serial_fp32_valu": ser,
                 "p50_ms": mix["p50_ms"], "p99_ms": mix["p99_ms"]}
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline: oracle on one frame")
        cpu = cpu_baseline()
    res = {
        "metric": METRIC,
        "value": main_res["queries_per_s"],
        "unit": "queries/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "settle_s": args.settle_s,
        "ms_per_step": main_res["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp32": "f32", "fp16": "f16", "bf16": "bf16", "fp32_valu": "f32"}[args.form],
        "data": "synthetic",
        "config": {"workload": f"1920x1080 frame: {N_QUERIES} queries (encode + inference) and "
                               f"{N_TRAIN_BATCHES}x{TRAIN_BATCH}-record training steps, {args.form} form",
                   "width": WIDTH, "n_hidden": N_HIDDEN, "queries": N_QUERIES,
                   "train_batches": N_TRAIN_BATCHES, "train_batch": TRAIN_BATCH, "form": args.form,
                   "products": {"fp32": "FP32 weights and activations on the FP32 matrix cores "
                                        "(v_mfma_f32_16x16x4_f32), not the vector ALUs",
                                "fp16": "FP16 matrix cores, FP32 accumulation",
                                "bf16": "BF16 matrix cores, FP32 accumulation",
                                "fp32_valu": "FP32 on the vector ALUs, no matrix instructions"}[args.form],
                   "training_records": ("raw, encoded inside the training kernels" if RAW_TRAIN[args.form]
                                        else "encoded by a separate pass, then trained")},
        "train_samples_per_s": main_res["train_samples_per_s"],
        "components_ms": main_res["components_ms"],
        "unfused_ms": main_res["unfused_ms"],
        "mlp_only_queries_per_s": main_res["mlp_only_queries_per_s"],
        "train_only_samples_per_s": main_res["train_only_samples_per_s"],
        "frame_tflops": main_res["frame_tflops"],
        "query_pass_by_preset_ms": main_res["query_pass_by_preset_ms"],
        "roofline": main_res["roofline"],
        "frame_roofline": main_res["frame_roofline"],
        "cpu_baseline": cpu,
        "forms": forms,
        "serve": serve,
        # the paper's own timings on its GPU (half precision), context only: not this
        # metric's baseline, hence vs_baseline stays null
        "paper_context": {
            "gpu": "RTX 3090", "precision": "fp16", "query_pass_ms": 1.59, "train_4_steps_ms": 1.11,
            "frame_ms": 2.70,
            "frame_time_ratio_fp16": (2.70 / forms["fp16"]["ms_per_step"]) if "fp16" in forms else None,
            "frame_time_ratio_bf16": (2.70 / forms["bf16"]["ms_per_step"]) if "bf16" in forms else None,
        },
    }
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()

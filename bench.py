#!/usr/bin/env python3
"""Benchmark of the hybrid tree attention verify call on one MI355X.

One "step" is one pass of the whole hot path -- tree mask, split-KV attention over the
cached keys, masked tree attention, LSE merge -- through ls_hybrid_tree_attn, on synthetic
inputs of the headline shape (8B-class GQA, 32k-token prefix, 64 tree tokens, bf16), already
resident in HBM.  K/V are rotated over enough independent copies (>= 1 GiB) that no call
finds its keys in the 256 MB Infinity Cache left there by an earlier call.

Prints ONE JSON line.  `value` is microseconds per verify call (whole job, wall clock over
the timed steps).  `roofline` is for the dominant kernel (the cached-key attention), timed
alone with HIP events on the stream it runs on.  `cpu_baseline` is the CPU oracle timed on
the host cores for the same workload.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published
MFMA_BF16_PEAK_TFLOPS = 2500.0  # MI355X dense bf16, published

# HBM bytes per launch of the cached-key kernel (fetched + written) from the rocprofv3 FETCH_SIZE /
# WRITE_SIZE runs summarised in profiles/whole_call_kernels_mi355x.md, scaled by the copy calibration.
# Hardware counters cannot be read while this script runs: the figure is copied from that
# profile and labelled so in the output; None for workloads without a committed profile.
PROFILED_TRAFFIC_BYTES = {"C3": 138834985 + 17079706,       # fetched + written by the cached-key kernel on its own
                          "B3": 146517174 + 9060352, "C5": 779084476 + 36045005, "L3": 151416787 + 17040486,
                          "C2": 38203094 + 8519885, "C4": 270950050 + 2129920}
PROFILED_TRAFFIC_SOURCE = ("profiles/whole_call_kernels_mi355x.md (rocprofv3 --pmc FETCH_SIZE and WRITE_SIZE of the cached-key "
                           "kernel launched alone, scaled by the copy calibration; not this run)")
PREWARM_SECONDS = 0.35         # untimed calls before --warmup: the shader clock needs ~0.2 s of work to settle


def algorithmic_bytes_prefix(w, prefix_lens):
    """Bytes the cached-key kernel must move per launch: K and V rows of every KV head once,
    plus the queries.  Split partials are overhead and not counted."""
    e = 4 if w.dtype == "f32" else 2
    total = 0
    for p in prefix_lens:
        total += 2 * w.n_kv_heads * int(p) * w.head_dim * e + w.n_q_heads * w.n_tree * w.head_dim * e
    return total


def algorithmic_bytes_call(w, prefix_lens):
    e = 4 if w.dtype == "f32" else 2
    total = 0
    for p in prefix_lens:
        total += (2 * w.n_kv_heads * int(p) * w.head_dim * e + 2 * w.n_kv_heads * w.n_tree * w.head_dim * e +
                  2 * w.n_q_heads * w.n_tree * w.head_dim * e + w.n_q_heads * w.n_tree * 4 + w.n_tree * 4)
    return total


def flops_prefix(w, prefix_lens):
    return sum(4 * w.n_q_heads * w.n_tree * int(p) * w.head_dim for p in prefix_lens)


def bench_accept_commit(args, w):
    """Workloads of kind "accept": greedy tree acceptance followed by the KV commit of the accepted
    path, timed as one step.  Both kernels are latency-bound (a tree has at most 128 nodes)."""
    import numpy as np
    import torch

    from paper_2502_17421_amd import binding as ls
    from paper_2502_17421_amd import synth

    rng = np.random.default_rng(w.seed)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[w.dtype]
    e = 4 if w.dtype == "f32" else 2
    cap = w.prefix_hi + w.n_tree
    parents, draft, target, plens = [], [], [], []
    for b in range(w.batch):
        par = synth.tree_constrained(rng, w.n_tree, w.max_depth, w.max_children)
        d, g = synth.make_tokens(rng, par, 32000, 0.7)
        parents.append(par), draft.append(d), target.append(g)
        plens.append(int(rng.integers(w.prefix_lo, w.prefix_hi + 1)))
    parents, draft, target = np.stack(parents), np.stack(draft), np.stack(target)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    kc = torch.zeros((w.batch, w.n_kv_heads, cap, w.head_dim), dtype=dt, device="cuda")
    vc = torch.zeros_like(kc)
    kt = torch.randn((w.batch, w.n_kv_heads, w.n_tree, w.head_dim), device="cuda").to(dt)
    vt = torch.randn((w.batch, w.n_kv_heads, w.n_tree, w.head_dim), device="cuda").to(dt)
    q = torch.zeros((w.batch, w.n_q_heads, w.n_tree, w.head_dim), dtype=dt, device="cuda")
    desc = ls.make_desc(q, kc, vc, kt, vt, q, cap)
    d_par, d_draft, d_target, d_plens = dev(parents), dev(draft), dev(target), dev(plens)
    path = torch.empty((w.batch, w.n_tree), dtype=torch.int32, device="cuda")
    n = torch.empty((w.batch,), dtype=torch.int32, device="cuda")
    nxt, new_lens, err = torch.empty_like(n), torch.empty_like(n), torch.empty_like(n)
    stream = torch.cuda.current_stream()

    def step():
        ls.ls_tree_accept_greedy(d_par, d_draft, d_target, path, n, nxt, err, stream=stream)
        ls.ls_kv_commit(desc, kt, vt, path, n, d_plens, kc, vc, new_lens, err, stream=stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    us = (time.perf_counter() - t0) * 1e6 / args.steps
    lens = n.cpu().numpy()
    moved = int(lens.sum()) * 2 * w.n_kv_heads * w.head_dim * e * 2   # K and V rows, read + written
    cpu = None
    if not args.no_cpu_baseline:
        import oracle   # test infrastructure; imported for this leg only
        reps = 2000
        t0 = time.perf_counter()
        for _ in range(reps):
            for b in range(w.batch):
                oracle.tree_accept_greedy(parents[b], draft[b], target[b])
        cpu = {"value": (time.perf_counter() - t0) * 1e6 / reps, "unit": "us per acceptance of the batch", "cores": 1,
               "kind": "oracle", "sample": f"{reps} repetitions of the acceptance walk over the same {w.batch} tree(s)"}
        for b in range(w.batch):
            rp, rn, _ = oracle.tree_accept_greedy(parents[b], draft[b], target[b])
            assert rn == lens[b] and rp.tolist() == path[b].cpu().tolist()
    print(json.dumps({
        "metric": f"us per acceptance + KV commit (workload {w.name})", "value": us, "unit": "us", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": us * 1e-3, "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "int32 / " + w.dtype, "data": "synthetic",
        "config": {"workload": f"{w.name}: batch {w.batch}, {w.n_kv_heads} kv heads, head_dim {w.head_dim}, n_tree "
                               f"{w.n_tree}, accepted path lengths {lens.tolist()}"},
        "roofline": {"bound": "hbm", "achieved": moved / us * 1e-3, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": moved / us * 1e-3 / HBM_PEAK_GBS, "traffic": None,
                     "note": "two launches of a few microseconds each: launch latency, not bandwidth, sets the time"},
        "cpu_baseline": cpu}))


class ClockSampler:
    """Samples the shader clock and board power the driver reports (sysfs) while a timed region runs."""

    def __init__(self, period_s=0.001):
        import glob
        import threading
        self.sclk_files = glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk")[:1]
        self.power_files = glob.glob("/sys/class/drm/card*/device/hwmon/*/power1_input")[:1]
        self.period, self.sclk, self.power = period_s, [], []
        self._stop = threading.Event()
        self._thread = threading.Thread(target=self._run, daemon=True)

    def _run(self):
        while not self._stop.is_set():
            try:
                for f in self.sclk_files:
                    for line in open(f).read().splitlines():
                        if line.rstrip().endswith("*"):
                            self.sclk.append(int("".join(ch for ch in line.split(":")[1] if ch.isdigit())))
                for f in self.power_files:
                    self.power.append(int(open(f).read()) / 1e6)
            except (OSError, ValueError, IndexError):
                pass
            self._stop.wait(self.period)

    def __enter__(self):
        self._thread.start()
        return self

    def __exit__(self, *exc):
        self._stop.set()
        self._thread.join(timeout=1.0)

    def summary(self):
        def stats(v):
            v = sorted(v)
            return {"n": len(v), "min": v[0], "median": v[len(v) // 2], "max": v[-1]} if v else None
        return {"sclk_mhz": stats(self.sclk), "power_w": stats(self.power),
                "source": "sysfs pp_dpm_sclk / hwmon power1_input, sampled from the start of the pre-warm to the end "
                          "of the timed steps"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    # Whatever --warmup says, PREWARM_SECONDS of untimed calls run first (the first calls after
    # start-up run about 15 % slower while the clocks ramp): a short run gives the same figure
    # as a long one.
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=100)
    ap.add_argument("--workload", default="C3",
                    help="C1..C5 (the headline metric is quoted on C3); D1, D2: cross-attention over the cache only; "
                         "A3, A5: greedy acceptance + KV commit; W1: draft self-attention; H3: C3 in fp16; "
                         "L3: C3 with a 256-node tree; B3: C3 with the 68-node beam tree")
    ap.add_argument("--page-size", type=int, default=0,
                    help="keep the cache in shuffled pages of this many rows and call ls_hybrid_tree_attn_paged")
    ap.add_argument("--single-launch", action="store_true",
                    help="time ls_hybrid_tree_attn_fused (the workgroups of a query block share its merge) instead "
                         "of the two-launch call")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-hot", action="store_true", help="skip the timing with one K/V copy (cache-resident)")
    ap.add_argument("--token-major", action="store_true",
                    help="store Q, K, V and out as [B,L,H,D] (each head's row a run of D elements) and pass strides")
    ap.add_argument("--no-graph", action="store_true",
                    help="skip the timing of replays of a HIP graph that holds one cycle over the K/V copies")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run 10 device copies of 512 MiB (reference for scaling rocprofv3 FETCH_SIZE / WRITE_SIZE)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        sys.exit("bench.py: this build runs on one GPU only (no sharding, no collectives); use --gpus 1")

    import numpy as np
    import torch

    import ctypes

    from paper_2502_17421_amd import binding as ls
    from paper_2502_17421_amd import build as ls_build
    from paper_2502_17421_amd import synth
    from paper_2502_17421_amd.device_batch import DeviceBatch

    if not os.path.exists(ls.LIB_PATH):
        ls_build.build_library()
    if not os.path.exists(ls_build.PROBE_LIB_PATH):
        ls_build.build_probe_library()
    ls.lib()
    probe = ctypes.CDLL(ls_build.PROBE_LIB_PATH)   # measurement helpers, a library of their own
    probe.ls_probe_stream_read.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p]
    probe.ls_probe_mfma_loop.argtypes = [ctypes.c_int32, ctypes.c_void_p, ctypes.POINTER(ctypes.c_int64), ctypes.c_void_p]
    probe.ls_probe_mfma_loop_varied.argtypes = probe.ls_probe_mfma_loop.argtypes
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)

    if args.copy_calibration:
        n = 512 << 20
        src = torch.full((n,), 3, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_calibration": {"bytes_read_per_copy": n, "bytes_written_per_copy": n, "copies": 10}}))
        return

    w = synth.WORKLOADS[args.workload]
    if w.kind == "accept":
        return bench_accept_commit(args, w)
    batch = synth.make_batch(w, "iid")
    db = DeviceBatch(batch, token_major=args.token_major)
    plens = batch.prefix_lens.tolist()

    # cold-cache rotation: independent K/V copies totalling >= 1 GiB
    kv_bytes = db.k_cache.numel() * db.k_cache.element_size() * 2
    n_rot = max(2, -(-(1 << 30) // kv_bytes))
    # (a copy keeps the storage order of its source: same strides for every copy)
    same_order = lambda x: torch.empty_strided(x.shape, x.stride(), dtype=x.dtype, device=x.device).copy_(x)
    k_rot = [db.k_cache] + [same_order(db.k_cache) for _ in range(n_rot - 1)]
    v_rot = [db.v_cache] + [same_order(db.v_cache) for _ in range(n_rot - 1)]
    ws = torch.empty(ls.ls_workspace_bytes(db.desc), dtype=torch.uint8, device="cuda")
    ls.ls_workspace_init(ws)   # the arrival counters of --single-launch; nothing else reads them
    n_splits = ls.ls_prefix_num_splits(db.desc)
    stream = torch.cuda.current_stream()

    table = None
    if args.page_size:
        # the same rows scattered over shuffled pages [page, Hkv, page_size, D]; one table for all copies
        ps = args.page_size
        assert w.kind == "verify" and batch.max_prefix_len % ps == 0, "paged timing: whole pages, verify workloads"
        assert not args.token_major, "paged timing keeps each page head-major"
        per_seq = batch.max_prefix_len // ps
        n_pages = w.batch * per_seq
        perm = torch.randperm(n_pages, generator=torch.Generator().manual_seed(w.seed)).cuda()
        table = perm.view(w.batch, per_seq).to(torch.int32).contiguous()

        def to_pages(x):   # [B,Hkv,P,D] -> [B*P/ps, Hkv, ps, D] in table order
            b, h, pl, d = x.shape
            pages = x.view(b, h, per_seq, ps, d).permute(0, 2, 1, 3, 4).reshape(n_pages, h, ps, d)
            out_pages = torch.empty_like(pages)
            out_pages[perm] = pages
            return out_pages

        k_rot_c, v_rot_c = k_rot, v_rot      # the contiguous copies still serve the kernel-alone timing
        k_rot = [to_pages(x) for x in k_rot]
        v_rot = [to_pages(x) for x in v_rot]
        paged_desc = ls.make_desc(db.q, k_rot[0], v_rot[0], db.k_tree, db.v_tree, db.out, batch.max_prefix_len)

    def call(i, r=None, stream=stream):
        r = i % n_rot if r is None else r
        if table is not None:
            ls.ls_hybrid_tree_attn_paged(paged_desc, db.q, k_rot[r], v_rot[r], table, args.page_size, db.prefix_lens,
                                         db.k_tree, db.v_tree, db.parents, db.out, db.lse, ws, stream=stream)
        elif w.kind == "cross":  # cached keys only: the draft model's cross-attention over the target cache
            ls.ls_cache_attn(db.desc, db.q, k_rot[r], v_rot[r], db.prefix_lens, db.out, db.lse, ws, stream=stream)
        elif args.single_launch:
            ls.ls_hybrid_tree_attn_fused(db.desc, db.q, k_rot[r], v_rot[r], db.prefix_lens, db.k_tree, db.v_tree,
                                         db.parents, db.out, db.lse, ws, stream=stream)
        else:
            ls.ls_hybrid_tree_attn(db.desc, db.q, k_rot[r], v_rot[r], db.prefix_lens, db.k_tree, db.v_tree,
                                   db.parents, db.out, db.lse, ws, stream=stream)

    def prewarm(fn):
        """Untimed calls for PREWARM_SECONDS; returns how many were made."""
        n, t_end = 0, time.perf_counter() + PREWARM_SECONDS
        while time.perf_counter() < t_end:
            for _ in range(50):
                fn(n)
                n += 1
            torch.cuda.synchronize()
        return n

    with ClockSampler() as sampler:
        prewarm_calls = prewarm(call)
        for i in range(args.warmup):
            call(i)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(args.steps):
            call(i)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
    us_per_call = wall / args.steps * 1e6

    # per-call latency distribution (events around each call)
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    for i, (a, b) in enumerate(evs):
        a.record(stream)
        call(i)
        b.record(stream)
    torch.cuda.synchronize()
    lat = np.asarray([a.elapsed_time(b) * 1e3 for a, b in evs])

    # the dominant kernel alone, in the configuration the whole call launches it in (library
    # split count, partials in the problem's dtype): HIP events on its stream around the whole
    # timed region of back-to-back launches, so the per-launch figure excludes the ~6 us that an
    # event pair around a single launch adds on this stack
    part_dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[w.dtype]
    o_part = torch.empty((w.batch, w.n_q_heads, n_splits, w.n_tree, w.head_dim), dtype=part_dt, device="cuda")
    l_part = torch.empty((w.batch, w.n_q_heads, n_splits, w.n_tree), dtype=torch.float32, device="cuda")

    kc_alone, vc_alone = (k_rot_c, v_rot_c) if table is not None else (k_rot, v_rot)

    def prefix_only(i):
        r = i % n_rot
        ls.ls_prefix_attn_splitkv(db.desc, db.q, kc_alone[r], vc_alone[r], db.prefix_lens, 0, o_part, l_part,
                                  stream=stream)

    prewarm(prefix_only)
    for i in range(args.warmup):
        prefix_only(i)
    torch.cuda.synchronize()
    k0, k1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    k0.record(stream)
    for i in range(args.steps):
        prefix_only(i)
    k1.record(stream)
    torch.cuda.synchronize()
    kernel_us = k0.elapsed_time(k1) * 1e3 / args.steps
    for i, (a, b) in enumerate(evs):
        a.record(stream)
        prefix_only(i)
        b.record(stream)
    torch.cuda.synchronize()
    klat = np.asarray([a.elapsed_time(b) * 1e3 for a, b in evs])

    hot_us = None
    if not args.no_hot:
        prewarm(lambda i: call(i, 0))
        for i in range(args.warmup):
            call(i, 0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(args.steps):
            call(i, 0)
        torch.cuda.synchronize()
        hot_us = (time.perf_counter() - t0) / args.steps * 1e6

    graph_us = None
    if not args.no_graph:
        # one cycle over the K/V copies recorded once; a replay issues it with no host work per call
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            cap = torch.cuda.current_stream()
            for r in range(n_rot):
                call(r, r, cap)
        reps = max(1, args.steps // n_rot)
        prewarm(lambda i: g.replay() if i % n_rot == 0 else None)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            g.replay()
        torch.cuda.synchronize()
        graph_us = (time.perf_counter() - t0) / (reps * n_rot) * 1e6

    # what this card reaches in practice: a pure streaming read of 1 GiB, a bf16 MFMA issue loop
    buf = torch.full((1 << 30,), 1, dtype=torch.uint8, device="cuda")
    sink = torch.zeros(64, dtype=torch.float32, device="cuda")
    p0, p1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    raw_stream = ctypes.c_void_p(stream.cuda_stream)

    def stream_read():
        assert probe.ls_probe_stream_read(ctypes.c_void_p(buf.data_ptr()), buf.numel(), ctypes.c_void_p(sink.data_ptr()),
                                          raw_stream) == 0

    def mfma_loop(iters):
        fl_out = ctypes.c_int64(0)
        assert probe.ls_probe_mfma_loop(iters, ctypes.c_void_p(sink.data_ptr()), ctypes.byref(fl_out), raw_stream) == 0
        return int(fl_out.value)

    for _ in range(3):
        stream_read()
    p0.record(stream)
    for _ in range(10):
        stream_read()
    p1.record(stream)
    torch.cuda.synchronize()
    read_gbs = 10 * buf.numel() / (p0.elapsed_time(p1) * 1e-3) / 1e9
    del buf
    mfma_loop(2000)
    p0.record(stream)
    mf = mfma_loop(20000)
    p1.record(stream)
    torch.cuda.synchronize()
    mfma_tflops = mf / (p0.elapsed_time(p1) * 1e-3) / 1e12
    # the same loop kept up for about half a second (the board settles at a lower clock under load
    # that lasts; the short run above is over before it does): rate of the last fifth
    n_sus = max(10, int(0.5 / (p0.elapsed_time(p1) * 1e-3)))
    for _ in range(n_sus - n_sus // 5):
        mfma_loop(20000)
    p0.record(stream)
    for _ in range(n_sus // 5):
        mf = mfma_loop(20000)
    p1.record(stream)
    torch.cuda.synchronize()
    mfma_sustained = (n_sus // 5) * mf / (p0.elapsed_time(p1) * 1e-3) / 1e12
    # and on operands that vary from lane to lane and instruction to instruction, as real keys
    # and values do (constant operands draw far less power): sustained rate again
    def mfma_loop_varied(iters):
        fl_out = ctypes.c_int64(0)
        assert probe.ls_probe_mfma_loop_varied(iters, ctypes.c_void_p(sink.data_ptr()), ctypes.byref(fl_out),
                                               raw_stream) == 0
        return int(fl_out.value)

    for _ in range(n_sus - n_sus // 5):
        mfma_loop_varied(20000)
    p0.record(stream)
    for _ in range(n_sus // 5):
        mf = mfma_loop_varied(20000)
    p1.record(stream)
    torch.cuda.synchronize()
    mfma_varied = (n_sus // 5) * mf / (p0.elapsed_time(p1) * 1e-3) / 1e12
    practical = {"stream_read_gbs": read_gbs, "mfma_bf16_issue_loop_tflops": mfma_tflops,
                 "mfma_bf16_issue_loop_sustained_tflops": mfma_sustained,
                 "mfma_bf16_issue_loop_varied_operands_sustained_tflops": mfma_varied}

    bytes_prefix = algorithmic_bytes_prefix(w, plens)
    bytes_call = algorithmic_bytes_call(w, plens)
    fl = flops_prefix(w, plens)
    t_hbm = bytes_prefix / (HBM_PEAK_GBS * 1e9) * 1e6
    t_mfma = fl / (MFMA_BF16_PEAK_TFLOPS * 1e12) * 1e6
    if w.dtype != "f32" and t_mfma > t_hbm:
        roof = {"bound": "mfma", "achieved": fl / kernel_us / 1e6, "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s"}
    else:
        roof = {"bound": "hbm", "achieved": bytes_prefix / kernel_us / 1e3, "peak": HBM_PEAK_GBS, "unit": "GB/s"}
    roof["frac"] = roof["achieved"] / roof["peak"]
    roof["traffic"] = PROFILED_TRAFFIC_BYTES.get(w.name) if table is None and not args.token_major else None
    roof["traffic_source"] = PROFILED_TRAFFIC_SOURCE if roof["traffic"] is not None else None
    roof["frac_of_practical_peak"] = roof["achieved"] / (read_gbs if roof["bound"] == "hbm" else mfma_tflops)
    roof["kernel"] = "prefix_mfma_kernel (ls_prefix_attn_splitkv)"
    roof["kernel_us"] = kernel_us
    roof["kernel_us_single_launch_event_pair_median"] = float(np.median(klat))
    roof["algorithmic_bytes"] = bytes_prefix
    roof["algorithmic_flops"] = fl
    roof["hbm_gbs"] = bytes_prefix / kernel_us / 1e3
    roof["mfma_tflops"] = fl / kernel_us / 1e6

    cpu = None
    if not args.no_cpu_baseline:
        import oracle   # test infrastructure; imported for this leg only

        def oracle_full(batch, rows_per_seq, rng, **kw):
            for sq in batch.seqs:
                hq, t, _ = sq.q.shape
                flat = rng.choice(hq * t, size=min(rows_per_seq, hq * t), replace=False)
                rows = np.stack([flat // t, flat % t], axis=1).astype(np.int32)
                oracle.attn_rows(sq.q, sq.k_cache, sq.v_cache, sq.k_tree, sq.v_tree, sq.parents, rows=rows, **kw)

        budget = 12.0
        rows_total = w.batch * w.n_q_heads * w.n_tree
        rng = np.random.default_rng(7)
        # a first small sample sizes the run: the whole call if it fits the budget, else a row sample
        t0 = time.perf_counter()
        okw = {"use_tree": False} if w.kind == "cross" else {}
        oracle_full(batch, rows_per_seq=16, rng=rng, **okw)
        per_row = (time.perf_counter() - t0) / (16 * w.batch)
        n_rows = int(min(w.n_q_heads * w.n_tree, max(16, budget / per_row / w.batch)))
        t0 = time.perf_counter()
        oracle_full(batch, rows_per_seq=n_rows, rng=rng, **okw)
        dt = time.perf_counter() - t0
        cpu = {"value": dt / (n_rows * w.batch) * rows_total * 1e6, "unit": "us per verify call", "cores": oracle.num_threads(),
               "kind": "oracle",
               "sample": f"{n_rows * w.batch} of {rows_total} query rows of {w.name} (uniform sample per sequence), "
                         f"{dt:.2f} s measured, scaled to all rows"}

    out = {
        "metric": "us per verify call (hybrid tree attention, 32k-token prefix)" if w.name == "C3" else
                  (f"us per cross-attention call over the cache (workload {w.name})" if w.kind == "cross" else
                   f"us per verify call (hybrid tree attention, workload {w.name})"),
        "value": us_per_call,
        "unit": "us",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "prewarm_calls": prewarm_calls,
        "ms_per_step": us_per_call / 1e3,
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": "synthetic",
        "config": {"workload": f"{w.name}: batch {w.batch}, {w.n_q_heads} q heads / {w.n_kv_heads} kv heads, head_dim "
                               f"{w.head_dim}, prefix {plens}, n_tree {w.n_tree}, seed {w.seed}",
                   "kv_layout": ("[B,P,Hkv,D] (token-major)" if args.token_major else "[B,Hkv,P,D]") if table is None else f"shuffled pages [page,Hkv,{args.page_size},D]", "n_splits": n_splits, "launches": 1 if args.single_launch else 2, "kv_rotation_copies": n_rot,
                   "kv_rotation_bytes": n_rot * kv_bytes},
        "call_us": {"mean_wall": us_per_call, "event_min": float(lat.min()), "event_median": float(np.median(lat)),
                    "event_p90": float(np.percentile(lat, 90))},
        "call_hbm_gbs": bytes_call / us_per_call / 1e3,
        "call_tflops": fl / us_per_call / 1e6,
        "hot_cache_us": hot_us,
        "graph_replay_us": graph_us,
        "practical_peaks": practical,
        "clocks": sampler.summary(),
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()

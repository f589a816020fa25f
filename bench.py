"""Benchmark of the barrier-free collectives on one MI355X.

Headline (one JSON line on stdout; the results of every section go to stderr,
where the last line, "all sections: {...}", holds them all):
  * p50 microseconds per AllReduce at 16 KiB per rank: 8 virtual ranks,
    bfloat16, batch 1 x hidden 8192, normal(0,1) inputs, the library's
    default algorithm for that size (one-shot, 8-byte packets), `--steps`
    back-to-back calls with the epoch incremented (a "step" is one such call).
    Per-call latency is the interval between consecutive calls' completion
    times, taken inside the kernels from the 100 MHz constant clock; it
    includes launch and dispatch.  The launches are queued from C behind a
    short spin kernel, so the GPU, not Python, sets the pace; the same is done
    for the floor below.  (The mean with one Python launch per call is
    reported too, as python_launched_mean_us.)
  * the single-GPU floor measured the same way: back-to-back launches of a
    kernel with the same grid whose only work is one dependent HBM round
    trip (ratio = p50 / floor p50).
  * HBM GB/s at 64 MiB per rank (8 ranks, binary32, two-shot with 128-byte
    line packets): algorithmic bytes per call / average kernel time, the time
    taken with HIP events on the stream the kernels run on.
  * the CPU oracle timed on the host on a bounded sample of the 16 KiB
    workload (cpu_baseline).

Options: --gpus must be 1 (the virtual ranks share one GPU).
"""
from __future__ import annotations

import argparse
import hashlib
import re
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
TICK_US = 0.01  # 100 MHz constant clock


def log(msg: str) -> None:
    print(msg, file=sys.stderr, flush=True)


def _code_only(text: str) -> str:
    """C++ source without its comments and blank lines (string literals in
    these headers hold no comment markers)."""
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    text = re.sub(r"//[^\n]*", "", text)
    return "\n".join(line.rstrip() for line in text.splitlines() if line.strip())


def kernel_source_hash() -> str:
    """Hash of the device code (kernels, primitives, slot layout), comments
    left out: a counter summary stays valid across comment edits."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2607_16100_amd", "csrc")
    for name in ("ll_device.hpp", "ll_kernels.hpp", "ll_layout.hpp", "ll_iter.hpp", "ll_ring.hpp"):
        with open(os.path.join(csrc, name), encoding="utf-8") as f:
            h.update(name.encode())
            h.update(_code_only(f.read()).encode())
    return h.hexdigest()[:16]


def pct(a, q):
    return float(np.percentile(np.asarray(a, dtype=np.float64), q))


# ----------------------------------------------------------------------------
HOLD_TICKS = 3_000_000  # 30 ms: long enough for the host to queue a batch of launches


def stamp_stats(stamps, steps, grid):
    a = stamps.view(steps, 2, grid).cpu().numpy().astype(np.int64)
    starts = a[:, 0, :].min(axis=1)
    ends = a[:, 1, :].max(axis=1)
    intervals = np.diff(ends) * TICK_US
    spans = (ends - starts) * TICK_US
    return intervals, spans


def gpu_paced(torch, ll, launch_batch, steps, grid, batch=2000):
    """Per-call completion intervals of `steps` back-to-back launches, queued
    behind a short spin kernel so that the GPU, not the host, sets the pace.
    `launch_batch(first, count, stamps_ptr, stride)` queues `count` launches."""
    s = torch.cuda.current_stream().cuda_stream
    iv_all, sp_all = [], []
    done = 0
    while done < steps:
        cnt = min(batch, steps - done)
        stamps = torch.zeros(cnt * 2 * grid, dtype=torch.int64, device="cuda")
        ll.check(ll.ll_probe_spin(HOLD_TICKS, s), "spin")
        launch_batch(done, cnt, stamps.data_ptr(), 2 * grid)
        torch.cuda.synchronize()
        iv, sp = stamp_stats(stamps, cnt, grid)
        iv_all.append(iv)
        sp_all.append(sp)
        done += cnt
    return np.concatenate(iv_all), np.concatenate(sp_all)


def stamp_free_mean(torch, ll, launch_batch, steps, batch=2000):
    """Mean time per call of `steps` back-to-back launches without any stamps,
    queued behind the spin kernel like gpu_paced: HIP events on the launch
    stream, recorded after the spin kernel and after the last launch."""
    s = torch.cuda.current_stream()
    total_ms, done = 0.0, 0
    while done < steps:
        cnt = min(batch, steps - done)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ll.check(ll.ll_probe_spin(HOLD_TICKS, s.cuda_stream), "spin")
        e0.record(s)
        launch_batch(done, cnt, 0, 0)
        e1.record(s)
        torch.cuda.synchronize()
        total_ms += e0.elapsed_time(e1)
        done += cnt
    return total_ms * 1000.0 / steps


def bench_headline(torch, ll, steps, warmup):
    from paper_2607_16100_amd import workloads as wl
    from paper_2607_16100_amd.region import SymRegion

    p, n = 8, 8192
    x = wl.normal(p, n, "bf16", sigma=1.0, seed=0)
    reg = SymRegion(p, n, "bf16")
    reg.init()
    reg.write_inputs(x)
    s = reg.stream_handle()
    # the configuration's path, named explicitly: one-shot with 8-byte packets
    # (AUTO takes the line one-shot here, reported below with the other formats)
    algo = ll.LL_ALGO_ONESHOT_WAVES
    epoch = [1]

    shape = ll.Options(report=True)  # collects the launch shape

    def queue(first, count, stamps_ptr, stride):
        ll.check(ll.ll_bench_allreduce(reg.base, reg.rank_stride, reg.out_ptr, n, ll.LL_BF16, p, epoch[0], count,
                                       algo, shape, stamps_ptr, stride, s), "bench_allreduce")
        epoch[0] += count

    queue(0, warmup, 0, 0)
    torch.cuda.synchronize()
    grid, threads = shape.grid, shape.threads
    t0 = time.perf_counter()
    intervals, spans = gpu_paced(torch, ll, queue, steps, grid)
    wall = time.perf_counter() - t0
    ll.check(ll.ll_check(s), "headline")
    # the same GPU-paced batch without the per-workgroup stamps (HIP events)
    stampfree = stamp_free_mean(torch, ll, queue, steps)
    ll.check(ll.ll_check(s), "headline")
    # the same calls launched one at a time from Python (host-paced), for context
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    host_steps = min(steps, 2000)
    ev0.record()
    for _ in range(host_steps):
        ll.check(ll.ll_allreduce_algo(reg.base, reg.rank_stride, reg.out_ptr, n, ll.LL_BF16, ll.LL_SUM, p, epoch[0], s,
                                      algo))
        epoch[0] += 1
    ev1.record()
    torch.cuda.synchronize()
    host_mean = ev0.elapsed_time(ev1) * 1000.0 / host_steps
    ll.check(ll.ll_check(s), "headline")
    # the last call's output, checked against the oracle by the CPU-baseline leg
    HEADLINE_OUTPUT["bits"] = reg.read_out(p * n, np.uint16).reshape(p, n)
    # the same workload through AUTO and the other packet formats (context);
    # their epochs continue after the ones used above
    reg.epoch = epoch[0] - 1
    variants = {}
    for name in ("auto", "oneshot_sentinel_waves", "oneshot_line_waves", "twoshot_waves"):
        r = paced_collective(torch, ll, reg, "ar", n, ll.ALGOS[name], min(steps, 5000), 100)
        variants[name] = {"p50_us": r["p50_us"], "p99_us": r["p99_us"]}
    epochs = reg.epoch
    graph = bench_graph_replay(torch, ll, reg, n, p, grid, threads)
    return {
        "algorithm": "oneshot_waves", "variants": variants,
        "p50_us": pct(intervals, 50), "p99_us": pct(intervals, 99), "mean_us": float(np.mean(intervals)),
        "span_p50_us": pct(spans, 50), "stamp_free_mean_us": stampfree, "python_launched_mean_us": host_mean,
        "wall_s": wall, "grid": grid, "threads": threads, "epochs": epochs, "graph_replay": graph,
        "exchange_probe": bench_exchange_probe(torch, ll, reg, n, p, steps),
    }


def bench_graph_replay(torch, ll, reg, n, p, grid, threads, calls=1000, reps=5):
    """The headline call captured `calls` times into a HIP graph (epochs 1 ..
    calls; a captured call keeps its epoch, so the region is reset eagerly
    before every replay) and replayed `reps` times: mean per call from HIP
    events around each replay, and every replay's output (the buffer zeroed
    first) compared with the eager result.  Beside it the empty kernel with
    the same grid, captured and replayed the same way.  Context for serving
    loops that replay graphs; the headline stays the eager back-to-back p50."""
    try:
        want = reg.read_out(p * n, np.uint16)
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):  # the capture stream's status word, before capture
            reg.init(side)
            ll.check(reg.allreduce(n, "oneshot_waves", epoch=1), "graph warm-up")
        torch.cuda.synchronize()
        ll.check(ll.ll_check(side.cuda_stream), "graph warm-up")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            for i in range(calls):
                ll.check(reg.allreduce(n, "oneshot_waves", epoch=1 + i), "graph capture")
        g_empty = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g_empty, stream=side):
            for _ in range(calls):
                ll.check(ll.ll_probe_empty(grid, threads, 0, side.cuda_stream), "graph capture")
        torch.cuda.synchronize()
        per_call, empty, exact = [], [], True
        for _ in range(reps):
            reg.out.zero_()
            reg.init()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            g.replay()
            e1.record()
            torch.cuda.synchronize()
            ll.check(ll.ll_check(side.cuda_stream), "graph replay")
            per_call.append(e0.elapsed_time(e1) * 1000.0 / calls)
            exact = exact and bool(np.array_equal(reg.read_out(p * n, np.uint16), want))
            e0.record()
            g_empty.replay()
            e1.record()
            torch.cuda.synchronize()
            empty.append(e0.elapsed_time(e1) * 1000.0 / calls)
        reg.init()
        torch.cuda.synchronize()
        return {"calls_per_replay": calls, "replays": reps, "mean_us_per_call": float(np.median(per_call)),
                "empty_kernel_mean_us": float(np.median(empty)), "bit_exact_every_replay": exact}
    except Exception as e:  # context only: never lose the benchmark line over it
        return {"error": repr(e)}


def bench_exchange_probe(torch, ll, reg, n, p, steps):
    """The minimal-exchange probe on the headline's region, grid and packet
    volume (load, one packet store to one peer, poll, one output store per
    wave; no LDS, barrier or sum): stamped p50 interval and stamp-free mean,
    measured like the collective."""
    s = reg.stream_handle()

    shape = {}

    def queue(first, count, stamps_ptr, stride):
        st, shape["grid"] = ll.ll_bench_exchange(reg.base, reg.rank_stride, reg.out_ptr, n, ll.LL_BF16, p,
                                                 reg.epoch + 1, count, stamps_ptr, stride, s)
        ll.check(st, "bench_exchange")
        reg.epoch += count

    queue(0, 200, 0, 0)
    torch.cuda.synchronize()
    grid, threads = shape["grid"], 64 * p
    iv, sp = gpu_paced(torch, ll, queue, steps, grid)
    mean = stamp_free_mean(torch, ll, queue, steps)
    ll.check(ll.ll_check(s), "exchange probe")
    return {"p50_us": pct(iv, 50), "p99_us": pct(iv, 99), "span_p50_us": pct(sp, 50), "stamp_free_mean_us": mean,
            "grid": grid, "threads": threads}


HEADLINE_OUTPUT = {}


def bench_floor(torch, ll, steps, warmup, grid, threads):
    """Back-to-back floor kernels with the collective's grid, each loading a
    line nobody has touched for a long time (1 GiB table, larger than the
    256 MiB last-level cache) and storing it; and empty kernels."""
    words = (1 << 30) // 8
    chase = torch.zeros(words, dtype=torch.int64, device="cuda")
    sink = torch.zeros(16, dtype=torch.int64, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    step_lines = 4099
    pos = [0]

    def q_floor(first, count, stamps_ptr, stride):
        ll.check(ll.ll_bench_floor(chase.data_ptr(), words, pos[0], step_lines, sink.data_ptr(), grid, threads, count,
                                   stamps_ptr, stride, s), "bench_floor")
        pos[0] += count * step_lines

    def q_empty(first, count, stamps_ptr, stride):
        ll.check(ll.ll_bench_empty(grid, threads, count, stamps_ptr, stride, s), "bench_empty")

    out = {}
    for name, fn in (("floor", q_floor), ("empty", q_empty)):
        fn(0, warmup, 0, 0)
        torch.cuda.synchronize()
        iv, sp = gpu_paced(torch, ll, fn, steps, grid)
        out[name] = {"p50_us": pct(iv, 50), "p99_us": pct(iv, 99), "span_p50_us": pct(sp, 50),
                     "stamp_free_mean_us": stamp_free_mean(torch, ll, fn, steps)}
    # dependent-load latency of cold lines: chase through a table, after evicting caches
    line_words = 16
    perm = np.random.default_rng(1).permutation(words // line_words // 64)[:4096] * 64 * line_words
    nxt = np.roll(perm, -1)
    chase.index_copy_(0, torch.from_numpy(perm.astype(np.int64)).cuda(), torch.from_numpy(nxt.astype(np.int64)).cuda())
    junk = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    junk.fill_(1)
    del junk
    res = torch.zeros(3, dtype=torch.int64, device="cuda")
    ll.check(ll.ll_probe_chase(chase.data_ptr(), words, int(perm[0]), 2000, res.data_ptr(), s), "chase")
    torch.cuda.synchronize()
    r = res.cpu().numpy()
    out["hbm_dependent_load_us"] = float(r[0]) * TICK_US / 2000
    out["hbm_dependent_load_cycles"] = float(r[1]) / 2000
    # the floor composed from its two parts (empty-kernel interval plus one
    # dependent HBM load); the directly measured floor above is the denominator
    out["composed_p50_us"] = out["empty"]["p50_us"] + out["hbm_dependent_load_us"]
    del chase
    return out


def paced_collective(torch, ll, reg, kind, count, code, steps, warmup, flags=0):
    """p50/p99 call-to-call interval (GPU-paced) of one collective on a region.
    kind: "ar" (count elements, code = ll_algo), "rs" (recvcount, code =
    ll_proto), "ag" (sendcount, code = ll_proto); flags: LL_OPT_* of the calls."""
    s = reg.stream_handle()
    fn = {"ar": ll.ll_bench_allreduce, "rs": ll.ll_bench_reduce_scatter, "ag": ll.ll_bench_allgather}[kind]
    shape = ll.Options(flags=flags, report=True)

    def queue(first, cnt, stamps_ptr, stride):
        e = reg.epoch + 1
        ll.check(fn(reg.base, reg.rank_stride, reg.out_ptr, count, reg.dt, reg.nranks, e, cnt, code, shape,
                    stamps_ptr, stride, s), kind)
        reg.epoch += cnt

    queue(0, warmup, 0, 0)
    torch.cuda.synchronize()
    grid, threads = shape.grid, shape.threads
    iv, sp = gpu_paced(torch, ll, queue, steps, grid)
    ll.check(ll.ll_check(s), kind)
    return {"p50_us": pct(iv, 50), "p99_us": pct(iv, 99), "span_p50_us": pct(sp, 50), "grid": grid,
            "threads": threads}


def bench_rooted(torch, ll, steps):
    """Broadcast and Reduce, 8 ranks, bf16, 16 KiB and 1 MiB per rank, root 0."""
    from paper_2607_16100_amd import workloads as wl
    from paper_2607_16100_amd.region import SymRegion

    out = {}
    p = 8
    for n in (8192, 1 << 19):
        reg = SymRegion(p, n, "bf16")
        reg.init()
        reg.write_inputs(wl.normal(p, n, "bf16", seed=0))
        s = reg.stream_handle()
        for kind, code in (("broadcast", 0), ("reduce", 1)):
            for proto in ("packet8", "line128", "sentinel"):
                shape = ll.Options(report=True)

                def queue(first, cnt, stamps_ptr, stride, code=code, proto=proto, shape=shape):
                    ll.check(ll.ll_bench_rooted(code, reg.base, reg.rank_stride, reg.out_ptr, n, reg.dt, 0, p,
                                                reg.epoch + 1, cnt, ll.PROTOS[proto], shape, stamps_ptr, stride, s),
                             kind)
                    reg.epoch += cnt

                queue(0, 20, 0, 0)
                torch.cuda.synchronize()
                grid, threads = shape.grid, shape.threads
                iv, sp = gpu_paced(torch, ll, queue, steps, grid)
                ll.check(ll.ll_check(s), kind)
                out[f"{kind}_{n * 2 >> 10}KiB_{proto}"] = {"p50_us": pct(iv, 50), "p99_us": pct(iv, 99)}
        del reg
    return out


def bound_us(floor_p50_us, p, n, esize):
    """Lower bound of one AllReduce call: the latency floor plus the time the
    bytes no algorithm can avoid -- every rank reads its input and writes its
    output once -- take at the HBM peak."""
    if not floor_p50_us:
        return None
    return floor_p50_us + 2 * p * n * esize / (PEAK_HBM_GBS * 1e3)


def bench_c3(torch, ll, steps, floor_p50_us=None):
    """1 MiB per rank (batch 64 x hidden 8192 bf16, 8 ranks): two-shot against
    one-shot, each with its fraction of the floor + bytes/peak bound; then AUTO
    (flag formats only, and with the sentinel allowed) over 128 KiB .. 8 MiB
    per rank (batch 8 .. 512)."""
    from paper_2607_16100_amd import workloads as wl
    from paper_2607_16100_amd.region import SymRegion

    p, n = 8, 64 * 8192
    reg = SymRegion(p, n, "bf16")
    reg.init()
    reg.write_inputs(wl.normal(p, n, "bf16", sigma=0.5, seed=0))
    out = {}
    for algo in ("twoshot", "twoshot_line", "twoshot_waves", "twoshot_line_waves", "twoshot_sentinel",
                 "twoshot_sentinel_waves", "twoshot_sentinel_out", "twoshot_atomic", "oneshot", "oneshot_line",
                 "oneshot_sentinel", "auto"):
        out[algo] = paced_collective(torch, ll, reg, "ar", n, ll.ALGOS[algo], steps, 20)
    out["auto_sentinel_allowed"] = paced_collective(torch, ll, reg, "ar", n, ll.ALGOS["auto"], steps, 20,
                                                    flags=ll.LL_OPT_AUTO_SENTINEL)
    b = bound_us(floor_p50_us, p, n, 2)
    for r in out.values():
        r["bound_us"] = round(b, 3) if b else None
        r["frac_of_bound"] = round(b / r["p50_us"], 4) if b else None
    del reg
    sizes = {}
    for batch in (8, 16, 32, 64, 128, 256, 512):
        m = batch * 8192
        reg = SymRegion(p, m, "bf16")
        reg.init()
        reg.write_inputs(wl.normal(p, m, "bf16", sigma=0.5, seed=batch))
        st = steps if batch <= 64 else max(200, steps // 4)
        row = {"bytes_per_rank": m * 2}
        bb = bound_us(floor_p50_us, p, m, 2)
        row["bound_us"] = round(bb, 3) if bb else None
        for key, flags in (("auto", 0), ("auto_sentinel_allowed", ll.LL_OPT_AUTO_SENTINEL)):
            r = paced_collective(torch, ll, reg, "ar", m, ll.ALGOS["auto"], st, 20, flags=flags)
            row[key] = {"p50_us": r["p50_us"], "p99_us": r["p99_us"],
                        "frac_of_bound": round(bb / r["p50_us"], 4) if bb else None}
        sizes[f"{m * 2 >> 10}KiB"] = row
        log(json.dumps({f"{m * 2 >> 10}KiB": row}))
        del reg
    out["auto_by_size"] = sizes
    return out


def bench_c5(torch, ll, steps):
    """Stand-alone ReduceScatter and AllGather, bf16, hidden 7168 x batch {1, 16, 256}, 8 and 4 ranks."""
    from paper_2607_16100_amd import workloads as wl
    from paper_2607_16100_amd.region import SymRegion

    out = {}
    for p in (8, 4):
        for b in (1, 16, 256):
            total = 7168 * b
            m = total // p
            reg = SymRegion(p, total, "bf16", out_elems=p * total)
            reg.init()
            reg.write_inputs(wl.normal(p, total, "bf16", seed=0))
            for proto in ("auto", "packet8", "line128", "sentinel"):
                out[f"rs_p{p}_b{b}_{proto}"] = paced_collective(torch, ll, reg, "rs", m, ll.PROTOS[proto], steps, 20)
                out[f"ag_p{p}_b{b}_{proto}"] = paced_collective(torch, ll, reg, "ag", m, ll.PROTOS[proto], steps, 20)
            del reg
    return out


def bench_scratch(torch, ll, iters=10, warmup=3):
    """The paper's scratch-size study (Sec. VIII, "Impact of Scratch
    Buffer"): a 32 MiB f32 message per rank over 8 ranks through bounded
    scratch regions whose iterations hold 256 KiB .. 32 MiB per rank; mean
    time per call (HIP events on the launch stream)."""
    from paper_2607_16100_amd.region import ScratchRegion

    p, n = 8, (32 << 20) // 4
    out = {}
    for it_kib in (256, 512, 1024, 2048, 4096, 8192, 16384, 32768):
        reg = ScratchRegion(p, n, "f32", iter_bytes=it_kib << 10)
        reg.init()
        g = torch.Generator(device="cuda")
        g.manual_seed(0)
        reg.inp.view(torch.float32).copy_(torch.rand(p * n, generator=g, device="cuda") * 2 - 1)
        stream = torch.cuda.current_stream()
        row = {"iter_kib": it_kib, "scratch_slice_bytes": reg.scratch_stride}
        for algo in ("oneshot", "oneshot_line", "oneshot_sentinel", "twoshot", "twoshot_line", "twoshot_sentinel",
                     "twoshot_waves", "twoshot_line_waves", "twoshot_sentinel_waves", "auto"):
            for _ in range(warmup):
                ll.check(reg.allreduce(n, algo), algo)
            ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            ev0.record(stream)
            for _ in range(iters):
                ll.check(reg.allreduce(n, algo), algo)
            ev1.record(stream)
            torch.cuda.synchronize()
            ll.check(ll.ll_check(stream.cuda_stream), algo)
            row[algo] = round(ev0.elapsed_time(ev1) * 1000.0 / iters, 2)
            row["iterations"] = reg.last_iters
        out[f"{it_kib}KiB"] = row
        log(json.dumps(row))
        del reg
    return out


def bench_sweep(torch, ll, path, floor_p50_us=None):
    """C4: 8 ranks, binary32, 2 .. 2^26 elements per rank; p50/p99 and GB/s of
    every algorithm at every size (written to `path` as JSON lines), each with
    its ratio to the latency floor and its fraction of the HBM peak."""
    from paper_2607_16100_amd.region import SymRegion

    p = 8
    big = 1 << 26
    reg = SymRegion(p, big, "f32", out_elems=p * big)
    reg.init()
    g = torch.Generator(device="cuda")
    g.manual_seed(0)
    rows = torch.rand((p, big), generator=g, device="cuda", dtype=torch.float32) * 2 - 1
    reg.write_inputs_device(rows.view(torch.uint8).view(p, big * 4))
    del rows
    # warm the chip up first: the first size would otherwise run on cold clocks
    paced_collective(torch, ll, reg, "ar", 2, ll.ALGOS["auto"], 2000, 20)
    with open(path, "w") as f:
        for k in range(1, 27):
            n = 1 << k
            steps = 2000 if n * 4 <= (1 << 20) else (200 if n * 4 <= (16 << 20) else 20)
            for algo in ("auto", "oneshot_waves", "oneshot_sentinel_waves", "oneshot_line_waves", "oneshot", "oneshot_line",
                         "oneshot_sentinel", "twoshot_waves", "twoshot_sentinel_waves", "twoshot_line_waves", "twoshot", "twoshot_line",
                         "twoshot_sentinel", "twoshot_sentinel_out", "twoshot_atomic"):
                if algo in ("oneshot_waves", "oneshot_sentinel_waves", "oneshot_line_waves") and n * 4 > (1 << 20):
                    continue
                if algo in ("twoshot_atomic", "twoshot_sentinel_out") and n < 4:
                    continue
                r = paced_collective(torch, ll, reg, "ar", n, ll.ALGOS[algo], steps, min(20, steps))
                gbps = (moved_bytes(algo, p, n, 4) / r["p50_us"] / 1e3) if algo != "auto" else None
                b = bound_us(floor_p50_us, p, n, 4)
                r.update({"elements": n, "bytes_per_rank": n * 4, "algo": algo, "algorithmic_gbps_p50": gbps,
                          "hbm_frac_p50": gbps / PEAK_HBM_GBS if gbps else None,
                          "ratio_to_floor": r["p50_us"] / floor_p50_us if floor_p50_us else None,
                          "bound_us": b, "frac_of_bound": b / r["p50_us"] if b else None})
                f.write(json.dumps(r) + "\n")
                f.flush()
                log(f"sweep n={n} {algo} p50={r['p50_us']:.2f}")
    return path


def bench_sol_pieces(torch, ll):
    """The paper's speed-of-light pieces (Sec. VI) measured on one chip."""
    s = torch.cuda.current_stream().cuda_stream
    buf = torch.zeros(1024, dtype=torch.int32, device="cuda")
    out = torch.zeros(7, dtype=torch.int64, device="cuda")
    iters = 2000
    ll.check(ll.ll_probe_fence_l2(buf.data_ptr(), iters, out.data_ptr(), s), "fence")
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    fence_us = o[0] * TICK_US / iters
    sc1_us = o[2] * TICK_US / iters
    flags = torch.zeros(2048, dtype=torch.int32, device="cuda")
    pp = torch.zeros(3, dtype=torch.int64, device="cuda")
    rounds = 2000
    ll.check(ll.ll_probe_pingpong(flags.data_ptr(), rounds, 8, 1, 10_000_000, pp.data_ptr(), s), "pingpong")
    torch.cuda.synchronize()
    q = pp.cpu().numpy()
    done = int(q[1])
    ping_us = (q[0] * TICK_US / done) if done else float("nan")
    remote = (ping_us - 2 * fence_us) / 2
    ids = torch.zeros(64, dtype=torch.int32, device="cuda")
    ll.check(ll.ll_probe_xcd(ids.data_ptr(), 64, 64, s), "xcd")
    torch.cuda.synchronize()
    xcd = ids.cpu().numpy().tolist()
    return {
        "fence_us": fence_us, "coherent_load_us": sc1_us, "pingpong_us": ping_us, "pingpong_rounds": done,
        "remote_store_us": remote, "sol_us": 2 * fence_us + remote,
        "xcd_of_workgroup_0_15": xcd[:16],
    }


RING_MIN_BYTES = {"line128": 7680 << 10, "packet8": 5 << 20}  # all ranks' inputs from which a two-shot runs on the ring (8 ranks)


def moved_bytes(algo, p, count, esize):
    """The algorithmic bytes of one AllReduce call: the flagged two-shot
    algorithms run on the ring kernels at the bandwidth-bound sizes."""
    from paper_2607_16100_amd import bytemodel

    if algo in ("twoshot", "twoshot_line", "twoshot_waves", "twoshot_line_waves"):
        proto = "line128" if "_line" in algo else "packet8"
        if p * count * esize >= RING_MIN_BYTES[proto]:
            return bytemodel.ring_allreduce_bytes(proto, p, count, esize)
    return bytemodel.allreduce_bytes(algo, p, count, esize)


def bench_bandwidth(torch, ll, count, algos, iters=20, warmup=3):
    """Average kernel time (HIP events on the launch stream) and GB/s at `count`
    binary32 elements per rank, 8 ranks."""
    from paper_2607_16100_amd import bytemodel
    from paper_2607_16100_amd import workloads as wl
    from paper_2607_16100_amd.region import SymRegion

    p = 8
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # fresh device allocations, as for the copy reference
    reg = SymRegion(p, count, "f32", out_elems=p * count)
    reg.init()
    # inputs generated on the device from a seeded torch generator (the values
    # do not affect timing; parity at this size is covered by the tests)
    g = torch.Generator(device="cuda")
    g.manual_seed(0)
    rows = (torch.rand((p, count), generator=g, device="cuda", dtype=torch.float32) * 2 - 1)
    reg.write_inputs_device(rows.view(torch.uint8).view(p, count * 4))
    del rows
    stream = torch.cuda.current_stream()
    res = {}
    for algo in algos:
        shape = ll.Options(report=True)
        for _ in range(warmup):
            ll.check(reg.allreduce(count, algo, opt=shape), algo)
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        ev0.record(stream)
        for _ in range(iters):
            ll.check(reg.allreduce(count, algo), algo)
        ev1.record(stream)
        torch.cuda.synchronize()
        ll.check(ll.ll_check(stream.cuda_stream), algo)
        us = ev0.elapsed_time(ev1) * 1000.0 / iters
        nbytes = moved_bytes(algo, p, count, 4)
        useful = bytemodel.useful_bytes(p, count, 4)
        grid, threads = shape.grid, shape.threads
        res[algo] = {"kernel_us": us, "algorithmic_bytes": nbytes, "gbps": nbytes / us / 1e3,
                     "useful_gbps": useful / us / 1e3, "grid": grid, "threads": threads}
    del reg
    return res


def bench_copy(torch, ll, nbytes=1 << 30, iters=20, placements=3):
    """HBM bandwidth of plain streaming kernels over `nbytes`: torch's
    device-to-device copy, and the library's streaming probe (16-byte
    non-temporal loads and stores, grid-stride) as a copy, a read and a write,
    each at the best over grid sizes and, for the copy, over `placements`
    separately allocated source/destination pairs (where the two buffers
    sit moves a copy's rate by up to 10 %).  This is the rate a simple kernel
    reaches on this GPU, the practical ceiling under the 8 TB/s peak."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # fresh device allocations, not blocks the earlier legs left cached
    pairs = []
    for _ in range(placements):
        src = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        dst = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        src.fill_(1)
        pairs.append((src, dst))
    src, dst = pairs[0]
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(iters):
        dst.copy_(src)
    e1.record(stream)
    torch.cuda.synchronize()
    us = e0.elapsed_time(e1) * 1000.0 / iters
    res = {"bytes": nbytes, "kernel_us": us, "gbps": 2.0 * nbytes / us / 1e3}
    s = stream.cuda_stream
    probe = {}
    grids = (512, 768, 1024, 1536, 2048, 4096, 8192, 16384)
    for mode, name, moved in ((0, "copy", 2), (1, "read", 1), (2, "write", 1)):
        best = None
        shapes = [(0, g) for g in grids] + ([(i, g) for i in range(1, placements) for g in (512, 1024, 2048)]
                                            if mode == 0 else [])
        for pair, grid in shapes:
            a, b = pairs[pair]
            ll.check(ll.ll_probe_stream(a.data_ptr(), b.data_ptr(), nbytes, mode, grid, 256, s), "stream")
            e0.record(stream)
            for _ in range(iters):
                ll.check(ll.ll_probe_stream(a.data_ptr(), b.data_ptr(), nbytes, mode, grid, 256, s), "stream")
            e1.record(stream)
            torch.cuda.synchronize()
            t = e0.elapsed_time(e1) * 1000.0 / iters
            gbps = moved * nbytes / t / 1e3
            if best is None or gbps > best["gbps"]:
                best = {"gbps": gbps, "kernel_us": t, "grid": grid, "threads": 256, "placement": pair}
        probe[name] = best
    res["streaming_probe"] = probe
    del pairs, src, dst
    return res


def bench_cpu_baseline(seconds: float):
    import oracle
    from paper_2607_16100_amd import workloads as wl

    x = wl.normal(8, 8192, "bf16", sigma=1.0, seed=0)
    times = []
    want = None
    t_end = time.perf_counter() + seconds
    while time.perf_counter() < t_end:
        t0 = time.perf_counter()
        want = oracle.allreduce(x)
        times.append(time.perf_counter() - t0)
    med = float(np.median(times))
    res = {"value": med * 1e6, "unit": "us", "cores": 1, "kind": "oracle",
           "sample": f"8 ranks x 8192 bf16 (the 16 KiB workload) reduced {len(times)} times in ~{seconds:.0f} s "
                     f"by the single-threaded C oracle; median per call",
           "gbps_read_inputs_write_output": (8 * 8192 * 2 + 8192 * 2) / med / 1e9,
           "host_cores_available": len(os.sched_getaffinity(0))}
    got = HEADLINE_OUTPUT.get("bits")
    if got is not None:  # the headline's last GPU result against the oracle's
        res["headline_bit_exact"] = bool(np.array_equal(got, want))
    res["bandwidth_workload"] = bench_cpu_all_cores(seconds / 2)
    return res


def bench_cpu_all_cores(seconds: float):
    """The same C oracle on the 64 MiB-per-rank binary32 workload (8 ranks),
    once on one thread and then on every host core: the elements are split
    into contiguous column blocks, one per thread, and each block is reduced
    by an unchanged oracle call, so the per-element order is untouched and the
    result is bit-identical.  ctypes releases the GIL for the calls."""
    import oracle
    from concurrent.futures import ThreadPoolExecutor
    from paper_2607_16100_amd import workloads as wl

    p, n = 8, 16 << 20
    x = wl.uniform(p, n, "f32", seed=0)
    t0 = time.perf_counter()
    one = oracle.allreduce(x)
    t_one = time.perf_counter() - t0
    cores = max(1, min(16, len(os.sched_getaffinity(0))))
    edges = [(n * i // cores) // 64 * 64 for i in range(cores)] + [n]
    blocks = [np.ascontiguousarray(x[:, edges[i]:edges[i + 1]]) for i in range(cores)]
    del x
    times, outs = [], None
    with ThreadPoolExecutor(max_workers=cores) as pool:
        t_end = time.perf_counter() + seconds
        while time.perf_counter() < t_end or not times:
            t0 = time.perf_counter()
            outs = list(pool.map(oracle.allreduce, blocks))
            times.append(time.perf_counter() - t0)
    same = all(np.array_equal(outs[i], one[:, edges[i]:edges[i + 1]]) for i in range(cores))
    med = float(np.median(times))
    traffic = (p * n * 4 + n * 4) / 1e9  # every input read once, one output row written
    return {"bytes_per_rank": n * 4, "one_core_us": t_one * 1e6, "one_core_gbps": traffic / t_one,
            "all_cores_us": med * 1e6, "all_cores_gbps": traffic / med, "cores": cores,
            "calls": len(times), "bit_identical": bool(same),
            "sample": "8 ranks x 16 Mi binary32 uniform[-1,1); one single-threaded call, then the median "
                      "of repeated calls split into one contiguous column block per core"}


# The 64 MiB leg's kernel: what AUTO runs for 64 MiB of binary32 per rank at 8
# ranks (the line two-shot on the ring kernel).
BW_ALGO = "twoshot_line_waves"
BW_KERNEL = "k_ring<ProtoLine, f32, 8, AllReduce> (64 MiB per rank, 8 ranks)"
BW_COUNTERS = "ring_f32_64MiB_p8_counters.txt"


def traffic_from_profiles(kernel_hash: str, grid_threads: int):
    """HBM bytes per launch from the committed counter summary (rocprofv3
    FETCH_SIZE and WRITE_SIZE, scaled by what they read for a 1 GiB copy), if
    it was taken from the current device code with the same launch grid."""
    path = os.path.join(ROOT, "profiles", BW_COUNTERS)
    if not os.path.exists(path):
        return None
    try:
        with open(path) as f:
            d = json.load(f)
    except (OSError, ValueError):
        return None
    if d.get("kernel_source_hash") != kernel_hash or d.get("grid_size_threads") != grid_threads:
        return None
    return d.get("hbm_bytes_per_launch")


def result_line(result, steps, warmup):
    """The JSON line of a run: the headline, its bounds and the CPU baseline.  The
    sections' own results stay out of it (main logs them): with all of them the
    line grew past 16 KB, more than a record of the run's last output holds."""
    h = result.get("headline", {})
    fl = result.get("floor", {}).get("floor", {})
    c3 = result.get("c3")
    bw = result.get("bw", {}).get(BW_ALGO)
    khash = kernel_source_hash()
    roofline = None
    if bw:
        roofline = {"bound": "hbm", "achieved": round(bw["gbps"], 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                    "frac": round(bw["gbps"] / PEAK_HBM_GBS, 4),
                    "traffic": traffic_from_profiles(khash, bw["grid"] * bw["threads"]),
                    "kernel": BW_KERNEL,
                    "kernel_us": round(bw["kernel_us"], 2), "algorithmic_bytes": bw["algorithmic_bytes"]}
        if roofline["traffic"]:
            # the counters' bytes (FETCH_SIZE + WRITE_SIZE, calibrated) over the same kernel time
            roofline["traffic_gbps"] = round(roofline["traffic"] / bw["kernel_us"] / 1e3, 1)
        probe = result.get("copy", {}).get("streaming_probe", {}).get("copy")
        if probe:
            # the best plain streaming copy on the same GPU: what a simple kernel reaches
            roofline["copy_ceiling_gbps"] = round(probe["gbps"], 1)
            roofline["frac_of_copy_ceiling"] = round(bw["gbps"] / probe["gbps"], 4)
    if h and fl:
        ex = h.get("exchange_probe", {})
        lat = {"bound": "latency floor: back-to-back launches of a kernel with the same grid doing one dependent "
                        "HBM load (empty-kernel launch + one HBM round trip)",
               "kernel": "k_oneshot_tile<ProtoLL, bf16, 8> (16 KiB per rank, 8 ranks, one tile per workgroup)",
               "p50_us": round(h["p50_us"], 3), "floor_p50_us": round(fl["p50_us"], 3),
               "ratio_to_floor": round(h["p50_us"] / fl["p50_us"], 3), "target_ratio": 1.5,
               "composed_floor_us": round(result["floor"].get("composed_p50_us", float("nan")), 3),
               "kernel_span_p50_us": round(h["span_p50_us"], 3),
               "floor_span_p50_us": round(fl["span_p50_us"], 3),
               "stamp_free_mean_us": round(h["stamp_free_mean_us"], 3),
               "floor_stamp_free_mean_us": round(fl["stamp_free_mean_us"], 3),
               "ratio_to_floor_stamp_free": round(h["stamp_free_mean_us"] / fl["stamp_free_mean_us"], 3)}
        if ex:
            lat.update({"exchange_probe_p50_us": round(ex["p50_us"], 3),
                        "exchange_probe_stamp_free_mean_us": round(ex["stamp_free_mean_us"], 3),
                        "ratio_to_exchange_probe": round(h["p50_us"] / ex["p50_us"], 3)})
        if roofline is None:
            roofline = {"bound": "latency", "achieved": lat["p50_us"], "peak": lat["floor_p50_us"], "unit": "us",
                        "frac": round(lat["floor_p50_us"] / lat["p50_us"], 4), "traffic": None}
        roofline["latency"] = lat
    return {
        "metric": "p50 µs per AllReduce at 16 KB (P=8, bf16) + HBM GB/s at 64 MB",
        "value": round(h["p50_us"], 3) if h else None,
        "unit": "µs",
        "n_gpus": 1,
        "steps": steps,
        "warmup": warmup,
        "ms_per_step": round(h["mean_us"] / 1000.0, 6) if h else None,
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "AllReduce sum, 8 virtual ranks on one GPU, bf16 batch 1 x hidden 8192 "
                               "(16 KiB per rank), one-shot 8-byte packets (one wave per peer), back-to-back calls",
                   "ranks": 8, "elements_per_rank": 8192, "element_type": "bf16", "accumulate": "f32",
                   "parallelism": "8 virtual ranks / 1 GPU"},
        "p99_us": round(h["p99_us"], 3) if h else None,
        "floor_p50_us": round(fl["p50_us"], 3) if fl else None,
        "ratio_to_floor": round(h["p50_us"] / fl["p50_us"], 3) if (h and fl) else None,
        "hbm_gbps_64MB": round(bw["gbps"], 1) if bw else None,
        "c3_1MiB": ({k: {"p50_us": round(c3[k]["p50_us"], 3), "frac_of_bound": c3[k]["frac_of_bound"]}
                     for k in ("auto", "auto_sentinel_allowed")} | {"bound_us": c3["auto"]["bound_us"]}) if c3 else None,
        "roofline": roofline,
        "cpu_baseline": result.get("cpu"),
        "kernel_source_hash": khash,
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10000)
    ap.add_argument("--warmup", type=int, default=200)
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--bw-iters", type=int, default=20)
    ap.add_argument("--only", default="", help="comma list of sections: headline,floor,sol,bw,c3,c5,rooted,scratch,copy,cpu")
    ap.add_argument("--sweep", default="", help="also run the full C4 size sweep, writing JSON lines to this file")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: the P virtual ranks share one GPU; --gpus {args.gpus} is not supported "
              f"(only one GPU is used; sharding over several GPUs is a design, not code)", file=sys.stderr)
        sys.exit(2)
    only = set(x for x in args.only.split(",") if x)

    def want(sec):
        return not only or sec in only

    import torch

    from paper_2607_16100_amd import llcoll as ll

    torch.cuda.set_device(0)
    props = torch.cuda.get_device_properties(0)
    log(f"device: {props.name} {getattr(props, 'gcnArchName', '')} CUs={props.multi_processor_count}")
    result = {}
    result["device"] = {"name": props.name, "arch": getattr(props, "gcnArchName", ""),
                        "compute_units": props.multi_processor_count, "hbm_bytes": props.total_memory,
                        "hip_runtime": getattr(torch.version, "hip", None), "torch": torch.__version__}
    if want("headline"):
        log("headline: 16 KiB bf16 one-shot, 8 ranks")
        result["headline"] = bench_headline(torch, ll, args.steps, args.warmup)
        log(json.dumps(result["headline"]))
    grid = result.get("headline", {}).get("grid", 64)
    threads = result.get("headline", {}).get("threads", 256)
    if want("floor"):
        log("floor")
        result["floor"] = bench_floor(torch, ll, args.steps, args.warmup, grid, threads)
        log(json.dumps(result["floor"]))
    if want("sol"):
        log("speed-of-light pieces")
        result["sol"] = bench_sol_pieces(torch, ll)
        log(json.dumps(result["sol"]))
    if want("bw"):
        log("bandwidth at 64 MiB per rank")
        result["bw"] = bench_bandwidth(torch, ll, 16 << 20, ["twoshot_line_waves", "twoshot_line", "twoshot",
                                                                "twoshot_sentinel", "twoshot_sentinel_waves",
                                                                "twoshot_sentinel_out", "twoshot_atomic",
                                                                "oneshot_line", "oneshot", "oneshot_sentinel"],
                                       iters=args.bw_iters)
        log(json.dumps(result["bw"]))
    if want("copy"):
        log("device copy reference (right after the bandwidth leg, in the same state of the chip)")
        result["copy"] = bench_copy(torch, ll)
        log(json.dumps(result["copy"]))
    if want("c3"):
        log("C3: 1 MiB bf16, two-shot vs one-shot")
        result["c3"] = bench_c3(torch, ll, min(args.steps, 2000), result.get("floor", {}).get("floor", {}).get("p50_us"))
        log(json.dumps(result["c3"]))
    if want("c5"):
        log("C5: reduce-scatter / all-gather")
        result["c5"] = bench_c5(torch, ll, min(args.steps, 1000))
        log(json.dumps(result["c5"]))
    if want("rooted"):
        log("Broadcast / Reduce")
        result["rooted"] = bench_rooted(torch, ll, min(args.steps, 1000))
        log(json.dumps(result["rooted"]))
    if want("scratch"):
        log("scratch-size study: 32 MiB f32, 8 ranks")
        result["scratch"] = bench_scratch(torch, ll)
    if args.sweep:
        log("C4 sweep")
        fl0 = result.get("floor", {}).get("floor", {}).get("p50_us")
        result["sweep_file"] = bench_sweep(torch, ll, args.sweep, fl0)
    if want("cpu"):
        log("cpu baseline")
        result["cpu"] = bench_cpu_baseline(args.cpu_seconds)
        log(json.dumps(result["cpu"]))

    log("all sections: " + json.dumps(result))
    print(json.dumps(result_line(result, args.steps, args.warmup)), flush=True)


if __name__ == "__main__":
    main()

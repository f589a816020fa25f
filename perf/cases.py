"""Performance cases: the collectives as a program calls them, from one tiny
AllReduce to 64 MiB per rank.

A case names an operation ("op"), the rank count, the element type and the
per-rank element count of its input ("count"; ReduceScatter reduces "count"
elements per rank and returns count / ranks of them; AllGather sends "count"),
and options where the operation has any:

  allreduce       SymRegion.allreduce, the algorithm left to the library;
                  "sentinel": the data never holds the sentinel dword, so the
                  call allows sentinel mode
  decode_graph    "calls" AllReduces of one region captured into a HIP graph,
                  as a serving loop captures its decode step; a pass resets
                  the region and replays the graph
  reduce_scatter, allgather, broadcast, reduce
                  the stand-alone collectives, packet format left to the library
  buffered        AllReduce of buffers outside the region through a bounded
                  scratch of iterations of "iter_kib" KiB per rank
  static          the same through the scratch the library holds
"""
import math

import torch

from paper_2607_16100_amd import llcoll as ll
from paper_2607_16100_amd.region import ScratchRegion, SymRegion

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "bf16": 2}
MAX_BYTES = 64 << 20  # per rank, of input or output


def listed():
    return [
        # the smallest real message: 4 ranks, 4 KiB each, one call after another
        {"name": "ar_4k_f32_p4", "op": "allreduce", "ranks": 4, "dtype": "f32", "count": 1024, "sentinel": False},
        # tensor-parallel decode at batch 1, hidden 8192: two calls a layer, 32 layers, captured
        {"name": "decode_b1_graph", "op": "decode_graph", "ranks": 8, "dtype": "bf16", "count": 8192, "calls": 64},
        # the same at batch 64 (1 MiB per rank), 8 layers
        {"name": "decode_b64_graph", "op": "decode_graph", "ranks": 8, "dtype": "bf16", "count": 64 * 8192, "calls": 16},
        # a ragged batch of tokens at a rank count that divides nothing
        {"name": "ar_ragged_bf16_p7", "op": "allreduce", "ranks": 7, "dtype": "bf16", "count": 301 * 4104, "sentinel": False},
        # tensor-parallel prefill: 1024 tokens, hidden 8192 (16 MiB per rank)
        {"name": "ar_prefill_bf16_p8", "op": "allreduce", "ranks": 8, "dtype": "bf16", "count": 1024 * 8192, "sentinel": False},
        # the largest: a gradient bucket of 64 MiB of binary32 per rank
        {"name": "ar_64m_f32_p8", "op": "allreduce", "ranks": 8, "dtype": "f32", "count": 16 << 20, "sentinel": False},
        # sequence-parallel halves at hidden 7168, batch 256
        {"name": "rs_b256_bf16_p8", "op": "reduce_scatter", "ranks": 8, "dtype": "bf16", "count": 256 * 7168},
        {"name": "ag_b256_bf16_p8", "op": "allgather", "ranks": 8, "dtype": "bf16", "count": 256 * 7168 // 8},
        # sharded weights gathered whole: 7168 x 2048 per rank at 4 ranks
        {"name": "ag_28m_bf16_p4", "op": "allgather", "ranks": 4, "dtype": "bf16", "count": 2048 * 7168 // 4},
        # weights from one rank to all, and a metric or gradient summed on one rank
        {"name": "bcast_16m_bf16_p8", "op": "broadcast", "ranks": 8, "dtype": "bf16", "count": 8 << 20, "root": 3},
        {"name": "reduce_4m_f32_p6", "op": "reduce", "ranks": 6, "dtype": "f32", "count": 1024 * 1024 + 6, "root": 2},
        # a large message through a small scratch
        {"name": "buffered_32m_f32_p8", "op": "buffered", "ranks": 8, "dtype": "f32", "count": 8 << 20, "iter_kib": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["allreduce"] * 5 + ["decode_graph"] * 2 + ["reduce_scatter", "allgather", "broadcast", "reduce",
                                                               "buffered", "static"])
    p = rng.choice([2, 3, 4, 5, 6, 7, 8, 8])
    dtype = rng.choice(["f32", "bf16"])
    es = BYTES[dtype]
    case = {"op": op, "ranks": p, "dtype": dtype}
    top = {"allreduce": MAX_BYTES, "decode_graph": 2 << 20, "reduce_scatter": 16 << 20, "allgather": (16 << 20) // p,
           "broadcast": 32 << 20, "reduce": 16 << 20, "buffered": 32 << 20, "static": 8 << 20}[op]
    count = max(2, _log(rng, 64, top) // es)
    if rng.random() < 0.6:
        count = max(8, count // 8 * 8)  # whole 16-byte rows of bfloat16, as hidden sizes give
    if op == "reduce_scatter":
        count = max(1, count // p) * p
    if op == "allreduce":
        case["sentinel"] = rng.random() < 0.3
    if op == "decode_graph":
        case["calls"] = rng.choice([8, 16, 32])
    if op in ("broadcast", "reduce"):
        case["root"] = rng.randrange(p)
    if op == "buffered":
        case["iter_kib"] = rng.choice([256, 512, 1024, 2048, 4096])
    case["count"] = count
    return case


def _inputs(case, seed):
    """[ranks, count] on the GPU: activations and gradients are about normal."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(case["ranks"], case["count"], generator=g, device="cuda", dtype=torch.float32)
    return x.to(TORCH[case["dtype"]])


def _out_elems(case):
    """Elements of all ranks' outputs of one call."""
    p, n = case["ranks"], case["count"]
    return {"reduce_scatter": n, "allgather": p * p * n, "reduce": n}.get(case["op"], p * n)


def prepare(case, seed):
    p, n, dtype, op = case["ranks"], case["count"], case["dtype"], case["op"]
    x = _inputs(case, seed)
    st = {"case": case}
    if op in ("buffered", "static"):
        if op == "buffered":
            reg = ScratchRegion(p, n, dtype, iter_bytes=case["iter_kib"] * 1024)
            reg.init()
            reg.inp[: p * n * BYTES[dtype]].view(TORCH[dtype]).copy_(x.view(-1))
            st["reg"] = reg
            st["out"] = reg.out[: p * n * BYTES[dtype]].view(TORCH[dtype]).view(p, n)
        else:
            st["in"] = x.contiguous()
            st["out"] = torch.empty_like(x)
        return st
    reg = SymRegion(p, n, dtype, out_elems=max(1, _out_elems(case)))
    reg.init()
    reg.write_inputs_device(x.view(torch.uint8).view(p, -1))
    st["reg"] = reg
    st["out"] = reg.out[: _out_elems(case) * BYTES[dtype]].view(TORCH[dtype])
    if op == "allreduce":
        st["opt"] = ll.Options(flags=ll.LL_OPT_AUTO_SENTINEL) if case["sentinel"] else None
    if op == "decode_graph":
        _capture(st, case, reg)
    return st


def _capture(st, case, reg):
    p, n, dt = case["ranks"], case["count"], ll.DTYPES[case["dtype"]]
    outs = torch.empty(case["calls"], p, -(-n // 8) * 8, dtype=TORCH[case["dtype"]], device="cuda")
    call_bytes = outs[0].numel() * outs.element_size()

    def call(i, epoch, stream):
        # the P outputs of a call lie back to back
        ll.check(ll.ll_allreduce(reg.base, reg.rank_stride, outs.data_ptr() + i * call_bytes, n, dt, ll.LL_SUM, p, epoch,
                                 stream), "ll_allreduce")

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # one call before the capture, for the library's lazy set-up
        call(0, 1, side.cuda_stream)
        reg.init(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for i in range(case["calls"]):
            call(i, 1 + i, side.cuda_stream)
    st["graph"] = graph
    st["out"] = outs.view(case["calls"], -1)[:, : p * n].view(case["calls"], p, n)


def run(st):
    case = st["case"]
    op, n = case["op"], case["count"]
    if op == "allreduce":
        ll.check(st["reg"].allreduce(n, opt=st["opt"]))
    elif op == "decode_graph":
        st["reg"].init()
        st["graph"].replay()
    elif op == "reduce_scatter":
        ll.check(st["reg"].reduce_scatter(n // case["ranks"]))
    elif op == "allgather":
        ll.check(st["reg"].allgather(n))
    elif op == "broadcast":
        ll.check(st["reg"].broadcast(n, case["root"]))
    elif op == "reduce":
        ll.check(st["reg"].reduce(n, case["root"]))
    elif op == "buffered":
        ll.check(st["reg"].allreduce(n))
    else:
        stream = torch.cuda.current_stream().cuda_stream
        ll.check(ll.ll_allreduce_static(st["in"].data_ptr(), st["out"].data_ptr(), n, ll.DTYPES[case["dtype"]],
                                        ll.LL_SUM, case["ranks"], stream, ll.LL_ALGO_AUTO)[0])
    return st["out"]


def work(case):
    """Every rank's input read once and every rank's output written once (a
    Broadcast reads the root's input only)."""
    p, n, es = case["ranks"], case["count"], BYTES[case["dtype"]]
    calls = case.get("calls", 1)
    read = n if case["op"] == "broadcast" else p * n
    adds = 0 if case["op"] in ("broadcast", "allgather") else (p - 1) * n
    return {"bytes": calls * (read + _out_elems(case)) * es, "flops": calls * adds}


def tolerance(case):
    # the sum is ordered by rank, in binary32, rounded once: one right answer
    return "exact"


def exact(case, seed):
    p, n, op = case["ranks"], case["count"], case["op"]
    x = _inputs(case, seed).double()
    if op == "broadcast":
        return x[case["root"]].repeat(p)
    if op == "allgather":
        return x.view(-1).repeat(p)
    s = x.sum(0)
    if op in ("reduce_scatter", "reduce"):
        return s
    if op == "decode_graph":
        return s.expand(case["calls"], p, n)
    if op == "allreduce":
        return s.repeat(p)
    return s.expand(p, n)

"""GPU parity of the ring kernels (the bandwidth-bound sizes) against the CPU
oracle: the edges of their sizes, tiles and chunks, every collective and
flagged format, calls mixed with other kernels on one region, graph replays
and muted ranks."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2607_16100_amd import workloads as wl  # noqa: E402

if torch.cuda.is_available():
    from paper_2607_16100_amd import llcoll as ll  # noqa: E402
    from paper_2607_16100_amd.region import ScratchRegion, SymRegion  # noqa: E402
    from test_edge_gpu import assert_same, edge_inputs  # noqa: E402
else:  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

NP = {"f32": np.uint32, "bf16": np.uint16}
ES = {"f32": 4, "bf16": 2}
KIB, MIB = 1 << 10, 1 << 20
RING_THREADS = 128


def stream():
    return torch.cuda.current_stream().cuda_stream


def opts(**kw):
    kw.setdefault("poll_timeout", 20_000_000)
    return ll.Options(report=True, **kw)


def call(reg, op, n, p, root, opt, **kw):
    f = {"allreduce": lambda: reg.allreduce(n, opt=opt, **kw), "reduce_scatter": lambda: reg.reduce_scatter(n // p, opt=opt, **kw),
         "allgather": lambda: reg.allgather(n, opt=opt, **kw), "broadcast": lambda: reg.broadcast(n, root, opt=opt, **kw),
         "reduce": lambda: reg.reduce(n, root, opt=opt, **kw)}[op]
    return f()


def want_of(op, x, root):
    return {"allreduce": lambda: oracle.allreduce(x), "reduce_scatter": lambda: oracle.reduce_scatter(x),
            "allgather": lambda: oracle.allgather(x), "broadcast": lambda: oracle.broadcast(x, root),
            "reduce": lambda: oracle.reduce(x, root)}[op]().reshape(-1)


def out_elems(op, p, n):
    return {"reduce_scatter": n, "allgather": p * p * n, "reduce": n}.get(op, p * n)


def check(reg, op, n, p, dtype, root, ring, what, opt=None, **kw):
    print(what, flush=True)
    x = wl.uniform(p, n, dtype, seed=n % 1009 + p)
    reg.write_inputs(x)
    reg.out.fill_(0xA5)
    opt = opt or opts()
    if p == 2:  # its wave-per-peer kernels have workgroups of the ring's size: read the region
        reg.init()
    assert call(reg, op, n, p, root, opt, **kw) == ll.LL_OK, what
    assert ll.ll_check(stream()) == ll.LL_OK, what
    if p != 2:
        assert (opt.threads == RING_THREADS) == ring, f"{what}: on a workgroup of {opt.threads} threads"
    else:
        packet8 = kw.get("proto") == "packet8" or kw.get("algo") == "twoshot_waves"
        st, offs = ll.ll_slice_layout(reg.rank_stride, p)
        area = reg.sym.view(p, -1)[:, offs[1 if packet8 else 2]:offs[2 if packet8 else 3]]
        assert went_round_the_ring(area, op, n, dtype, packet8, reg.epoch, root) == ring, what
    total = out_elems(op, p, n)
    got = reg.read_out(total, NP[dtype])
    bad = np.flatnonzero(got != want_of(op, x, root))
    assert bad.size == 0, f"{what}: {bad.size} elements differ, first at {bad[0]}"
    if total * ES[dtype] < reg.out.numel():
        assert (reg.out[total * ES[dtype]:total * ES[dtype] + 4096] == 0xA5).all(), f"{what}: wrote past the outputs"


def went_round_the_ring(area, op, n, dtype, packet8, epoch, root=0):
    """Whether a 2-rank call whose packet area was clear before it ran on a ring
    kernel, from what it left there: on the ring every wave's completion block
    holds the epoch and nothing else (another kernel leaves the area clear there,
    or payload); a ReduceScatter has none, and leaves the area clear behind the
    ring, where another kernel's slot still has packets."""
    p, mode, es = 2, list(FIRST).index(op), ES[dtype]
    chunk = {"reduce_scatter": n // p * es, "allgather": n * es}.get(op, -(-(-(-n // p)) // (16 // es)) * 16)
    tiles = -(-chunk // (512 if packet8 else 960))
    waves_per_cu = 8 if op == "allgather" else 16
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    st, (_, waves, slot, flags) = ll.ll_ring_shape(p, mode, tiles, area.shape[1], 2, waves_per_cu * cus // 2 // p)
    assert st == ll.LL_OK
    if op == "reduce_scatter":
        assert slot < tiles * 1024  # or the other kernel's slot would end inside the ring's
        return not bool(area[:, slot:tiles * 1024].any())
    blocks = area[:, flags:flags + waves * 64].cpu().numpy().view(np.uint32).reshape(p, waves, 16)
    if op == "reduce":  # only the root is told
        blocks = blocks[root:root + 1]
    return bool((blocks[..., 15] == epoch).all() and not blocks[..., :15].any())


def scratch_area(d, packet8):
    """Byte range of the flagged sub-buffers in a 2-rank scratch slice for iterations of d bytes."""
    chunk = (-(-d // 2) + 4 + 15) // 16 * 16
    a8, a128 = (max(f(d), 2 * f(chunk)) for f in (lambda b: -(-(-(-b // 4) * 8) // 256) * 256,
                                                  lambda b: -(-(-(-b // 4)) // 240) * 1024))
    return (0, 2 * a8) if packet8 else (2 * a8, 2 * a8 + 2 * a128)


# First size in bytes on the ring, by rank count, whether the stream has an odd
# number of bfloat16 elements, and packet format (per rank; AllGather: sent).
NEVER = 1 << 40


def first_rooted(p, odd, line):
    if p == 8:
        return (256 if line else 192) * KIB if odd else 128 * KIB
    return None


def first_reduce(p, odd, line):
    by = {7: 2304 if line and odd else 2048, 6: 2096 if line else 2048, 5: 3072 if line else 2560, 4: 2048, 2: 16384,
          3: 16384 if line else NEVER}
    return first_rooted(p, odd, line) or by[p] * KIB


FIRST = {
    "allreduce": lambda p, odd=False, line=True: -(-((7680 if p == 8 and not odd else 7168) if line else
                                                     (6656 if p == 8 and odd else 5120)) * KIB // p),
    "reduce_scatter": lambda p, odd=False, line=True: NEVER if p == 2 and not line and not odd else
    -(-(38 if p == 6 and not line else 32) * MIB // p),
    "allgather": lambda p, odd=False, line=True: -(-(256 if line or not odd or p > 4 else 1600 if p == 2 else 512) * KIB // p),
    "broadcast": lambda p, odd=False, line=True: first_rooted(p, odd, line) or (MIB if p >= 4 else 4 * MIB),
    "reduce": lambda p, odd=False, line=True: first_reduce(p, odd, line),
}


@pytest.mark.parametrize("op", list(FIRST))
@pytest.mark.parametrize("p,dtype", [(2, "bf16"), (3, "f32"), (4, "bf16"), (5, "f32"), (7, "bf16"), (8, "f32")])
def test_sizes_at_the_edges(op, p, dtype):
    """Just below and at the first ring size, and above it: whole tiles, a
    word more and less, ragged chunks, a last chunk of one word."""
    es = ES[dtype]
    unit = p if op == "reduce_scatter" else 1  # ReduceScatter inputs are P equal chunks
    even = 2 if dtype == "bf16" else 1          # whole words
    first = -(-FIRST[op](p) // es)
    first = -(-first // (unit * even)) * unit * even
    tile = 960 // es * (1 if op == "allgather" else p)  # one more tile in every chunk
    top = first + 40 * tile
    tiles = -(-first // tile)
    sizes = [first - unit * even, first, first + unit * even, tile * (tiles + 1) // (unit * even) * unit * even,
             top - 3 * unit * even, top]
    if op == "allreduce":  # chunks are rounded up to 16 bytes: the last one is short
        c = -(-top // p) // (16 // es) * (16 // es)
        sizes.append((p - 1) * c + even)
    reg = SymRegion(p, top, dtype, out_elems=out_elems(op, p, top) + 4096)
    reg.init()
    for root in ((p - 1, 1) if op in ("broadcast", "reduce") else (0,)):
        for i, n in enumerate(sizes):
            ring = i > 0
            check(reg, op, n, p, dtype, root, ring if n >= first else False, f"{op} P={p} {dtype} n={n} root={root}")
        # the same size with a tuning field set, which the ring kernels leave to the others
        check(reg, op, first, p, dtype, root, False, f"{op} P={p} {dtype} n={first} root={root} tuned", opts(pipeline_lag=2))


@pytest.mark.parametrize("op", list(FIRST))
@pytest.mark.parametrize("proto", ["packet8", "line128"])
def test_named_formats_and_many_steps(op, proto):
    """8-byte packets and lines, at a size where the ring goes round several
    times, and a region that holds that format only."""
    p, dtype = 8, "bf16"
    n = {"allreduce": 10 * MIB + 6, "reduce_scatter": 8 * MIB, "allgather": MIB + 2}.get(op, 10 * MIB + 6)
    algo = "twoshot_waves" if proto == "packet8" else "twoshot_line_waves"
    reg = SymRegion(p, n, dtype, out_elems=out_elems(op, p, n) + 4096, sized_for=algo)
    reg.init()
    for k in range(2):
        kw = {"algo": algo} if op == "allreduce" else {"proto": proto}
        check(reg, op, n, p, dtype, 5, True, f"{op} {proto} call {k}", **kw)


@pytest.mark.parametrize("op", list(FIRST))
@pytest.mark.parametrize("p", [2, 3, 6, 7, 8])
def test_streams_that_start_and_end_on_half_a_word(op, p):
    """Odd bfloat16 counts: rows of odd ranks start on half a word, and a
    stream's last element is half of one.  The half word at every place of a
    lane, at a tile's and a chunk's first and last word, and in 8-byte packets."""
    unit = p if op == "reduce_scatter" else 1
    base = -(-FIRST[op](p, odd=True) // 2 // unit) | 1  # elements of a chunk (ReduceScatter) or of the message
    tile = 480 * (1 if op in ("allgather", "reduce_scatter") else p)
    top = base // tile * tile + 3 * tile
    counts = [base, base + 2, base + 4, base + 6, top - 1, top + 1]
    reg = SymRegion(p, (top + 8) * unit, "bf16", out_elems=out_elems(op, p, (top + 8) * unit) + 4096)
    reg.init()
    for m in counts:
        check(reg, op, m * unit, p, "bf16", p - 1, True, f"{op} P={p} odd count {m}")
    kw = {"algo": "twoshot_waves"} if op == "allreduce" else {"proto": "packet8"}
    for m in (counts[0], counts[1]):
        ring = 2 * m * unit >= FIRST[op](p, odd=True, line=False)
        check(reg, op, m * unit, p, "bf16", 0, ring, f"{op} P={p} odd count {m} packet8", **kw)


@pytest.mark.parametrize("op,p,odd,line", [
    ("allreduce", 8, True, False), ("reduce_scatter", 6, False, False), ("reduce_scatter", 2, False, False),
    ("allgather", 2, True, False), ("allgather", 4, True, False), ("broadcast", 8, True, True),
    ("broadcast", 8, True, False), ("reduce", 8, True, True), ("reduce", 7, True, True), ("reduce", 6, False, True),
    ("reduce", 5, False, False), ("reduce", 3, False, False)])
def test_first_sizes_that_differ_by_format_and_odd_streams(op, p, odd, line):
    """Just below and at the first size on the ring; a large message where the
    ring never serves."""
    unit = p if op == "reduce_scatter" else 1
    first = FIRST[op](p, odd, line)
    never = first >= NEVER
    m = -(-(20 * MIB if never else first) // (2 * unit))
    m += (m + odd) % 2
    reg = SymRegion(p, m * unit, "bf16", out_elems=out_elems(op, p, m * unit) + 4096)
    reg.init()
    kw = {"algo": "twoshot_line_waves" if line else "twoshot_waves"} if op == "allreduce" else {
        "proto": "line128" if line else "packet8"}
    for k, ring in ((m - 2, False), (m, not never)):
        check(reg, op, k * unit, p, "bf16", p - 1, ring, f"{op} P={p} odd={odd} {kw} {k * unit} elements", **kw)


def test_ring_and_other_kernels_share_a_region():
    """Calls of every kind and size in turn on one region, epochs one apart
    and up to the last one: no call takes another's packets for its own."""
    p, dtype = 8, "f32"
    n = 4 * MIB // 4
    reg = SymRegion(p, n, dtype, out_elems=p * p * n // 8 + 4096)
    reg.init()
    plan = [("allreduce", n, {}), ("allreduce", 4096, {}), ("allreduce", 16384, {"algo": "oneshot_line_waves"}),
            ("allreduce", n, {}), ("broadcast", n - 1, {}), ("allreduce", 65536, {"algo": "twoshot_line"}),
            ("reduce", n - 2, {}), ("allgather", n // 8, {}), ("allreduce", n, {"algo": "twoshot_waves"}),
            ("reduce_scatter", n, {}), ("allreduce", 30001, {}), ("allgather", n // 8 - 1, {"proto": "packet8"}),
            ("allreduce", n - 5, {})]
    for start in (0, 0xFFFFFFFF - len(plan)):
        reg.epoch = start
        for op, m, kw in plan:
            x = wl.normal(p, m, dtype, seed=m % 77 + reg.epoch % 5)
            reg.write_inputs(x)
            print(op, m, kw, reg.epoch, flush=True)
            assert call(reg, op, m, p, 2, opts(), **kw) == ll.LL_OK
            assert ll.ll_check(stream()) == ll.LL_OK
            got = reg.read_out(out_elems(op, p, m), NP[dtype])
            assert np.array_equal(got, want_of(op, x, 2)), f"{op} {m} {kw} epoch {reg.epoch}"
    assert reg.epoch == 0xFFFFFFFF


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("p,dtype,iter_bytes", [(2, "f32", 4096), (5, "bf16", 8192), (7, "f32", 20000), (8, "bf16", 1 << 18),
                                                (3, "odd", 6000), (8, "odd", 1 << 18)])
def test_bounded_scratch_goes_round_the_ring(p, dtype, iter_bytes, in_place):
    """Scratch regions that hold a few waves' rings: dozens to hundreds of
    steps, two calls, from epoch 1."""
    odd = 1 if dtype == "odd" else 0
    dtype = "bf16" if odd else dtype
    es = ES[dtype]
    n = 120 * iter_bytes // es + 2 + odd
    if iter_bytes > 65536:
        n = 9 * iter_bytes // es + 14 + odd
    reg = ScratchRegion(p, n, dtype, iter_bytes=iter_bytes, in_place=in_place)
    reg.init()
    for k, algo in enumerate(("auto", "twoshot_waves", "twoshot_line", "auto")):
        x = wl.normal(p, n, dtype, seed=10 * k + p)
        reg.write_inputs(x)
        opt = opts()
        if p == 2:  # as in check()
            reg.init()
        print(f"P={p} {dtype} {iter_bytes} in_place={in_place} {algo}", flush=True)
        assert reg.allreduce(n, algo, opt=opt) == ll.LL_OK
        assert ll.ll_check(stream()) == ll.LL_OK
        assert opt.threads == RING_THREADS and reg.last_iters > 1
        if p == 2:
            packet8 = algo == "twoshot_waves"
            lo, hi = scratch_area(reg.iter_bytes, packet8)
            assert went_round_the_ring(reg.scratch.view(p, -1)[:, lo:hi], "allreduce", n, dtype, packet8,
                                       reg.epoch - reg.last_iters + 1)
        assert np.array_equal(reg.read_out(p * n, NP[dtype]).reshape(p, n), oracle.allreduce(x)), algo


@pytest.mark.parametrize("op", ["allreduce", "reduce_scatter", "reduce"])
@pytest.mark.parametrize("p,dtype", [(3, "f32"), (8, "f32"), (8, "bf16")])
def test_infinities_nan_and_overflow(op, p, dtype):
    """The edges of IEEE arithmetic and of the rounding to bfloat16 (the columns
    of test_edge_gpu.py, repeated over the whole message) on the ring kernels."""
    es = ES[dtype]
    n = -(-FIRST[op](p) // es // (2 * p)) * 2 * p + 2 * p
    cols = edge_inputs(p, dtype, repeat=1)
    x = np.ascontiguousarray(np.tile(cols, (1, -(-n // cols.shape[1])))[:, :n])
    reg = SymRegion(p, n, dtype, out_elems=out_elems(op, p, n))
    reg.init()
    reg.write_inputs(x)
    opt = opts()
    print(op, p, dtype, n, flush=True)
    assert call(reg, op, n, p, 1, opt) == ll.LL_OK
    assert ll.ll_check(stream()) == ll.LL_OK
    assert opt.threads == RING_THREADS
    assert_same(reg.read_out(out_elems(op, p, n), NP[dtype]), want_of(op, x, 1), f"{op} P={p} {dtype}")


@pytest.mark.parametrize("op", list(FIRST))
def test_muted_rank_times_out(op):
    """A rank that publishes nothing is noticed by its peers, and the region
    works again after ll_init."""
    p, dtype, root = 8, "bf16", 1
    n = {"reduce_scatter": 16 * MIB}.get(op, MIB)
    reg = SymRegion(p, n, dtype, out_elems=out_elems(op, p, n))
    reg.init()
    mute = root if op == "broadcast" else 6
    reg.write_inputs(wl.normal(p, n, dtype, seed=3))
    print(op, "muted", flush=True)
    assert call(reg, op, n, p, root, opts(poll_timeout=200_000, mute_rank=mute)) == ll.LL_OK
    assert ll.ll_check(stream()) == ll.LL_ERR_TIMEOUT
    # the first wait to expire is a peer's, for the muted rank, or the muted
    # rank's own, for the outputs its peers cannot finish
    rank, missing, _ = ll.ll_last_timeout()
    assert missing == 1 << mute if rank != mute else missing
    reg.init()
    check(reg, op, n, p, dtype, root, True, f"{op} after the timeout")


@pytest.mark.parametrize("op,n", [("allreduce", 2 * MIB), ("allgather", 65536), ("broadcast", 65536 * 3), ("reduce", MIB)])
def test_graph_replays(op, n):
    """Captured ring calls replayed several times, the region reset and new
    inputs written before each replay."""
    p, dtype = 8, "bf16"
    reg = SymRegion(p, n, dtype, out_elems=out_elems(op, p, n))
    reg.init()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert call(reg, op, n, p, 3, None) == ll.LL_OK
    torch.cuda.synchronize()
    reg.init(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for i in range(3):
            assert call(reg, op, n, p, 3, None, epoch=1 + i) == ll.LL_OK
    for rep in range(3):
        x = wl.normal(p, n, dtype, sigma=10.0 ** (rep - 1), seed=40 + rep)
        print(op, "replay", rep, flush=True)
        reg.write_inputs(x)
        reg.init()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert ll.ll_check(side.cuda_stream) == ll.LL_OK
        assert np.array_equal(reg.read_out(out_elems(op, p, n), NP[dtype]), want_of(op, x, 3)), f"{op} replay {rep}"


@pytest.mark.parametrize("n,algo,ring_algo", [(16384, "auto", "auto"), (4096, "auto", "twoshot_waves"),
                                              (16384, "oneshot_line", "twoshot_line")])
def test_static_call_captured_before_a_ring_call_runs_after_it(n, algo, ring_algo):
    """ll_allreduce_static takes its epoch when it is called: a captured call
    is replayed after an eager call with a later epoch that went round the ring
    more than once over the same positions.  The captured call must not take
    any of that call's packets for its own."""
    p, big = 8, 4 * MIB // 4
    dev = lambda bits: torch.from_numpy(np.ascontiguousarray(bits).view(np.uint8).reshape(-1).copy()).cuda()  # noqa: E731
    x, y = wl.normal(p, n, "f32", seed=5), wl.normal(p, big, "f32", seed=6)
    xin, yin = dev(x), dev(y)
    xout, yout = torch.zeros_like(xin), torch.zeros_like(yin)

    def static(inp, out, m, name, s):
        st, used = ll.ll_allreduce_static(inp.data_ptr(), out.data_ptr(), m, ll.LL_F32, ll.LL_SUM, p, s, ll.ALGOS[name])
        assert st == ll.LL_OK, ll.ll_strerror(st)
        return used

    side = torch.cuda.Stream()
    static(xin, xout, n, algo, side.cuda_stream)  # lazy set-up, before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        assert static(xin, xout, n, algo, side.cuda_stream) == 1
    torch.cuda.synchronize()
    xout.zero_()
    print(f"static {algo} n={n} captured, {ring_algo} in between", flush=True)
    assert static(yin, yout, big, ring_algo, stream()) > 1
    assert ll.ll_check(stream()) == ll.LL_OK
    graph.replay()
    torch.cuda.synchronize()
    assert ll.ll_check(side.cuda_stream) == ll.LL_OK
    assert np.array_equal(yout.cpu().numpy().view(np.uint32).reshape(p, big), oracle.allreduce(y))
    assert np.array_equal(xout.cpu().numpy().view(np.uint32).reshape(p, n), oracle.allreduce(x))


@pytest.mark.parametrize("iter_bytes,sentinel,tuning,named", [
    (8192, False, {"pipeline_lag": 2}, "twoshot_waves"),            # a call the ring kernels do not serve
    (65536, True, {"pipeline_lag": 2}, "twoshot_sentinel_waves"),
    (1024, False, {}, "twoshot_waves"),                             # a scratch too small for a workgroup's ring
    (1024, True, {}, "twoshot_waves"),
    (8192, False, {}, "twoshot_line_waves"),                        # on the ring
    (65536, True, {}, "twoshot_line_waves")])
def test_bounded_scratch_auto_takes_the_ring_only_where_it_runs(iter_bytes, sentinel, tuning, named):
    """AUTO in several iterations: the ring kernel's format where it serves the
    call, and otherwise the algorithm measured for the iteration's size.  The
    scratch holds the same bytes after the call as after the named algorithm's."""
    p, dtype = 8, "bf16"
    n = 5 * iter_bytes // 2 + 6
    images = {}
    for algo in ("auto", named):
        reg = ScratchRegion(p, n, dtype, iter_bytes=iter_bytes)
        reg.init()
        x = wl.normal(p, n, dtype, seed=12)
        reg.write_inputs(x)
        flags = ll.LL_OPT_AUTO_SENTINEL if sentinel else 0
        print(f"{algo} {iter_bytes} sentinel={sentinel} {tuning}", flush=True)
        assert reg.allreduce(n, algo, opt=opts(flags=flags, **tuning)) == ll.LL_OK
        assert ll.ll_check(stream()) == ll.LL_OK
        assert reg.last_iters > 1
        assert np.array_equal(reg.read_out(p * n, NP[dtype]).reshape(p, n), oracle.allreduce(x)), algo
        images[algo] = reg.scratch.cpu().numpy().copy()
    assert np.array_equal(images["auto"], images[named])


@pytest.mark.parametrize("tuning,proto,ring", [({}, "line128", True), ({"clear_slots": 2}, "sentinel", False)])
def test_allgather_with_sentinel_units_allowed(tuning, proto, ring):
    """AUTO with sentinel units allowed, from the ring AllGather's size on: the
    ring kernel where it serves the call, otherwise sentinel units.  The
    region holds the same bytes after the call as after the named format's."""
    p, n, dtype = 8, 64 * KIB, "bf16"
    images = []
    for name, flags in (("auto", ll.LL_OPT_AUTO_SENTINEL), (proto, 0)):
        reg = SymRegion(p, n, dtype)
        reg.sym.zero_()
        reg.init()
        check(reg, "allgather", n, p, dtype, 0, ring, f"allgather {name} {tuning}", opts(flags=flags, **tuning), proto=name)
        images.append(reg.sym.cpu().numpy().copy())
    assert np.array_equal(*images)

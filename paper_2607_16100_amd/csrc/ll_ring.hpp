// Ring kernels: the collectives at the sizes that are bound by bandwidth.
//
// AllReduce (two-shot), ReduceScatter, AllGather, Broadcast and Reduce with
// 128-byte lines or 8-byte packets.  What bounds them is the fabric between
// the XCDs and the memory side: reads and writes together run at about 6.6
// TB/s when packets are written by one XCD and read by another, whatever the
// number of waves, and writes that leave the 256 MiB memory-side cache cost
// HBM bandwidth on top.  So the kernels move as few bytes as the exchange
// allows, and keep what they move in the cache:
//  - No gather through scratch.  The owner of a reduced chunk stores it
//    straight into every rank's output, and at its end tells every peer so
//    with one completion flag per wave.  A gather through packets writes and
//    reads each result once more per peer: 64 MiB of binary32 per rank at 8
//    ranks moves 3.3 GB with it and 2.1 GB without.
//  - A ring of packets.  A wave reuses kRingEntries positions of 1 KiB per
//    peer instead of a slot position per tile, so the packets of a call of any
//    size live in at most 56 MiB at 8 ranks, which that cache can hold (a
//    Broadcast's packets have a position per tile and grow with the message).  Each
//    peer's packets are the credit to go on (see kRingEntries), so a ring needs no
//    counter, no barrier and no second buffer; a bounded-scratch call needs no
//    iterations.
//  - Waves that work alone.  A wave takes a tile of every chunk: it sends P-1
//    tiles and reduces one, all in registers, with no LDS and no workgroup
//    barrier, and its next tile's packets go out before it waits.
// Measured (8 ranks, bfloat16 unless said, back-to-back calls on one region,
// against the kernels that pass the result through scratch): AllReduce 1 MiB 10.7
// -> 9.6 us, 4 MiB 31.4 -> 21.9, 16 MiB 124 -> 78 (86 from a program's calls on
// changing inputs), 64 MiB of binary32 504 -> 317; AllGather 448 KiB sent 17.5 ->
// 8.0; Broadcast 16 MiB 146 -> 42; Reduce 16 MiB 147 -> 62; bounded scratch, 32 MiB
// in 1 MiB iterations 339 -> 163.  The figures beside single choices below compare
// two forms in the same run.
//
// Grid = P * W workgroups of kRingThreads threads; workgroup b serves rank
// r = b % P, and its waves are numbered g = (b / P) * waves + wave, G of them
// a rank.  A chunk is cut into tiles of one wave each (ProtoLine: 960 payload
// bytes in 1 KiB of packets; ProtoLL: 512 payload bytes in 1 KiB); wave g of
// every rank handles tiles g, g + G, g + 2 G, ... of every chunk, its steps.
// The host keeps the grid resident, and every wait is bounded.
//
// Modes: AllReduce and Reduce cut the message into P chunks (the last ones
// may be short or empty) and rank r reduces chunk r for every rank's output or
// for the root's; ReduceScatter has P chunks of equal length and keeps chunk r;
// AllGather sends no packets, rank r stores its input as block r of every
// output; Broadcast cuts the root's message into P chunks, sends chunk r to
// rank r as packets, and rank r stores it into every output, so that every
// rank's CUs carry the copies and not the root's alone.
#pragma once

#include "ll_device.hpp"
#include "ll_kernels.hpp"
#include "ll_layout.hpp"

namespace llc {

using layout::RingMode;
using layout::RING_AG;
using layout::RING_AR;
using layout::RING_BCAST;
using layout::RING_REDUCE;
using layout::RING_RS;

// Ring positions of a wave in each of its slots.  In its step s a wave
// publishes tile s and then reduces tile s - 1.  So when it publishes tile s,
// it has every peer's tile s - 2, which the peer published after it had
// reduced tile s - 4: position s % 4 has been read and is free again.
//
// The flag must tell a position's tiles apart although the caller gives a
// call one epoch: the tiles of a position carry the epoch and 0 in turn
// (layout::ring_flag).  The first time round a position holds another call's
// flag or 0, neither of which is the epoch; from then on it holds the other
// value of the two, because its reader has seen it there, so a 0 is never
// waited for where one was left before the call.  Neither value can be taken
// for another call's epoch, whichever of the two calls runs first: a call
// captured into a graph runs after calls that were given later epochs.
constexpr uint32_t kRingEntries = (uint32_t)layout::kRingEntries;
static_assert(kRingEntries == 4, "a publish one step ahead needs four positions");
// Waves are independent; two to a workgroup spread a 1 MiB call over the CUs
// more evenly than four (9.2 against 10.0 us) and cost less to dispatch than
// single ones (64 MiB: 308 against 317 us).
constexpr int kRingThreads = 128;

struct RingArgs {
  char *sym;            // region base; rank r's slice at sym + r * stride
  uint64_t stride;
  const char *in;       // rank r's input at in + r * in_stride
  uint64_t in_stride;
  char *out;            // rank q's output at out + q * out_pitch
  uint64_t out_pitch;
  uint64_t area;        // offset of the ring slots in every slice
  uint64_t flags;       // offset of the completion flags in every slice
  uint64_t timeout;     // flag-wait budget, 100 MHz ticks
  uint32_t *status;
  uint64_t *stamps;
  uint32_t total;       // bytes of the stream the P chunks make up (at most kRingMaxBytes)
  uint32_t chunk;       // bytes of a chunk (the last ones may be short or empty)
  uint32_t slot;        // bytes of a ring slot
  uint32_t tiles;       // tiles per chunk
  uint32_t waves;       // G: waves per rank
  uint32_t epoch;
  int32_t mute;         // rank that publishes nothing (test hook), or -1
  uint32_t root;
  uint32_t grid;
};

typedef void (*ring_fn)(RingArgs);

template <class Pr>
struct RingTile {
  static constexpr uint32_t kPayload = Pr::kLanes == 64 ? 960 : Pr::kUnitWords * 4 * 64;
  static constexpr uint32_t kPackets = 1024;
};

__device__ __forceinline__ RingArgs pin_args(const RingArgs &k) {
  RingArgs a;
  a.sym = in_sgpr(k.sym);
  a.stride = in_sgpr(k.stride);
  a.in = in_sgpr(k.in);
  a.in_stride = in_sgpr(k.in_stride);
  a.out = in_sgpr(k.out);
  a.out_pitch = in_sgpr(k.out_pitch);
  a.area = in_sgpr(k.area);
  a.flags = in_sgpr(k.flags);
  a.timeout = in_sgpr(k.timeout);
  a.status = in_sgpr(k.status);
  a.stamps = in_sgpr(k.stamps);
  a.total = in_sgpr(k.total);
  a.chunk = in_sgpr(k.chunk);
  a.slot = in_sgpr(k.slot);
  a.tiles = in_sgpr(k.tiles);
  a.waves = in_sgpr(k.waves);
  a.epoch = in_sgpr(k.epoch);
  a.mute = in_sgpr(k.mute);
  a.root = in_sgpr(k.root);
  a.grid = in_sgpr(k.grid);
  return a;
}

// Odd: streams with an odd number of bfloat16 elements.  Rows then start on
// half a word for every other rank, which 16-byte buffer accesses take at some
// cost (a copy with such stores runs at two thirds of the speed), and end in
// half a word, which goes as 2 bytes of its own so that nothing outside the
// row is read or written.
template <class Pr, int DT, int P, int Mode, bool Odd>
__global__ __launch_bounds__(kRingThreads) void k_ring(RingArgs ka) {
  const RingArgs a = pin_args(ka);
  const uint64_t t_start = a.stamps != nullptr ? now_ticks() : 0;
  constexpr uint32_t TB = RingTile<Pr>::kPayload, PB = RingTile<Pr>::kPackets;
  constexpr int NW = Pr::kMaxWords;
  constexpr uint32_t kNowhere = 0x80000000u;  // past every resource, also with a stream offset added to it
  // Outputs are written through to the coherence point (a peer's completion
  // flag stands for them) and not read again: 16 MiB with the streaming hint
  // 79 us, without it 82; inputs are loaded without it (64 MiB: 306 against
  // 310 us, 4 MiB 22.8 against 28.7), packets neither stored nor polled with it
  // (64 MiB: 397 us).
  constexpr int kOut = kSC1 | kNT;
  const uint32_t r = blockIdx.x % P;
  const uint32_t lane = threadIdx.x & 63;
  const int sub = Pr::kLanes == 64 ? (int)lane : 0;
  const uint32_t g = uniform_u32((blockIdx.x / P) * (kRingThreads / 64) + (threadIdx.x >> 6));
  const uint32_t G = a.waves;
  const uint32_t steps = g < a.tiles ? (a.tiles - g + G - 1) / G : 0;
  // the lane's payload within a tile
  uint32_t po = lane * NW * 4;
  if constexpr (Pr::kLanes == 64) po = lane < 60 ? lane * 16 : kNowhere;
  const bool publish = (int)r != a.mute;
  const bool sends = Mode != RING_BCAST || r == a.root;  // Broadcast: only the root has packets to send
  const uint32_t want = Mode == RING_BCAST ? (r == a.root ? 0u : 1u << a.root) : ((1u << P) - 1u) & ~(1u << r);
  const rsrc_t in_rs = make_rsrc(a.in + (uint64_t)r * a.in_stride, Mode == RING_AG ? a.chunk : a.total);
  char *const slice_r = a.sym + (uint64_t)r * a.stride;
  const rsrc_t ring_rs = make_rsrc(slice_r + a.area, (P - 1) * a.slot);
  const uint32_t my_chunk = r * a.chunk;
  const uint32_t my_end = my_chunk + a.chunk < a.total ? my_chunk + a.chunk : (my_chunk < a.total ? a.total : my_chunk);
  WaitBudget budget(a.timeout, a.status);
  bool dead = false;  // a wait has expired: the wave waits no more

  auto chunk_len = [&](uint32_t c) -> uint32_t {
    const uint32_t at = c * a.chunk;
    return at >= a.total ? 0u : (a.total - at < a.chunk ? a.total - at : a.chunk);
  };
  // Odd: which of the lane's words at byte `at` of a chunk of `len` bytes is the
  // half word at its end (0..NW-1); NW or more: none.
  auto tail_word = [&](uint32_t len, uint32_t at) -> uint32_t {
    return (len & 2u) != 0 && po != kNowhere ? ((len & ~3u) - (po + at)) / 4 : kNowhere;
  };
  // The lane's words at byte `at` of chunk c of the rank's input (AllGather: of
  // its input).
  auto load_tile = [&](uint32_t c, uint32_t at) -> u32x4 {
    u32x4 v = {0u, 0u, 0u, 0u};
    rsrc_t rs = in_rs;
    uint32_t off = po + at, len = 0;
    if constexpr (Odd) {
      len = Mode == RING_AG ? a.chunk : chunk_len(c);
      rs = make_rsrc(a.in + (uint64_t)r * a.in_stride + (Mode == RING_AG ? 0 : (uint64_t)c * a.chunk), len & ~3u);
    } else {
      off += Mode == RING_AG ? 0 : c * a.chunk;
    }
    if constexpr (NW == 2) {
      const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
      v.x = w.x;
      v.y = w.y;
    } else {
      v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    }
    if constexpr (Odd) {
      const uint32_t j = tail_word(len, at);
      const rsrc_t rt = make_rsrc(a.in + (uint64_t)r * a.in_stride + (Mode == RING_AG ? 0 : (uint64_t)c * a.chunk), len);
      const uint32_t h = __builtin_amdgcn_raw_buffer_load_b16(rt, (int)(j < NW ? len - 2 : kNowhere), 0, 0);
      v.x = j == 0 ? h : v.x;
      v.y = j == 1 ? h : v.y;
      if constexpr (NW == 4) {
        v.z = j == 2 ? h : v.z;
        v.w = j == 3 ? h : v.w;
      }
    }
    return v;
  };
  auto flag_of = [&](uint32_t s) -> uint32_t {
    return Mode == RING_BCAST ? a.epoch : layout::ring_flag(a.epoch, s);
  };
  // A Broadcast has no packets coming back as credit: every tile has a
  // position of its own.
  auto pos_of = [&](uint32_t s) -> uint32_t {
    return uniform_u32((g + (Mode == RING_BCAST ? s : s % kRingEntries) * G) * PB);
  };
  // The result of the wave's tile at byte `at` of chunk r, to its output(s).
  auto store_out = [&](uint32_t at, u32x4 v) {
    v = Pr::start_store(v, sub);
    const uint32_t j = Odd ? tail_word(my_end - my_chunk, at) : 0;
    const uint32_t half = j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t q = (r + k) % P;
      if (Mode == RING_RS && k > 0) break;
      if (Mode == RING_REDUCE && k > 0) break;
      const uint32_t to = Mode == RING_REDUCE ? a.root : q;
      const bool to_it = publish || to == r;
      // Odd: the resource starts at the chunk, so that its whole words count
      // from there
      char *const row = a.out + (uint64_t)to * a.out_pitch + (Odd ? my_chunk : 0u);
      const uint32_t end = my_end - (Odd ? my_chunk : 0u);
      const int off = (int)(po + at + (Odd ? 0u : my_chunk));
      const rsrc_t rd = make_rsrc(row, to_it ? (Odd ? end & ~3u : end) : 0u);
      if constexpr (Odd)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)half, make_rsrc(row, to_it ? end : 0u),
                                              (int)(j < NW ? end - 2 : kNowhere), 0, kOut);
      if constexpr (NW == 2) {
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, rd, off, 0, kOut);
      } else {
        __builtin_amdgcn_raw_buffer_store_b128(v, rd, off, 0, kOut);
      }
    }
  };

  if constexpr (Mode == RING_AG) {
    for (uint32_t s = 0; s < steps; ++s) {
      const uint32_t at = (g + s * G) * TB;
      store_out(at, Pr::finish_load(load_tile(r, at), sub));
    }
  } else {
    u32x4 own = {0u, 0u, 0u, 0u};
    for (uint32_t s = 0; s <= steps; ++s) {
      const u32x4 mine = own;  // the own tile of step s - 1
      if (s < steps && sends) {
        const uint32_t at = (g + s * G) * TB;
        // A wave that has not sent yet goes before waves that poll: 1 MiB
        // 11.0 -> 10.0 us, 16 MiB 91 -> 82 us.
        __builtin_amdgcn_s_setprio(3);
        u32x4 x[P];  // x[k]: the tile of chunk (r + k) % P
#pragma unroll
        for (int k = 0; k < P; ++k) x[k] = load_tile((r + k) % P, at);
        // The ring position goes into the vector offset, not into a scalar
        // offset register: with one, the compiler lets the instruction after a
        // 16-byte buffer store overwrite the store's data registers, and the
        // last lanes of the store have then carried the new contents.
        const uint32_t off = publish ? pos_of(s) + lane * 16 : kNowhere;
        const uint32_t f = flag_of(s);
#pragma unroll
        for (int k = 1; k < P; ++k) {
          const uint32_t q = (r + k) % P;
          char *dst = a.sym + (uint64_t)q * a.stride + a.area + (uint64_t)(r - (r > q ? 1u : 0u)) * a.slot;
          st_pkt(make_rsrc(dst, a.slot), off, Pr::pack(Pr::finish_load(x[k], sub), f, sub));
        }
        own = Pr::finish_load(x[0], sub);
      }
      __builtin_amdgcn_s_setprio(0);
      if (s == 0) continue;
      // ---- tile s - 1: poll the peers' packets, reduce, store
      const uint32_t off = pos_of(s - 1) + lane * 16;
      const uint32_t f = flag_of(s - 1);
      u32x4 got[P];
#pragma unroll
      for (int q = 0; q < P; ++q) got[q] = u32x4{0u, 0u, 0u, 0u};
      uint32_t pend = want;
      uint32_t spins = 0;
      while (true) {
        compiler_fence();
#pragma unroll
        for (uint32_t q = 0; q < P; ++q)
          if (pend & (1u << q)) got[q] = ld_pkt(ring_rs, off, (q - (q > r ? 1u : 0u)) * a.slot);
        uint32_t late = 0;
#pragma unroll
        for (uint32_t q = 0; q < P; ++q) {
          const bool ready = Pr::ready(got[q], f);
          late |= (__builtin_amdgcn_ballot_w64(!ready) != 0 ? 1u : 0u) << q;
        }
        pend = late & want;
        if (pend == 0 || dead) break;
        if ((++spins & 15) == 0 && budget.expired()) {
          budget.report((int)r, pend, a.epoch);
          dead = true;
          break;
        }
      }
      u32x4 res = mine;
      if constexpr (Mode == RING_BCAST) {
#pragma unroll
        for (uint32_t q = 0; q < P; ++q)
          if (q == a.root && q != r) res = Pr::unpack(got[q], sub);
      } else {
#pragma unroll
        for (int q = 0; q < P; ++q) got[q] = Pr::unpack(got[q], sub);
        res = reduce_ordered<Pr, DT, P>(got, mine, (int)r);
      }
      store_out((g + (s - 1) * G) * TB, res);
    }
  }
  // Completion: the wave's stores into the peers' outputs are acknowledged at
  // the device's coherence point, then one flag goes to every peer that
  // received some; a rank is done when wave g of every peer has said so.
  if constexpr (Mode != RING_RS) {
    wait_vm_all();
    compiler_fence();
    const bool peer = lane < P && lane != r;
    if (peer && publish && (Mode != RING_REDUCE || lane == a.root)) {
      uint32_t *f = (uint32_t *)(a.sym + (uint64_t)lane * a.stride + a.flags +
                                 ((uint64_t)(r - (r > lane ? 1u : 0u)) * G + g) * 64 + 60);
      __hip_atomic_store(f, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t *f =
        (const uint32_t *)(slice_r + a.flags + ((uint64_t)(lane - (lane > r ? 1u : 0u)) * G + g) * 64 + 60);
    bool pend = peer && (Mode != RING_REDUCE || r == a.root);
    uint32_t spins = 0;
    while (true) {
      if (pend && __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch) pend = false;
      const uint64_t still = __builtin_amdgcn_ballot_w64(pend);
      if (still == 0 || dead) break;
      if ((++spins & 15) == 0 && budget.expired()) {
        if (lane == 0) budget.report((int)r, (uint32_t)still, a.epoch);
        break;
      }
    }
  }
  if (a.stamps != nullptr) {
    __syncthreads();
    if (threadIdx.x == 0) {
      a.stamps[blockIdx.x] = t_start;
      a.stamps[a.grid + blockIdx.x] = now_ticks();
    }
  }
}

}  // namespace llc

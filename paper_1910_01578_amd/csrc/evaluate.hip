// Simulated run time of sampled placements: in-order list scheduling of each
// graph on D devices with transfer costs, and the per-device memory check that
// makes a placement invalid (Section 4.1's run time and invalid placements;
// Section 2's placement "with and without simulation").
//
// Every device runs its ops one at a time in node-id order.  For op v placed
// on device p:  ready = max over predecessors u of finish(u) + [p_u != p] *
// out_xfer[u];  start = max(ready, free[p]);  finish(v) = start + op_cost[v];
// free[p] = finish(v).  A graph's run time is its largest finish time.
//
// The recurrence is a longest path: finish(v) = cost(v) + max over the edges
// into v, where "the op before v on its device" is one more edge.  Windows of
// 64 nodes are solved one after another, lane = node, one work-group per
// (graph, sample): the lanes of a window repeat
//   finish(v) = max(finish(v), finish(u) + weight(u -> v))
// over the edges inside the window until no lane changes.  The graph is
// acyclic, so the fixed point is the schedule, exact in integers.  Plain edges
// need as many repeats as the longest chain has edges (up to 64); edges that
// skip 2 to 16 ops along a device's chain and 2 to 8 along each op's latest
// predecessor, formed by pointer doubling, cut that to about 5 - 11.
//
// Four waves share the work: while wave 0 solves window w, wave 1 forms window
// w + 2's edge lists, wave 3 its device chains and wave 2 the arrival times at
// window w + 1 from nodes before window w.  Finish times of the last R nodes stay in
// LDS; older ones of graphs longer than R nodes are read back from a global
// copy.  What bounds it is wave 0's chain of LDS
// round trips: about 280 cycles a repeat and 7 - 10 repeats plus 900 cycles a
// window.  52,000 ops, 64 samples: 1.12 ms a call (op by op on one wave: 30.4 ms);
// 2,500 ops, 16 samples: 77 us (933 us).  Edges beyond the four slots of a node are
// read from memory again in each round over them; 20,000 ops, 64 samples, op by op
// before: 3 predecessors each 0.61 ms (14.1), 8 1.9 ms (33.6), 99 21.7 ms (400).
//
// Times below 2^26 units (they share a word with the device or a lane number),
// saturating; a graph with a finish time of 2^26 or more gets the result -1.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "host_plan.h"
#include "kernels.h"

namespace gdp {

namespace {

constexpr int kWin = 64;                        // nodes per window, one per lane
constexpr unsigned kTimeLimit = 1u << 26;
constexpr int kSlots = 4;                       // edges per node and kind held as lane pointers
constexpr unsigned kNone = 0xffu;               // an unused slot
// A chain of this many latest predecessors inside a window makes its skip edges
// worth their permutes: layered graphs stay below it (their repeats do not fall
// with the skips), operator chains are far above (48 -> 11 repeats at 2,500 ops).
constexpr int kDeep = 10;
constexpr int kDeepBit = 64;

static_assert(kWin == kEvalWindow, "evaluator window");

// What the two preparation-free arrays hold for every sample alike:
//   node header  {cost, out_xfer, internal slots, near slots}: four bytes each,
//                the lane of a predecessor in the node's own window (slot 0 the
//                latest) and in the window before it
//   window       {first record, old records, first extra record, extra records << 7 | deep << 6 | slots in use}
//   records of a window's in-edges: the old ones (predecessors before the
//                previous window) from the front, the extra ones (beyond the
//                slots) from the back; {u relative to the graph | big << 31,
//                min(out_xfer[u], 2^26 - 1) << 6 | lane of v}
__device__ __forceinline__ int2 make_record(int u_rel, int x, int lane_v) {
  const bool big = x >= (int)kTimeLimit;
  return make_int2(u_rel | (big ? (int)0x80000000u : 0),
                   (int)(((big ? kTimeLimit - 1u : (unsigned)x) << 6) | (unsigned)lane_v));
}

__global__ __launch_bounds__(256) void k_window_lists(const int* __restrict__ in_ptr, const int* __restrict__ in_idx,
                                                      const int* __restrict__ op_cost,
                                                      const int* __restrict__ out_xfer, GraphTable wt,
                                                      int4* __restrict__ hdr, int4* __restrict__ win,
                                                      int2* __restrict__ rec) {
  __shared__ int ptr[kWin + 1], best[kWin], cin[kWin], cnear[kWin];
  __shared__ unsigned char slot_in[kWin][kSlots], slot_near[kWin][kSlots];
  __shared__ int n_old, n_extra, m_in, m_near, deep;
  const int w = blockIdx.x, t = threadIdx.x;
  const int g = graph_of_block(wt, w);
  const int g0 = wt.ptr[g], v0 = g0 + (w - wt.blk[g]) * kWin;
  const int cnt = min(kWin, wt.ptr[g + 1] - v0);
  if (t <= kWin) ptr[t] = in_ptr[v0 + min(t, cnt)];
  if (t < kWin) {
    best[t] = cin[t] = cnear[t] = 0;
    for (int q = 0; q < kSlots; ++q) slot_in[t][q] = slot_near[t][q] = (unsigned char)kNone;
  }
  if (t == 0) n_old = n_extra = m_in = m_near = deep = 0;
  __syncthreads();
  const int rb = ptr[0], re = ptr[cnt];
  auto lane_of = [&](int e) {                   // largest lane with ptr[lane] <= e
    int lo = 0, hi = cnt - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (ptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  for (int e = rb + t; e < re; e += 256) {
    const int u = in_idx[e], lv = lane_of(e);
    if (u >= v0 && u < v0 + lv) atomicMax(&best[lv], u - v0 + 1);
  }
  __syncthreads();
  for (int e = rb + t; e < re; e += 256) {
    const int u = in_idx[e], lv = lane_of(e);
    if (u < g0 || u >= v0 + lv) continue;       // not a predecessor in this graph (invalid input)
    bool extra = false;
    if (u >= v0) {
      const int s = u - v0 + 1 == best[lv] ? 0 : 1 + atomicAdd(&cin[lv], 1);
      if (s < kSlots) slot_in[lv][s] = (unsigned char)(u - v0);
      else extra = true;
    } else if (u >= v0 - kWin) {
      const int s = atomicAdd(&cnear[lv], 1);
      if (s < kSlots) slot_near[lv][s] = (unsigned char)(u - v0 + kWin);
      else extra = true;
    }
    const int2 r = make_record(u - g0, out_xfer[u], lv);
    if (extra) rec[re - 1 - atomicAdd(&n_extra, 1)] = r;
    else if (u < v0 - kWin) rec[rb + atomicAdd(&n_old, 1)] = r;
  }
  __syncthreads();
  if (t < cnt) {
    atomicMax(&m_in, best[t] > 0 ? min(1 + cin[t], kSlots) : 0);
    atomicMax(&m_near, min(cnear[t], kSlots));
    auto bytes = [](const unsigned char* b) { return (int)(b[0] | b[1] << 8 | b[2] << 16 | (unsigned)b[3] << 24); };
    int u = t, steps = 0;                       // steps back along the latest predecessors
    while (steps < kDeep && best[u] > 0) {
      u = best[u] - 1;
      ++steps;
    }
    if (steps == kDeep) deep = 1;
    hdr[v0 + t] = make_int4(op_cost[v0 + t], out_xfer[v0 + t], bytes(slot_in[t]), bytes(slot_near[t]));
  }
  __syncthreads();
  if (t == 0) win[w] = make_int4(rb, n_old, re - n_extra, n_extra << 7 | (deep ? kDeepBit : 0) | m_near << 3 | m_in);
}

struct EvalArgs {
  const int* placements;   // [K, N]
  const int* op_mem;       // [N]
  const int4* hdr;         // [N]
  const int4* win;         // [windows]
  const int2* rec;         // [E]
  unsigned* far;           // [K, far_stride] finish times and devices of every node
  size_t far_stride;
  int n, D, K, dev_bits;
  double time_unit;
  int64_t* makespan;       // [G, K]
  unsigned char* valid;    // [G, K]
  float* run_time;         // [G, K] or null
};

struct CapTable {
  long long cap[GDP_MAX_GRAPHS];
};

// A finish time and the device it ran on share one word: time << 6 | device.
__device__ __forceinline__ unsigned pack(unsigned t, unsigned low) { return (t << 6) | low; }
// A global load that waits for itself: a node older than the ring.  Written as
// inline assembly so that the compiler cannot merge it with the ring's LDS read
// into one generic (flat) load.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ unsigned load_wait(const unsigned* p) {
  unsigned w;
  asm volatile("global_load_dword %0, %1, off\n\ts_waitcnt vmcnt(0)" : "=v"(w) : "v"(p) : "memory");
  return w;
}
#pragma clang diagnostic pop
// The value of v in lane sel (0 .. 63).
__device__ __forceinline__ unsigned lane_at(unsigned v, unsigned sel) {
  return (unsigned)__builtin_amdgcn_ds_bpermute((int)(sel << 2), (int)v);
}

// One window's edge lists per lane; an edge is weight << 6 | lane of its source
// (weights include the cost of the node itself, but for the near edges).  An
// absent edge is the lane itself with weight 0.
struct Lists {
  uint4 in;                // edges from the node's own window
  uint4 near;              // edges from the window before (~0: none)
  uint4 chain;             // 1, 2, 4 and 8 ops back on the node's device
  uint4 skip;              // 2, 4 and 8 steps back along the latest predecessors; cost << 6 | device
  unsigned chain16;        // 16 ops back on the device
  uint4 w;                 // the same in every lane: slots in use, first and last extra record, 0
  uint2 last;              // the same in every lane: the lanes that are the last of their device
};
struct WinBuf {
  uint4 in[kWin], near[kWin], chain[kWin], skip[kWin];
  unsigned chain16[kWin];
  uint4 w;
  uint2 last;
};

constexpr int kMemSpread = 8;    // copies of the per-device memory sums (fewer lanes on one address)

template <int R>
__global__ __launch_bounds__(256) void k_list_schedule(EvalArgs a, GraphTable wt, CapTable caps) {
  __shared__ unsigned ring[R];                  // packed (finish, device) of the last R nodes
  __shared__ __attribute__((aligned(16))) WinBuf buf[2];
  __shared__ unsigned ready[2][kWin];           // latest arrivals from old nodes
  __shared__ unsigned flds[kWin];               // finish times during the repeats
  __shared__ unsigned fbuf[2 * kWin];           // finish times of this window and the one before (extra records)
  __shared__ unsigned arr[kWin];
  __shared__ unsigned dev_free[GDP_MAX_DEVICES];
  __shared__ unsigned long long mem[GDP_MAX_DEVICES][kMemSpread];
  __shared__ int side_wrapped;
  const int lane = threadIdx.x & 63;
  // wave 0 solves, wave 1 forms edges and their skips, wave 2 old nodes' arrivals and
  // the memory sums, wave 3 the device chains
  const int role = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = blockIdx.x / a.K, k = blockIdx.x % a.K;
  const int g0 = wt.ptr[g], ng = wt.ptr[g + 1] - g0;
  const int w0 = wt.blk[g], nw = wt.blk[g + 1] - w0;
  const int* prow = a.placements + (size_t)k * a.n + g0;
  const int4* hrow = a.hdr + g0;
  const int* mrow = a.op_mem + g0;
  unsigned* far = a.far + (size_t)k * a.far_stride + g0;
  const bool use_far = ng > R;                  // nodes older than the ring are read back
  if (threadIdx.x < GDP_MAX_DEVICES) dev_free[threadIdx.x] = 0u;
  for (int i = threadIdx.x; i < GDP_MAX_DEVICES * kMemSpread; i += 256) (&mem[0][0])[i] = 0ull;
  if (threadIdx.x == 0) side_wrapped = 0;
  bool wrapped = false;
  auto device_of = [&](int p) { return p >= 0 && p < a.D ? (unsigned)p : 0u; };
  // the window's own 64 nodes: placement or any per-node word, loaded a window ahead
  auto place_of = [&](int w) { return w * kWin + lane < ng ? prow[w * kWin + lane] : -1; };
  // (a vector load: a scalar one would share the counter that LDS results are waited on with)
  int vzero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
  auto win_of = [&](int w) { return w < nw ? a.win[w0 + w + vzero] : make_int4(0, 0, 0, 0); };

  // Both of a window's edge waves: what a successor needs of a node (out_xfer and
  // device in one word), and the edge word of source word `src` in lane l.
  auto own_of = [&](int4 h, unsigned p) { return pack(min((unsigned)h.y, kTimeLimit - 1u), p); };
  auto moves = [&](unsigned src, unsigned l, unsigned p) { return l != kNone && (src & 63u) != p; };

  // ---- wave 1: window w's own edges into buf[w & 1] ----------------------------
  int4 l_hdr = make_int4(0, 0, -1, -1), l_win = make_int4(0, 0, 0, 0);
  int l_p = -1;
  auto load_lists = [&](int w) {
    l_hdr = w * kWin + lane < ng ? hrow[w * kWin + lane] : make_int4(0, 0, -1, -1);
    l_p = place_of(w);
    l_win = win_of(w);
  };
  auto form_lists = [&](int w) {
    const int4 h = l_hdr, wn = l_win;          // wn: the same in every lane
    const unsigned p = device_of(l_p);
    load_lists(w + 1);
    WinBuf& B = buf[w & 1];
    const bool live = w * kWin + lane < ng;
    const unsigned cost = min((unsigned)h.x, kTimeLimit - 1u);
    wrapped |= live && (unsigned)h.x >= kTimeLimit;
    const unsigned own = own_of(h, p);
    unsigned in[kSlots], src[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) src[q] = lane_at(own, ((unsigned)h.z >> (8 * q)) & 63u);
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      const unsigned l = ((unsigned)h.z >> (8 * q)) & 0xffu;
      const unsigned wgt = (moves(src[q], l, p) ? src[q] >> 6 : 0u) + cost;
      wrapped |= l != kNone && wgt >= kTimeLimit;
      in[q] = l == kNone ? (unsigned)lane : pack(min(wgt, kTimeLimit - 1u), l);
    }
    const uint64_t bigs = __ballot((unsigned)h.y >= kTimeLimit);
    if (bigs != 0ull) {                        // transfers of 2^26 and more
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const unsigned l = ((unsigned)h.z >> (8 * q)) & 0xffu;
        wrapped |= moves(src[q], l, p) && ((bigs >> (l & 63u)) & 1ull);
      }
    }
    // skips of 2, 4 and 8 along the latest predecessors, where the window uses them
    unsigned sk[3] = {0u, 0u, 0u};
    if (__builtin_amdgcn_readfirstlane(wn.w) & kDeepBit) {
      unsigned sp = in[0] & 63u, ss = in[0] >> 6;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const unsigned s2 = lane_at(ss, sp), sp2 = lane_at(sp, sp);
        ss += s2;
        sp = sp2;
        wrapped |= ss >= kTimeLimit;
        ss = min(ss, kTimeLimit - 1u);
        sk[i] = pack(ss, sp);
      }
    }
    B.in[lane] = make_uint4(in[0], in[1], in[2], in[3]);
    B.skip[lane] = make_uint4(sk[0], sk[1], sk[2], pack(cost, p));
    if (lane == 0) B.w = make_uint4((unsigned)wn.w & 127u, (unsigned)wn.z, (unsigned)(wn.z + (wn.w >> 7)), 0u);
  };

  // ---- wave 3: window w's device chains and edges from window w - 1 -------------
  int4 c_hdr = make_int4(0, 0, -1, -1);
  int c_p = -1;
  unsigned prev_own = 0u;
  uint64_t prev_bigs = 0ull;
  auto load_chains = [&](int w) {
    c_hdr = w * kWin + lane < ng ? hrow[w * kWin + lane] : make_int4(0, 0, -1, -1);
    c_p = place_of(w);
  };
  auto form_chains = [&](int w) {
    const int4 h = c_hdr;
    const unsigned p = device_of(c_p), cost = min((unsigned)h.x, kTimeLimit - 1u);
    load_chains(w + 1);
    WinBuf& B = buf[w & 1];
    const bool live = w * kWin + lane < ng;
    unsigned nr[kSlots], src[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) src[q] = lane_at(prev_own, ((unsigned)h.w >> (8 * q)) & 63u);
    uint64_t same = __ballot(live);             // lanes on the same device
    for (int b = 0; b < a.dev_bits; ++b) {
      const bool bit = (p >> b) & 1u;
      const uint64_t m = __ballot(bit);
      same &= bit ? m : ~m;
    }
    const uint64_t below = same & ((1ull << lane) - 1ull);
    const uint64_t last = __ballot(live && (same >> lane) == 1ull);
    const bool chained = live && below;
    unsigned cp = chained ? 63u - (unsigned)__builtin_clzll(below) : (unsigned)lane;
    unsigned cs = chained ? cost : 0u;
    unsigned ch[5];
    ch[0] = pack(cs, cp);
#pragma unroll
    for (int i = 1; i < 5; ++i) {               // 2, 4, 8 and 16 ops back
      const unsigned c2 = lane_at(cs, cp), cp2 = lane_at(cp, cp);
      cs += c2;
      cp = cp2;
      wrapped |= cs >= kTimeLimit;
      cs = min(cs, kTimeLimit - 1u);
      ch[i] = pack(cs, cp);
    }
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      const unsigned l = ((unsigned)h.w >> (8 * q)) & 0xffu;
      const bool moved = moves(src[q], l, p);
      nr[q] = l == kNone ? ~0u : pack(moved ? src[q] >> 6 : 0u, l);
      if (prev_bigs != 0ull) wrapped |= moved && ((prev_bigs >> (l & 63u)) & 1ull);
    }
    B.near[lane] = make_uint4(nr[0], nr[1], nr[2], nr[3]);
    B.chain[lane] = make_uint4(ch[0], ch[1], ch[2], ch[3]);
    B.chain16[lane] = ch[4];
    if (lane == 0) B.last = make_uint2((unsigned)last, (unsigned)(last >> 32));
    prev_own = own_of(h, p);
    prev_bigs = __ballot((unsigned)h.y >= kTimeLimit);
  };

  // ---- wave 2: arrivals at window w from the nodes before window w - 1 --------
  constexpr int kAhead = 3;                     // record chunks of 64 loaded a window ahead
  int2 o_rec[kAhead];
  int4 o_win = make_int4(0, 0, 0, 0), o_next = make_int4(0, 0, 0, 0);
  int o_p = -1, o_m = 0;
  auto load_old = [&](int w) {                  // window w's placements, sums and records, window w + 1's extent
    o_p = place_of(w);
    o_m = w * kWin + lane < ng ? mrow[w * kWin + lane] : 0;
    o_win = o_next;
    o_next = win_of(w + 1);
#pragma unroll
    for (int c = 0; c < kAhead; ++c) {
      o_rec[c] = make_int2(0, 0);
      if (c * kWave + lane < o_win.y) o_rec[c] = a.rec[o_win.x + c * kWave + lane];
    }
  };
  auto old_arrivals = [&](int w) {
    int2 rc[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) rc[c] = o_rec[c];
    const int pr = o_p, m = o_m;
    const unsigned p = device_of(pr);
    const int base = __builtin_amdgcn_readfirstlane(o_win.x), n_old = __builtin_amdgcn_readfirstlane(o_win.y);
    load_old(w + 1);
    unsigned* rdy = ready[w & 1];
    const int v0 = w * kWin;
    rdy[lane] = 0u;
    unsigned pv[kAhead], word[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) {
      pv[c] = lane_at(p, (unsigned)rc[c].y & 63u);
      word[c] = ring[rc[c].x & (R - 1)];
    }
    // the solver is writing window w - 1 into the ring; nodes R and more behind v0 are in memory
    auto arrive = [&](int2 r, bool ok, unsigned dv, unsigned wd) {
      const int u = r.x & 0x7fffffff;
      if (use_far && ok && u < v0 - R) wd = load_wait(&far[u]);
      const bool moved = ok && (wd & 63u) != dv;
      wrapped |= moved && r.x < 0;
      if (ok) atomicMax(&rdy[(unsigned)r.y & 63u], (wd >> 6) + (moved ? (unsigned)r.y >> 6 : 0u));
    };
#pragma unroll
    for (int c = 0; c < kAhead; ++c)
      if (c * kWave < n_old) arrive(rc[c], c * kWave + lane < n_old, pv[c], word[c]);
    for (int e0 = kAhead * kWave; e0 < n_old; e0 += kWave) {
      int2 r = make_int2(0, 0);
      if (e0 + lane < n_old) r = a.rec[base + e0 + lane];
      arrive(r, e0 + lane < n_old, lane_at(p, (unsigned)r.y & 63u), ring[r.x & (R - 1)]);
    }
    if (pr >= 0 && pr < a.D) atomicAdd(&mem[p][lane & (kMemSpread - 1)], (unsigned long long)(uint32_t)m);
  };

  // ---- wave 0: the fixed point of window w -------------------------------------
  unsigned mk = 0u, fprev = 0u;
  Lists now, next;
  auto read_lists = [&](int w) {
    const WinBuf& B = buf[w & 1];
    next.w = B.w;
    next.last = B.last;
    next.in = B.in[lane];
    next.near = B.near[lane];
    next.chain = B.chain[lane];
    next.skip = B.skip[lane];
    next.chain16 = B.chain16[lane];
  };
  auto solve_window = [&](int w) {
    const uint4 in = now.in, nr = now.near, ch = now.chain, sk = now.skip;
    const unsigned cost = sk.w >> 6, p = sk.w & 63u;
    const unsigned c16 = now.chain16;
    const int slots = __builtin_amdgcn_readfirstlane((int)now.w.x);
    const int x0 = __builtin_amdgcn_readfirstlane((int)now.w.y), x1 = __builtin_amdgcn_readfirstlane((int)now.w.z);
    const int n_in = slots & 7, n_near = (slots >> 3) & 7;
    const bool deep = (slots & kDeepBit) != 0;
    const uint64_t last = (uint64_t)now.last.y << 32 | now.last.x;
    const int v0 = w * kWin;
    const bool live = v0 + lane < ng;
    // flds still holds the previous window's finish times
    const unsigned t0 = flds[nr.x & 63u], t1 = flds[nr.y & 63u];
    unsigned r = max(ready[w & 1][lane], dev_free[p]);
    r = max(r, max(nr.x == ~0u ? 0u : t0 + (nr.x >> 6), nr.y == ~0u ? 0u : t1 + (nr.y >> 6)));
    if (n_near > 2) {
      const unsigned t2 = flds[nr.z & 63u], t3 = flds[nr.w & 63u];
      r = max(r, max(nr.z == ~0u ? 0u : t2 + (nr.z >> 6), nr.w == ~0u ? 0u : t3 + (nr.w >> 6)));
    }
    // the next window's lists arrive during this one's repeats
    if (w + 1 < nw) read_lists(w + 1);
    unsigned f = live ? min(r + cost, kTimeLimit) : 0u;
    // Repeats: every lane's edges read in one round, from a copy of f in LDS (a
    // permute per edge: 322 cycles a repeat at 11 edges against 290).  At most
    // 63 edges of less than 2^26 each on top of 2^26: no wrap-around before
    // the clamp that follows.
    auto repeat = [&](auto edges, auto skips) {
      constexpr int NE = decltype(edges)::value;      // slots in use
      constexpr bool SK = decltype(skips)::value;
      bool again = true;
      while (again) {
        flds[lane] = f;
        __builtin_amdgcn_wave_barrier();
        const unsigned h0 = flds[ch.x & 63u], h1 = flds[ch.y & 63u], h2 = flds[ch.z & 63u], h3 = flds[ch.w & 63u],
                       h4 = flds[c16 & 63u];
        unsigned e[kSlots], k[3];
        e[0] = flds[in.x & 63u];
        if constexpr (SK) {
          k[0] = flds[sk.x & 63u];
          k[1] = flds[sk.y & 63u];
          k[2] = flds[sk.z & 63u];
        }
        if constexpr (NE > 1) e[1] = flds[in.y & 63u];
        if constexpr (NE > 2) {
          e[2] = flds[in.z & 63u];
          e[3] = flds[in.w & 63u];
        }
        unsigned best = max(max(h0 + (ch.x >> 6), h1 + (ch.y >> 6)), max(h2 + (ch.z >> 6), h3 + (ch.w >> 6)));
        best = max(best, max(h4 + (c16 >> 6), e[0] + (in.x >> 6)));
        if constexpr (SK) best = max(best, max(k[0] + (sk.x >> 6), max(k[1] + (sk.y >> 6), k[2] + (sk.z >> 6))));
        if constexpr (NE > 1) best = max(best, e[1] + (in.y >> 6));
        if constexpr (NE > 2) best = max(best, max(e[2] + (in.z >> 6), e[3] + (in.w >> 6)));
        again = __any(best > f);
        f = max(f, best);
        __builtin_amdgcn_wave_barrier();
      }
      f = min(f, kTimeLimit);
    };
    auto relax = [&]() {
      using std::bool_constant;
      using std::integral_constant;
      if (deep) {
        if (n_in == 1) repeat(integral_constant<int, 1>(), bool_constant<true>());
        else repeat(integral_constant<int, kSlots>(), bool_constant<true>());
      } else {
        if (n_in <= 1) repeat(integral_constant<int, 1>(), bool_constant<false>());
        else if (n_in == 2) repeat(integral_constant<int, 2>(), bool_constant<false>());
        else repeat(integral_constant<int, kSlots>(), bool_constant<false>());
      }
    };
    relax();
    while (x1 > x0) {
      // edges beyond the slots: by records, through LDS
      const unsigned old = f;
      fbuf[lane] = fprev;
      fbuf[kWin + lane] = f;
      arr[lane] = 0u;
      __builtin_amdgcn_wave_barrier();
      for (int e = x0 + lane; e < x1; e += kWave) {
        const int2 q = a.rec[e];
        const int u = q.x & 0x7fffffff;
        const unsigned lv = (unsigned)q.y & 63u;
        const bool moved = device_of(prow[u]) != device_of(prow[v0 + (int)lv]);
        wrapped |= moved && q.x < 0;
        atomicMax(&arr[lv], fbuf[u - v0 + kWin] + (moved ? (unsigned)q.y >> 6 : 0u));
      }
      __builtin_amdgcn_wave_barrier();
      if (live) f = max(f, min(arr[lane] + cost, kTimeLimit));
      if (!__any(f != old)) break;
      relax();
    }
    wrapped |= f >= kTimeLimit;               // (then flds, not clamped, no longer matters)
    mk = max(mk, f);
    if ((last >> lane) & 1ull) dev_free[p] = f;
    const unsigned word = pack(f & (kTimeLimit - 1u), p);
    if (live) ring[(v0 + lane) & (R - 1)] = word;
    if (use_far) {
      // at most one store in flight: the previous window's is complete, so
      // that a read-back of nodes R and more behind finds them written
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (live) far[v0 + lane] = word;
    }
    fprev = f;
    now = next;
  };

  if (threadIdx.x < kWin) flds[threadIdx.x] = 0u;
  if (role == 1) load_lists(0);
  if (role == 3) load_chains(0);
  if (role == 2) {
    o_next = win_of(0);
    load_old(0);
  }
  __syncthreads();                              // the tables above are cleared
  if (role == 1) {
    form_lists(0);
    if (nw > 1) form_lists(1);
  } else if (role == 3) {
    form_chains(0);
    if (nw > 1) form_chains(1);
  } else if (role == 2) {
    old_arrivals(0);
  }
  __syncthreads();
  if (role == 0) {
    read_lists(0);
    now = next;
  }
  __syncthreads();                              // buf[0] is free for window 2
  for (int w = 0; w < nw; ++w) {
    if (role == 0) solve_window(w);
    else if (role == 1 && w + 2 < nw) form_lists(w + 2);
    else if (role == 2 && w + 1 < nw) old_arrivals(w + 1);
    else if (role == 3 && w + 2 < nw) form_chains(w + 2);
    __syncthreads();
  }
  if (role != 0 && __any(wrapped) && lane == 0) side_wrapped = 1;
  __syncthreads();
  if (role != 0) return;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mk = max(mk, (unsigned)__shfl_xor((int)mk, o, kWave));
  const bool over = __any(wrapped) || side_wrapped != 0;
  unsigned long long held = 0ull;
  if (lane < a.D)
    for (int i = 0; i < kMemSpread; ++i) held += mem[lane][i];
  const bool ok = __all(held <= (unsigned long long)caps.cap[g]);
  if (lane != 0) return;
  const size_t o = (size_t)g * a.K + k;
  const int64_t m = over ? (int64_t)-1 : (int64_t)mk;
  a.makespan[o] = m;
  a.valid[o] = ok ? 1 : 0;
  if (a.run_time) a.run_time[o] = (float)((double)m * a.time_unit);
}

}  // namespace

// Work-groups per CU follow from the ring in LDS (R words, kBesideRing bytes
// beside it): the longest ring with which every (graph, sample) still runs at once
// (256, 512 and 768 of them), a shorter one (more read-backs) as they multiply, and
// never longer than the longest graph needs.  What counts is that they run at once.
// 52,000 ops, rings of 32,768 / 16,384 / 8,192 / 4,096, us: 256 samples 1,174 / 1,130 /
// 1,131 / 1,111, 512 samples 2,285 / 1,205 / 1,191 / 1,171, 1,024 samples 4,521 / 2,339 /
// 2,247 / 1,348.  Between the lengths that do, read-backs decide: 40,000 ops of which each
// reads three up to 12,000 back, 512 samples: 1,641 / 891 / 932 / 992 us.
constexpr int kBesideRing = 15 * 1024, kLds = 160 * 1024, kCus = 256;
int eval_ring(const int32_t* graph_ptr, int G, int K) {
  int most = 0;
  for (int g = 0; g < G; ++g) most = std::max(most, graph_ptr[g + 1] - graph_ptr[g]);
  const int64_t groups = (int64_t)G * K;
  int r = 32768;
  while (r > kEvalMinRing && (r / 2 >= most || groups > (int64_t)kCus * (kLds / (4 * r + kBesideRing)))) r /= 2;
  return r;
}

hipError_t launch_evaluate(const EvalLaunch& L, hipStream_t s) {
  hipLaunchKernelGGL(k_window_lists, dim3(L.blocks), dim3(256), 0, s, L.in_ptr, L.in_idx, L.op_cost, L.out_xfer,
                     *L.table, reinterpret_cast<int4*>(L.hdr), reinterpret_cast<int4*>(L.win),
                     reinterpret_cast<int2*>(L.rec));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  EvalArgs a;
  a.placements = L.placements;
  a.op_mem = L.op_mem;
  a.hdr = reinterpret_cast<const int4*>(L.hdr);
  a.win = reinterpret_cast<const int4*>(L.win);
  a.rec = reinterpret_cast<const int2*>(L.rec);
  a.far = L.far;
  a.far_stride = L.far_stride;
  a.n = L.n;
  a.D = L.D;
  a.K = L.K;
  a.dev_bits = 0;
  while ((1 << a.dev_bits) < L.D) ++a.dev_bits;
  a.time_unit = L.time_unit;
  a.makespan = L.makespan;
  a.valid = L.valid;
  a.run_time = L.run_time;
  const GraphTable& wt = *L.table;
  CapTable caps;
  for (int i = 0; i < GDP_MAX_GRAPHS; ++i) caps.cap[i] = i < wt.n ? L.mem_cap[i] : 0;
  const dim3 grid((unsigned)wt.n * (unsigned)L.K), block(256);
  switch (eval_ring(wt.ptr, wt.n, L.K)) {
    case 32768: hipLaunchKernelGGL((k_list_schedule<32768>), grid, block, 0, s, a, wt, caps); break;
    case 16384: hipLaunchKernelGGL((k_list_schedule<16384>), grid, block, 0, s, a, wt, caps); break;
    case 8192: hipLaunchKernelGGL((k_list_schedule<8192>), grid, block, 0, s, a, wt, caps); break;
    default: hipLaunchKernelGGL((k_list_schedule<kEvalMinRing>), grid, block, 0, s, a, wt, caps); break;
  }
  return hipGetLastError();
}

}  // namespace gdp

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
// skip 2, 4 and 8 ops along a device's chain and along each op's latest
// predecessor, formed by pointer doubling, cut that to about 5 - 11.
//
// Two waves share the work: wave 1 forms window w + 1's edge lists (static
// ones from the records below, the skips, and the arrival times from nodes
// finished before window w) while wave 0 solves window w.  Finish times of the
// last R nodes stay in LDS; older ones of graphs longer than R nodes are read
// back from a global copy.  What bounds it is wave 0's chain of LDS lane
// permutes.  One sample at 52,000 nodes on 8 devices takes what 64 take, as
// every sample has its own compute unit.
//
// Times below 2^26 units (they share a word with the device or a lane number),
// saturating; a graph with a finish time of 2^26 or more gets the result -1.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace gdp {

namespace {

constexpr int kWin = 64;                        // nodes per window, one per lane
constexpr unsigned kTimeLimit = 1u << 26;
constexpr int kSlots = 4;                       // edges per node and kind held as lane pointers
constexpr unsigned kNone = 0xffu;               // an unused slot

static_assert(kWin == kEvalWindow, "evaluator window");

// What the two preparation-free arrays hold for every sample alike:
//   node header  {cost, out_xfer, internal slots, near slots}: four bytes each,
//                the lane of a predecessor in the node's own window (slot 0 the
//                latest) and in the window before it
//   window       {first record, old records, first extra record, extra records << 6 | slots in use}
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
  __shared__ int n_old, n_extra, m_in, m_near;
  const int w = blockIdx.x, t = threadIdx.x;
  const int g = graph_of_block(wt, w);
  const int g0 = wt.ptr[g], v0 = g0 + (w - wt.blk[g]) * kWin;
  const int cnt = min(kWin, wt.ptr[g + 1] - v0);
  if (t <= kWin) ptr[t] = in_ptr[v0 + min(t, cnt)];
  if (t < kWin) {
    best[t] = cin[t] = cnear[t] = 0;
    for (int q = 0; q < kSlots; ++q) slot_in[t][q] = slot_near[t][q] = (unsigned char)kNone;
  }
  if (t == 0) n_old = n_extra = m_in = m_near = 0;
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
    hdr[v0 + t] = make_int4(op_cost[v0 + t], out_xfer[v0 + t], bytes(slot_in[t]), bytes(slot_near[t]));
  }
  __syncthreads();
  if (t == 0) win[w] = make_int4(rb, n_old, re - n_extra, n_extra << 6 | m_near << 3 | m_in);
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

// What wave 1 hands wave 0 for one window, per lane; an edge is weight << 6 |
// lane of its source (weights include the cost of the node itself, but for the
// near edges).  An absent edge is the lane itself with weight 0.
struct WinBuf {
  uint4 in[kWin];          // edges from the node's own window
  uint4 near[kWin];        // edges from the window before (~0: none)
  uint4 chain[kWin];       // 1, 2, 4 and 8 ops back on the node's device
  uint4 skip[kWin];        // 2, 4 and 8 steps back along the latest predecessors; cost << 6 | device
  unsigned ready[kWin];    // latest arrival from older nodes
  unsigned last_lo, last_hi;   // lanes that are the last of their device
  int slots, extra0, extra1;   // slots in use; the extra records
};

constexpr int kMemSpread = 8;    // copies of the per-device memory sums (fewer lanes on one address)

template <int R>
__global__ __launch_bounds__(128) void k_list_schedule(EvalArgs a, GraphTable wt, CapTable caps) {
  __shared__ unsigned ring[R];                  // packed (finish, device) of the last R nodes
  __shared__ __attribute__((aligned(16))) WinBuf buf[2];
  __shared__ unsigned fbuf[2 * kWin];           // finish times of this window and the one before (extra records)
  __shared__ unsigned arr[kWin];
  __shared__ unsigned dev_free[GDP_MAX_DEVICES];
  __shared__ unsigned long long mem[GDP_MAX_DEVICES][kMemSpread];
  __shared__ int side_wrapped;
  const int lane = threadIdx.x & 63;
  const bool solver = threadIdx.x < kWave;      // wave 0 solves, wave 1 prepares
  const int g = blockIdx.x / a.K, k = blockIdx.x % a.K;
  const int g0 = wt.ptr[g], ng = wt.ptr[g + 1] - g0;
  const int w0 = wt.blk[g], nw = wt.blk[g + 1] - w0;
  const int* prow = a.placements + (size_t)k * a.n + g0;
  const int4* hrow = a.hdr + g0;
  const int* mrow = a.op_mem + g0;
  unsigned* far = a.far + (size_t)k * a.far_stride + g0;
  const bool use_far = ng > R;                  // nodes older than the ring are read back
  if (threadIdx.x < GDP_MAX_DEVICES) dev_free[threadIdx.x] = 0u;
  for (int i = threadIdx.x; i < GDP_MAX_DEVICES * kMemSpread; i += 128) (&mem[0][0])[i] = 0ull;
  if (threadIdx.x == 0) side_wrapped = 0;
  bool wrapped = false;

  // wave 1: inputs of the window being prepared (nxt) and of the one before it
  struct Side {
    int4 h;
    unsigned p;        // device (0 where the placement is out of range)
    bool counted;      // a real node on a device in range
    int m;
  };
  auto load_side = [&](int w) {
    Side s = {make_int4(0, 0, -1, -1), 0u, false, 0};
    const int v = w * kWin + lane;
    if (w < nw && v < ng) {
      s.h = hrow[v];
      const int p = prow[v];
      s.counted = p >= 0 && p < a.D;
      s.p = s.counted ? (unsigned)p : 0u;
      s.m = mrow[v];
    }
    return s;
  };
  constexpr int kAhead = 3;                     // record chunks of 64 loaded a window ahead
  int2 rq[kAhead];
  int4 wq = make_int4(0, 0, 0, 0);
  Side cur, nxt;
  unsigned prev_p = 0u, prev_x = 0u;
  auto load_win = [&](int w) {
    wq = w < nw ? a.win[w0 + w] : make_int4(0, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < kAhead; ++c)
      if (c * kWave + lane < wq.y) rq[c] = a.rec[wq.x + c * kWave + lane];
  };

  // wave 1: window w's lists into buf[w & 1]; every node before window w - 1 is final
  auto prepare = [&](int w) {
    WinBuf& B = buf[w & 1];
    cur = nxt;
    const int4 wn = make_int4(__builtin_amdgcn_readfirstlane(wq.x), __builtin_amdgcn_readfirstlane(wq.y),
                              __builtin_amdgcn_readfirstlane(wq.z), __builtin_amdgcn_readfirstlane(wq.w));
    int2 rc[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) rc[c] = rq[c];
    nxt = load_side(w + 1);
    load_win(w + 1);
    const int v0 = w * kWin;
    const bool live = v0 + lane < ng;
    const unsigned p = cur.p;
    unsigned cost = (unsigned)cur.h.x, xfer = (unsigned)cur.h.y;
    if (cost >= kTimeLimit) { wrapped |= live; cost = kTimeLimit - 1u; }
    // device chain: the previous and the following lanes on the same device
    uint64_t same = __ballot(live);
    for (int b = 0; b < a.dev_bits; ++b) {
      const bool bit = (p >> b) & 1u;
      const uint64_t m = __ballot(bit);
      same &= bit ? m : ~m;
    }
    const uint64_t below = same & ((1ull << lane) - 1ull);
    const uint64_t last = __ballot(live && (same >> lane) == 1ull);
    unsigned ptr = live && below ? 63u - (unsigned)__builtin_clzll(below) : (unsigned)lane;
    unsigned sum = live && below ? cost : 0u;
    unsigned ch[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i > 0) {
        const unsigned s2 = lane_at(sum, ptr);
        ptr = lane_at(ptr, ptr);
        sum += s2;
        if (sum >= kTimeLimit) { wrapped = true; sum = kTimeLimit - 1u; }
      }
      ch[i] = pack(sum, ptr);
    }
    // edges from this window and from the one before
    unsigned in[kSlots], nr[kSlots];
    const int n_in = wn.w & 7, n_near = (wn.w >> 3) & 7;
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
      in[q] = (unsigned)lane;
      nr[q] = ~0u;
      if (q < n_in) {
        const unsigned l = ((unsigned)cur.h.z >> (8 * q)) & 0xffu;
        const unsigned pu = lane_at(p, l & 63u), xu = lane_at(xfer, l & 63u);
        if (l != kNone) {
          unsigned wgt = pu != p ? xu : 0u;
          if (wgt >= kTimeLimit) wgt = kTimeLimit;
          wgt += cost;
          if (wgt >= kTimeLimit) { wrapped = true; wgt = kTimeLimit - 1u; }
          in[q] = pack(wgt, l);
        }
      }
      if (q < n_near) {
        const unsigned l = ((unsigned)cur.h.w >> (8 * q)) & 0xffu;
        const unsigned pu = lane_at(prev_p, l & 63u), xu = lane_at(prev_x, l & 63u);
        if (l != kNone) {
          unsigned wgt = pu != p ? xu : 0u;
          if (wgt >= kTimeLimit) { wrapped = true; wgt = kTimeLimit - 1u; }
          nr[q] = pack(wgt, l);
        }
      }
    }
    // skips along the latest predecessors
    unsigned sk[3];
    ptr = in[0] & 63u;
    sum = in[0] >> 6;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (n_in > 0) {
        const unsigned s2 = lane_at(sum, ptr);
        ptr = lane_at(ptr, ptr);
        sum += s2;
        if (sum >= kTimeLimit) { wrapped = true; sum = kTimeLimit - 1u; }
      }
      sk[i] = pack(sum, ptr);
    }
    B.in[lane] = make_uint4(in[0], in[1], in[2], in[3]);
    B.near[lane] = make_uint4(nr[0], nr[1], nr[2], nr[3]);
    B.chain[lane] = make_uint4(ch[0], ch[1], ch[2], ch[3]);
    B.skip[lane] = make_uint4(sk[0], sk[1], sk[2], pack(cost, p));
    B.ready[lane] = 0u;
    if (lane == 0) {
      B.last_lo = (unsigned)last;
      B.last_hi = (unsigned)(last >> 32);
      B.slots = wn.w & 63;
      B.extra0 = wn.z;
      B.extra1 = wn.z + (wn.w >> 6);
    }
    // arrivals from old nodes
    for (int c = 0; c * kWave < wn.y; ++c) {
      const int e = c * kWave + lane;
      const bool ok = e < wn.y;
      int2 r = make_int2(0, 0);
      if (c < kAhead) {
        r = c == 0 ? rc[0] : c == 1 ? rc[1] : rc[2];
      } else if (ok) {
        r = a.rec[wn.x + e];
      }
      const int u = r.x & 0x7fffffff;
      const unsigned lv = (unsigned)r.y & 63u, x = (unsigned)r.y >> 6;
      const unsigned pv = lane_at(p, lv);
      if (ok) {
        // the solver is writing window w - 1 into the ring
        unsigned word;
        if (u >= v0 - R) word = ring[u & (R - 1)];
        else word = load_wait(&far[u]);
        const bool moved = (word & 63u) != pv;
        if (moved && r.x < 0) wrapped = true;
        atomicMax(&B.ready[lv], (word >> 6) + (moved ? x : 0u));
      }
    }
    if (cur.counted) atomicAdd(&mem[p][lane & (kMemSpread - 1)], (unsigned long long)(uint32_t)cur.m);
    prev_p = p;
    prev_x = xfer;
  };

  if (!solver) {
    nxt = load_side(0);
    load_win(0);
  }
  __syncthreads();                              // the tables above are cleared
  if (!solver) prepare(0);
  unsigned mk = 0u, fprev = 0u;
  __syncthreads();
  for (int w = 0; w < nw; ++w) {
    if (!solver) {
      if (w + 1 < nw) prepare(w + 1);
    } else {
      const WinBuf& B = buf[w & 1];
      const uint4 in = B.in[lane], ch = B.chain[lane], sk = B.skip[lane];
      const unsigned cost = sk.w >> 6, p = sk.w & 63u;
      const int slots = __builtin_amdgcn_readfirstlane(B.slots);
      const int n_in = slots & 7, n_near = slots >> 3;
      const int x0 = __builtin_amdgcn_readfirstlane(B.extra0), x1 = __builtin_amdgcn_readfirstlane(B.extra1);
      const int v0 = w * kWin;
      const bool live = v0 + lane < ng;
      unsigned r = max(B.ready[lane], dev_free[p]);
      if (n_near > 0) {
        const uint4 nr = B.near[lane];
        const unsigned t0 = lane_at(fprev, nr.x & 63u), t1 = lane_at(fprev, nr.y & 63u);
        r = max(r, nr.x == ~0u ? 0u : t0 + (nr.x >> 6));
        r = max(r, nr.y == ~0u ? 0u : t1 + (nr.y >> 6));
        if (n_near > 2) {
          const unsigned t2 = lane_at(fprev, nr.z & 63u), t3 = lane_at(fprev, nr.w & 63u);
          r = max(r, nr.z == ~0u ? 0u : t2 + (nr.z >> 6));
          r = max(r, nr.w == ~0u ? 0u : t3 + (nr.w >> 6));
        }
      }
      unsigned f = live ? min(r + cost, kTimeLimit) : 0u;
      if (x1 > x0) fbuf[lane] = fprev;
      // the fixed point
      const unsigned a0 = in.x & 63u, a1 = in.y & 63u, a2 = in.z & 63u, a3 = in.w & 63u;
      const unsigned c0 = ch.x & 63u, c1 = ch.y & 63u, c2 = ch.z & 63u, c3 = ch.w & 63u;
      const unsigned s0 = sk.x & 63u, s1 = sk.y & 63u, s2 = sk.z & 63u;
      bool again = true;
      while (again) {
        const unsigned old = f;
        const unsigned h0 = lane_at(f, c0), h1 = lane_at(f, c1), h2 = lane_at(f, c2), h3 = lane_at(f, c3);
        unsigned best = max(max(h0 + (ch.x >> 6), h1 + (ch.y >> 6)), max(h2 + (ch.z >> 6), h3 + (ch.w >> 6)));
        if (n_in > 0) {
          const unsigned e0 = lane_at(old, a0), k0 = lane_at(old, s0), k1 = lane_at(old, s1), k2 = lane_at(old, s2);
          best = max(best, max(max(e0 + (in.x >> 6), k0 + (sk.x >> 6)), max(k1 + (sk.y >> 6), k2 + (sk.z >> 6))));
          if (n_in > 1) {
            const unsigned e1 = lane_at(old, a1), e2 = lane_at(old, a2), e3 = lane_at(old, a3);
            best = max(best, max(e1 + (in.y >> 6), max(e2 + (in.z >> 6), e3 + (in.w >> 6))));
          }
        }
        f = min(max(f, best), kTimeLimit);
        if (x1 > x0) {
          // edges beyond the slots: by records, through LDS
          fbuf[kWin + lane] = f;
          arr[lane] = 0u;
          __builtin_amdgcn_wave_barrier();
          for (int e = x0 + lane; e < x1; e += kWave) {
            const int2 q = a.rec[e];
            const int u = q.x & 0x7fffffff;
            const unsigned lv = (unsigned)q.y & 63u;
            const int pu = prow[u], pv = prow[v0 + (int)lv];
            const unsigned du = pu >= 0 && pu < a.D ? (unsigned)pu : 0u, dv = pv >= 0 && pv < a.D ? (unsigned)pv : 0u;
            if (du != dv && q.x < 0) wrapped = true;
            atomicMax(&arr[lv], fbuf[u - v0 + kWin] + (du != dv ? (unsigned)q.y >> 6 : 0u));
          }
          __builtin_amdgcn_wave_barrier();
          const unsigned t = arr[lane];
          if (t != 0u) f = max(f, min(t + cost, kTimeLimit));
        }
        again = __any(f != old);
      }
      wrapped |= f >= kTimeLimit;
      mk = max(mk, f);
      const uint64_t last = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(B.last_hi) << 32 |
                            (unsigned)__builtin_amdgcn_readfirstlane(B.last_lo);
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
    }
    __syncthreads();
  }
  if (!solver && __any(wrapped) && lane == 0) side_wrapped = 1;
  __syncthreads();
  if (!solver) return;
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

// Work-groups per CU follow from the ring in LDS (R words, 14 KB beside it):
// the longest ring while every (graph, sample) still has a CU of its own, a
// shorter one (more read-backs, several work-groups per CU) as they multiply,
// and never longer than the longest graph needs.
int eval_ring(const int32_t* graph_ptr, int G, int K) {
  int most = 0;
  for (int g = 0; g < G; ++g) most = std::max(most, graph_ptr[g + 1] - graph_ptr[g]);
  const int64_t groups = (int64_t)G * K;
  int r = groups <= 256 ? 32768 : groups <= 512 ? 16384 : groups <= 1024 ? 8192 : 4096;
  while (r > 4096 && r / 2 >= most) r /= 2;
  return r;
}

hipError_t launch_evaluate(const EvalLaunch& L, hipStream_t s) {
  hipLaunchKernelGGL(k_window_lists, dim3(L.windows), dim3(256), 0, s, L.in_ptr, L.in_idx, L.op_cost, L.out_xfer,
                     *L.window_table, reinterpret_cast<int4*>(L.hdr), reinterpret_cast<int4*>(L.win),
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
  const GraphTable& wt = *L.window_table;
  CapTable caps;
  for (int i = 0; i < GDP_MAX_GRAPHS; ++i) caps.cap[i] = i < wt.n ? L.mem_cap[i] : 0;
  const dim3 grid((unsigned)wt.n * (unsigned)L.K), block(128);
  switch (eval_ring(wt.ptr, wt.n, L.K)) {
    case 32768: hipLaunchKernelGGL((k_list_schedule<32768>), grid, block, 0, s, a, wt, caps); break;
    case 16384: hipLaunchKernelGGL((k_list_schedule<16384>), grid, block, 0, s, a, wt, caps); break;
    case 8192: hipLaunchKernelGGL((k_list_schedule<8192>), grid, block, 0, s, a, wt, caps); break;
    default: hipLaunchKernelGGL((k_list_schedule<4096>), grid, block, 0, s, a, wt, caps); break;
  }
  return hipGetLastError();
}

}  // namespace gdp

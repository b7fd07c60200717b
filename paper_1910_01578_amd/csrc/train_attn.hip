// Segment attention of the update step, forward and backward, in fp32 accuracy
// on the bf16 matrix cores.  Band form: the queries of a segment [seg0, seg1) of
// graph g attend to keys [max(g_start, seg0 - mem_len), seg1).  qkv: [n, 3d]
// (Q | K | V, heads contiguous).
//
// Every fp32 operand, the probabilities and their gradients included, is the
// exact sum of three bf16 values; a product of two operands is formed from the
// six pairs of weight 2^-16 and above (the rest is up to 2^-24 of it), as the
// update step's dense products are.
//
// A work-group is 4 waves and one head; it owns 64 COLS queries (forward, dQ)
// or keys (dK, dV) of one segment, 16 COLS a wave, one per lane column.  The
// other side passes through LDS in tiles of 64 rows, split into planes on the
// way; while one tile is worked on, the next is split into a second buffer and
// the one after is loaded.  Scores are formed transposed (S^T = K Q^T, or S =
// Q K^T for the key side), so that a lane's accumulator holds 4 tile rows of its
// own column, rows 4 (lane / 16) + r of each block of 16.  The next product
// contracts over those rows with its k slots ordered {16 b + 4 g + i, then 16
// (b + 1) + 4 g + i}, so that a lane's own values are its B operand; the A
// operand is the transposed tile, read by ds_read_b64_tr_b16 from the row-major
// planes.  Scores are kept in log2 units (the register operand is pre-multiplied
// by log2(e) / sqrt(d_h)).
//
// What bounds it: the vector ALU (exponentials, splits) and the matrix
// instructions together.  52,000 rows, 8 heads of 32, segments and memory of 512
// (16x16x4 fp32 instructions before): forward 597 -> 315 us, dQ 853 -> 409 us,
// dK and dV 1,554 -> 657 us.
//
// The gradients of W_q and W_k are small differences of large sums (a row's ds
// add up to zero), so what the forward divides by and sums has to agree with what
// the backward forms: the denominators are summed as trees, O and dQ add each 32
// rows in one rounding, the log-sum-exp stays in log2 units.  Error of these two
// gradients against float64 with the forward's own ReLU signs, d_h = 32, 6,000
// nodes: 2.0e-4 without these, 9.7e-5 with them (fp32 instructions: 1.3e-4).
//
// For the same reason the backward keeps a1 b1 on a sum of its own (dO . v, dQ, dK,
// dV): an instruction drops the low bits of what is small beside its sum towards
// minus infinity, dO . v then leans against Dq in every row alike, and the rows'
// sums keep that.  Same error at 52,000 nodes, last layer: 6.5e-5 with all pairs on
// one sum, 5.6e-6 so (fp32 instructions: 6.1e-6); backward of 6 layers 15.1 -> 15.6
// ms.  The forward's scores and their copies in the backward lean alike for all
// keys of a query, which the softmax cancels.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "host_plan.h"
#include "train_kernels.h"
#include "train_planes.h"

namespace gdp {
namespace tr {

namespace {

constexpr int kAttnTile = 64;    // rows staged per tile
constexpr float kLog2e = 1.4426950408889634f;

// The segment rows [r0, r1) of work block b (segments split into blocks of
// `rows` rows; gt.blk the per-graph prefix of blocks).
struct SegRows {
  int gs, ge, seg0, seg1, r0, r1;
};
__device__ __forceinline__ SegRows seg_rows(const GraphTable& gt, int b, int seg, int rows) {
  const int g = graph_of_block(gt, b);
  const int per = (seg + rows - 1) / rows;
  const int local = b - gt.blk[g];
  SegRows s;
  s.gs = gt.ptr[g];
  s.ge = gt.ptr[g + 1];
  s.seg0 = s.gs + (local / per) * seg;
  s.seg1 = min(s.seg0 + seg, s.ge);
  s.r0 = s.seg0 + (local % per) * rows;
  s.r1 = min(s.r0 + rows, s.seg1);
  return s;
}

// 2^x by the hardware instruction (results below 2^-126 are 0).
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// c += the five plane pairs of a b below a1 b1, smallest first.
__device__ __forceinline__ f32x4 mma_low(const Planes& a, const Planes& b, f32x4 c) {
  c = mma(a.p[2], b.p[0], c);
  c = mma(a.p[1], b.p[1], c);
  c = mma(a.p[0], b.p[2], c);
  c = mma(a.p[1], b.p[0], c);
  return mma(a.p[0], b.p[1], c);
}
__device__ __forceinline__ f32x4 mma_top(const Planes& a, const Planes& b, f32x4 c) { return mma(a.p[0], b.p[0], c); }
__device__ __forceinline__ f32x4 add4(f32x4 a, f32x4 b) {
#pragma unroll
  for (int r = 0; r < 4; ++r) a[r] += b[r];
  return a;
}

// ds_read_b64_tr_b16: within each group of 16 lanes, destination lane 4q + p
// receives in slot e element p of the 8-byte word addressed by source lane
// 4e + q.
__device__ __forceinline__ uint2 read_tr16(const char* p) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
  const bf16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
      (__attribute__((address_space(3))) bf16x4_t*)((__attribute__((address_space(3))) char*)p));
  return __builtin_bit_cast(uint2, v);
}

// A 64-row tile of one head's columns as three bf16 planes in LDS.
template <int DH>
struct Tile {
  static constexpr int G = DH / 8;                          // 16-byte granules per row
  static constexpr int kPlane = kAttnTile * DH * 2;
  static constexpr int kBytes = 3 * kPlane;
  static constexpr int U = kAttnTile * G > 256 ? kAttnTile * G / 256 : 1;
  // Byte offset of granule g of a row: eight consecutive rows of a fragment read
  // fall in distinct granules modulo 128 bytes.
  static __device__ __forceinline__ int at(int row, int g) {
    if constexpr (DH == 16) return row * 32 + ((g ^ ((row >> 2) & 1)) << 4);
    else if constexpr (DH == 32) return row * 64 + ((g ^ (((row >> 2) ^ (row >> 1)) & 3)) << 4);
    else return row * 128 + ((g ^ (row & 7)) << 4);
  }
  float v[U][8];
  static __device__ __forceinline__ int unit(int u) { return ((int)threadIdx.x + 256 * u) % (kAttnTile * G); }
  // rows [t0, t0 + 64) of src's columns [c0, c0 + DH); rows at or past t1 copy row t1 - 1
  __device__ __forceinline__ void load(const float* src, int ld, int c0, int t0, int t1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(unit(u) / G, t1 - 1 - t0);
      const float* p = src + (size_t)t0 * ld + c0 + (unsigned)(r * ld + unit(u) % G * 8);
      const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
      v[u][0] = a.x; v[u][1] = a.y; v[u][2] = a.z; v[u][3] = a.w;
      v[u][4] = b.x; v[u][5] = b.y; v[u][6] = b.z; v[u][7] = b.w;
    }
  }
  __device__ __forceinline__ void store(char* s) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Planes p = split8(v[u]);
      const int o = at(unit(u) / G, unit(u) % G);
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8*>(s + q * kPlane + o) = p.p[q];
    }
  }
  static __device__ __forceinline__ bf16x8 granule(const char* s, int plane, int row, int g) {
    return *reinterpret_cast<const bf16x8*>(s + plane * kPlane + at(row, g));
  }
};

// A lane's operand for products over the head dimension: its own row's DH
// values, 8 per lane group and k step.  With DH = 16 one instruction covers two
// plane pairs: lane groups 0, 1 hold one plane's 16 values, groups 2, 3 another's;
// the two largest products have an instruction each (twice one half), as smaller
// ones beside them would lose their last bits (gradients of W_q and W_k 1.6e-4 ->
// 7e-5, 4,000 nodes; a fourth instruction, 2.5 % of that update).
template <int DH>
struct RowOperand {
  static constexpr int NK = DH == 64 ? 2 : 1;
  Planes k[NK];
  __device__ __forceinline__ void load(const float* src, size_t ld, int v, bool ok, int c0, int g4, float mul) {
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      float t[8];
      const float* p = src + (size_t)(ok ? v : 0) * ld + c0 + (DH == 16 ? (g4 & 1) * 8 : s * 32 + g4 * 8);
#pragma unroll
      for (int i = 0; i < 8; i += 4) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok) a = *reinterpret_cast<const float4*>(p + i);
        t[i] = a.x * mul; t[i + 1] = a.y * mul; t[i + 2] = a.z * mul; t[i + 3] = a.w * mul;
      }
      k[s] = split8(t);
    }
    if constexpr (DH == 16) {      // B planes of the pairs (a3 b1 | a1 b3), (a2 b2 | a1 b2) and (a b1/2 | a b1/2)
      const Planes o = k[0];
      k[0].p[0] = g4 >= 2 ? o.p[2] : o.p[0];
#pragma unroll
      for (int i = 0; i < 8; ++i) k[0].p[2][i] = (bf16)((float)o.p[0][i] * 0.5f);
    }
  }
};

// acc[c] = tile rows [row0, row0 + 16) . the columns' rows, over the head dimension.
// APART: a1 b1 on a sum of its own.
template <bool APART, int DH, int COLS>
__device__ __forceinline__ void dot_rows(f32x4 (&acc)[COLS], const char* tile, int row0, const RowOperand<DH> (&y)[COLS],
                                         int col, int g4) {
  using T = Tile<DH>;
  f32x4 low[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) acc[c] = low[c] = zero4();
  if constexpr (DH == 16) {
    const bool up = g4 >= 2;
    const bf16x8 a31 = T::granule(tile, up ? 0 : 2, row0 + col, g4 & 1), a21 = T::granule(tile, up ? 0 : 1, row0 + col, g4 & 1),
                 a2 = T::granule(tile, 1, row0 + col, g4 & 1), a1 = T::granule(tile, 0, row0 + col, g4 & 1);
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      low[c] = mma(a31, y[c].k[0].p[0], low[c]);
      low[c] = mma(a21, y[c].k[0].p[1], low[c]);
      low[c] = mma(a2, y[c].k[0].p[2], low[c]);
      acc[c] = mma(a1, y[c].k[0].p[2], APART ? acc[c] : low[c]);
    }
  } else {
#pragma unroll
    for (int s = 0; s < RowOperand<DH>::NK; ++s) {
      Planes a;
#pragma unroll
      for (int q = 0; q < 3; ++q) a.p[q] = T::granule(tile, q, row0 + col, s * 4 + g4);
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        if constexpr (APART) {
          low[c] = mma_low(a, y[c].k[s], low[c]);
          acc[c] = mma_top(a, y[c].k[s], acc[c]);
        } else {
          acc[c] = mma_top(a, y[c].k[s], mma_low(a, y[c].k[s], acc[c]));
        }
      }
    }
  }
  if constexpr (APART) {
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[c] = add4(acc[c], low[c]);
  }
}

// tile^T . w over the tile's rows [row0, row0 + 32), to add(db, c, a, w[c]) for
// every 16 head dims from 16 db and every column; w[c]: the lane's values of rows
// row0 + 4 g4 + i and row0 + 16 + 4 g4 + i.
template <int DH, int COLS, typename Add>
__device__ __forceinline__ void acc_rows(const char* tile, int row0, const Planes (&w)[COLS], int col, int g4, Add add) {
  using T = Tile<DH>;
#pragma unroll
  for (int db = 0; db < DH / 16; ++db) {
    Planes a;
    const int r = row0 + 4 * g4 + (col >> 2), dim = 16 * db + 4 * (col & 3);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint2 lo = read_tr16(tile + q * T::kPlane + T::at(r, dim / 8) + (dim % 8) * 2);
      const uint2 hi = read_tr16(tile + q * T::kPlane + T::at(r + 16, dim / 8) + (dim % 8) * 2);
      a.p[q] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
#pragma unroll
    for (int c = 0; c < COLS; ++c) add(db, c, a, w[c]);
  }
}

template <int DH>
constexpr int buffers() { return DH == 64 ? 1 : 2; }

// Two arrays' tiles through LDS: next(i) says where tile i starts and ends,
// work(x, y, i) uses it.  With one buffer (d_h = 64) a tile is written between
// two barriers, with two it is written beside the tile before it.
template <int DH, typename Load, typename Work>
__device__ __forceinline__ void for_tiles(char* lds, int tiles, Load load, Work work) {
  constexpr int NB = buffers<DH>(), kBuf = 2 * Tile<DH>::kBytes;
  Tile<DH> x, y;
  load(x, y, 0);
  if constexpr (NB == 2) {
    x.store(lds);
    y.store(lds + Tile<DH>::kBytes);
    load(x, y, min(1, tiles - 1));
  }
  for (int i = 0; i < tiles; ++i) {
    __syncthreads();
    char* cur = lds + (NB == 2 ? (i & 1) * kBuf : 0);
    if constexpr (NB == 2) {
      char* nxt = lds + ((i + 1) & 1) * kBuf;
      x.store(nxt);
      y.store(nxt + Tile<DH>::kBytes);
      load(x, y, min(i + 2, tiles - 1));
    } else {
      x.store(cur);
      y.store(cur + Tile<DH>::kBytes);
      load(x, y, min(i + 1, tiles - 1));
      __syncthreads();
    }
    work(cur, cur + Tile<DH>::kBytes, i);
  }
}

// What the matrix instructions cannot form because an operand is infinite, or rounds
// to a bf16 infinity, and so has no planes: a result that is not finite is formed
// again, one row after another in fp32.  Once it is NaN it stays so.
template <int DH>
__device__ __forceinline__ float dot_fp32(const float* x, const float* y, float mul) {
  float t = 0.f;
  for (int i = 0; i < DH; ++i) t = fmaf(x[i] * mul, y[i], t);
  return t;
}
// The lane's values 16 db + 4 g4 + r: o += w * row.
template <int DB>
__device__ __forceinline__ void add_row_fp32(f32x4 (&o)[DB], float w, const float* row, int g4) {
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    const float4 v = *reinterpret_cast<const float4*>(row + db * 16 + 4 * g4);
    o[db][0] = fmaf(w, v.x, o[db][0]);
    o[db][1] = fmaf(w, v.y, o[db][1]);
    o[db][2] = fmaf(w, v.z, o[db][2]);
    o[db][3] = fmaf(w, v.w, o[db][3]);
  }
}
template <int DB, int COLS>
__device__ __forceinline__ bool finite_column(const f32x4 (&o)[DB][COLS], int c) {
  float any = 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 4; ++r) any = fmaf(o[db][c][r], 0.f, any);
  return any == any;
}
// Query q's attention over keys [k0, k1): m, the sum of 2^(s - m) and the weighted values.
template <int DH>
__device__ __forceinline__ void attend_fp32(const float* __restrict__ qkv, int ld, int d, int q, int k0, int k1, int c0,
                                            int g4, float mul, float& m, float& sum, f32x4 (&o)[DH / 16]) {
  auto score = [&](int j) { return dot_fp32<DH>(qkv + (size_t)q * ld + c0, qkv + (size_t)j * ld + d + c0, mul); };
  m = -INFINITY;
  sum = 0.f;
#pragma unroll
  for (int db = 0; db < DH / 16; ++db) o[db] = zero4();
  for (int j = k0; j < k1 && sum == sum; ++j) {
    const float s = score(j);
    m = fmaxf(m, s);
    if (s != s) sum = s;
  }
  for (int j = k0; j < k1 && sum == sum; ++j) {
    const float p = exp2f(score(j) - m);
    sum += p;
    add_row_fp32<DH / 16>(o, p, qkv + (size_t)j * ld + 2 * d + c0, g4);
  }
}
// Query q's dQ (less the scale) over keys [k0, k1), from its log-sum-exp L and Dq.
template <int DH>
__device__ __forceinline__ void query_grad_fp32(const float* __restrict__ qkv, const float* __restrict__ dO, int ld, int d,
                                                int q, int k0, int k1, int c0, int g4, float mul, float L, float Dq,
                                                f32x4 (&dq)[DH / 16]) {
#pragma unroll
  for (int db = 0; db < DH / 16; ++db) dq[db] = zero4();
  float w = 0.f;
  for (int j = k0; j < k1 && w == w; ++j) {
    const float* k = qkv + (size_t)j * ld + d + c0;
    const float s = dot_fp32<DH>(qkv + (size_t)q * ld + c0, k, mul), dp = dot_fp32<DH>(dO + (size_t)q * d + c0, k + d, 1.0f);
    w = exp2f(s - L) * (dp - Dq);
    add_row_fp32<DH / 16>(dq, w, k, g4);
  }
}
// A key's dK (less the scale) and dV from the queries of the segments from seg0
// that hold it in their band, up to `end`.
template <int DH>
__device__ __forceinline__ void key_grad_fp32(const float* __restrict__ qkv, const float* __restrict__ dO,
                                              const float* __restrict__ Dq, const float* __restrict__ lse, int ld, int d,
                                              int heads, int head, int key, int seg0, int seg, int mem, int end, int c0,
                                              int g4, float mul, f32x4 (&dk)[DH / 16], f32x4 (&dv)[DH / 16]) {
#pragma unroll
  for (int db = 0; db < DH / 16; ++db) dk[db] = dv[db] = zero4();
  const float* k = qkv + (size_t)key * ld + d + c0;
  float w = 0.f;
  for (int i = seg0; i < end && w == w; ++i) {
    const int sg0 = seg0 + (i - seg0) / seg * seg;
    if (sg0 > seg0 && key < sg0 - mem) break;
    const float *q = qkv + (size_t)i * ld + c0, *g = dO + (size_t)i * d + c0;
    const float p = exp2f(dot_fp32<DH>(k, q, mul) - lse[(size_t)i * heads + head]);
    w = p * (dot_fp32<DH>(g, k + d, 1.0f) - Dq[(size_t)i * heads + head]);
    add_row_fp32<DH / 16>(dv, p, g, g4);
    add_row_fp32<DH / 16>(dk, w, q, g4);
  }
}

template <int DH, int COLS>
__global__ __launch_bounds__(256) void k_attn_fwd(const float* __restrict__ qkv, int d, int heads, int seg, int mem,
                                                  GraphTable gt, float scale, float* __restrict__ o,
                                                  float* __restrict__ lse) {
  constexpr int DB = DH / 16;
  __shared__ __attribute__((aligned(16))) char lds[buffers<DH>() * 2 * Tile<DH>::kBytes];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g4 = lane >> 4;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int head = logical % heads, c0 = head * DH;
  const SegRows b = seg_rows(gt, logical / heads, seg, 64 * COLS);
  const int ld = 3 * d;
  const int k0 = max(b.gs, b.seg0 - mem), k1 = b.seg1;
  RowOperand<DH> qf[COLS];
  f32x4 oacc[DB][COLS];
  float m[COLS], lsum[COLS];
  int q[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    q[c] = b.r0 + (wave * COLS + c) * 16 + col;
    qf[c].load(qkv, ld, q[c], q[c] < b.r1, c0, g4, scale * kLog2e);
    m[c] = -INFINITY;
    lsum[c] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db][c] = zero4();
  }
  for_tiles<DH>(
      lds, (k1 - k0 + kAttnTile - 1) / kAttnTile,
      [&](Tile<DH>& x, Tile<DH>& y, int i) {
        x.load(qkv, ld, d + c0, k0 + i * kAttnTile, k1);
        y.load(qkv, ld, 2 * d + c0, k0 + i * kAttnTile, k1);
      },
      [&](const char* sK, const char* sV, int i) {
        const int t0 = k0 + i * kAttnTile;
        f32x4 s[4][COLS];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) dot_rows<false, DH, COLS>(s[kb], sK, kb * 16, qf, col, g4);
        if (t0 + kAttnTile > k1) {
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int c = 0; c < COLS; ++c)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (t0 + kb * 16 + 4 * g4 + r >= k1) s[kb][c][r] = -INFINITY;
        }
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
          float tmax = -INFINITY;
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) tmax = fmaxf(tmax, s[kb][c][r]);
          tmax = fmaxf(tmax, xor_shfl(tmax, 16));
          tmax = fmaxf(tmax, xor_shfl(tmax, 32));
          const float mn = fmaxf(m[c], tmax);
          const float corr = exp2_fast(m[c] - mn);
          m[c] = mn;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) oacc[db][c][r] *= corr;
          float sum[4];
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s[kb][c][r] = exp2_fast(s[kb][c][r] - mn);
            sum[kb] = (s[kb][c][0] + s[kb][c][1]) + (s[kb][c][2] + s[kb][c][3]);
          }
          lsum[c] = lsum[c] * corr + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          Planes p[COLS];
#pragma unroll
          for (int c = 0; c < COLS; ++c) {
            float t[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              t[r] = s[2 * h][c][r];
              t[4 + r] = s[2 * h + 1][c][r];
            }
            p[c] = split8(t);
          }
          acc_rows<DH, COLS>(sV, 32 * h, p, col, g4, [&](int db, int c, const Planes& a, const Planes& w) {
            oacc[db][c] = add4(oacc[db][c], mma_top(a, w, mma_low(a, w, zero4())));
          });
        }
      });
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    lsum[c] += xor_shfl(lsum[c], 16);
    lsum[c] += xor_shfl(lsum[c], 32);
    if (q[c] >= b.r1) continue;
    if (!(lsum[c] * 0.f == 0.f) || !finite_column(oacc, c)) {
      f32x4 t[DB];
      attend_fp32<DH>(qkv, ld, d, q[c], k0, k1, c0, g4, scale * kLog2e, m[c], lsum[c], t);
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db][c] = t[db];
    }
    const float inv = 1.0f / lsum[c];
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<float4*>(o + (size_t)q[c] * d + c0 + db * 16 + 4 * g4) =
          make_float4(oacc[db][c][0] * inv, oacc[db][c][1] * inv, oacc[db][c][2] * inv, oacc[db][c][3] * inv);
    if (g4 == 0) lse[(size_t)q[c] * heads + head] = m[c] + log2f(lsum[c]);
  }
}

// dQ for the work-group's queries: p = exp(s - lse) (lse in log2 units), ds = p (dO . v - Dq),
// dq = scale * sum_j ds_j k_j (into the Q columns of dqkv, row stride lddq).
template <int DH, int COLS>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_q(const float* __restrict__ qkv, const float* __restrict__ dO,
                                                    const float* __restrict__ Dq, const float* __restrict__ lse,
                                                    int d, int heads, int seg, int mem, GraphTable gt, float scale,
                                                    float* __restrict__ dqkv, int lddq) {
  constexpr int DB = DH / 16;
  __shared__ __attribute__((aligned(16))) char lds[buffers<DH>() * 2 * Tile<DH>::kBytes];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g4 = lane >> 4;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int head = logical % heads, c0 = head * DH;
  const SegRows b = seg_rows(gt, logical / heads, seg, 64 * COLS);
  const int ld = 3 * d;
  const int k0 = max(b.gs, b.seg0 - mem), k1 = b.seg1;
  RowOperand<DH> qf[COLS], df[COLS];
  float L2[COLS], Dv[COLS];
  f32x4 dq[DB][COLS];
  int q[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    q[c] = b.r0 + (wave * COLS + c) * 16 + col;
    const bool ok = q[c] < b.r1;
    qf[c].load(qkv, ld, q[c], ok, c0, g4, scale * kLog2e);
    df[c].load(dO, d, q[c], ok, c0, g4, 1.0f);
    L2[c] = ok ? lse[(size_t)q[c] * heads + head] : 0.f;
    Dv[c] = ok ? Dq[(size_t)q[c] * heads + head] : 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) dq[db][c] = zero4();
  }
  for_tiles<DH>(
      lds, (k1 - k0 + kAttnTile - 1) / kAttnTile,
      [&](Tile<DH>& x, Tile<DH>& y, int i) {
        x.load(qkv, ld, d + c0, k0 + i * kAttnTile, k1);
        y.load(qkv, ld, 2 * d + c0, k0 + i * kAttnTile, k1);
      },
      [&](const char* sK, const char* sV, int i) {
        const int left = k1 - (k0 + i * kAttnTile);
        auto tile = [&](auto ragged) {                     // ragged: keys past the segment's end in the tile
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            float t[COLS][8];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int row0 = 32 * h + 16 * e;
              f32x4 s[COLS], dp[COLS];
              dot_rows<false, DH, COLS>(s, sK, row0, qf, col, g4);
              dot_rows<true, DH, COLS>(dp, sV, row0, df, col, g4);
#pragma unroll
              for (int c = 0; c < COLS; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const float w = exp2_fast(s[c][r] - L2[c]) * (dp[c][r] - Dv[c]);
                  t[c][4 * e + r] = !decltype(ragged)::value || row0 + 4 * g4 + r < left ? w : 0.f;
                }
            }
            Planes w[COLS];
#pragma unroll
            for (int c = 0; c < COLS; ++c) w[c] = split8(t[c]);
            acc_rows<DH, COLS>(sK, 32 * h, w, col, g4, [&](int db, int c, const Planes& a, const Planes& x) {
              dq[db][c] = add4(dq[db][c], add4(mma_top(a, x, zero4()), mma_low(a, x, zero4())));
            });
          }
        };
        if (left >= kAttnTile) tile(std::false_type());
        else tile(std::true_type());
      });
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    if (q[c] >= b.r1) continue;
    if (!finite_column(dq, c)) {
      f32x4 t[DB];
      query_grad_fp32<DH>(qkv, dO, ld, d, q[c], k0, k1, c0, g4, scale * kLog2e, L2[c], Dv[c], t);
#pragma unroll
      for (int db = 0; db < DB; ++db) dq[db][c] = t[db];
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<float4*>(dqkv + (size_t)q[c] * lddq + c0 + db * 16 + 4 * g4) =
          make_float4(dq[db][c][0] * scale, dq[db][c][1] * scale, dq[db][c][2] * scale, dq[db][c][3] * scale);
  }
}

// dK, dV for the work-group's keys: first from the queries of their own segment
// (live: the key's row receives that gradient), then also from the later
// segments whose memory holds them (all: that part stops at the projection
// weights, as the memory passes no gradient to its rows).
template <int DH, int COLS>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_kv(const float* __restrict__ qkv, const float* __restrict__ dO,
                                                     const float* __restrict__ Dq, const float* __restrict__ lse,
                                                     int d, int heads, int seg, int mem, GraphTable gt, float scale,
                                                     float* __restrict__ dqkv_live, int ldl,
                                                     float* __restrict__ dkv_all, int lda) {
  constexpr int DB = DH / 16, NB = buffers<DH>();
  __shared__ __attribute__((aligned(16))) char lds[NB * 2 * Tile<DH>::kBytes];
  __shared__ float sL[2][kAttnTile], sDq[2][kAttnTile];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g4 = lane >> 4;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int head = logical % heads, c0 = head * DH;
  const SegRows b = seg_rows(gt, logical / heads, seg, 64 * COLS);
  const int ld = 3 * d;
  RowOperand<DH> kf[COLS], vf[COLS];
  f32x4 dk[DB][COLS], dv[DB][COLS];
  int key[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    key[c] = b.r0 + (wave * COLS + c) * 16 + col;
    const bool ok = key[c] < b.r1;
    kf[c].load(qkv, ld, key[c], ok, d + c0, g4, scale * kLog2e);
    vf[c].load(qkv, ld, key[c], ok, 2 * d + c0, g4, 1.0f);
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[db][c] = dv[db][c] = zero4();
  }
  // the key's own segment, then later segments whose band starts before r1
  const int per = (seg + kAttnTile - 1) / kAttnTile;       // tiles of a whole segment
  int last = b.seg0 + seg;                                 // end of the segments that see these keys
  while (last < b.ge && last - mem < b.r1) last += seg;
  const int own = (b.seg1 - b.seg0 + kAttnTile - 1) / kAttnTile;
  const int end = min(last, b.ge);
  int tiles = own;
  if (end > b.seg0 + seg) {
    const int more = end - (b.seg0 + seg), whole = more / seg, rest = more - whole * seg;
    tiles += whole * per + (rest + kAttnTile - 1) / kAttnTile;
  }
  auto seg_of = [&](int i) { return b.seg0 + (i < own ? 0 : 1 + (i - own) / per) * seg; };
  auto row_of = [&](int i) { return seg_of(i) + (i < own ? i : (i - own) % per) * kAttnTile; };
  auto store_key = [&](const f32x4& k4, const f32x4& v4, int at, int db, float* out, int ldo, int first) {
    float* p = out + (size_t)at * ldo + first + c0 + db * 16 + 4 * g4;
    *reinterpret_cast<float4*>(p) = make_float4(k4[0] * scale, k4[1] * scale, k4[2] * scale, k4[3] * scale);
    *reinterpret_cast<float4*>(p + d) = make_float4(v4[0], v4[1], v4[2], v4[3]);
  };
  auto store = [&](float* out, int ldo, int first) {
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      if (key[c] >= b.r1) continue;
#pragma unroll
      for (int db = 0; db < DB; ++db) store_key(dk[db][c], dv[db][c], key[c], db, out, ldo, first);
    }
  };
  // lse (waves 0, 2) and Dq (waves 1, 3) of a tile's queries, one value per lane
  float aux = 0.f;
  const float* aux_src = (wave & 1) ? Dq : lse;
  auto aux_load = [&](int i) {
    const int sg1 = min(seg_of(i) + seg, b.ge);
    aux = aux_src[(size_t)min(row_of(i) + lane, sg1 - 1) * heads + head];
  };
  auto aux_store = [&](int buf) { ((wave & 1) ? sDq[buf] : sL[buf])[lane] = aux; };
  aux_load(0);
  aux_store(0);
  for_tiles<DH>(
      lds, tiles,
      [&](Tile<DH>& x, Tile<DH>& y, int i) {
        const int t0 = row_of(i), sg1 = min(seg_of(i) + seg, b.ge);
        x.load(qkv, ld, c0, t0, sg1);
        y.load(dO, d, c0, t0, sg1);
      },
      [&](const char* sQ, const char* sD, int i) {
        if (i == own) store(dqkv_live, ldl, d);            // the own segment is complete
        const int t0 = row_of(i), sg0 = seg_of(i), sg1 = min(sg0 + seg, b.ge);
        const float* L = sL[i & 1];
        const float* Dd = sDq[i & 1];
        aux_load(min(i + 1, tiles - 1));
        auto tile = [&](auto masked) {                     // masked: not every (query, key) of the tile is in the band
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            float p[COLS][8], ds[COLS][8];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int row0 = 32 * h + 16 * e;
              f32x4 s[COLS], dp[COLS];
              dot_rows<true, DH, COLS>(s, sQ, row0, kf, col, g4);
              dot_rows<true, DH, COLS>(dp, sD, row0, vf, col, g4);
              const float4 l4 = *reinterpret_cast<const float4*>(L + row0 + 4 * g4);
              const float4 d4 = *reinterpret_cast<const float4*>(Dd + row0 + 4 * g4);
              const float lr[4] = {l4.x, l4.y, l4.z, l4.w}, dr[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
              for (int c = 0; c < COLS; ++c) {
                const bool seen = i < own || key[c] >= sg0 - mem;   // the band of segment sg0 holds the key
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  float w = exp2_fast(s[c][r] - lr[r]);
                  if (decltype(masked)::value && !(seen && t0 + row0 + 4 * g4 + r < sg1)) w = 0.f;
                  p[c][4 * e + r] = w;
                  ds[c][4 * e + r] = w * (dp[c][r] - dr[r]);
                }
              }
            }
            Planes w[COLS];
#pragma unroll
            for (int c = 0; c < COLS; ++c) w[c] = split8(p[c]);
            acc_rows<DH, COLS>(sD, 32 * h, w, col, g4, [&](int db, int c, const Planes& a, const Planes& x) {
              dv[db][c] = add4(mma_top(a, x, dv[db][c]), mma_low(a, x, zero4()));
            });
#pragma unroll
            for (int c = 0; c < COLS; ++c) w[c] = split8(ds[c]);
            acc_rows<DH, COLS>(sQ, 32 * h, w, col, g4, [&](int db, int c, const Planes& a, const Planes& x) {
              dk[db][c] = add4(mma_top(a, x, dk[db][c]), mma_low(a, x, zero4()));
            });
          }
        };
        if (t0 + kAttnTile <= sg1 && (i < own || b.r0 >= sg0 - mem)) tile(std::false_type());
        else tile(std::true_type());
        aux_store((i + 1) & 1);
      });
  if (tiles == own) store(dqkv_live, ldl, d);
  store(dkv_all, lda, 0);
  // (a sum that was not finite after the own segment is not now)
  unsigned again = 0;
#pragma unroll
  for (int c = 0; c < COLS; ++c)
    if (key[c] < b.r1 && !(finite_column(dk, c) && finite_column(dv, c))) again |= 1u << c;
  for (; again; again &= again - 1) {
    const int at = b.r0 + (wave * COLS + __builtin_ctz(again)) * 16 + col;
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {
      f32x4 tk[DB], tv[DB];
      key_grad_fp32<DH>(qkv, dO, Dq, lse, ld, d, heads, head, at, b.seg0, seg, mem, part ? end : b.seg1, c0, g4,
                        scale * kLog2e, tk, tv);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        if (part) store_key(tk[db], tv[db], at, db, dkv_all, lda, 0);
        else store_key(tk[db], tv[db], at, db, dqkv_live, ldl, d);
      }
    }
  }
}

// Dq[v][h] = dO[v] . O[v] over the head's columns, one thread per (v, h).
template <int DH>
__global__ void k_attn_dq_rowdot(const float* __restrict__ dO, const float* __restrict__ O, int n, int d, int heads,
                                 float* __restrict__ Dq) {
  const size_t total = (size_t)n * heads;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const size_t base = (i / heads) * d + (i % heads) * DH;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < DH; t += 4) {
      const float4 a = *reinterpret_cast<const float4*>(dO + base + t);
      const float4 c = *reinterpret_cast<const float4*>(O + base + t);
      s[0] = fmaf(a.x, c.x, s[0]);
      s[1] = fmaf(a.y, c.y, s[1]);
      s[2] = fmaf(a.z, c.z, s[2]);
      s[3] = fmaf(a.w, c.w, s[3]);
    }
    Dq[i] = (s[0] + s[1]) + (s[2] + s[3]);
  }
}

// The attention blocks of every graph: segments in blocks of `rows` rows.
int attn_table(const GraphTable& gt, int seg, int rows, GraphTable* t) {
  *t = gt;
  return prefix_blocks_attention(t->ptr, t->n, seg, rows, t->blk);
}

// Two columns a lane (128 rows a work-group) halve the tile reads per product,
// where segments fill such blocks and d_h = 64 does not run out of registers.
bool two_columns(int dh, int seg) { return dh <= 32 && (seg % 128 == 0 || seg >= 512); }

}  // namespace

hipError_t launch_attn_fwd(const float* qkv, int n, int d, int heads, int seg, int mem, const GraphTable& gt,
                           float* o, float* lse, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int dh = d / heads;
  const float scale = 1.0f / sqrtf((float)dh);
  const bool two = two_columns(dh, seg);
  GraphTable t;
  const int blocks = attn_table(gt, seg, two ? 128 : 64, &t);
  dim3 grid(blocks * heads), block(256);
#define GDP_ATTN_FWD(DH, COLS) \
  hipLaunchKernelGGL((k_attn_fwd<DH, COLS>), grid, block, 0, s, qkv, d, heads, seg, mem, t, scale, o, lse)
  if (dh == 16 && two) GDP_ATTN_FWD(16, 2);
  else if (dh == 16) GDP_ATTN_FWD(16, 1);
  else if (dh == 32 && two) GDP_ATTN_FWD(32, 2);
  else if (dh == 32) GDP_ATTN_FWD(32, 1);
  else if (dh == 64) GDP_ATTN_FWD(64, 1);
  else return hipErrorInvalidValue;
#undef GDP_ATTN_FWD
  return hipGetLastError();
}

hipError_t launch_attn_bwd(const float* qkv, const float* O, const float* dO, const float* lse, int n, int d,
                           int heads, int seg, int mem, const GraphTable& gt, float* Dq, float* dqkv_live,
                           float* dkv_all, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int dh = d / heads;
  const float scale = 1.0f / sqrtf((float)dh);
  const bool two = two_columns(dh, seg);
  GraphTable t;
  const int blocks = attn_table(gt, seg, two ? 128 : 64, &t);
  const unsigned rd_blocks = (unsigned)std::min<size_t>(((size_t)n * heads + 255) / 256, 8192);
  dim3 grid(blocks * heads), block(256);
#define GDP_ATTN_BWD(DH, COLS)                                                                                      \
  do {                                                                                                              \
    hipLaunchKernelGGL((k_attn_dq_rowdot<DH>), dim3(rd_blocks), dim3(256), 0, s, dO, O, n, d, heads, Dq);           \
    hipLaunchKernelGGL((k_attn_bwd_q<DH, COLS>), grid, block, 0, s, qkv, dO, (const float*)Dq, lse, d, heads, seg,  \
                       mem, t, scale, dqkv_live, 3 * d);                                                            \
    hipLaunchKernelGGL((k_attn_bwd_kv<DH, COLS>), grid, block, 0, s, qkv, dO, (const float*)Dq, lse, d, heads, seg, \
                       mem, t, scale, dqkv_live, 3 * d, dkv_all, 2 * d);                                            \
  } while (0)
  if (dh == 16 && two) GDP_ATTN_BWD(16, 2);
  else if (dh == 16) GDP_ATTN_BWD(16, 1);
  else if (dh == 32 && two) GDP_ATTN_BWD(32, 2);
  else if (dh == 32) GDP_ATTN_BWD(32, 1);
  else if (dh == 64) GDP_ATTN_BWD(64, 1);
  else return hipErrorInvalidValue;
#undef GDP_ATTN_BWD
  return hipGetLastError();
}

}  // namespace tr
}  // namespace gdp

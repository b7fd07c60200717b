// The update step's dense products, C(m, n) = epi(sum_k A(m, k) B(k, n)), in
// fp32 accuracy on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values (8 significant bits
// each), a = a1 + a2 + a3 by repeated round-to-nearest, and the product of two
// bf16 values is exact in fp32.  With a bf16 B (the weights of a bf16 policy)
// the three products a1 b + a2 b + a3 b are the whole product; with an fp32 B
// the six products of weight 2^-16 and above are formed (|a2| is up to 2^-8 of |a|
// and |a3| up to 2^-17, so of the three left out a2 b3 and a3 b2 are up to 2^-25 of
// |a b| each, all three 2^-24).  Accumulation is the matrix cores' fp32.  The
// bf16 instructions do 16 times the work of the fp32 ones per cycle, so three
// products cost 3/16 and six 3/8 of the fp32 instructions.
//
// The products below a1 b1 go to sums of their own.  Where an instruction's sum
// and its products differ much in size, the low bits of the smaller are dropped
// towards minus infinity: with all products on one sum a result leans by 1e-8 of
// its root mean square (k = 256, normal operands; apart: 1e-10).  A gradient adds
// up such results over all rows, and the lean with them: at 52,000 rows column
// sums were off by 1.6e-6 (three products) and 3.1e-6 (six), apart 9e-8 (fp32
// instructions 2.8e-7).
//
// A work-group (4 waves, 2 x 2) owns a BM x BM tile of C, each wave a (BM/2)^2
// block.  k advances in steps of KS through two LDS buffers: while a wave's
// matrix instructions work on step s from one, its vector ALU splits step s + 1
// into bf16 planes for the other, and the loads of step s + 3 go out into the
// registers that frees (the memory's latency is two steps).  One barrier a step.
// KS is 32 (16x16x32 instructions) for 64 x 64 tiles and 16 (32x32x16; half the
// LDS, and registers for both sums) for 128 x 128 ones.  Planes are [row][KS k];
// the 16-byte granules of a row are permuted so that eight consecutive rows of a
// fragment read fall in distinct granules modulo 128 bytes.  Products are formed
// transposed, so a lane holds 4 consecutive n of one m.  With splits > 1 each split of k writes its raw sums
// to partial[z]; k_gemm_reduce adds them in split order, in double, and applies
// the epilogue.
//
// What bounds it: the split's vector work, the LDS traffic and the matrix
// instructions of a step are about equal (600 - 800 cycles each), and two
// work-groups a CU overlap them in part.  At 52,000 rows, 16x16x4 fp32
// instructions before and this kernel now: weight gradient (256 x 1024) 332 ->
// 143 us, input gradient (1,024 columns, bf16 weights, ReLU') now 181 us (151
// TFLOP/s); relative error against float64 2.9e-7 -> 8.9e-8 (k = 256), 5.6e-7 ->
// 2.4e-7 (weight gradient).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "host_plan.h"
#include "lds_dma.h"
#include "train_kernels.h"
#include "train_planes.h"

namespace gdp {
namespace tr {

namespace {

template <typename T> constexpr int planes() { return sizeof(T) == 2 ? 1 : 3; }

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + expf(-z)); }

// Byte offset of 16-byte granule g (8 k values) of a tile row.  32-byte rows: any
// 8 and any 16 aligned rows of a granule are distinct modulo 128 and 256 bytes
// (with row bit 2 alone, 8 only: weight gradients 93 against 91.5 us on average).
template <int KS>
__device__ __forceinline__ int tile_at(int row, int g) {
  if constexpr (KS == 32) return row * 64 + ((g ^ (((row >> 2) ^ (row >> 1)) & 3)) << 4);
  else return row * 32 + ((g ^ (((row >> 2) ^ (row >> 3)) & 1)) << 4);
}

// Eight values as 1 or 3 bf16 planes of 16 bytes at byte offset `at`, planes
// `plane` bytes apart.
__device__ __forceinline__ void store_planes(char* s, int at, int plane, const float (&v)[8]) {
  const Planes o = split8(v);
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8*>(s + q * plane + at) = o.p[q];
}
__device__ __forceinline__ void store_planes(char* s, int at, int plane, const bf16 (&v)[8]) {
  (void)plane;
  bf16x8 p;
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = v[i];
  *reinterpret_cast<bf16x8*>(s + at) = p;
}

template <typename T, int N> struct alignas(sizeof(T) * N) Pack { T v[N]; };

// A tile of R rows x KS k in registers: element (r, k) = p[r * sr + k * sk].
// KF: sk == 1, a unit is one row's 8 consecutive k.  Else sr == 1 and a unit is
// 8 k of one row (fp32; a wave's lanes hold consecutive rows) or of two rows
// (bf16).  Loads are unconditional, so that they stay in flight across the
// steps: rows at or past rmax are copies of the last one (their results are not
// stored), k at or past kmax of the last k, which zero_tail() clears.  VEC:
// aligned for vector loads, and with KF every step is whole (host-checked).
template <typename T, int R, int KS, bool KF, bool VEC>
struct Stage {
  static constexpr int G = KS / 8;                          // granules per row
  static constexpr int P = !KF && sizeof(T) == 2 ? 2 : 1;   // rows per unit
  static constexpr int kUnits = R / P * G;                  // fewer than 256: threads share units
  static constexpr int U = (kUnits + 255) / 256;
  T v[U][P][8];
  static __device__ __forceinline__ int unit(int u) {
    return ((int)threadIdx.x + 256 * u) % (kUnits < 256 ? kUnits : 256 * U);
  }
  static __device__ __forceinline__ int row(int u) { return KF ? unit(u) / G : unit(u) % (R / P) * P; }
  static __device__ __forceinline__ int gran(int u) { return KF ? unit(u) % G : unit(u) / (R / P); }
  // base: element (r0, k0), rows and ks the rows and k left from there (at least 1)
  __device__ __forceinline__ void load(const T* base, long sr, long sk, int rows, int ks) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (VEC && KF) {
        const T* q = base + (unsigned)__mul24(min(row(u), rows - 1), (int)sr) + gran(u) * 8;
        constexpr int N = 16 / sizeof(T);
#pragma unroll
        for (int h = 0; h < 8; h += N) {
          const Pack<T, N> t = *reinterpret_cast<const Pack<T, N>*>(q + h);
#pragma unroll
          for (int i = 0; i < N; ++i) v[u][0][h + i] = t.v[i];
        }
      } else if constexpr (VEC) {
        const int r = min(row(u), rows - P);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const Pack<T, P> t =
              *reinterpret_cast<const Pack<T, P>*>(base + (unsigned)(__mul24(min(gran(u) * 8 + i, ks - 1), (int)sk) + r));
#pragma unroll
          for (int h = 0; h < P; ++h) v[u][h][i] = t.v[h];
        }
      } else {
#pragma unroll
        for (int h = 0; h < P; ++h)
#pragma unroll
          for (int i = 0; i < 8; ++i)
            v[u][h][i] = base[(size_t)min(row(u) + h, rows - 1) * sr + (size_t)min(gran(u) * 8 + i, ks - 1) * sk];
      }
    }
  }
  __device__ __forceinline__ void zero_tail(int ks) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < P; ++h)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (gran(u) * 8 + i >= ks) v[u][h][i] = (T)0.f;
  }
  // the unit's 8 values added up (one unit of one row per thread)
  __device__ __forceinline__ float sum8() const {
    static_assert(U == 1 && P == 1, "one row per thread");
    const T(&a)[8] = v[0][0];
    return (((float)a[0] + (float)a[1]) + ((float)a[2] + (float)a[3])) + (((float)a[4] + (float)a[5]) + ((float)a[6] + (float)a[7]));
  }
  __device__ __forceinline__ void store(char* s) const {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < P; ++h) store_planes(s, tile_at<KS>(row(u) + h, gran(u)), R * KS * 2, v[u][h]);
  }
};

// The epilogue as a compile-time set of operations.
enum Epi { E_RAW = 0, E_BIAS = 1, E_RELU = 2, E_SIGMOID = 4, E_MASK = 8, E_RES = 16, E_ACC = 32 };

template <typename TA, typename TB>
int epi_of(const GemmStrided<TA, TB>& g) {
  return (g.bias_f || g.bias_h ? E_BIAS : 0) | (g.act == ACT_RELU ? E_RELU : g.act == ACT_SIGMOID ? E_SIGMOID : 0) |
         (g.mask ? E_MASK : 0) | (g.res ? E_RES : 0) | (g.accumulate ? E_ACC : 0);
}

// What the epilogue reads for N consecutive columns from (m, n).  A kernel reads
// it for all of its results before it stores the first: the stores may alias
// these arrays, so a load behind a store cannot start early, and each of a lane's
// 16 results would take a memory round trip of its own (52,000 rows, both with all
// planes on one sum: ReLU' mask of 1,024 columns 172 -> 157 us, bias and ReLU 143 ->
// 137 us).
template <int EPI, int N>
struct EpiIn {
  float bias[N];
  Pack<float, N> mask, res, old;
  template <typename TA, typename TB>
  __device__ __forceinline__ void load(const GemmStrided<TA, TB>& g, int m, int n) {
    if constexpr ((EPI & E_BIAS) != 0) {
#pragma unroll
      for (int r = 0; r < N; ++r) bias[r] = sizeof(TB) == 2 ? (float)g.bias_h[n + r] : g.bias_f[n + r];
    }
    if constexpr ((EPI & E_MASK) != 0) mask = *reinterpret_cast<const Pack<float, N>*>(g.mask + (size_t)m * g.ldm + n);
    if constexpr ((EPI & E_RES) != 0) res = *reinterpret_cast<const Pack<float, N>*>(g.res + (size_t)m * g.ldr + n);
    if constexpr ((EPI & E_ACC) != 0) old = *reinterpret_cast<const Pack<float, N>*>(g.c + (size_t)m * g.ldc + n);
  }
};

template <int EPI, int N, typename TA, typename TB>
__device__ __forceinline__ void epilogue(const GemmStrided<TA, TB>& g, int m, int n, const EpiIn<EPI, N>& in, float (&v)[N]) {
  Pack<float, N> t;
#pragma unroll
  for (int r = 0; r < N; ++r) {
    if constexpr ((EPI & E_BIAS) != 0) v[r] += in.bias[r];
    if constexpr ((EPI & E_RELU) != 0) v[r] = fmaxf(v[r], 0.f);
    if constexpr ((EPI & E_SIGMOID) != 0) v[r] = sigmoidf_(v[r]);
    if constexpr ((EPI & E_MASK) != 0) v[r] = in.mask.v[r] > 0.f ? v[r] : 0.f;
    if constexpr ((EPI & E_RES) != 0) v[r] += in.res.v[r];
    if constexpr ((EPI & E_ACC) != 0) v[r] += in.old.v[r];
    t.v[r] = v[r];
  }
  *reinterpret_cast<Pack<float, N>*>(g.c + (size_t)m * g.ldc + n) = t;
}
template <int EPI, int N, typename TA, typename TB>
__device__ __forceinline__ void epilogue(const GemmStrided<TA, TB>& g, int m, int n, float (&v)[N]) {
  EpiIn<EPI, N> in;
  in.load(g, m, n);
  epilogue<EPI, N>(g, m, n, in, v);
}

}  // namespace

// sum over [k0, k1) of A(m, k) B(k, n), one product at a time in fp32.
template <typename TA, typename TB>
__device__ __forceinline__ float dot_fp32(const GemmStrided<TA, TB>& g, int m, int n, int k0, int k1) {
  const TA* a = g.a + (size_t)m * g.sam;
  const TB* b = g.b + (size_t)n * g.sbn;
  float t = 0.f;
  for (int k = k0; k < k1 && t == t; k += 8) {             // NaN stays NaN
    float x[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const size_t q = (size_t)min(k + i, k1 - 1);
      x[i] = (float)a[q * g.sak];
      y[i] = (float)b[q * g.sbk];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (k + i < k1) t = fmaf(x[i], y[i], t);
  }
  return t;
}
// The results of a lane's R x C blocks of E that are not finite, formed again by
// dot(i, j, e): where an operand is infinite or rounds to a bf16 infinity (from
// 3.396e38), its planes and those of what it meets give inf - inf or inf * 0.
template <int R, int C, int E, typename Acc, typename Dot>
__device__ __forceinline__ void form_again(Acc (&acc)[R][C], Dot dot) {
  static_assert(R * C * E <= 64, "one bit a result");
  float any = 0.f;                                         // NaN if one is not finite
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int e = 0; e < E; ++e) any = fmaf(acc[i][j][e], 0.f, any);
  if (any == any) return;
  uint64_t todo = 0;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (!isfinite(acc[i][j][e])) todo |= 1ull << ((i * C + j) * E + e);
  while (todo) {
    const int at = __builtin_ctzll(todo);
    todo &= todo - 1;
    const float t = dot(at / E / C, at / E % C, at % E);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (at == (i * C + j) * E + e) acc[i][j][e] = t;
  }
}

// VEC: vector loads and float4 stores are aligned (host-checked).
template <typename TA, typename TB, int BM, bool AKF, bool BKF, bool VEC, int EPI>
__global__ __launch_bounds__(256, 2) void k_gemm_split(GemmStrided<TA, TB> g, int k_per_split, float* partial, int nt,
                                                    int mt) {
  constexpr int KS = BM == 64 ? 32 : 16;
  constexpr int MT = KS == 32 ? 16 : 32;                 // rows and columns of one matrix instruction
  constexpr int WT = BM / 2, NB = WT / MT, PA = planes<TA>(), PB = planes<TB>();
  constexpr int kPlane = BM * KS * 2, kBuf = (PA + PB) * kPlane;
  typedef float acc_t __attribute__((ext_vector_type(MT * MT / 64)));
  __shared__ __attribute__((aligned(16))) char lds[2 * kBuf];
  static_assert(BM <= kVecRows && KS <= kVecRows, "rows indexed by a 24-bit product");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane % MT, gr = lane / MT;
  const int mw = (wave >> 1) * WT, nw = (wave & 1) * WT;
  // consecutive tiles of a row block share its rows of A: keep them on one XCD
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int n0 = (tile % nt) * BM, m0 = (tile / nt % mt) * BM, z = tile / (nt * mt);
  const int kb = z * k_per_split, ke = min(g.K, kb + k_per_split);
  acc_t acc[NB][NB], low[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < MT * MT / 64; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
  Stage<TA, BM, KS, AKF, VEC> la[2];
  Stage<TB, BM, KS, BKF, VEC> lb[2];
  auto load = [&](auto set, int k) {                     // past the end: the last step again
    k = min(k, kb + (ke - kb - 1) / KS * KS);
    la[set].load(g.a + (size_t)m0 * g.sam + (size_t)k * g.sak, g.sam, g.sak, g.M - m0, ke - k);
    lb[set].load(g.b + (size_t)n0 * g.sbn + (size_t)k * g.sbk, g.sbn, g.sbk, g.N - n0, ke - k);
  };
  double rowsum = 0.0;                                   // a weight gradient's bias: the sums of A's rows over k
  auto split = [&](auto set, int buf) {
    if constexpr (!AKF) rowsum += (double)la[set].sum8();
    la[set].store(lds + buf * kBuf);
    lb[set].store(lds + buf * kBuf + PA * kPlane);
  };
  auto step = [&](auto s, int k) {                       // step k from buffer s; step k + KS into the other
    constexpr int S = decltype(s)::value;
    const char* sA = lds + S * kBuf;
    const char* sB = sA + PA * kPlane;
    constexpr std::integral_constant<int, 1 - S> other{};
    if (k + 2 * KS > ke) {                               // the last step, and one more after an odd number
      la[1 - S].zero_tail(ke - k - KS);
      lb[1 - S].zero_tail(ke - k - KS);
    }
    bf16x8 fb[NB][PB], fa[NB][PA];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int p = 0; p < PB; ++p)
        fb[j][p] = *reinterpret_cast<const bf16x8*>(sB + p * kPlane + tile_at<KS>(nw + MT * j + col, gr));
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int p = 0; p < PA; ++p)
        fa[i][p] = *reinterpret_cast<const bf16x8*>(sA + p * kPlane + tile_at<KS>(mw + MT * i + col, gr));
    split(other, 1 - S);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      // smallest products first
#pragma unroll
      for (int w = 2; w >= 0; --w)
#pragma unroll
        for (int pa = w; pa >= 0; --pa) {
          const int pb = w - pa;
          if (pa >= PA || pb >= PB) continue;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            acc_t& c = w > 0 ? low[i][j] : acc[i][j];
            if constexpr (MT == 16) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][pb], fa[i][pa], c, 0, 0, 0);
            else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j][pb], fa[i][pa], c, 0, 0, 0);
          }
        }
    load(other, k + 3 * KS);
    if constexpr (KS == 16) {
      // Fragment reads first, then the split's vector work in the shadow of the
      // matrix instructions (201 -> 184 us for 1024 x 256 over 52,000 rows; the
      // other shape's compiler order is as good).
      __builtin_amdgcn_sched_group_barrier(0x100, NB * (PA + PB), 0);
#pragma unroll
      for (int i = 0; i < NB * NB * (PA * PB == 9 ? 6 : PA * PB); ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
      }
    }
    __syncthreads();
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  load(c0, kb);
  load(c1, kb + KS);
  if (kb + KS > ke) {
    la[0].zero_tail(ke - kb);
    lb[0].zero_tail(ke - kb);
  }
  split(c0, 0);
  load(c0, kb + 2 * KS);
  __syncthreads();
  for (int k = kb; k < ke; k += 2 * KS) {
    step(c0, k);
    step(c1, k + KS);
  }
  if constexpr (!AKF) {
    if (g.rowsum && n0 == 0) {                           // the k granules of a row, in order
      double* red = reinterpret_cast<double*>(lds);
      red[threadIdx.x] = rowsum;
      __syncthreads();
      const int m = m0 + (int)threadIdx.x;
      if (threadIdx.x < BM && m < g.M) {
        double t = 0.0;
        for (int q = 0; q < 256 / BM; ++q) t += red[threadIdx.x + q * BM];
        if (partial) partial[(size_t)gridDim.x / (nt * mt) * g.M * g.N + (size_t)z * g.M + m] = (float)t;
        else g.rowsum[m] = (float)t;
      }
    }
  }
  // lane: row mw + MT i + col of C, groups of 4 columns
  constexpr int NQ = MT * MT / 256;
  auto row_of = [&](int i) { return m0 + mw + MT * i + col; };
  auto col_of = [&](int j, int q) { return n0 + nw + MT * j + (MT == 16 ? 4 * gr : 8 * q + 4 * gr); };
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < MT * MT / 64; ++r) acc[i][j][r] += low[i][j][r];
  if constexpr (PA * PB > 1)
    form_again<NB, NB, MT * MT / 64>(acc, [&](int i, int j, int r) {
      return dot_fp32(g, min(row_of(i), g.M - 1), min(col_of(j, r / 4) + r % 4, g.N - 1), kb, ke);
    });
  EpiIn<EPI, 4> in[VEC ? NB : 1][VEC ? NB : 1][VEC ? NQ : 1];
  if constexpr (VEC && EPI != E_RAW) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) in[i][j][q].load(g, min(row_of(i), g.M - 1), min(col_of(j, q), g.N - 4));
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int m = row_of(i), n = col_of(j, q);
        if (m >= g.M || n >= g.N) continue;
        float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        float* o = partial + ((size_t)z * g.M + m) * g.N + n;
        if constexpr (VEC) {
          if (partial) *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
          else epilogue<EPI, 4>(g, m, n, in[i][j][q], v);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (n + r >= g.N) break;
            float w[1] = {v[r]};
            if (partial) o[r] = v[r];
            else epilogue<EPI, 1>(g, m, n + r, w);
          }
        }
      }
}

// ---------------------------------------------------------------------------
// x W^T for many rows and bf16 weights with k their fast dimension: a work-group
// owns 128 rows and 128 columns, a wave 32 rows and all 128 columns.  A wave's
// rows go from memory straight to its registers in fragment layout (eight
// consecutive k a lane), two steps ahead, and are split there; only the weights
// pass through LDS, by direct loads into a ring of three buffers, two steps
// ahead.  So LDS moves 40 KB a step of 32 instead of 96.  In the kernel above and
// here, 52,000 rows, us: 256 to 1,024 columns 126 -> 121 (ReLU), 1,024 to 256 131 -> 121
// (residual), 256 to 768 84 -> 80; 16,384 rows of 128 to 512 16.4 -> 15.5; the same error
// (8.9e-8 at k = 256, 1.9e-7 at k = 1,024).
// ---------------------------------------------------------------------------
constexpr int kLinTile = 128, kLinStep = 32;

template <int EPI>
__global__ __launch_bounds__(256, 2) void k_linear_split(GemmStrided<float, bf16> g, int nt) {
  __shared__ __attribute__((aligned(16))) bf16 ring[3][kLinTile * kLinStep];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g4 = lane >> 4;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int n0 = (tile % nt) * kLinTile, m0 = (tile / nt) * kLinTile;
  const int steps = g.K / kLinStep;                      // even (host-checked)
  const bf16* w = g.b + (size_t)n0 * g.sbn;
  auto fetch = [&](int s) {                              // step s's weights (past the end: the last step's again)
    const dma::DmaTile<bf16, kLinTile, kLinStep, 4> t(ring[s % 3], w + min(s, steps - 1) * kLinStep, (int)g.sbn, kLinTile - 1);
    t.all();
  };
  const float* row[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    row[i] = g.a + (size_t)min(m0 + wave * 32 + i * 16 + col, g.M - 1) * g.sam + g4 * 8;
  float raw[2][2][8];
  auto load = [&](auto set, int s) {
    const int k = min(s, steps - 1) * kLinStep;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float4 a = *reinterpret_cast<const float4*>(row[i] + k), b = *reinterpret_cast<const float4*>(row[i] + k + 4);
      float(&v)[8] = raw[set][i];
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
      v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
  };
  f32x4 acc[2][8], low[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = low[i][j] = zero4();
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  fetch(0);
  load(c0, 0);
  fetch(1);
  load(c1, 1);
  auto step = [&](auto set, int s) {
    // step s's weights are in: younger are step s's rows, step s + 1's weights and
    // rows (4 + 2 + 4 loads)
    dma::wait_vm_barrier<10>();
    fetch(s + 2);
    Planes fa[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = split8(raw[set][i]);
    load(set, s + 2);
    const bf16* b = ring[s % 3];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bf16x8 fb = *reinterpret_cast<const bf16x8*>(&b[dma::swz<bf16, kLinStep>(16 * j + col, g4 * 8)]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa[i].p[2], low[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa[i].p[0], acc[i][j], 0, 0, 0);
        low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa[i].p[1], low[i][j], 0, 0, 0);
      }
    }
  };
  for (int s = 0; s < steps; s += 2) {
    step(c0, s);
    step(c1, s + 1);
  }
  dma::wait_loads_then_barrier();                        // no direct load outlives the work-group
  auto row_of = [&](int i) { return m0 + wave * 32 + i * 16 + col; };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] += low[i][j][r];
  form_again<2, 8, 4>(acc, [&](int i, int j, int r) {
    return dot_fp32(g, min(row_of(i), g.M - 1), n0 + 16 * j + 4 * g4 + r, 0, g.K);
  });
  EpiIn<EPI, 4> in[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) in[i][j].load(g, min(row_of(i), g.M - 1), n0 + 16 * j + 4 * g4);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int m = row_of(i), n = n0 + 16 * j + 4 * g4;
      if (m >= g.M) continue;
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = acc[i][j][r];
      epilogue<EPI, 4>(g, m, n, in[i][j], v);
    }
}

// 64 x V consecutive elements of C per work-group, each wave a quarter of the
// splits, the quarters combined in order (then, in the last work-groups, 256 row
// sums each).
template <typename TA, typename TB, int V>
__global__ __launch_bounds__(256) void k_gemm_reduce(GemmStrided<TA, TB> g, int splits, const float* partial, int blocks) {
  __shared__ double run[4][64 * V];
  const size_t mn = (size_t)g.M * g.N;
  if ((int)blockIdx.x >= blocks) {
    const int m = ((int)blockIdx.x - blocks) * 256 + (int)threadIdx.x;
    if (m >= g.M) return;
    double t = 0.0;
    const float* p = partial + splits * mn + m;
    int z = 0;
    for (; z + 8 <= splits; z += 8) {
      float q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = p[(size_t)(z + u) * g.M];
#pragma unroll
      for (int u = 0; u < 8; ++u) t += (double)q[u];
    }
    for (; z < splits; ++z) t += (double)p[(size_t)z * g.M];
    g.rowsum[m] = (float)t;
    return;
  }
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  const size_t i = (blockIdx.x * (size_t)64 + lane) * V;
  const size_t at = i < mn ? i : 0;
  const int per = (splits + 3) / 4;
  int z = min(splits, part * per);
  const int ze = min(splits, z + per);
  double t[V];   // the splits' sums added in double: long reductions (k = rows) keep fp32 accuracy
#pragma unroll
  for (int r = 0; r < V; ++r) t[r] = 0.0;
  for (; z + 8 <= ze; z += 8) {
    Pack<float, V> q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = *reinterpret_cast<const Pack<float, V>*>(partial + (z + u) * mn + at);
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int r = 0; r < V; ++r) t[r] += (double)q[u].v[r];
  }
  for (; z < ze; ++z) {
    const Pack<float, V> q = *reinterpret_cast<const Pack<float, V>*>(partial + z * mn + at);
#pragma unroll
    for (int r = 0; r < V; ++r) t[r] += (double)q.v[r];
  }
#pragma unroll
  for (int r = 0; r < V; ++r) run[part][r * 64 + lane] = t[r];
  __syncthreads();
  if (part != 0 || i >= mn) return;
  float v[V];
#pragma unroll
  for (int r = 0; r < V; ++r)
    v[r] = (float)(((run[0][r * 64 + lane] + run[1][r * 64 + lane]) + run[2][r * 64 + lane]) + run[3][r * 64 + lane]);
  epilogue<E_RAW, V>(g, (int)(i / g.N), (int)(i % g.N), v);
}

namespace {

// Vectors of `bytes` bytes along the fast dimension are aligned when the base
// and the other dimension's stride are multiples of them.
template <typename T>
bool vec_aligned(const T* p, long stride, int bytes) {
  return ((uintptr_t)p % bytes) == 0 && (stride * (long)sizeof(T)) % bytes == 0;
}

template <typename TA, typename TB, bool AKF, bool BKF, bool VEC, int EPI>
hipError_t launch_epi(const GemmStrided<TA, TB>& g, int bm, int splits, int kps, float* part, hipStream_t s) {
  const int nt = (g.N + bm - 1) / bm, mt = (g.M + bm - 1) / bm;
  const dim3 grid((unsigned)nt * mt * splits), block(256);
  if constexpr (VEC) {
    if (bm == 128) {
      hipLaunchKernelGGL((k_gemm_split<TA, TB, 128, AKF, BKF, VEC, EPI>), grid, block, 0, s, g, kps, part, nt, mt);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_gemm_split<TA, TB, 64, AKF, BKF, VEC, EPI>), grid, block, 0, s, g, kps, part, nt, mt);
  return hipGetLastError();
}

template <typename TA, typename TB, bool AKF, bool BKF, int EPI>
hipError_t launch_form(const GemmStrided<TA, TB>& g, int bm, int splits, int kps, float* part, bool vec, hipStream_t s) {
  return vec ? launch_epi<TA, TB, AKF, BKF, true, EPI>(g, bm, splits, kps, part, s)
             : launch_epi<TA, TB, AKF, BKF, false, EPI>(g, bm, splits, kps, part, s);
}

}  // namespace

template <typename TA, typename TB>
hipError_t launch_gemm_strided(const GemmStrided<TA, TB>& g, float* partial, size_t partial_floats, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  // vector loads along the operands' fast dimension and float4 columns of c
  const bool akf = g.sak == 1, bkf = g.sbk == 1;
  bool vec = g.N % 4 == 0 && g.N >= 4 && g.M >= 2 && g.K >= 1;
  vec = vec && (akf ? g.K % 32 == 0 && vec_aligned(g.a, g.sam, 16) : vec_aligned(g.a, g.sak, 2 * sizeof(TA)));
  vec = vec && (bkf ? g.K % 32 == 0 && vec_aligned(g.b, g.sbn, 16) : vec_aligned(g.b, g.sbk, 2 * sizeof(TB)));
  vec = vec && vec_stride(akf ? g.sam : g.sak) && vec_stride(bkf ? g.sbn : g.sbk);
  vec = vec && (!partial || vec_aligned(partial, 0, 16));
  vec = vec && (vec_aligned(g.c, g.ldc, 16) && (!g.mask || vec_aligned(g.mask, g.ldm, 16)) &&
                (!g.res || vec_aligned(g.res, g.ldr, 16)));
  if (!akf) vec = vec && g.M % 2 == 0;          // row pairs
  int bm = 64, splits = 1;
  if (akf) {
    // 128 x 128 tiles when they give at least two work-groups per CU, else 64 x 64.
    // 64 / 128, 256 to 256 columns, us, at 256, 512 and 768 tiles of 128: x W^T 13.6 /
    // 15.0, 23.0 / 22.2, 32.2 / 30.5, with fp32 weights 19.9 / 19.9, 34.2 / 30.8, 48.5 /
    // 43.2; dY W 18.9 / 16.5, 30.8 / 24.6, 43.0 / 34.4 (its line would be 256).
    const long tiles128 = (long)((g.M + 127) / 128) * ((g.N + 127) / 128);
    if (vec && tiles128 >= 512) bm = 128;
  } else {
    // A weight gradient: few tiles, long k (the rows).  Pieces of k of 256 to
    // kMostRows rows, each summed in fp32, the pieces added in double; as many as
    // make rounds of two work-groups per CU cheapest (at 52,000 rows a step of
    // 16 takes 1.4 us with the chip full; the pieces' sums cost their traffic).
    // With 1,000 - 52,000 rows and 64 x 64 to 256 x 1,024 gradients the number chosen
    // is within 1 % of the best of ten (29,000 rows, 128 x 512: 61 us, one tenth as
    // many pieces 689 us).
    constexpr int kMostRows = 2048, kLeastRows = 256;
    if (vec && g.M >= 128 && g.N >= 128) bm = 128;
    const long tiles = (long)((g.M + bm - 1) / bm) * ((g.N + bm - 1) / bm);
    const long most = partial ? std::min<long>(std::max(1, g.K / kLeastRows), std::max<long>(1, (long)(partial_floats / ((size_t)g.M * (g.N + 1))))) : 1;
    double best = 0.0;
    for (long n = partial ? std::min<long>(most, (g.K + kMostRows - 1) / kMostRows) : 1; n <= most; ++n) {
      const double rows = std::max(1.0, std::ceil((double)g.K / n));
      const double rounds = std::ceil(tiles * n / 512.0);
      const double us = rounds * (rows / 16 * 1.4 * (bm == 128 ? 1.0 : 0.4) + 8.0) + (n > 1 ? n * (double)g.M * g.N * 8e-6 / 5.0 : 0.0);
      if (best == 0.0 || us < best) {
        best = us;
        splits = (int)n;
      }
    }
  }
  const int kps = splits > 1 ? (((g.K + splits - 1) / splits + 31) / 32) * 32 : std::max(g.K, 1);
  splits = splits > 1 ? (g.K + kps - 1) / kps : 1;
  float* part = splits > 1 ? partial : nullptr;
  const int epi = epi_of(g);
  // Many rows by bf16 weights, where its 128 x 128 tiles give two work-groups per
  // CU: k_linear_split (as above: 13.0, 20.5 and 29.2 us).
  if constexpr (std::is_same<TA, float>::value && std::is_same<TB, bf16>::value) {
    const long tiles = (long)((g.M + kLinTile - 1) / kLinTile) * (g.N / kLinTile);
    if (akf && bkf && vec && g.N % kLinTile == 0 && g.K % (2 * kLinStep) == 0 && tiles >= 512) {
      const dim3 grid((unsigned)tiles), block(256);
#define GDP_LINEAR_CASE(E) \
  case E: hipLaunchKernelGGL((k_linear_split<E>), grid, block, 0, s, g, g.N / kLinTile); return hipGetLastError()
      switch (epi) {
        GDP_LINEAR_CASE(E_BIAS);
        GDP_LINEAR_CASE(E_BIAS | E_RELU);
        GDP_LINEAR_CASE(E_BIAS | E_SIGMOID);
        GDP_LINEAR_CASE(E_BIAS | E_RES);
        GDP_LINEAR_CASE(E_ACC);
      }
#undef GDP_LINEAR_CASE
    }
  }
  // The forms in use: a linear layer, its input gradient, its weight gradient.
  hipError_t e = hipErrorInvalidValue;
#define GDP_GEMM_CASE(E, AKF, BKF) \
  case E: e = launch_form<TA, TB, AKF, BKF, E>(g, bm, splits, kps, part, vec, s); break
  if (akf && bkf) {
    if constexpr (std::is_same<TA, float>::value) {
      switch (epi) {
        GDP_GEMM_CASE(E_BIAS | E_RELU, true, true);
        GDP_GEMM_CASE(E_BIAS | E_RES, true, true);
        GDP_GEMM_CASE(E_ACC, true, true);
      }
    }
    switch (epi) {                              // bf16 features too
      GDP_GEMM_CASE(E_BIAS, true, true);
      GDP_GEMM_CASE(E_BIAS | E_SIGMOID, true, true);
    }
  } else if (akf && g.sbn == 1) {
    if constexpr (std::is_same<TA, float>::value) {
      switch (epi) {
        GDP_GEMM_CASE(E_RAW, true, false);
        GDP_GEMM_CASE(E_MASK, true, false);
        GDP_GEMM_CASE(E_RES, true, false);
        GDP_GEMM_CASE(E_ACC, true, false);
      }
    }
  } else if (g.sam == 1 && g.sbn == 1) {
    if constexpr (std::is_same<TA, float>::value) {
      switch (epi) {
        GDP_GEMM_CASE(E_RAW, false, false);
      }
    }
  }
#undef GDP_GEMM_CASE
  if (e != hipSuccess || splits == 1) return e;
  const int v = vec ? 4 : 1;
  const int blocks = (int)(((size_t)g.M * g.N / v + 63) / 64);
  const dim3 rgrid((unsigned)(blocks + (g.rowsum ? (g.M + 255) / 256 : 0)));
  if (vec) hipLaunchKernelGGL((k_gemm_reduce<TA, TB, 4>), rgrid, dim3(256), 0, s, g, splits, (const float*)partial, blocks);
  else hipLaunchKernelGGL((k_gemm_reduce<TA, TB, 1>), rgrid, dim3(256), 0, s, g, splits, (const float*)partial, blocks);
  return hipGetLastError();
}

#define GDP_GEMM_INST(TA, TB) \
  template hipError_t launch_gemm_strided<TA, TB>(const GemmStrided<TA, TB>&, float*, size_t, hipStream_t);
GDP_GEMM_INST(float, float)
GDP_GEMM_INST(float, bf16)
GDP_GEMM_INST(bf16, bf16)
#undef GDP_GEMM_INST

}  // namespace tr
}  // namespace gdp

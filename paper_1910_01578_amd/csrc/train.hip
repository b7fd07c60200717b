// Kernels of the policy's update step (Section 3: Eq. 1 optimised with PPO;
// Section 3.1: the graph embedding network trains jointly with the placement
// network; Section 3.2: the cached segment memory passes no gradient): the
// training forward pass that keeps every intermediate, the backward pass and
// the Adam update, but for the dense products (train_gemm.hip) and the attention
// (train_attn.hip).  Everything here computes in fp32 (weights and inputs of
// bf16 problems are widened on load), with fixed summation orders, so results
// are deterministic.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"
#include "host_plan.h"
#include "train_kernels.h"

namespace gdp {
namespace tr {

__device__ __forceinline__ float ld(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ld(const bf16* p, size_t i) { return (float)p[i]; }

// V = width / 64 consecutive columns of a row a lane.
template <int V>
struct alignas(4 * V) Cols {
  float v[V];
};
template <int V>
__device__ __forceinline__ Cols<V> load_cols(const float* row, int lane) {
  return *reinterpret_cast<const Cols<V>*>(row + lane * V);
}
template <int V>
__device__ __forceinline__ void store_cols(float* row, int lane, const Cols<V>& c) {
  *reinterpret_cast<Cols<V>*>(row + lane * V) = c;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// The rows [r0, r1) of chunk `chunk` (kColChunkRows rows, none across graphs).
__device__ __forceinline__ int chunk_rows(const GraphTable& ct, int chunk, int& r0, int& r1) {
  const int g = graph_of_block(ct, chunk);
  r0 = ct.ptr[g] + (chunk - ct.blk[g]) * kColChunkRows;
  r1 = min(r0 + kColChunkRows, ct.ptr[g + 1]);
  return g;
}

// Four waves' column sums a, b of a chunk, added in wave order into partial[chunk][2][64 V].
template <int V>
__device__ __forceinline__ void chunk_sums(const Cols<V>& a, const Cols<V>& b, int chunk, float* partial) {
  __shared__ float red[4][2][64 * V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  store_cols<V>(red[wave][0], lane, a);
  store_cols<V>(red[wave][1], lane, b);
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * 64 * V; i += 256) {
    const float* r = &red[0][0][0] + i;
    partial[(size_t)chunk * 128 * V + i] = (r[0] + r[128 * V]) + (r[256 * V] + r[384 * V]);
  }
}

// out0[g][c], out1[g][c] = the graph's chunk sums (columns 0 .. C - 1 and C .. 2C - 1)
// added in double: 64 columns x 16 runs of chunks per work-group, the runs
// combined in order.  mean: divided by the graph's rows.
__global__ __launch_bounds__(1024) void k_chunks_final(const float* partial, int C, int cols, GraphTable ct, float* out0,
                                                       float* out1, int mean) {
  __shared__ double run[16][64];
  const int g = blockIdx.y;
  const int cl = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + cl;
  const int k0 = ct.blk[g], k1 = ct.blk[g + 1];
  const int per = (k1 - k0 + 15) / 16;
  const int ka = min(k1, k0 + part * per), kz = min(k1, ka + per);
  double t = 0.0;
  int k = ka;
  for (; k + 8 <= kz; k += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(k + u) * cols + c];
#pragma unroll
    for (int u = 0; u < 8; ++u) t += (double)v[u];
  }
  for (; k < kz; ++k) t += (double)partial[(size_t)k * cols + c];
  run[part][cl] = t;
  __syncthreads();
  if (part != 0) return;
  t = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) t += run[u][cl];
  float v = (float)t;
  if (mean) v /= (float)(ct.ptr[g + 1] - ct.ptr[g]);
  if (c < C) out0[(size_t)g * C + c] = v;
  else out1[(size_t)g * C + c - C] = v;
}
static hipError_t launch_chunks_final(const float* partial, int C, int cols, const GraphTable& ct, float* out0,
                                      float* out1, bool mean, hipStream_t s) {
  hipLaunchKernelGGL(k_chunks_final, dim3(cols / 64, ct.n), dim3(1024), 0, s, partial, C, cols, ct, out0, out1,
                     mean ? 1 : 0);
  return hipGetLastError();
}

#define GDP_BY_WIDTH(d, GO)                 \
  switch (d) {                              \
    case 64: GO(1); break;                  \
    case 128: GO(2); break;                 \
    case 256: GO(4); break;                 \
    default: return hipErrorInvalidValue;   \
  }

// ---------------------------------------------------------------------------
// Row-wise kernels: one wavefront per row, the row in registers.  Bound by
// memory (52,000 rows of 256: forward 107 MB, 30 us at the copy rate of 5 TB/s
// less the launch; backward 160 MB and the gains' sums in the same pass).
// ---------------------------------------------------------------------------
template <int V>
__device__ __forceinline__ float row_stats(const Cols<V>& x, float& mu) {
  constexpr float inv = 1.0f / (64 * V);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) s += x.v[i];
  mu = wave_sum(s) * inv;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const float t = x.v[i] - mu;
    q += t * t;
  }
  return 1.0f / sqrtf(wave_sum(q) * inv + 1e-5f);
}

// out = LN(r) * g + b  (eps 1e-5, biased variance); 16 rows a work-group
template <typename T, int V>
__global__ __launch_bounds__(256) void k_ln_fwd(const float* __restrict__ r, int n, const T* g, const T* b,
                                                float* __restrict__ out) {
  constexpr int d = 64 * V;
  const int row0 = blockIdx.x * 16 + (threadIdx.x >> 6) * 4, lane = threadIdx.x & 63;
  Cols<V> gn, sh, x[4];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    gn.v[i] = ld(g, lane * V + i);
    sh.v[i] = ld(b, lane * V + i);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = load_cols<V>(r + (size_t)min(row0 + k, n - 1) * d, lane);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (row0 + k >= n) return;
    float mu;
    const float rstd = row_stats<V>(x[k], mu);
    Cols<V> y;
#pragma unroll
    for (int i = 0; i < V; ++i) y.v[i] = (x[k].v[i] - mu) * rstd * gn.v[i] + sh.v[i];
    store_cols<V>(out + (size_t)(row0 + k) * d, lane, y);
  }
}

// LayerNorm backward for out = LN(r) g + b and upstream dout: dr, and the
// chunk's sums of dout * xhat and dout (the gain's and shift's gradients).
template <typename T, int V>
__global__ __launch_bounds__(256) void k_ln_bwd(const float* __restrict__ r, const float* __restrict__ dout, const T* g,
                                                GraphTable ct, float* __restrict__ dr, float* partial) {
  constexpr int d = 64 * V;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int r0, r1;
  chunk_rows(ct, blockIdx.x, r0, r1);
  Cols<V> gn, sg, sb;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    gn.v[i] = ld(g, lane * V + i);
    sg.v[i] = sb.v[i] = 0.f;
  }
  for (int row = r0 + wave * 2; row < r1; row += 8) {     // two rows at a time
    Cols<V> x[2], dy[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const size_t at = (size_t)min(row + k, r1 - 1) * d;
      x[k] = load_cols<V>(r + at, lane);
      dy[k] = load_cols<V>(dout + at, lane);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (row + k >= r1) break;
      float mu;
      const float rstd = row_stats<V>(x[k], mu);
      float s1 = 0.f, s2 = 0.f;
      Cols<V> xh, gd, o;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        xh.v[i] = (x[k].v[i] - mu) * rstd;
        gd.v[i] = dy[k].v[i] * gn.v[i];
        s1 += gd.v[i];
        s2 += gd.v[i] * xh.v[i];
        sg.v[i] += dy[k].v[i] * xh.v[i];
        sb.v[i] += dy[k].v[i];
      }
      s1 = wave_sum(s1) * (1.0f / d);
      s2 = wave_sum(s2) * (1.0f / d);
#pragma unroll
      for (int i = 0; i < V; ++i) o.v[i] = rstd * (gd.v[i] - s1 - xh.v[i] * s2);
      store_cols<V>(dr + (size_t)(row + k) * d, lane, o);
    }
  }
  chunk_sums<V>(sg, sb, blockIdx.x, partial);
}

template <typename T>
hipError_t launch_ln_fwd(const float* r, int n, int d, const T* g, const T* b, float* out, hipStream_t s) {
#define GO(V) hipLaunchKernelGGL((k_ln_fwd<T, V>), dim3((n + 15) / 16), dim3(256), 0, s, r, n, g, b, out)
  GDP_BY_WIDTH(d, GO)
#undef GO
  return hipGetLastError();
}
template <typename T>
hipError_t launch_ln_bwd(const float* r, const float* dout, int d, const T* g, const GraphTable& rows, int chunks,
                         float* dr, float* dg, float* db, float* partial, hipStream_t s) {
#define GO(V) hipLaunchKernelGGL((k_ln_bwd<T, V>), dim3(chunks), dim3(256), 0, s, r, dout, g, rows, dr, partial)
  GDP_BY_WIDTH(d, GO)
#undef GO
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_chunks_final(partial, d, 2 * d, rows, dg, db, false, s);
}
template hipError_t launch_ln_fwd<float>(const float*, int, int, const float*, const float*, float*, hipStream_t);
template hipError_t launch_ln_fwd<bf16>(const float*, int, int, const bf16*, const bf16*, float*, hipStream_t);
template hipError_t launch_ln_bwd<float>(const float*, const float*, int, const float*, const GraphTable&, int, float*,
                                         float*, float*, float*, hipStream_t);
template hipError_t launch_ln_bwd<bf16>(const float*, const float*, int, const bf16*, const GraphTable&, int, float*,
                                        float*, float*, float*, hipStream_t);

// ---------------------------------------------------------------------------
// FiLM (Eq. 4).
// ---------------------------------------------------------------------------
// y[v][c] = gamma[g(v)][c] * x[v][c] + beta[g(v)][c], 16 bytes a thread (d is a
// multiple of 4, so a thread's columns are of one node)
__global__ __launch_bounds__(256) void k_film_apply(const float4* __restrict__ x, size_t n4, int d4,
                                                    const float* __restrict__ gamma, const float* __restrict__ beta,
                                                    GraphTable gt, float4* __restrict__ y) {
  const size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
  if (i >= n4) return;
  const int v = (int)(i / d4), c = (int)(i % d4) * 4;
  const size_t at = (size_t)graph_of_node(gt, v) * d4 * 4 + c;
  const float4 t = x[i], gm = *reinterpret_cast<const float4*>(gamma + at), bt = *reinterpret_cast<const float4*>(beta + at);
  y[i] = make_float4(gm.x * t.x + bt.x, gm.y * t.y + bt.y, gm.z * t.z + bt.z, gm.w * t.w + bt.w);
}
hipError_t launch_film_apply(const float* x, int n, int d, const float* gamma, const float* beta, const GraphTable& gt,
                             float* y, hipStream_t s) {
  const size_t n4 = (size_t)n * d / 4;
  hipLaunchKernelGGL(k_film_apply, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const float4*>(x), n4, d / 4, gamma, beta, gt, reinterpret_cast<float4*>(y));
  return hipGetLastError();
}

template <int V>
__global__ __launch_bounds__(256) void k_film_bwd(const float* __restrict__ dy, const float* __restrict__ x,
                                                  const float* gamma, GraphTable ct, float* __restrict__ dx,
                                                  float* partial) {
  constexpr int d = 64 * V;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int r0, r1;
  const int g = chunk_rows(ct, blockIdx.x, r0, r1);
  const Cols<V> gm = load_cols<V>(gamma + (size_t)g * d, lane);
  Cols<V> sg, sb;
#pragma unroll
  for (int i = 0; i < V; ++i) sg.v[i] = sb.v[i] = 0.f;
  for (int row = r0 + wave * 4; row < r1; row += 16) {    // four rows at a time
    Cols<V> xr[4], yr[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t at = (size_t)min(row + k, r1 - 1) * d;
      xr[k] = load_cols<V>(x + at, lane);
      yr[k] = load_cols<V>(dy + at, lane);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (row + k >= r1) break;
      Cols<V> o;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        sg.v[i] += yr[k].v[i] * xr[k].v[i];
        sb.v[i] += yr[k].v[i];
        o.v[i] = gm.v[i] * yr[k].v[i];
      }
      store_cols<V>(dx + (size_t)(row + k) * d, lane, o);
    }
  }
  chunk_sums<V>(sg, sb, blockIdx.x, partial);
}
hipError_t launch_film_bwd(const float* dy, const float* x, int d, const float* gamma, const GraphTable& ct, int chunks,
                           float* dx, float* dgamma, float* dbeta, float* partial, hipStream_t s) {
#define GO(V) hipLaunchKernelGGL((k_film_bwd<V>), dim3(chunks), dim3(256), 0, s, dy, x, gamma, ct, dx, partial)
  GDP_BY_WIDTH(d, GO)
#undef GO
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_chunks_final(partial, d, 2 * d, ct, dgamma, dbeta, false, s);
}

// dW_l[c][h] = sum_g dfilm_l[g][c] x0[g][h] and db_l[c] = sum_g dfilm_l[g][c], for
// gamma's and beta's weights of every layer (blockIdx.y = 2 l + which); a
// work-group per c.
__global__ __launch_bounds__(256) void k_film_wgrad(FilmWeightGrads gr, const float* __restrict__ dfilm,
                                                    const float* __restrict__ x0, int G, int d, int H) {
  const int l = blockIdx.y >> 1, c = blockIdx.x;
  const bool beta = blockIdx.y & 1;
  const float* df = dfilm + (size_t)blockIdx.y * G * d + c;
  float* w = (beta ? gr.wb[l] : gr.wg[l]) + (size_t)c * H;
  for (int h = threadIdx.x; h < H; h += 256) {
    double t = 0.0;
    for (int g = 0; g < G; ++g) t += (double)df[(size_t)g * d] * (double)x0[(size_t)g * H + h];
    w[h] = (float)t;
  }
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int g = 0; g < G; ++g) t += (double)df[(size_t)g * d];
    (beta ? gr.bb[l] : gr.bg[l])[c] = (float)t;
  }
}

// dx0[g][h] = sum over layers, gamma and beta, c of dfilm[g][c] W[c][h]: 64
// columns x 16 runs of c per work-group, the runs combined in order.
template <typename T>
__global__ __launch_bounds__(1024) void k_film_dx0(FilmLayers<T> w, int layers, const float* __restrict__ dfilm, int G,
                                                   int d, int H, float* __restrict__ dx0) {
  __shared__ double run[16][64];
  const int cl = threadIdx.x & 63, part = threadIdx.x >> 6, h = blockIdx.x * 64 + cl, g = blockIdx.y;
  const int per = d / 16;
  double t = 0.0;
  for (int q = 0; q < 2 * layers; ++q) {
    const T* W = ((q & 1) ? w.wb[q >> 1] : w.wg[q >> 1]) + (size_t)part * per * H + h;
    const float* df = dfilm + ((size_t)q * G + g) * d + part * per;
    for (int c = 0; c < per; c += 4) {
      float a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = df[c + u];
        b[u] = ld(W, (size_t)(c + u) * H);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) t += (double)a[u] * (double)b[u];
    }
  }
  run[part][cl] = t;
  __syncthreads();
  if (part != 0) return;
  t = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) t += run[u][cl];
  dx0[(size_t)g * H + h] = (float)t;
}
template <typename T>
hipError_t launch_film_weights_bwd(const FilmLayers<T>& w, const FilmWeightGrads& gr, int layers, const float* dfilm,
                                   const float* x0, int G, int d, int H, float* dx0, hipStream_t s) {
  hipLaunchKernelGGL(k_film_wgrad, dim3(d, 2 * layers), dim3(256), 0, s, gr, dfilm, x0, G, d, H);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_film_dx0<T>), dim3(H / 64, G), dim3(1024), 0, s, w, layers, dfilm, G, d, H, dx0);
  return hipGetLastError();
}
template hipError_t launch_film_weights_bwd<float>(const FilmLayers<float>&, const FilmWeightGrads&, int, const float*,
                                                   const float*, int, int, int, float*, hipStream_t);
template hipError_t launch_film_weights_bwd<bf16>(const FilmLayers<bf16>&, const FilmWeightGrads&, int, const float*,
                                                  const float*, int, int, int, float*, hipStream_t);

// ---------------------------------------------------------------------------
// Elementwise kernels and the mean pool.
// ---------------------------------------------------------------------------
__global__ void k_mask_pos(const float4* a, const float4* b, size_t n4, float4* out) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n4; i += (size_t)gridDim.x * blockDim.x) {
    float4 v = a[i];
    const float4 m = b[i];
    v.x = m.x > 0.f ? v.x : 0.f;
    v.y = m.y > 0.f ? v.y : 0.f;
    v.z = m.z > 0.f ? v.z : 0.f;
    v.w = m.w > 0.f ? v.w : 0.f;
    out[i] = v;
  }
}
hipError_t launch_mask_pos(const float* a, const float* b, size_t n, float* out, hipStream_t s) {
  const size_t n4 = n / 4;                      // rows of 64 columns and more
  const unsigned blocks = (unsigned)std::min<size_t>((n4 + 255) / 256, 8192);
  hipLaunchKernelGGL(k_mask_pos, dim3(std::max(1u, blocks)), dim3(256), 0, s, reinterpret_cast<const float4*>(a),
                     reinterpret_cast<const float4*>(b), n4, reinterpret_cast<float4*>(out));
  return hipGetLastError();
}

// dh[v][c] += dx0[g(v)][c] / n_g  (the mean pool's backward)
__global__ void k_meanpool_bwd(const float* dx0, int n, int H, GraphTable gt, float* dh) {
  const size_t total = (size_t)n * H;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int v = (int)(i / H), c = (int)(i % H);
    const int g = graph_of_node(gt, v);
    dh[i] += dx0[(size_t)g * H + c] / (float)(gt.ptr[g + 1] - gt.ptr[g]);
  }
}
hipError_t launch_meanpool_bwd(const float* dx0, int n, int H, const GraphTable& gt, float* dh, hipStream_t s) {
  const size_t total = (size_t)n * H;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_meanpool_bwd, dim3(blocks), dim3(256), 0, s, dx0, n, H, gt, dh);
  return hipGetLastError();
}

// x0[g] = mean over the rows of graph g: its chunks' column sums, then the chunks.
template <int V>
__global__ __launch_bounds__(256) void k_chunk_colsum(const float* __restrict__ h, GraphTable ct, float* partial) {
  constexpr int H = 64 * V;
  __shared__ float red[4][H];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int r0, r1;
  chunk_rows(ct, blockIdx.x, r0, r1);
  Cols<V> t;
#pragma unroll
  for (int i = 0; i < V; ++i) t.v[i] = 0.f;
  for (int row = r0 + wave * 4; row < r1; row += 16) {
    Cols<V> x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = load_cols<V>(h + (size_t)min(row + k, r1 - 1) * H, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (row + k < r1)
#pragma unroll
        for (int i = 0; i < V; ++i) t.v[i] += x[k].v[i];
  }
  store_cols<V>(red[wave], lane, t);
  __syncthreads();
  if (threadIdx.x < H)
    partial[(size_t)blockIdx.x * H + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}
hipError_t launch_meanpool_f32(const float* h, int H, const GraphTable& ct, int chunks, float* partial, float* x0,
                               hipStream_t s) {
#define GO(V) hipLaunchKernelGGL((k_chunk_colsum<V>), dim3(chunks), dim3(256), 0, s, h, ct, partial)
  GDP_BY_WIDTH(H, GO)
#undef GO
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_chunks_final(partial, H, H, ct, x0, nullptr, true, s);
}

// ---------------------------------------------------------------------------
// Eq. 2's max-pool with the winning neighbour of every element (ties: the
// lowest node id), and its backward: dP[u][c] = sum over the neighbours v of u
// (out-edges in CSR order, then in-edges in ascending order) whose element c
// was won by u of dA[v][c].  u in S(v) implies v in N(u), so every v that
// selected u is visited.
// ---------------------------------------------------------------------------
//
// 16 V lanes own a node (V = H / 64), each four columns; neighbours four at a
// time, so that their rows are in flight together.
template <int V>
__global__ __launch_bounds__(256) void k_gather_max_arg(const float* __restrict__ P, const int* __restrict__ s_ptr,
                                                        const int* __restrict__ s_idx, int n, float* __restrict__ A,
                                                        int* __restrict__ arg) {
  constexpr int H = 64 * V, LPR = 16 * V;
  const int v = (int)((blockIdx.x * 256 + threadIdx.x) / LPR), c = (int)(threadIdx.x % LPR) * 4;
  if (v >= n) return;
  float best[4] = {0.f, 0.f, 0.f, 0.f};
  int who[4] = {-1, -1, -1, -1};
  const int e0 = s_ptr[v], e1 = s_ptr[v + 1];
  for (int e = e0; e < e1; e += 4) {
    int u[4];
    float4 p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = s_idx[min(e + k, e1 - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = *reinterpret_cast<const float4*>(P + (size_t)u[k] * H + c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (e + k >= e1) break;
      const float q[4] = {p[k].x, p[k].y, p[k].z, p[k].w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (who[i] < 0 || q[i] > best[i] || (q[i] == best[i] && u[k] < who[i])) {
          best[i] = q[i];
          who[i] = u[k];
        }
    }
  }
  *reinterpret_cast<float4*>(A + (size_t)v * H + c) = make_float4(best[0], best[1], best[2], best[3]);
  *reinterpret_cast<int4*>(arg + (size_t)v * H + c) = make_int4(who[0], who[1], who[2], who[3]);
}
hipError_t launch_gather_max_arg(const float* P, const int* s_ptr, const int* s_idx, int n, int H, float* A, int* arg,
                                 hipStream_t s) {
#define GO(V) \
  hipLaunchKernelGGL((k_gather_max_arg<V>), dim3((unsigned)(((size_t)n * 16 * V + 255) / 256)), dim3(256), 0, s, P, s_ptr, s_idx, n, A, arg)
  GDP_BY_WIDTH(H, GO)
#undef GO
  return hipGetLastError();
}

template <int V>
__global__ __launch_bounds__(256) void k_gather_max_bwd(const float* __restrict__ dA, const int* __restrict__ arg,
                                                        const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
                                                        const int* __restrict__ in_ptr, const int* __restrict__ in_idx,
                                                        const float* __restrict__ P, int n, float* __restrict__ dZ) {
  constexpr int H = 64 * V, LPR = 16 * V;
  const int u = (int)((blockIdx.x * 256 + threadIdx.x) / LPR), c = (int)(threadIdx.x % LPR) * 4;
  if (u >= n) return;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  auto edges = [&](const int* __restrict__ idx, int e0, int e1) {
    for (int e = e0; e < e1; e += 4) {
      int v[4];
      int4 w[4];
      float4 g[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = idx[min(e + k, e1 - 1)];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        w[k] = *reinterpret_cast<const int4*>(arg + (size_t)v[k] * H + c);
        g[k] = *reinterpret_cast<const float4*>(dA + (size_t)v[k] * H + c);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (e + k >= e1) break;
        if (w[k].x == u) s[0] += g[k].x;
        if (w[k].y == u) s[1] += g[k].y;
        if (w[k].z == u) s[2] += g[k].z;
        if (w[k].w == u) s[3] += g[k].w;
      }
    }
  };
  edges(col_idx, row_ptr[u], row_ptr[u + 1]);
  edges(in_idx, in_ptr[u], in_ptr[u + 1]);
  const float4 p = *reinterpret_cast<const float4*>(P + (size_t)u * H + c);
  *reinterpret_cast<float4*>(dZ + (size_t)u * H + c) =
      make_float4(s[0] * p.x * (1.0f - p.x), s[1] * p.y * (1.0f - p.y), s[2] * p.z * (1.0f - p.z), s[3] * p.w * (1.0f - p.w));
}
hipError_t launch_gather_max_bwd(const float* dA, const int* arg, const int* row_ptr, const int* col_idx,
                                 const int* in_ptr, const int* in_idx, const float* P, int n, int H, float* dZ,
                                 hipStream_t s) {
#define GO(V)                                                                                                        \
  hipLaunchKernelGGL((k_gather_max_bwd<V>), dim3((unsigned)(((size_t)n * 16 * V + 255) / 256)), dim3(256), 0, s, dA, \
                     arg, row_ptr, col_idx, in_ptr, in_idx, P, n, dZ)
  GDP_BY_WIDTH(H, GO)
#undef GO
  return hipGetLastError();
}

// Sorts each in-edge row ascending (rows filled by atomics come in any order),
// so the backward's sums run in a fixed order.  16 lanes a row: each entry's
// place is the number of smaller ones (ids differ), counted over the row in
// registers (up to 16 entries) or in LDS (up to kSortLds); longer rows by
// insertion on one lane.
constexpr int kSortLds = 256;
__global__ __launch_bounds__(256) void k_sort_rows(const int* ptr, int n, int* idx) {
  __shared__ int rows[16][kSortLds];
  const int grp = threadIdx.x >> 4, sub = threadIdx.x & 15;
  const int v = blockIdx.x * 16 + grp;
  const int a = v < n ? ptr[v] : 0, b = v < n ? ptr[v + 1] : 0, len = b - a;
  if (len > kSortLds) {
    if (sub == 0)
      for (int i = a + 1; i < b; ++i) {
        const int x = idx[i];
        int j = i - 1;
        while (j >= a && idx[j] > x) {
          idx[j + 1] = idx[j];
          --j;
        }
        idx[j + 1] = x;
      }
    return;
  }
  if (len < 2) return;
  // a row's lanes are in one wave: the LDS writes below precede its reads
  for (int i = sub; i < len; i += 16) rows[grp][i] = idx[a + i];
  __builtin_amdgcn_wave_barrier();
  for (int i = sub; i < len; i += 16) {
    const int x = rows[grp][i];
    int place = 0;
    for (int j = 0; j < len; ++j) {
      const int y = rows[grp][j];
      place += y < x || (y == x && j < i) ? 1 : 0;
    }
    idx[a + place] = x;
  }
}
hipError_t launch_sort_rows(const int* ptr, int n, int* idx, hipStream_t s) {
  hipLaunchKernelGGL(k_sort_rows, dim3((n + 15) / 16), dim3(256), 0, s, ptr, n, idx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adam (Kingma and Ba, 2015): fp32 master weights and moments; the dtype copy
// the kernels read is rewritten from the master.  Many small tensors in one
// launch: a launch of its own costs each more than its work.
// ---------------------------------------------------------------------------
constexpr int kAdamBlock = 2048;                // elements per work-group
struct AdamTable {
  int n;
  int blk[kAdamTensors + 1];                    // work-groups before each tensor
  gdp_adam_tensor t[kAdamTensors];
};
template <typename T>
__global__ __launch_bounds__(256) void k_adam(AdamTable a, float lr, float b1, float b2, float eps, float c1, float c2) {
  int lo = 0, hi = a.n - 1;                     // largest tensor with blk[i] <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.blk[mid] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const gdp_adam_tensor t = a.t[lo];
  T* param = static_cast<T*>(t.param);
  const int64_t i0 = (int64_t)((int)blockIdx.x - a.blk[lo]) * kAdamBlock;
  const int64_t i1 = i0 + kAdamBlock < t.n ? i0 + kAdamBlock : t.n;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const float g = t.grad[i];
    const float mi = b1 * t.m[i] + (1.0f - b1) * g;
    const float vi = b2 * t.v[i] + (1.0f - b2) * g * g;
    t.m[i] = mi;
    t.v[i] = vi;
    const float w = t.master[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    t.master[i] = w;
    param[i] = from_f32<T>(w);
  }
}
hipError_t launch_adam(const gdp_adam_tensor* t, int n_tensors, bool to_bf16, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t s) {
  AdamTable a;
  a.n = 0;
  int64_t blocks = 0;
  for (int i = 0; i < n_tensors && a.n < kAdamTensors; ++i) {
    if (t[i].n == 0) continue;
    a.blk[a.n] = (int)blocks;
    a.t[a.n++] = t[i];
    blocks += (t[i].n + kAdamBlock - 1) / kAdamBlock;
  }
  if (a.n == 0) return hipSuccess;
  a.blk[a.n] = (int)blocks;
  const dim3 grid((unsigned)blocks), block(256);
  if (to_bf16) hipLaunchKernelGGL((k_adam<bf16>), grid, block, 0, s, a, lr, b1, b2, eps, c1, c2);
  else hipLaunchKernelGGL((k_adam<float>), grid, block, 0, s, a, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace tr
}  // namespace gdp

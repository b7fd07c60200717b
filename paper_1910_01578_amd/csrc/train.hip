// Kernels of the policy's update step (Section 3: Eq. 1 optimised with PPO;
// Section 3.1: the graph embedding network trains jointly with the placement
// network; Section 3.2: the cached segment memory passes no gradient): the
// training forward pass that keeps every intermediate, the backward pass and
// the Adam update.  Everything here computes in fp32 (weights and inputs of
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

// ---------------------------------------------------------------------------
// Column sums per graph: out[g][c] (+)= sum over rows v of graph g of
// A[v][c] (* B[v][c] when B is given), in a fixed order: 256-row chunks of
// each graph into partials, then each graph's chunks in order.
// ---------------------------------------------------------------------------
constexpr int kColRows = 256;

template <typename TA>
__global__ __launch_bounds__(256) void k_colsum_partial(const TA* a, int lda, const float* b, int ldb, int C,
                                                        GraphTable ct, float* partial) {
  const int chunk = blockIdx.y;
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  const int g = graph_of_block(ct, chunk);
  const int r0 = ct.ptr[g] + (chunk - ct.blk[g]) * kColRows;
  const int r1 = min(r0 + kColRows, ct.ptr[g + 1]);
  // eight interleaved partial sums (rows r0 + 8 i + u go to sum u), combined in order
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int r = r0;
  for (; r + 8 <= r1; r += 8) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      float v = ld(a, (size_t)(r + u) * lda + c);
      if (b) v *= b[(size_t)(r + u) * ldb + c];
      s[u] += v;
    }
  }
  for (; r < r1; ++r) {             // the last (at most 7) rows into sum 0
    float v = ld(a, (size_t)r * lda + c);
    if (b) v *= b[(size_t)r * ldb + c];
    s[0] += v;
  }
  partial[(size_t)chunk * C + c] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// out[g][c] (+)= the graph's chunk sums added in double; 64 columns x 4 chunk
// quarters per work-group, the quarters combined in order.
__global__ __launch_bounds__(256) void k_colsum_final(const float* partial, int C, GraphTable ct, float* out, int ldo,
                                                      int accumulate) {
  __shared__ double q4[4][64];
  const int g = blockIdx.y;
  const int cl = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + cl;
  const int k0 = ct.blk[g], k1 = ct.blk[g + 1];
  const int per = (k1 - k0 + 3) / 4;
  const int ka = k0 + part * per, kz = min(k1, ka + per);
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (c < C) {
    int k = ka;
    for (; k + 4 <= kz; k += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += (double)partial[(size_t)(k + u) * C + c];
    }
    for (; k < kz; ++k) s[0] += (double)partial[(size_t)k * C + c];
  }
  q4[part][cl] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (part == 0 && c < C) {
    const double t = (q4[0][cl] + q4[1][cl]) + (q4[2][cl] + q4[3][cl]);
    float* o = out + (size_t)g * ldo + c;
    *o = accumulate ? *o + (float)t : (float)t;
  }
}

template <typename TA>
hipError_t launch_colsum(const TA* a, int lda, const float* b, int ldb, int C, const GraphTable& ct, int chunks,
                         float* partial, float* out, int ldo, bool accumulate, hipStream_t s) {
  if (C <= 0 || chunks <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_colsum_partial<TA>), dim3((C + 255) / 256, chunks), dim3(256), 0, s, a, lda, b, ldb, C, ct,
                     partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_colsum_final, dim3((C + 63) / 64, ct.n), dim3(256), 0, s, (const float*)partial, C, ct, out,
                     ldo, accumulate ? 1 : 0);
  return hipGetLastError();
}
template hipError_t launch_colsum<float>(const float*, int, const float*, int, int, const GraphTable&, int, float*,
                                         float*, int, bool, hipStream_t);
template hipError_t launch_colsum<bf16>(const bf16*, int, const float*, int, int, const GraphTable&, int, float*,
                                        float*, int, bool, hipStream_t);

// ---------------------------------------------------------------------------
// Row-wise kernels: one wavefront per row of width d <= 1024.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// out = LN(r) * g + b  (eps 1e-5, biased variance)
template <typename T>
__global__ __launch_bounds__(256) void k_ln_fwd(const float* r, int n, int d, const T* g, const T* b, float* out) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  const float* x = r + (size_t)row * d;
  float s = 0.f;
  for (int c = lane; c < d; c += kWave) s += x[c];
  const float mu = wave_sum(s) / d;
  float q = 0.f;
  for (int c = lane; c < d; c += kWave) {
    const float t = x[c] - mu;
    q += t * t;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / d + 1e-5f);
  for (int c = lane; c < d; c += kWave) out[(size_t)row * d + c] = (x[c] - mu) * rstd * ld(g, c) + ld(b, c);
}

// LayerNorm backward for out = LN(r) g + b and upstream dout: dr, and the
// per-row terms of the gain gradient (dout * xhat) in xg.
template <typename T>
__global__ __launch_bounds__(256) void k_ln_bwd(const float* r, const float* dout, int n, int d, const T* g,
                                                float* dr, float* xg) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  const float* x = r + (size_t)row * d;
  const float* dy = dout + (size_t)row * d;
  float s = 0.f;
  for (int c = lane; c < d; c += kWave) s += x[c];
  const float mu = wave_sum(s) / d;
  float q = 0.f;
  for (int c = lane; c < d; c += kWave) {
    const float t = x[c] - mu;
    q += t * t;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / d + 1e-5f);
  float s1 = 0.f, s2 = 0.f;
  for (int c = lane; c < d; c += kWave) {
    const float xh = (x[c] - mu) * rstd;
    const float gd = dy[c] * ld(g, c);
    s1 += gd;
    s2 += gd * xh;
  }
  s1 = wave_sum(s1) / d;
  s2 = wave_sum(s2) / d;
  for (int c = lane; c < d; c += kWave) {
    const float xh = (x[c] - mu) * rstd;
    const float gd = dy[c] * ld(g, c);
    dr[(size_t)row * d + c] = rstd * (gd - s1 - xh * s2);
    xg[(size_t)row * d + c] = dy[c] * xh;
  }
}

template <typename T>
hipError_t launch_ln_fwd(const float* r, int n, int d, const T* g, const T* b, float* out, hipStream_t s) {
  hipLaunchKernelGGL((k_ln_fwd<T>), dim3((n + 3) / 4), dim3(256), 0, s, r, n, d, g, b, out);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_ln_bwd(const float* r, const float* dout, int n, int d, const T* g, float* dr, float* xg,
                         hipStream_t s) {
  hipLaunchKernelGGL((k_ln_bwd<T>), dim3((n + 3) / 4), dim3(256), 0, s, r, dout, n, d, g, dr, xg);
  return hipGetLastError();
}
template hipError_t launch_ln_fwd<float>(const float*, int, int, const float*, const float*, float*, hipStream_t);
template hipError_t launch_ln_fwd<bf16>(const float*, int, int, const bf16*, const bf16*, float*, hipStream_t);
template hipError_t launch_ln_bwd<float>(const float*, const float*, int, int, const float*, float*, float*,
                                         hipStream_t);
template hipError_t launch_ln_bwd<bf16>(const float*, const float*, int, int, const bf16*, float*, float*,
                                        hipStream_t);

// ---------------------------------------------------------------------------
// Elementwise kernels.
// ---------------------------------------------------------------------------
// y[v][c] = gamma[g(v)][c] * x[v][c] + beta[g(v)][c]  (gamma, beta [G][d]; null: identity)
template <typename TX>
__global__ void k_film_apply(const TX* x, int n, int d, const float* gamma, const float* beta, GraphTable gt,
                             float* y) {
  const size_t total = (size_t)n * d;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int v = (int)(i / d), c = (int)(i % d);
    float val = ld(x, i);
    if (gamma) {
      const int g = graph_of_node(gt, v);
      val = gamma[(size_t)g * d + c] * val + beta[(size_t)g * d + c];
    }
    y[i] = val;
  }
}
template <typename TX>
hipError_t launch_film_apply(const TX* x, int n, int d, const float* gamma, const float* beta, const GraphTable& gt,
                             float* y, hipStream_t s) {
  const size_t total = (size_t)n * d;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL((k_film_apply<TX>), dim3(blocks), dim3(256), 0, s, x, n, d, gamma, beta, gt, y);
  return hipGetLastError();
}
template hipError_t launch_film_apply<float>(const float*, int, int, const float*, const float*, const GraphTable&,
                                             float*, hipStream_t);
template hipError_t launch_film_apply<bf16>(const bf16*, int, int, const float*, const float*, const GraphTable&,
                                            float*, hipStream_t);

// Elementwise ops on n values: out = op(a, b, c).
__global__ void k_ew(int op, const float* a, const float* b, const float* c, size_t n, float* out) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    float r;
    switch (op) {
      case EW_ADD: r = a[i] + b[i]; break;                                 // a + b
      case EW_MASK_POS: r = b[i] > 0.f ? a[i] : 0.f; break;                // a where b > 0 (ReLU')
      case EW_SIGMOID_GRAD: r = a[i] * b[i] * (1.0f - b[i]); break;        // a * s (1 - s)
      case EW_SCALE_BY: r = a[i] * b[i]; break;                             // a * b
      default: r = 0.f;
    }
    out[i] = r;
  }
}
hipError_t launch_ew(int op, const float* a, const float* b, const float* c, size_t n, float* out, hipStream_t s) {
  const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_ew, dim3(std::max(1u, blocks)), dim3(256), 0, s, op, a, b, c, n, out);
  return hipGetLastError();
}

// dX[v][c] = gamma[g(v)][c] * dY[v][c]  (the input side of FiLM's backward)
__global__ void k_film_dx(const float* dy, int n, int d, const float* gamma, GraphTable gt, float* dx) {
  const size_t total = (size_t)n * d;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int v = (int)(i / d), c = (int)(i % d);
    const float gm = gamma ? gamma[(size_t)graph_of_node(gt, v) * d + c] : 1.0f;
    dx[i] = gm * dy[i];
  }
}
hipError_t launch_film_dx(const float* dy, int n, int d, const float* gamma, const GraphTable& gt, float* dx,
                          hipStream_t s) {
  const size_t total = (size_t)n * d;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_film_dx, dim3(blocks), dim3(256), 0, s, dy, n, d, gamma, gt, dx);
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

// x0[g][c] = mean over the rows of graph g: the graph's column sums (256-row
// chunks, then the chunks in order), divided by its node count.
__global__ void k_scale_rows_by_graph_size(float* x0, int H, GraphTable gt) {
  const int g = blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
  if (c < H) x0[(size_t)g * H + c] /= (float)(gt.ptr[g + 1] - gt.ptr[g]);
}
hipError_t launch_meanpool_f32(const float* h, int H, const GraphTable& chunks, int n_chunks, float* partial,
                               float* x0, hipStream_t s) {
  hipError_t e = launch_colsum<float>(h, H, nullptr, 0, H, chunks, n_chunks, partial, x0, H, false, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scale_rows_by_graph_size, dim3((H + 255) / 256, chunks.n), dim3(256), 0, s, x0, H, chunks);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Eq. 2's max-pool with the winning neighbour of every element (ties: the
// lowest node id), and its backward: dP[u][c] = sum over the neighbours v of u
// (out-edges in CSR order, then in-edges in ascending order) whose element c
// was won by u of dA[v][c].  u in S(v) implies v in N(u), so every v that
// selected u is visited.
// ---------------------------------------------------------------------------
__global__ void k_gather_max_arg(const float* P, const int* s_ptr, const int* s_idx, int n, int H, float* A,
                                 int* arg) {
  const size_t total = (size_t)n * H;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int v = (int)(i / H), c = (int)(i % H);
    float best = 0.f;
    int who = -1;
    for (int e = s_ptr[v]; e < s_ptr[v + 1]; ++e) {
      const int u = s_idx[e];
      const float p = P[(size_t)u * H + c];
      if (who < 0 || p > best || (p == best && u < who)) {
        best = p;
        who = u;
      }
    }
    A[i] = who < 0 ? 0.f : best;
    arg[i] = who;
  }
}
hipError_t launch_gather_max_arg(const float* P, const int* s_ptr, const int* s_idx, int n, int H, float* A, int* arg,
                                 hipStream_t s) {
  const size_t total = (size_t)n * H;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_gather_max_arg, dim3(blocks), dim3(256), 0, s, P, s_ptr, s_idx, n, H, A, arg);
  return hipGetLastError();
}

__global__ void k_gather_max_bwd(const float* dA, const int* arg, const int* row_ptr, const int* col_idx,
                                 const int* in_ptr, const int* in_idx, int n, int H, float* dP) {
  const size_t total = (size_t)n * H;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int u = (int)(i / H), c = (int)(i % H);
    float s = 0.f;
    for (int e = row_ptr[u]; e < row_ptr[u + 1]; ++e) {
      const int v = col_idx[e];
      if (arg[(size_t)v * H + c] == u) s += dA[(size_t)v * H + c];
    }
    for (int e = in_ptr[u]; e < in_ptr[u + 1]; ++e) {
      const int v = in_idx[e];
      if (arg[(size_t)v * H + c] == u) s += dA[(size_t)v * H + c];
    }
    dP[i] = s;
  }
}
hipError_t launch_gather_max_bwd(const float* dA, const int* arg, const int* row_ptr, const int* col_idx,
                                 const int* in_ptr, const int* in_idx, int n, int H, float* dP, hipStream_t s) {
  const size_t total = (size_t)n * H;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_gather_max_bwd, dim3(blocks), dim3(256), 0, s, dA, arg, row_ptr, col_idx, in_ptr, in_idx, n, H,
                     dP);
  return hipGetLastError();
}

// Sorts each in-edge row ascending (rows filled by atomics come in any order),
// so the backward's sums run in a fixed order.  Insertion sort per row.
__global__ void k_sort_rows(const int* ptr, int n, int* idx) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int a = ptr[v], b = ptr[v + 1];
  for (int i = a + 1; i < b; ++i) {
    const int x = idx[i];
    int j = i - 1;
    while (j >= a && idx[j] > x) {
      idx[j + 1] = idx[j];
      --j;
    }
    idx[j + 1] = x;
  }
}
hipError_t launch_sort_rows(const int* ptr, int n, int* idx, hipStream_t s) {
  hipLaunchKernelGGL(k_sort_rows, dim3((n + 255) / 256), dim3(256), 0, s, ptr, n, idx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adam (Kingma and Ba, 2015) on one parameter tensor: fp32 master weights and
// moments; the dtype copy the kernels read is rewritten from the master.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_adam(float* master, T* param, const float* grad, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float g = grad[i];
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float w = master[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    master[i] = w;
    param[i] = from_f32<T>(w);
  }
}
template <typename T>
hipError_t launch_adam(float* master, T* param, const float* grad, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, float c1, float c2, hipStream_t s) {
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL((k_adam<T>), dim3(std::max(1u, blocks)), dim3(256), 0, s, master, param, grad, m, v, n, lr, b1,
                     b2, eps, c1, c2);
  return hipGetLastError();
}
template hipError_t launch_adam<float>(float*, float*, const float*, float*, float*, int64_t, float, float, float,
                                       float, float, float, hipStream_t);
template hipError_t launch_adam<bf16>(float*, bf16*, const float*, float*, float*, int64_t, float, float, float,
                                      float, float, float, hipStream_t);

}  // namespace tr
}  // namespace gdp

// Launch interface of the update-step kernels: the training forward that keeps
// every intermediate, the backward pass and Adam.  train_gemm.hip (dense products)
// and train_attn.hip (attention) compute in fp32 accuracy on the bf16 matrix cores,
// train.hip (everything else) in fp32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"
#include "kernels.h"

namespace gdp {
namespace tr {

enum Act { ACT_NONE = 0, ACT_RELU = 1, ACT_SIGMOID = 2 };

// C(m, n) = epi(sum_k A(m, k) B(k, n)) with A(m, k) = a[m sam + k sak] and
// B(k, n) = b[k sbk + n sbn]; epi adds a bias over n (fp32 or bf16), applies
// act, zeroes where mask[m ldm + n] <= 0, adds res[m ldr + n], and writes or
// adds to c (c may be res, not the operands).
template <typename TA, typename TB>
struct GemmStrided {
  const TA* a;
  long sam, sak;
  const TB* b;
  long sbk, sbn;
  int M, N, K;
  float* c;
  long ldc;
  const float* bias_f = nullptr;
  const bf16* bias_h = nullptr;
  int act = ACT_NONE;
  const float* mask = nullptr;
  long ldm = 0;
  const float* res = nullptr;
  long ldr = 0;
  bool accumulate = false;
  float* rowsum = nullptr;   // weight gradients (a slow in k): out, [M], sum_k A(m, k)
};
// partial: scratch for split-k sums (partial_floats floats; null: no split).
template <typename TA, typename TB>
hipError_t launch_gemm_strided(const GemmStrided<TA, TB>& g, float* partial, size_t partial_floats, hipStream_t s);

// Row-wise kernels take widths of 64, 128 or 256.  Per-graph column sums run over
// kColChunkRows-row chunks (ct: the graphs and those chunks), added up in order.
constexpr int kColChunkRows = 64;

template <typename T>
hipError_t launch_ln_fwd(const float* r, int n, int d, const T* g, const T* b, float* out, hipStream_t s);
// LayerNorm backward: dr, and the gain's and shift's gradients.  rows: all rows
// as one graph; partial: chunks * 2 d floats.
template <typename T>
hipError_t launch_ln_bwd(const float* r, const float* dout, int d, const T* g, const GraphTable& rows, int chunks,
                         float* dr, float* dg, float* db, float* partial, hipStream_t s);

hipError_t launch_film_apply(const float* x, int n, int d, const float* gamma, const float* beta, const GraphTable& gt,
                             float* y, hipStream_t s);
// FiLM backward: dx = gamma dy, dgamma[g] = sum over graph g of dy x, dbeta[g] =
// sum of dy.  partial: chunks * 2 d floats.
hipError_t launch_film_bwd(const float* dy, const float* x, int d, const float* gamma, const GraphTable& ct, int chunks,
                           float* dx, float* dgamma, float* dbeta, float* partial, hipStream_t s);
// The FiLM weights' gradients of every layer and the graph embeddings' gradient
// dx0 [G, H], from dfilm ([L][2][G][d]: dgamma, then dbeta).
struct FilmWeightGrads {
  float* wg[kFilmLayersPerLaunch];
  float* bg[kFilmLayersPerLaunch];
  float* wb[kFilmLayersPerLaunch];
  float* bb[kFilmLayersPerLaunch];
};
template <typename T>
hipError_t launch_film_weights_bwd(const FilmLayers<T>& w, const FilmWeightGrads& gr, int layers, const float* dfilm,
                                   const float* x0, int G, int d, int H, float* dx0, hipStream_t s);

// out = a where b > 0, else 0 (ReLU').
hipError_t launch_mask_pos(const float* a, const float* b, size_t n, float* out, hipStream_t s);

// x0[g] = mean of graph g's rows of h; partial: chunks * H floats.
hipError_t launch_meanpool_f32(const float* h, int H, const GraphTable& ct, int chunks, float* partial, float* x0,
                               hipStream_t s);
hipError_t launch_meanpool_bwd(const float* dx0, int n, int H, const GraphTable& gt, float* dh, hipStream_t s);

hipError_t launch_gather_max_arg(const float* P, const int* s_ptr, const int* s_idx, int n, int H, float* A, int* arg,
                                 hipStream_t s);
// dZ = (the max-pool's backward of dA) P (1 - P): the gradient before the sigmoid.
hipError_t launch_gather_max_bwd(const float* dA, const int* arg, const int* row_ptr, const int* col_idx,
                                 const int* in_ptr, const int* in_idx, const float* P, int n, int H, float* dZ,
                                 hipStream_t s);
hipError_t launch_sort_rows(const int* ptr, int n, int* idx, hipStream_t s);

// qkv [n, 3d] fp32; o [n, d]; lse [n, heads] in log2 units.
hipError_t launch_attn_fwd(const float* qkv, int n, int d, int heads, int seg, int mem, const GraphTable& gt,
                           float* o, float* lse, hipStream_t s);
// dqkv_live [n, 3d]: dQ and the own-segment dK, dV; dkv_all [n, 2d]: those dK,
// dV plus what later segments' queries send to the row as memory; Dq [n, heads] scratch.
hipError_t launch_attn_bwd(const float* qkv, const float* O, const float* dO, const float* lse, int n, int d,
                           int heads, int seg, int mem, const GraphTable& gt, float* Dq, float* dqkv_live,
                           float* dkv_all, hipStream_t s);

// Adam on up to kAdamTensors tensors in one launch.
constexpr int kAdamTensors = 64;
hipError_t launch_adam(const gdp_adam_tensor* t, int n_tensors, bool to_bf16, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t s);

}  // namespace tr
}  // namespace gdp

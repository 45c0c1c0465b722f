// Dense surrogate BPTT of one layer -- the "Original" column of Table 1 -- on the matrix cores.
//
//   gate+delta  one thread per (b,j) walks t downward: G = eps * g(V) * 1[band] (or eps for the
//               readout), delta[t-1] = alpha delta[t] + G[t]; writes G and delta densely.
//   grad_in     [T*B, N_in] = delta [T*B, N_out] . W^T      (GEMM, both operands K-contiguous)
//   dW          [N_in, N_out] = trace^T [N_in, T*B] . G     (GEMM, K = T*B, split over K)
// Both products take float32 operands in three bf16 parts (gemm.hip): at 128000 rows x 1024 x 1024 1.52 ms
// each (176 TFLOP/s), where float32 MFMA tiles took 3.4 (dW) and 2.5 ms (grad_in); the dense backward of
// three such layers 17.2 -> 9.15 ms.
#include "common.h"

namespace snn {
namespace {

__device__ __forceinline__ float gate(float e, float v, float theta, float bth, float beta, bool readout) {
  if (readout) return e;
  const float d = fabsf(v - theta);
  if (!(d < bth)) return 0.0f;
  const float x = beta * d + 1.0f;
  return e / (x * x);
}

__global__ __launch_bounds__(256) void dense_gate_delta(const float* __restrict__ eps, const float* __restrict__ V,
                                                        int T, size_t BN_, float alpha, float theta, float bth,
                                                        float beta, int readout, float* __restrict__ Gd,
                                                        float* __restrict__ Dd) {
  const size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (k >= BN_) return;
  const bool ro = readout != 0;
  float d = 0.0f;
  Dd[(size_t)(T - 1) * BN_ + k] = 0.0f;
  constexpr int U = 4;
  int t = T - 1;
  for (; t >= U - 1; t -= U) {  // independent loads of U steps in flight
    float e[U], v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t o = (size_t)(t - u) * BN_ + k;
      e[u] = eps[o];
      v[u] = ro ? 0.0f : V[o];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tt = t - u;
      const float G = gate(e[u], v[u], theta, bth, beta, ro);
      Gd[(size_t)tt * BN_ + k] = G;
      if (tt > 0) {
        d = alpha * d + G;
        Dd[(size_t)(tt - 1) * BN_ + k] = d;
      }
    }
  }
  for (; t >= 0; --t) {
    const size_t o = (size_t)t * BN_ + k;
    const float G = gate(eps[o], ro ? 0.0f : V[o], theta, bth, beta, ro);
    Gd[o] = G;
    if (t > 0) {
      d = alpha * d + G;
      Dd[(size_t)(t - 1) * BN_ + k] = d;
    }
  }
}

__global__ void reduce_splits(const float* __restrict__ part, int n_split, size_t n, float* __restrict__ out) {
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    double s = 0.0;  // fixed order, rounded once
    for (int c = 0; c < n_split; ++c) s += (double)part[(size_t)c * n + k];
    out[k] = (float)s;
  }
}

// K slices of the dW product (88e12 multiply-adds a second at 1024 x 1024 x 128000).
int dw_splits(int TB, int N_in, int N_out) { return plan_splits(N_in, N_out, TB, 88e12).splits; }

}  // namespace
}  // namespace snn

using namespace snn;

extern "C" size_t snn_dense_backward_workspace(int T, int B, int N_in, int N_out) {
  if (bad_dim(T) || bad_dim(B) || bad_dim(N_in) || bad_dim(N_out)) return 0;
  if (too_big(T, B, N_in) || too_big(T, B, N_out)) return 0;
  const size_t TB = (size_t)T * B;
  Carve c(nullptr);
  c.take<float>(TB * N_out);  // G
  c.take<float>(TB * N_out);  // delta
  const int sp = dw_splits(T * B, N_in, N_out);
  if (sp > 1) c.take<float>((size_t)sp * N_in * N_out);
  return c.off;
}

extern "C" snn_status snn_dense_backward_ref(const float* W, const float* trace_in, const float* V,
                                             const float* eps_out, int T, int B, int N_in, int N_out, float alpha,
                                             float theta, float b_th, float beta, float* grad_in, float* dW,
                                             void* workspace, size_t workspace_bytes, void* stream) {
  if (!W || !trace_in || !eps_out || !dW || !workspace) return SNN_ERR_INVALID_ARG;
  if (bad_dim(T) || bad_dim(B) || bad_dim(N_in) || bad_dim(N_out)) return SNN_ERR_INVALID_ARG;
  if (too_big(T, B, N_in) || too_big(T, B, N_out)) return SNN_ERR_INVALID_ARG;
  if (bad_alpha(alpha) || isnan(theta) || isnan(b_th) || b_th < 0.0f || isnan(beta) || beta < 0.0f)
    return SNN_ERR_INVALID_ARG;
  const bool readout = isinf(theta) && theta > 0.0f;
  if (!readout && !V) return SNN_ERR_INVALID_ARG;
  if (workspace_bytes < snn_dense_backward_workspace(T, B, N_in, N_out)) return SNN_ERR_INVALID_ARG;

  hipStream_t s = static_cast<hipStream_t>(stream);
  const int TB = T * B;
  Carve ws(workspace);
  float* Gd = ws.take<float>((size_t)TB * N_out);
  float* Dd = ws.take<float>((size_t)TB * N_out);
  const int sp = dw_splits(TB, N_in, N_out);
  float* part = sp > 1 ? ws.take<float>((size_t)sp * N_in * N_out) : dW;

  const size_t BN_ = (size_t)B * N_out;
  hipLaunchKernelGGL(dense_gate_delta, dim3((unsigned)((BN_ + 255) / 256)), dim3(256), 0, s, eps_out, V, T, BN_,
                     alpha, theta, b_th, beta, readout ? 1 : 0, Gd, Dd);
  // dW[i][j] = sum_r trace[r][i] G[r][j]
  gemm_split_km(N_in, N_out, TB, trace_in, N_in, Gd, N_out, part, N_out, sp, (size_t)N_in * N_out, s);
  if (sp > 1) {
    const size_t n = (size_t)N_in * N_out;
    hipLaunchKernelGGL(reduce_splits, dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                       part, sp, n, dW);
  }
  if (grad_in)  // grad_in[r][i] = sum_j delta[r][j] W[i][j]
    gemm_split_kc(TB, N_in, N_out, Dd, N_out, W, N_out, grad_in, N_in, s);
  return launch_status();
}

// Readout cross-entropy (App. E) and the CSR of the entries the loss reads, so that the
// readout's backward runs through snn_sparse_backward like any other layer. The readout is
// the infinite-threshold LIF layer of Sec. 3; its derivative factor is 1.
//   mode 0: a[b,c] = max_t V_out[t,b,c] (first maximal t), entries = the arg-max positions
//   mode 1: a[b,c] = sum_t V_out[t,b,c], entries = every (t,b,c)
// eps = dL/da = (softmax(a) - onehot(label)) / B at each entry; loss = mean -log p[b,label].
//
// Two kernels: ce_sample (one block per sample: logits, softmax, per-sample loss, dL/da, and in mode
// 0 the sample's entries sorted by (arg-max step, class) with their running count per step) and
// ce_rows (mode 0: row pointers and entries of four time steps per block) or ce_fill_sum (mode 1).
// Both are bound by latency: V_out is 1 to 51 MB. The time axis of a sample is therefore spread over
// the block (one thread per (time residue, class), eight loads in flight) instead of one thread
// walking all T steps of a class, and the CSR needs no scan over T*B row counts: row (t, b) starts
// at sum_b' cum[b'][t] + sum_{b' < b} (cum[b'][t+1] - cum[b'][t]), cum[b][t] = classes of sample b
// whose arg-max step is before t. Against eight kernels with a thread per class walking time (29 us
// at T = 100, C = 10; 113 at T = 300, C = 10; 200 at T = 500, C = 100; a one-thread mean of 12 us):
// a 784 -> 200 -> 10 training step 262 -> 217 us, a 2312 -> 200 -> 10 backward at T = 300 1.750 ->
// 1.626 ms, the 3 x 1024 backward at T = 500, C = 100 2.34 -> 2.14 ms.
#include "common.h"

#include <climits>

namespace snn {
namespace {

constexpr int kThreads = 256;

// Running maximum over time of the strict comparison v > best from t = 0 on: the first maximal t.
// Partial maxima merge by (larger value, then earlier t); a NaN never wins a comparison.
__device__ __forceinline__ void max_merge(float& v, int& t, float v2, int t2) {
  if (v2 > v || (v2 == v && t2 < t)) {
    v = v2;
    t = t2;
  }
}

// Classes up to which a thread counts the entries before its own; with more, the sample's keys are sorted (two counts
// of C steps each took 188 us a call with 1000 classes and 21 ms with 16384, one sample; sorted 27 and 243 us).
constexpr int kRankMax = 128;

__host__ __device__ inline int sort_slots(int C) {
  if (C <= kRankMax) return C;
  int n = 2 * kRankMax;
  while (n < C) n <<= 1;
  return n;
}

// One block per sample b. Thread (tg, c) takes steps tg, tg + TG, ... of class c (classes past the
// block's width in further rounds); the TG partial results of a class meet in LDS.
template <int NT>
__global__ __launch_bounds__(NT) void ce_sample(const float* __restrict__ V, const int32_t* __restrict__ labels,
                                                int T, int B, int C, int mode, int32_t* __restrict__ tstar,
                                                float* __restrict__ dlda, float* __restrict__ loss_b,
                                                int32_t* __restrict__ cum, int32_t* __restrict__ sorted_c,
                                                float* __restrict__ sorted_d) {
  extern __shared__ float a[];                   // [C] logits
  int* ts = reinterpret_cast<int*>(a + C);       // arg-max steps [C]; then the sorted keys [sort_slots(C)]
  __shared__ __attribute__((aligned(8))) char part_raw[NT * 8];
  __shared__ float red[NT / kWave];
  float* pv = reinterpret_cast<float*>(part_raw);
  int* pt = reinterpret_cast<int*>(part_raw) + NT;
  double* pd = reinterpret_cast<double*>(part_raw);
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int w = tid / kWave;
  const int l = tid % kWave;
  const size_t step = (size_t)B * C;
  const int Cw = min(C, NT);  // classes of a round
  const int TG = NT / Cw;
  const int tg = tid / Cw;
  constexpr int kAhead = 8;
  for (int c0 = 0; c0 < C; c0 += Cw) {
    const int c = c0 + tid - tg * Cw;
    const bool on = tg < TG && c < C;
    const float* src = V + (size_t)b * C + (on ? c : 0);
    float best = -INFINITY;
    int bt = INT_MAX;
    double sum = 0.0;  // the logit of a sum over time, rounded once
    if (on) {
      for (int t0 = tg; t0 < T; t0 += kAhead * TG) {
        float v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = src[(size_t)min(t0 + u * TG, T - 1) * step];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int t = t0 + u * TG;
          if (t < T) {
            if (mode == 0) {
              if (v[u] > best) {
                best = v[u];
                bt = t;
              }
            } else {
              sum += (double)v[u];
            }
          }
        }
      }
    }
    if (mode == 0) {
      pv[tid] = best;
      pt[tid] = bt;
    } else {
      pd[tid] = sum;
    }
    __syncthreads();
    int half = 1;
    while (half < TG) half <<= 1;
    for (half >>= 1; half > 0; half >>= 1) {
      if (tg < half && tg + half < TG) {
        const int o = tid + half * Cw;
        if (mode == 0) {
          max_merge(best, bt, pv[o], pt[o]);
          pv[tid] = best;
          pt[tid] = bt;
        } else {
          sum += pd[o];
          pd[tid] = sum;
        }
      }
      __syncthreads();
    }
    if (on && tg == 0) {
      if (mode == 0) {
        const float v0 = src[0];
        if (isnan(v0) || bt == INT_MAX) {  // step 0 is the start of the comparison, whatever it holds
          best = v0;
          bt = 0;
        }
        a[c] = best;
        ts[c] = bt;
        tstar[(size_t)b * C + c] = bt;
      } else {
        a[c] = (float)sum;
      }
    }
    __syncthreads();
  }
  // max over classes, then the softmax's sum
  auto block_all = [&](float x, bool is_max) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const float o = __shfl_xor(x, off, kWave);
      x = is_max ? fmaxf(x, o) : x + o;
    }
    if (l == 0) red[w] = x;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int k = 1; k < NT / kWave; ++k) r = is_max ? fmaxf(r, red[k]) : r + red[k];
    __syncthreads();
    return r;
  };
  float m = -INFINITY;
  for (int c = tid; c < C; c += NT) m = fmaxf(m, a[c]);
  const float amax = block_all(m, true);
  float s = 0.0f;
  for (int c = tid; c < C; c += NT) s += expf(a[c] - amax);
  const float Z = block_all(s, false);
  const int y = labels[b];
  const bool ok = y >= 0 && y < C;
  const float invB = 1.0f / (float)B;
  if (tid == 0) loss_b[b] = ok ? (logf(Z) - (a[y] - amax)) : NAN;
  const auto grad = [&](int c) {
    const float p = expf(a[c] - amax) / Z;
    return (p - (c == y ? 1.0f : 0.0f)) * invB;
  };
  for (int c = tid; c < C; c += NT) dlda[(size_t)b * C + c] = grad(c);
  if (mode != 0) return;
  // the sample's entries by step, then class: keys step * C + class (below T * C < 2^31) in order
  if (C > kRankMax) {
    int* key = ts;
    for (int c = tid; c < C; c += NT) key[c] += (C - 1) * key[c] + c;
    const int n = sort_slots(C);
    for (int k = C + tid; k < n; k += NT) key[k] = INT_MAX;
    __syncthreads();
    for (int run = 2; run <= n; run <<= 1)  // bitonic
      for (int j = run >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < n / 2; i += NT) {
          const int lo = 2 * j * (i / j) + i % j;
          const int u = key[lo], v = key[lo + j];
          if ((u > v) == ((lo & run) == 0)) {
            key[lo] = v;
            key[lo + j] = u;
          }
        }
        __syncthreads();
      }
    for (int k = tid; k < C; k += NT) {
      const int c = key[k] % C;
      sorted_c[(size_t)b * C + k] = c;
      sorted_d[(size_t)b * C + k] = grad(c);
    }
  } else {
    int pos = 0, t = 0;
    if (tid < C) {  // C <= kRankMax <= NT
      t = ts[tid];
      for (int k = 0; k < C; ++k) pos += ts[k] < t || (ts[k] == t && k < tid);
      sorted_c[(size_t)b * C + pos] = tid;
      sorted_d[(size_t)b * C + pos] = grad(tid);
    }
    __syncthreads();
    if (tid < C) ts[pos] = t * C + tid;
    __syncthreads();
  }
  for (int t = tid; t <= T; t += NT) {  // classes with an arg-max step before t
    int lo = 0, hi = C;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (ts[mid] < t * C) lo = mid + 1; else hi = mid;
    }
    cum[(size_t)b * (T + 1) + t] = lo;
  }
}

// Mean of the per-sample losses by one wavefront (float64, fixed order).
__device__ __forceinline__ void mean_loss(const float* __restrict__ loss_b, int B, float* __restrict__ loss) {
  double s = 0.0;
  for (int b = lane_id(); b < B; b += kWave) s += (double)loss_b[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
  if (lane_id() == 0) *loss = (float)(s / (double)B);
}

// Row pointers and entries of kRowSteps time steps per block, one thread per sample (mode 0). ALONG (a row holds one
// entry and more on average): a step's entries of 256 samples are contiguous and the block copies them a thread per
// entry, which finds its sample by bisection, in gridDim.y shares.
constexpr int kRowSteps = 4;

template <bool ALONG>
__global__ __launch_bounds__(kThreads) void ce_rows(const int32_t* __restrict__ cum,
                                                    const int32_t* __restrict__ sorted_c,
                                                    const float* __restrict__ sorted_d,
                                                    const float* __restrict__ loss_b, int T, int B, int C,
                                                    int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
                                                    float* __restrict__ eps, float* __restrict__ loss) {
  __shared__ int red[kRowSteps][kThreads / kWave];
  __shared__ int first[ALONG ? kThreads : 1], from[ALONG ? kThreads : 1];
  const int tid = threadIdx.x;
  const int w = tid / kWave;
  const int l = tid % kWave;
  const int t0 = blockIdx.x * kRowSteps;
  auto load = [&](int b, int (&x)[kRowSteps + 1]) {
#pragma unroll
    for (int q = 0; q <= kRowSteps; ++q) x[q] = b < B ? cum[(size_t)b * (T + 1) + min(t0 + q, T)] : 0;
  };
  // entries of all samples before each step
  int base[kRowSteps] = {};
  for (int b = tid; b < B; b += kThreads) {
    int x[kRowSteps + 1];
    load(b, x);
#pragma unroll
    for (int q = 0; q < kRowSteps; ++q) base[q] += x[q];
  }
#pragma unroll
  for (int q = 0; q < kRowSteps; ++q) {
    base[q] = wave_sum_int(base[q]);
    if (l == 0) red[q][w] = base[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kRowSteps; ++q) {
    base[q] = 0;
    for (int k = 0; k < kThreads / kWave; ++k) base[q] += red[q][k];
  }
  for (int b0 = 0; b0 < B; b0 += kThreads) {
    const int b = b0 + tid;
    int x[kRowSteps + 1], ex[kRowSteps];
    load(b, x);
    __syncthreads();  // red is rewritten
#pragma unroll
    for (int q = 0; q < kRowSteps; ++q) {
      const int n = x[q + 1] - x[q];
      const int incl = wave_incl_scan(n);
      ex[q] = incl - n;
      if (l == kWave - 1) red[q][w] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRowSteps; ++q) {
      int before = 0, all = 0;
      for (int k = 0; k < kThreads / kWave; ++k) {
        before += k < w ? red[q][k] : 0;
        all += red[q][k];
      }
      const int row = base[q] + before + ex[q];
      const int begin = base[q];
      base[q] += all;
      if (ALONG) {
        if (b < B && t0 + q < T && blockIdx.y == 0) row_ptr[(size_t)(t0 + q) * B + b] = row;
        __syncthreads();  // first and from are rewritten
        first[tid] = row;
        from[tid] = x[q];
        __syncthreads();
        for (uint32_t u = begin + blockIdx.y * kThreads + tid; u < (uint32_t)(begin + all); u += gridDim.y * kThreads) {
          const int e = (int)u;  // (unsigned steps: the last may pass 2^31)
          int lo = 0, hi = kThreads - 1;  // the last sample that starts at or before e
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first[mid] <= e) lo = mid; else hi = mid - 1;
          }
          const size_t k = (size_t)(b0 + lo) * C + from[lo] + (e - first[lo]);
          col_idx[e] = sorted_c[k];
          eps[e] = sorted_d[k];
        }
      } else if (b < B && t0 + q < T) {
        row_ptr[(size_t)(t0 + q) * B + b] = row;
        for (int k = x[q]; k < x[q + 1]; ++k) {
          col_idx[row + k - x[q]] = sorted_c[(size_t)b * C + k];
          eps[row + k - x[q]] = sorted_d[(size_t)b * C + k];
        }
      }
    }
  }
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    if (tid == 0) row_ptr[(size_t)T * B] = B * C;
    if (w == 0) mean_loss(loss_b, B, loss);
  }
}

__global__ void ce_fill_sum(const float* __restrict__ dlda, const float* __restrict__ loss_b, int T, int B, int C,
                            int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx, float* __restrict__ eps,
                            float* __restrict__ loss) {
  const size_t n = (size_t)T * B * C;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const size_t r = k / C;
    const int c = (int)(k - r * C);
    const int b = (int)(r % B);
    col_idx[k] = c;
    eps[k] = dlda[(size_t)b * C + c];
    if (c == 0) row_ptr[r] = (int32_t)k;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) row_ptr[(size_t)T * B] = (int32_t)n;
    if (threadIdx.x < kWave) mean_loss(loss_b, B, loss);
  }
}

// dL/dV_out densely: dL/da at the arg-max time (mode 0) or at every t (mode 1), 0 elsewhere.
__global__ void ce_dense(const int32_t* __restrict__ tstar, const float* __restrict__ dlda, int T, int B, int C,
                         int mode, float* __restrict__ out) {
  const size_t n = (size_t)T * B * C;
  const size_t BC = (size_t)B * C;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const int t = (int)(k / BC);
    const size_t bc = k - (size_t)t * BC;
    out[k] = (mode == 1 || tstar[bc] == t) ? dlda[bc] : 0.0f;
  }
}

}  // namespace
}  // namespace snn

using namespace snn;

extern "C" size_t snn_readout_ce_workspace(int T, int B, int C, int mode) {
  if (bad_dim(T) || bad_dim(B) || bad_dim(C) || too_big(T, B, C) || (mode != 0 && mode != 1)) return 0;
  Carve c(nullptr);
  c.take<int32_t>((size_t)B * C);  // tstar
  c.take<float>((size_t)B * C);    // dL/da
  c.take<float>((size_t)B);        // per-sample loss
  if (mode == 0) {
    c.take<int32_t>((size_t)B * (T + 1));  // entries before each step, per sample
    c.take<int32_t>((size_t)B * C);        // classes in entry order
    c.take<float>((size_t)B * C);          // their dL/da
  }
  return c.off;
}

extern "C" snn_status snn_readout_ce(const float* V_out, const int32_t* labels, int T, int B, int C, int mode,
                                     int32_t* row_ptr, int32_t* col_idx, float* eps, float* loss,
                                     float* eps_dense, void* workspace, size_t workspace_bytes, void* stream) {
  if (!V_out || !labels || !row_ptr || !col_idx || !eps || !loss || !workspace) return SNN_ERR_INVALID_ARG;
  if (bad_dim(T) || bad_dim(B) || bad_dim(C) || too_big(T, B, C)) return SNN_ERR_INVALID_ARG;
  if (mode != 0 && mode != 1) return SNN_ERR_INVALID_ARG;
  if (workspace_bytes < snn_readout_ce_workspace(T, B, C, mode)) return SNN_ERR_INVALID_ARG;
  if ((size_t)C * sizeof(float) > 64 * 1024) return SNN_ERR_UNSUPPORTED;

  hipStream_t s = static_cast<hipStream_t>(stream);
  Carve ws(workspace);
  int32_t* tstar = ws.take<int32_t>((size_t)B * C);
  float* dlda = ws.take<float>((size_t)B * C);
  float* loss_b = ws.take<float>((size_t)B);
  int32_t* cum = nullptr;
  int32_t* sorted_c = nullptr;
  float* sorted_d = nullptr;
  if (mode == 0) {
    cum = ws.take<int32_t>((size_t)B * (T + 1));
    sorted_c = ws.take<int32_t>((size_t)B * C);
    sorted_d = ws.take<float>((size_t)B * C);
  }
  // 1024 threads per sample where a sample holds enough values for them
  const size_t lds = (size_t)C * sizeof(float) + (size_t)sort_slots(C) * sizeof(int);
  if ((int64_t)T * C >= 8192 || C > kThreads) {
    ensure_dynamic_lds((const void*)ce_sample<1024>, (int)lds);
    hipLaunchKernelGGL(ce_sample<1024>, dim3(B), dim3(1024), lds, s, V_out, labels, T, B, C, mode, tstar, dlda, loss_b,
                       cum, sorted_c, sorted_d);
  } else {
    hipLaunchKernelGGL(ce_sample<kThreads>, dim3(B), dim3(kThreads), lds, s, V_out, labels, T, B, C, mode, tstar, dlda,
                       loss_b, cum, sorted_c, sorted_d);
  }
  if (mode == 0) {
    const unsigned tb = (unsigned)((T + kRowSteps - 1) / kRowSteps);
    if (C >= T) {
      const unsigned shares = (unsigned)std::min<int64_t>(64, ((int64_t)B * C / tb + 16383) / 16384);
      hipLaunchKernelGGL(ce_rows<true>, dim3(tb, shares), dim3(kThreads), 0, s, cum, sorted_c, sorted_d, loss_b, T, B, C,
                         row_ptr, col_idx, eps, loss);
    } else {
      hipLaunchKernelGGL(ce_rows<false>, dim3(tb), dim3(kThreads), 0, s, cum, sorted_c, sorted_d, loss_b, T, B, C,
                         row_ptr, col_idx, eps, loss);
    }
  } else {
    const size_t n = (size_t)T * B * C;
    hipLaunchKernelGGL(ce_fill_sum, dim3((unsigned)std::min<size_t>((n + 255) / 256, 8192)), dim3(256), 0, s, dlda,
                       loss_b, T, B, C, row_ptr, col_idx, eps, loss);
  }
  if (eps_dense) {
    const size_t n = (size_t)T * B * C;
    hipLaunchKernelGGL(ce_dense, dim3((unsigned)std::min<size_t>((n + 255) / 256, 8192)), dim3(256), 0, s, tstar,
                       dlda, T, B, C, mode, eps_dense);
  }
  return launch_status();
}

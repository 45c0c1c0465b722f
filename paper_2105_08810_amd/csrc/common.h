// Shared host/device helpers of libsnn (internal header).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/snn.h"

namespace snn {

constexpr int kWave = 64;  // CDNA4 wavefront width

// ------------------------------------------------------------------ host-side checks

inline bool bad_dim(int x) { return x <= 0; }

// Element count of a [T,B,N] tensor must stay below 2^31 (int32 CSR offsets and indexing).
inline bool too_big(int T, int B, int N) {
  return (int64_t)T * (int64_t)B * (int64_t)N >= ((int64_t)1 << 31);
}

inline bool bad_alpha(float a) { return !(a > 0.0f && a <= 1.0f); }  // also rejects NaN

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline snn_status launch_status() {
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SNN_OK : SNN_ERR_HIP;
}

// Bump allocator over the caller's workspace.
struct Carve {
  char* base;
  size_t off = 0;
  explicit Carve(void* p) : base(static_cast<char*>(p)) {}
  template <class T>
  T* take(size_t n) {
    T* p = reinterpret_cast<T*>(base ? base + off : nullptr);
    off += align256(n * sizeof(T));
    return p;
  }
};

// Number of compute units of the current device (cached per process and device).
int cu_count();

// Raises a kernel's dynamic-LDS limit on the current device to at least `bytes`. The attribute
// is set once per device, kernel and size and remembered (thread-safe); later calls only look up.
void ensure_dynamic_lds(const void* kernel, int bytes);

// Sparse dW on the matrix cores (dw_mfma.hip), for 512 <= N_out <= 1024, N_in % 4 == 0 and at most
// 10% of the entries active.
struct MdwPlan {
  int n_win, n_itiles, n_chunks, wpc;  // windows of rows, input tiles, chunks of windows, windows per chunk
};
bool mdw_eligible(int T, int B, int N_in, int N_out, int64_t out_cap);
MdwPlan plan_mdw(int T, int B, int N_in, int N_out);
size_t mdw_workspace(int T, int B, int N_in, int N_out, int64_t out_cap);
// Structure-only part: sorts each window's entries by column quad into the workspace.
void mdw_enqueue_layout(int T, int B, int N_in, int N_out, const int32_t* out_row_ptr, const int32_t* out_col_idx,
                        int64_t out_cap, void* workspace, hipStream_t s);
// The rest (needs eps): G into the sorted entries, the accumulation, the chunk reduction into dW.
void mdw_enqueue_rest(const float* trace_in, int T, int B, int N_in, int N_out, const float* out_g, const float* eps_out,
                      int64_t out_cap, float* dW, void* workspace, hipStream_t s);

// Device-side choice between several ways to do a call's work, all enqueued: a kernel with a gate runs iff the
// CSR holds at least `least` and fewer than `under` entries. end NULL: it always runs. The entry arrays'
// allocated length is only an upper bound of the entries, and reading the count back would wait for the GPU.
struct Gate {
  const int32_t* end = nullptr;  // row_ptr[T * B]
  int64_t cap = 0;               // allocated entries
  int64_t least = 0;
  int64_t under = INT64_MAX;
};

__device__ __forceinline__ bool gate_open(const Gate& g) {
  if (!g.end) return true;
  int64_t n = *g.end;
  n = n < 0 ? 0 : (n > g.cap ? g.cap : n);  // malformed too: one way always runs
  return n >= g.least && n < g.under;
}

// Sparse dW by columns of row windows (dw_columns.hip): partial dW of n_chunks chunks (one chunk: dW itself).
struct ColsParts {
  float* part;
  int n_chunks;
};
bool cols_fits(int N_out);
void cols_seconds(int T, int B, int N_in, int N_out, double* fixed, double* per_entry);
size_t cols_workspace(int T, int B, int N_in, int N_out, int64_t out_cap);
ColsParts cols_enqueue(const float* trace_in, int T, int B, int N_in, int N_out, const int32_t* out_row_ptr,
                       const int32_t* out_col_idx, const float* out_g, const float* eps_out, int64_t out_cap, float* dW,
                       void* workspace, const Gate& gate, hipStream_t s);

// Dense float32 products (gemm.hip). K slice z of `splits` goes to C + z * c_split.
//   gemm_split_km  C = sum_k A[k, m] B[k, n], operands in three bf16 parts, float32 sums
//   gemm_split_kc  C = sum_k A[m, k] B[n, k], the same
//   gemm_f64_km    C = sum_k A[k, m] B[k, n], products and sums in float64
// plan_splits: the K slices of a km product whose whole rounds of blocks run at mac_rate multiply-adds a second,
// and the time this should take with the partials' sum.
struct SplitPlan {
  int splits;
  double seconds;
};
SplitPlan plan_splits(int M, int N, int K, double mac_rate);
void gemm_split_km(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc, int splits,
                   size_t c_split, hipStream_t s);
void gemm_split_kc(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc,
                   hipStream_t s);
// The elements (r, col_idx[e]) of C, as gemm_split_kc forms it, at the entries e < cap of a CSR over C's
// rows: out[e] (0 for a column outside [0, N)). What is not an entry is not written.
struct GatherOut {
  const int32_t* row_ptr = nullptr;  // [M + 1]
  const int32_t* col_idx = nullptr;
  int64_t cap = 0;
  float* out = nullptr;
};
void gemm_split_kc_gather(int M, int N, int K, const float* A, int lda, const float* B, int ldb, const GatherOut& to,
                          const Gate& gate, hipStream_t s);
void gemm_f64_km(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc, int splits,
                 size_t c_split, const Gate& gate, hipStream_t s);

// Exclusive scan of counts[0..n) into out[0..n] (out[n] = total) and *total64 = total.
// temp must hold scan_temp_elems(n) int32 values.
size_t scan_temp_elems(int n);
void launch_exclusive_scan(const int32_t* counts, int n, int32_t* out, int64_t* total64, int32_t* temp,
                           hipStream_t stream, const Gate& gate = Gate{});

// ------------------------------------------------------------------ device helpers

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Lanes below the calling lane that have bits set in mask.
__device__ __forceinline__ int mask_prefix(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Inclusive prefix over the wave's lanes.
__device__ __forceinline__ int wave_incl_scan(int v) {
  const int l = lane_id();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    int u = __shfl_up(v, off, kWave);
    if (l >= off) v += u;
  }
  return v;
}

}  // namespace snn

// Sparse dW of layers with many active entries: the entries of 128 rows sorted by column, a wavefront per 8
// columns x 128 inputs with its float64 sums in registers.
//
// dW[i][j] = sum over the entries (r, j) of trace[r][i] G[r][j]. Taken entry by entry in row order the sums
// have to be in LDS, and the float64 LDS atomics pace it (3.05e12 multiply-adds a second). Sorted by column
// inside a window of rows, an entry costs its wavefront one 8-byte LDS read per lane, three conversions, two
// float64 multiply-adds and half a scalar load of its record. Bound: vector instructions (six per record), and
// the latency of a batch (scalar load, then LDS), which eight wavefronts per SIMD hide: 16 wavefronts x 8
// columns per block 931 us for 2312 -> 200 at 76800 rows, 12% active (8 x 16: 1036, 12 x 10: 1009; the sort 37).
// dW there 1514 us entry by entry, 3.1 ms as a dense float64 product; 1024 -> 1024 at 128000 rows, 15% active:
// 4.35 ms dense, 3.24 so; 1500 -> 900 at 25600 rows, 15%: 2.06 dense, 1.01 so.
#include "common.h"

namespace snn {
namespace {

constexpr int kRows = 128;    // rows of a window (a column's mask: four words)
constexpr int kInputs = 128;  // inputs of a tile, two per lane
constexpr int kCols = 8;     // columns of a wavefront
constexpr int kWaves = 16;    // two blocks of 1024 threads per CU
constexpr int kThreads = kWaves * kWave;
constexpr int kBatch = 4;     // records taken together; a column's records are padded to whole batches (G = 0)
constexpr int kColsMax = 3200;
static_assert((5 * kColsMax + 1) * sizeof(int) <= 64 * 1024, "masks and starts fit the default LDS limit");
static_assert(kRows * kInputs * sizeof(float) <= 64 * 1024, "the tile fits the static LDS limit");

__device__ __forceinline__ int clamp_entry(int v, int64_t cap) { return (int)(v < 0 ? 0 : (v > cap ? cap : v)); }

struct ColRec {
  uint32_t off;  // byte offset of the row in the trace tile
  float g;
};

__host__ __device__ inline int64_t win_stride(int N_out) { return 4 * (((int64_t)N_out * (kBatch - 1) + 3) / 4 + 1); }
// First record of a window whose first entry is e0: whole batches, with room for every column's padding.
__host__ __device__ inline int64_t win_base(int win, int e0, int N_out) {
  return (((int64_t)e0 + 3) & ~(int64_t)3) + win * win_stride(N_out);
}
// Length of the record array: every window's entries and padding, and a batch read ahead past the last.
__host__ __device__ inline int64_t cols_records(int n_win, int N_out, int64_t cap) {
  return ((cap + 3) & ~(int64_t)3) + n_win * win_stride(N_out) + 2 * kBatch;
}
// Records that fit from `base` on, whole batches. With row pointers that do not decrease a window never needs more
// than there are; with others it may hold up to kRows records per column whatever the next window's base is, so
// starts and stores are bounded by this.
__host__ __device__ inline int win_room(int64_t recs, int64_t base) {
  const int64_t left = recs - 2 * kBatch - base;
  return (int)(left < 0 ? 0 : (left < (1 << 30) ? left : (1 << 30)));
}

__global__ __launch_bounds__(kThreads) void cols_layout(int TB, int N_out, const int32_t* __restrict__ rp,
                                                        const int32_t* __restrict__ col, const float* __restrict__ g,
                                                        const float* __restrict__ eps, int64_t cap,
                                                        int32_t* __restrict__ start, ColRec* __restrict__ rec,
                                                        int64_t recs, Gate gate) {
  extern __shared__ uint32_t mask[];  // [N_out][4] rows of each column, then [N_out + 1] starts
  __shared__ int red[kWaves];
  if (!gate_open(gate)) return;
  int* st = reinterpret_cast<int*>(mask + 4 * N_out);
  const int tid = threadIdx.x, w = tid / kWave, l = lane_id();
  const int win = blockIdx.x, r0 = win * kRows, nr = min(kRows, TB - r0);
  for (int k = tid; k < 4 * N_out; k += kThreads) mask[k] = 0u;
  __syncthreads();
  for (int row = w; row < nr; row += kWaves) {
    const int e1 = clamp_entry(rp[r0 + row + 1], cap);
    for (int e = clamp_entry(rp[r0 + row], cap) + l; e < e1; e += kWave) {
      const int j = col[e];
      if ((unsigned)j < (unsigned)N_out) atomicOr(&mask[4 * j + (row >> 5)], 1u << (row & 31));
    }
  }
  __syncthreads();
  const auto count = [&](int j) {
    return __popc(mask[4 * j]) + __popc(mask[4 * j + 1]) + __popc(mask[4 * j + 2]) + __popc(mask[4 * j + 3]);
  };
  const auto padded = [&](int j) { return (count(j) + kBatch - 1) / kBatch * kBatch; };
  const int per = (N_out + kThreads - 1) / kThreads;
  const int j0 = min(N_out, tid * per), j1 = min(N_out, j0 + per);
  int sum = 0;
  for (int j = j0; j < j1; ++j) sum += padded(j);
  const int incl = wave_incl_scan(sum);
  if (l == kWave - 1) red[w] = incl;
  __syncthreads();
  int base = incl - sum, all = 0;
  for (int k = 0; k < kWaves; ++k) {
    base += k < w ? red[k] : 0;
    all += red[k];
  }
  for (int j = j0; j < j1; ++j) {
    st[j] = base;
    base += padded(j);
  }
  if (tid == 0) st[N_out] = all;
  __syncthreads();
  const int64_t base0 = win_base(win, clamp_entry(rp[r0], cap), N_out);
  const int room = win_room(recs, base0);
  ColRec* dst = rec + base0;
  int32_t* sg = start + (size_t)win * (N_out + 1);
  for (int j = tid; j <= N_out; j += kThreads) sg[j] = min(st[j], room);
  for (int row = w; row < nr; row += kWaves) {
    const int e1 = clamp_entry(rp[r0 + row + 1], cap);
    for (int e = clamp_entry(rp[r0 + row], cap) + l; e < e1; e += kWave) {
      const int j = col[e];
      if ((unsigned)j >= (unsigned)N_out) continue;
      int pos = st[j];
      const int q = row >> 5;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t m = mask[4 * j + k];
        pos += k < q ? __popc(m) : (k == q ? __popc(m & ((1u << (row & 31)) - 1u)) : 0);
      }
      if (pos < room) dst[pos] = ColRec{(uint32_t)(row * kInputs * sizeof(float)), eps[e] * (g ? g[e] : 1.0f)};
    }
  }
  for (int j = tid; j < N_out; j += kThreads) {
    const int n = count(j);
    if (n % kBatch == 0) continue;
    int row = 0;  // the padding reads a row that the column reads anyway
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (mask[4 * j + k]) row = 32 * k + 31 - __clz(mask[4 * j + k]);
    const int end = min(st[j + 1], room);
    for (int k = st[j] + n; k < end; ++k) dst[k] = ColRec{(uint32_t)(row * kInputs * sizeof(float)), 0.0f};
  }
}

// Uniform addresses through the scalar cache (read-only here; written by earlier kernels).
typedef uint32_t Quad __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) Quad* ScalarQuads;
typedef const __attribute__((address_space(4))) int32_t* ScalarInts;

template <bool VEC>
__global__ __launch_bounds__(kThreads, 2 * kWaves / 4) void cols_dw(const float* __restrict__ trace, int TB, int N_in, int N_out,
                                                       const int32_t* __restrict__ rp, int64_t cap,
                                                       const int32_t* __restrict__ start,
                                                       const ColRec* __restrict__ rec, float* __restrict__ out,
                                                       int n_chunks, int n_itiles, int groups, int cpw, Gate gate) {
  __shared__ __attribute__((aligned(16))) float tile[kRows * kInputs];
  if (!gate_open(gate)) return;
  // the tiles of one chunk of windows run on one XCD and share its records and trace rows in that L2
  int id = blockIdx.x;
  const int nb = gridDim.x;
  if ((nb & 7) == 0) id = (id & 7) * (nb >> 3) + (id >> 3);
  const int tiles = n_itiles * groups;
  const int chunk = id / tiles, t = id % tiles;
  const int i0 = (t / groups) * kInputs;
  const int tid = threadIdx.x, l = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c0 = ((t % groups) * kWaves + w) * cpw;
  const int nc = min(cpw, N_out - c0);
  const int n_win = (TB + kRows - 1) / kRows;
  double acc[kCols][2];
#pragma unroll
  for (int c = 0; c < kCols; ++c) acc[c][0] = acc[c][1] = 0.0;
  const char* mine = reinterpret_cast<const char*>(tile) + 8 * l;
  for (int win = chunk; win < n_win; win += n_chunks) {
    __syncthreads();
#pragma unroll 2
    for (int x = tid; x < kRows * kInputs / 4; x += kThreads) {
      const int row = x / (kInputs / 4), c4 = 4 * (x % (kInputs / 4));
      const int r = win * kRows + row, i = i0 + c4;
      const float* src = trace + (size_t)min(r, TB - 1) * N_in;  // rows past the end have no entry
      float4 v;
      if (VEC && i + 4 <= N_in) v = *reinterpret_cast<const float4*>(src + i);
      else v = make_float4(src[min(i, N_in - 1)], src[min(i + 1, N_in - 1)], src[min(i + 2, N_in - 1)], src[min(i + 3, N_in - 1)]);
      *reinterpret_cast<float4*>(tile + row * kInputs + c4) = v;
    }
    __syncthreads();
    if (nc <= 0) continue;
    ScalarInts sp = (ScalarInts)(uintptr_t)(start + (size_t)win * (N_out + 1) + c0);
    const int e0 = __builtin_amdgcn_readfirstlane(clamp_entry(rp[win * kRows], cap));
    int at = sp[0];
    ScalarQuads p = (ScalarQuads)(uintptr_t)(rec + win_base(win, e0, N_out) + at);
    Quad a = p[0], b = p[1];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
      if (c < nc) {
        const int end = sp[c + 1];
        for (; at < end; at += kBatch) {
          p += 2;
          const Quad an = p[0], bn = p[1];  // the next batch (past the window's end: within the array, not used)
          const float2 t0 = *reinterpret_cast<const float2*>(mine + a.x);
          const float2 t1 = *reinterpret_cast<const float2*>(mine + a.z);
          const float2 t2 = *reinterpret_cast<const float2*>(mine + b.x);
          const float2 t3 = *reinterpret_cast<const float2*>(mine + b.z);
          const double g0 = (double)__uint_as_float(a.y), g1 = (double)__uint_as_float(a.w);
          const double g2 = (double)__uint_as_float(b.y), g3 = (double)__uint_as_float(b.w);
          acc[c][0] = fma(g0, (double)t0.x, acc[c][0]);
          acc[c][1] = fma(g0, (double)t0.y, acc[c][1]);
          acc[c][0] = fma(g1, (double)t1.x, acc[c][0]);
          acc[c][1] = fma(g1, (double)t1.y, acc[c][1]);
          acc[c][0] = fma(g2, (double)t2.x, acc[c][0]);
          acc[c][1] = fma(g2, (double)t2.y, acc[c][1]);
          acc[c][0] = fma(g3, (double)t3.x, acc[c][0]);
          acc[c][1] = fma(g3, (double)t3.y, acc[c][1]);
          a = an;
          b = bn;
        }
      }
    }
  }
  float* dst = out + (size_t)chunk * N_in * N_out;
#pragma unroll
  for (int c = 0; c < kCols; ++c)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = i0 + 2 * l + k;
      if (c < nc && i < N_in) dst[(size_t)i * N_out + c0 + c] = (float)acc[c][k];
    }
}

struct ColsPlan {
  int n_win, n_itiles, groups, cpw, n_chunks;
  size_t recs;
};

ColsPlan plan_cols(int T, int B, int N_in, int N_out, int64_t out_cap) {
  ColsPlan p{};
  p.n_win = (T * B + kRows - 1) / kRows;
  p.n_itiles = (N_in + kInputs - 1) / kInputs;
  p.groups = (N_out + kWaves * kCols - 1) / (kWaves * kCols);
  p.cpw = (N_out + kWaves * p.groups - 1) / (kWaves * p.groups);
  p.n_chunks = std::max(1, std::min({2 * cu_count() / (p.n_itiles * p.groups), p.n_win, 64}));  // one round of blocks
  p.recs = (size_t)cols_records(p.n_win, N_out, out_cap);
  return p;
}

}  // namespace

bool cols_fits(int N_out) { return N_out > 32 && N_out <= kColsMax; }

// The time this takes: launches and each window's barriers, the trace through LDS once per column group (6 TB/s from
// L2 and HBM), and 8e12 multiply-adds a second with 1.5 records of padding per column and window, both times what
// whole rounds of blocks and windows take over even shares. Within 10% of what 300 -> 300 to 1024 -> 1024 layers
// take at 4 to 50% active.
void cols_seconds(int T, int B, int N_in, int N_out, double* fixed, double* per_entry) {
  const double TB = (double)T * B, in = (double)((N_in + kInputs - 1) / kInputs * kInputs);
  const ColsPlan p = plan_cols(T, B, N_in, N_out, 0);
  const int tiles = p.n_itiles * p.groups, slots = 2 * cu_count();
  const double rounds = (double)((tiles * p.n_chunks + slots - 1) / slots) * ((p.n_win + p.n_chunks - 1) / p.n_chunks);
  const double even = (double)p.n_win * tiles / slots;
  *per_entry = in / 8e12 * std::max(1.0, rounds / even);
  *fixed = 60e-6 + p.groups * TB * in * 4.0 / 6e12 * std::max(1.0, rounds / even) + 1.5 * TB / kRows * N_out * *per_entry;
}

size_t cols_workspace(int T, int B, int N_in, int N_out, int64_t out_cap) {
  const ColsPlan p = plan_cols(T, B, N_in, N_out, out_cap);
  Carve c(nullptr);
  c.take<int32_t>((size_t)p.n_win * (N_out + 1) + 1);
  c.take<ColRec>(p.recs);
  if (p.n_chunks > 1) c.take<float>((size_t)p.n_chunks * N_in * N_out);
  return c.off;
}

ColsParts cols_enqueue(const float* trace_in, int T, int B, int N_in, int N_out, const int32_t* out_row_ptr,
                       const int32_t* out_col_idx, const float* out_g, const float* eps_out, int64_t out_cap, float* dW,
                       void* workspace, const Gate& gate, hipStream_t s) {
  const ColsPlan p = plan_cols(T, B, N_in, N_out, out_cap);
  Carve ws(workspace);
  int32_t* start = ws.take<int32_t>((size_t)p.n_win * (N_out + 1) + 1);
  ColRec* rec = ws.take<ColRec>(p.recs);
  float* part = p.n_chunks > 1 ? ws.take<float>((size_t)p.n_chunks * N_in * N_out) : dW;
  hipLaunchKernelGGL(cols_layout, dim3((unsigned)p.n_win), dim3(kThreads), (5 * (size_t)N_out + 1) * sizeof(int), s,
                     T * B, N_out, out_row_ptr, out_col_idx, out_g, eps_out, out_cap, start, rec,
                     (int64_t)p.recs, gate);
  const dim3 grid((unsigned)(p.n_itiles * p.groups * p.n_chunks));
  const bool vec = N_in % 4 == 0 && reinterpret_cast<uintptr_t>(trace_in) % 16 == 0;
  if (vec)
    hipLaunchKernelGGL(cols_dw<true>, grid, dim3(kThreads), 0, s, trace_in, T * B, N_in, N_out, out_row_ptr, out_cap,
                       start, rec, part, p.n_chunks, p.n_itiles, p.groups, p.cpw, gate);
  else
    hipLaunchKernelGGL(cols_dw<false>, grid, dim3(kThreads), 0, s, trace_in, T * B, N_in, N_out, out_row_ptr, out_cap,
                       start, rec, part, p.n_chunks, p.n_itiles, p.groups, p.cpw, gate);
  return {part, p.n_chunks};
}

}  // namespace snn

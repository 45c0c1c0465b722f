// LIF forward of one fully connected layer (Sec. 2.1): Eq. (lif) with V_rest = V_r = 0,
// V[0] = 0, the strict Heaviside of Eq. (spike_fn), and the input trace that Eq. (w_grad)
// reuses (the filtered input of Eq. (lif_unrolled)).
//
// The weighted input of a row (t, b) is I[t,b,:] = sum of W[i,:] over the row's spiking inputs,
// added in ascending i (the list of spiking inputs comes from ballots over the row's bytes), and
// the recurrence V[t+1] = (alpha V[t] + I[t]) - S_out[t], S_out[t] = V[t] > theta, walks time per
// neuron. Two forms:
//   lif_fused   (the default) one block per (sample, group of columns) walks time in tiles: its
//               wavefronts form a tile's weighted inputs two rows each into LDS, then every
//               thread runs its column's recurrence over the tile from LDS. V, S_out, the active
//               bitset and the input trace are written once; the weighted inputs never reach HBM.
//               The trace of the output spikes (the next layer's input trace) can be written
//               beside V from the spike bits the recurrence has in hand.
//   lif_gather + lif_scan  (widths whose bitset words straddle samples, W rows that are not
//               whole float4 columns, grids of fewer than two blocks per CU) one wavefront per row
//               parks I[t,b,:] in the slot of V[t+1,b,:]; then one thread per (b, j) runs the
//               recurrence over t, overwriting it with V[t+1], and one thread per (b, input) the
//               input trace.
// Float32 with separately rounded operations (__fmul_rn / __fadd_rn) and the ascending
// summation order make V a deterministic function of the inputs; both forms give the same bits.
#include "common.h"

namespace snn {
namespace {

// V and traces are stored non-temporally: each is a pass over memory that nothing reads again before the layer
// is done, and in L2 it would take the place of W's rows and of the spike rows that are read twice (2312 -> 200,
// T = 300, B = 256: forward 428 -> 321 us; 3 x 1024, T = 500: 1666 -> 1596; 5 x 300, T = 100: 266 -> 249). The
// spikes stay cached: the next layer reads them at once (stored so, the last of these takes 260).
typedef float Quad __attribute__((ext_vector_type(4)));

constexpr int kGatherWaves = 4;        // wavefronts (rows) per gather block
constexpr int kPiece = 4 * kWave;      // inputs per ballot piece (4 bytes per lane)
constexpr int kSegPieces = 4;          // pieces whose spike bytes are loaded together
constexpr int kScanThreads = 256;
constexpr int kScanAhead = 32;         // time steps loaded ahead in the scans

template <bool ALIGNED>
__device__ __forceinline__ uint32_t load4(const uint8_t* p, int i, int n) {
  if (ALIGNED) return i < n ? *reinterpret_cast<const uint32_t*>(p + i) : 0u;
  uint32_t x = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (i + q < n) x |= (uint32_t)p[i + q] << (8 * q);
  return x;
}

// The spike bytes of one segment of a row (kSegPieces pieces of 4 bytes per lane; bytes past
// N_in read as no spike).
template <bool ALIGNED>
__device__ __forceinline__ void load_segment(const uint8_t* __restrict__ row, int s0, int N_in,
                                             uint32_t (&x)[kSegPieces]) {
  const int l = lane_id();
#pragma unroll
  for (int c = 0; c < kSegPieces; ++c) x[c] = load4<ALIGNED>(row, s0 + c * kPiece + 4 * l, N_in);
}

// Ascending list (offsets inside the segment) of a segment's spiking inputs in lst; returns its
// length.
__device__ __forceinline__ int segment_list(const uint32_t (&x)[kSegPieces], uint16_t* lst) {
  const int l = lane_id();
  int base = 0;
#pragma unroll
  for (int c = 0; c < kSegPieces; ++c) {
    const bool a0 = (x[c] & 0xffu) != 0, a1 = (x[c] & 0xff00u) != 0, a2 = (x[c] & 0xff0000u) != 0,
               a3 = (x[c] & 0xff000000u) != 0;
    const uint64_t m0 = __ballot(a0), m1 = __ballot(a1), m2 = __ballot(a2), m3 = __ballot(a3);
    int pos = base + mask_prefix(m0) + mask_prefix(m1) + mask_prefix(m2) + mask_prefix(m3);
    const int o = c * kPiece + 4 * l;
    if (a0) lst[pos++] = (uint16_t)o;
    if (a1) lst[pos++] = (uint16_t)(o + 1);
    if (a2) lst[pos++] = (uint16_t)(o + 2);
    if (a3) lst[pos++] = (uint16_t)(o + 3);
    base += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
  }
  return base;
}

// Ascending list of a segment's spiking inputs as byte offsets inside their piece (piece c's
// entries at [starts[c], starts[c + 1]) of lst); returns its length.
__device__ __forceinline__ int segment_list8(const uint32_t (&x)[kSegPieces], uint8_t* lst, int (&starts)[kSegPieces]) {
  const int l = lane_id();
  int base = 0;
#pragma unroll
  for (int c = 0; c < kSegPieces; ++c) {
    starts[c] = base;
    const bool a0 = (x[c] & 0xffu) != 0, a1 = (x[c] & 0xff00u) != 0, a2 = (x[c] & 0xff0000u) != 0,
               a3 = (x[c] & 0xff000000u) != 0;
    const uint64_t m0 = __ballot(a0), m1 = __ballot(a1), m2 = __ballot(a2), m3 = __ballot(a3);
    int pos = base + mask_prefix(m0) + mask_prefix(m1) + mask_prefix(m2) + mask_prefix(m3);
    const int o = 4 * l;
    if (a0) lst[pos++] = (uint8_t)o;
    if (a1) lst[pos++] = (uint8_t)(o + 1);
    if (a2) lst[pos++] = (uint8_t)(o + 2);
    if (a3) lst[pos++] = (uint8_t)(o + 3);
    base += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
  }
  return base;
}

// Input index of list entry e (s0: the segment's first input).
__device__ __forceinline__ int list8_input(const uint8_t* lst, const int (&starts)[kSegPieces], int e, int s0) {
  const int c = (e >= starts[1]) + (e >= starts[2]) + (e >= starts[3]);
  return s0 + c * kPiece + (int)lst[e];
}

// The weighted input of one row (t, b) at NQ float4 column groups per lane: lane l sums columns
// col0 + 4 (l + 64 m) .. +3, m < NQ, over the row's spiking inputs in ascending i, from +0.0 with
// separately rounded adds. The row's spike bytes are read kSegPieces pieces at a time (all loads
// issued first), their spiking inputs listed in lst (LDS) in ascending order, and the list's W
// rows summed KB at a time (KB * NQ float4 loads in flight).
template <bool ALIGNED, bool VEC, int NQ, int KB>
__device__ __forceinline__ void row_input_sums(const uint8_t* __restrict__ row, const float* __restrict__ W, int N_in,
                                               int N_out, int col0, uint16_t* lst, float (&acc)[NQ][4]) {
  const int l = lane_id();
#pragma unroll
  for (int m = 0; m < NQ; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[m][q] = 0.0f;

  for (int s0 = 0; s0 < N_in; s0 += kSegPieces * kPiece) {
    uint32_t x[kSegPieces];
    load_segment<ALIGNED>(row, s0, N_in, x);
    const int n = segment_list(x, lst);
    __builtin_amdgcn_wave_barrier();
    // sums in ascending i, KB W rows in flight; positions past the list are clamped to its last
    // entry and their sums skipped by a select
    for (int k = 0; k < n; k += KB) {
      float4 wv[KB][NQ];
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int ii = s0 + (int)lst[min(k + u, n - 1)];
        const float* wr = W + (size_t)ii * N_out + col0;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          const int j = 4 * (l + kWave * m);
          const int jn = N_out - col0;  // columns of the row from col0 on
          if (VEC) {
            wv[u][m] = j < jn ? *reinterpret_cast<const float4*>(wr + j) : make_float4(0.f, 0.f, 0.f, 0.f);
          } else {
            wv[u][m].x = j < jn ? wr[j] : 0.0f;
            wv[u][m].y = j + 1 < jn ? wr[j + 1] : 0.0f;
            wv[u][m].z = j + 2 < jn ? wr[j + 2] : 0.0f;
            wv[u][m].w = j + 3 < jn ? wr[j + 3] : 0.0f;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const bool take = k + u < n;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          acc[m][0] = take ? __fadd_rn(acc[m][0], wv[u][m].x) : acc[m][0];
          acc[m][1] = take ? __fadd_rn(acc[m][1], wv[u][m].y) : acc[m][1];
          acc[m][2] = take ? __fadd_rn(acc[m][2], wv[u][m].z) : acc[m][2];
          acc[m][3] = take ? __fadd_rn(acc[m][3], wv[u][m].w) : acc[m][3];
        }
      }
    }
    __builtin_amdgcn_wave_barrier();  // the list is rewritten by the next segment
  }
}

// One wavefront per row (t, b), t < T - 1: the row's weighted input over every column, parked in
// the slot of V[t+1, b, :].
template <bool ALIGNED, bool VEC, int NQ>
__global__ __launch_bounds__(kGatherWaves * kWave) void lif_gather(const uint8_t* __restrict__ s_in,
                                                                   const float* __restrict__ W, int T, int B,
                                                                   int N_in, int N_out, float* __restrict__ V) {
  constexpr int kBatch = NQ >= 16 ? 1 : (NQ >= 8 ? 2 : 4);  // W rows in flight: kBatch * NQ float4 loads
  __shared__ uint16_t seg_list[kGatherWaves][kSegPieces * kPiece];
  const int w = threadIdx.x / kWave;
  const int l = lane_id();
  const long r = (long)blockIdx.x * kGatherWaves + w;  // row r = t * B + b, t < T - 1
  if (r >= (long)(T - 1) * B) return;
  float acc[NQ][4];
  row_input_sums<ALIGNED, VEC, NQ, kBatch>(s_in + (size_t)r * N_in, W, N_in, N_out, 0, seg_list[w], acc);
  float* dst = V + (size_t)(r + B) * N_out;  // slot of V[t+1, b, :]
#pragma unroll
  for (int m = 0; m < NQ; ++m) {
    const int j = 4 * (l + kWave * m);
    if (VEC) {
      if (j < N_out) *reinterpret_cast<float4*>(dst + j) = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (j + q < N_out) dst[j + q] = acc[m][q];
    }
  }
}

// lif_gather for layers of at most 32 outputs (readouts): a wavefront takes 64 / L rows, L lanes each (lane =
// column), so that one W load serves 64 / L rows; with a row per wavefront most lanes have no column. The L lanes
// of a row read LB of its bytes each, place the spiking inputs in the row's list by a scan over the lanes, and
// the lists are summed (ascending, kNarrowKb rows of W in flight) when one may overflow and at the end. Same
// sums in the same order as lif_gather. Bound: latency of the W rows, a list's length over kNarrowKb round
// trips. 12544 -> 10, T = 100, B = 256 (2349
// spikes in the longest row): 461 -> 150 us.
constexpr int kNarrowCols = 32;
constexpr int kNarrowFull = 512;  // entries from which a row's list is summed before more inputs are read
constexpr int kNarrowKb = 16;

template <int LB>
struct Bytes;
template <>
struct Bytes<4> { typedef uint32_t type; };
template <>
struct Bytes<8> { typedef uint2 type; };
template <>
struct Bytes<16> { typedef uint4 type; };

template <int LB, int L>
__global__ __launch_bounds__(kGatherWaves * kWave) void lif_gather_narrow(const uint8_t* __restrict__ s_in,
                                                                          const float* __restrict__ W, int T, int B,
                                                                          int N_in, int N_out, float* __restrict__ V) {
  constexpr int kRowsPerWave = kWave / L;
  constexpr int kCap = kNarrowFull + L * LB;
  constexpr int kAheadLoads = 4;
  static_assert(kCap % kNarrowKb == 0 && kNarrowKb % 8 == 0, "lists of whole batches, batches of whole 16-byte reads");
  __shared__ __attribute__((aligned(16))) uint16_t lists[kGatherWaves * kRowsPerWave][kCap];
  const int w = threadIdx.x / kWave;
  const int l = lane_id();
  const int g = l / L, li = l % L;
  const long rows = (long)(T - 1) * B;
  // a wavefront's rows lie a quarter (half) of the rows apart: activity clusters in time, and a wavefront takes as
  // long as its longest list
  const long wave_rows = (long)gridDim.x * kGatherWaves;
  const long r = (long)g * wave_rows + (long)blockIdx.x * kGatherWaves + w;
  const bool live = r < rows;
  const uint8_t* row = s_in + (size_t)(live ? r : 0) * N_in;
  uint16_t* lst = lists[w * kRowsPerWave + g];
  const int col = min(li, N_out - 1);
  float acc = 0.0f;
  int cnt = 0;  // entries in the row's list
  auto sum_list = [&]() {
    __builtin_amdgcn_wave_barrier();
    for (int k = 0; __ballot(k < cnt); k += kNarrowKb) {
      // eight entries a read (past the list: anything, clamped into W and not added)
      uint16_t i[kNarrowKb];
      const uint4* e = reinterpret_cast<const uint4*>(lst + min(k, kCap - kNarrowKb));
#pragma unroll
      for (int u = 0; u < kNarrowKb / 8; ++u) {
        const uint4 x = e[u];
        __builtin_memcpy(i + 8 * u, &x, sizeof(x));
      }
      float wv[kNarrowKb];
#pragma unroll
      for (int u = 0; u < kNarrowKb; ++u) wv[u] = W[(size_t)min((int)i[u], N_in - 1) * N_out + col];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kNarrowKb; ++u) acc = k + u < cnt ? __fadd_rn(acc, wv[u]) : acc;
    }
    cnt = 0;
    __builtin_amdgcn_wave_barrier();
  };
  typedef typename Bytes<LB>::type Piece;
  for (int i0 = 0; i0 < N_in; i0 += kAheadLoads * L * LB) {
    uint32_t x[kAheadLoads][LB / 4];
#pragma unroll
    for (int u = 0; u < kAheadLoads; ++u) {
      const int i = i0 + (u * L + li) * LB;  // N_in is a multiple of LB: a piece is in the row or past it
      const bool in = live && i < N_in;
      const Piece p = *reinterpret_cast<const Piece*>(row + (in ? i : 0));
      __builtin_memcpy(x[u], &p, LB);
#pragma unroll
      for (int q = 0; q < LB / 4; ++q) x[u][q] = in ? x[u][q] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kAheadLoads; ++u) {
      uint32_t mask = 0;  // bit k: byte k of the piece is a spike
#pragma unroll
      for (int q = 0; q < LB / 4; ++q) {
        const uint32_t y = x[u][q];
        const uint32_t high = ((((y & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y) >> 7) & 0x01010101u;
        mask |= ((high * 0x01020408u) >> 24 & 0xfu) << (4 * q);
      }
      if (__ballot(mask != 0) == 0) continue;
      const int n = __popc(mask);
      int incl = n;  // inclusive scan over the row's lanes
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);  // row_shr:1
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);  // row_shr:2
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);  // row_shr:4
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);  // row_shr:8
      if (L == 32) {
        const int low = __shfl(incl, (l & ~31) + 15, kWave);
        incl += li >= 16 ? low : 0;
      }
      int pos = cnt + incl - n;
      const int ib = i0 + (u * L + li) * LB;
      while (mask) {
        lst[pos++] = (uint16_t)(ib + __builtin_ctz(mask));
        mask &= mask - 1u;
      }
      cnt += __shfl(incl, (l & ~(L - 1)) + L - 1, kWave);
      if (__ballot(cnt > kNarrowFull)) sum_list();
    }
  }
  sum_list();
  if (live && li < N_out) V[(size_t)(r + B) * N_out + li] = acc;
}

// The input trace of input k = b * N_in + i over the whole time axis: trace[0] = 0,
// trace[t+1] = alpha trace[t] + S_in[t] (loads kScanAhead steps ahead). One input per lane, not
// four: four times the wavefronts for the same bytes, so that more of them overlap their load and
// store phases (T = 500, B = 256, 1024 inputs: 0.152 -> 0.123 ms beside the recurrence).
__device__ __forceinline__ void trace_walk(size_t k, const uint8_t* __restrict__ s_in, int T, int B, int N_in,
                                           float alpha, float* __restrict__ trace) {
  const size_t step = (size_t)B * N_in;
  if (k >= step) return;
  float tr = 0.0f;
  trace[k] = 0.0f;
  for (int t0 = 0; t0 < T - 1; t0 += kScanAhead) {
    const int np = min(kScanAhead, T - 1 - t0);
    uint32_t x[kScanAhead];
#pragma unroll
    for (int p = 0; p < kScanAhead; ++p) x[p] = s_in[(size_t)(t0 + min(p, np - 1)) * step + k];
#pragma unroll
    for (int p = 0; p < kScanAhead; ++p) {
      if (p < np) {
        tr = __fadd_rn(__fmul_rn(alpha, tr), x[p] ? 1.0f : 0.0f);
        __builtin_nontemporal_store(tr, trace + (size_t)(t0 + p + 1) * step + k);
      }
    }
  }
}

// The input trace of input quad k = b * ceil(N_in / 4) + quad over the whole time axis, as
// trace_walk (the trace blocks beside lif_fused's blocks: there four inputs per lane are faster,
// 0.326 against 0.340 ms at T = 100, B = 512, 2312 inputs).
template <bool ALIGNED>
__device__ __forceinline__ void trace_walk4(size_t k, const uint8_t* __restrict__ s_in, int T, int B, int N_in,
                                            float alpha, float* __restrict__ trace) {
  const int nq = (N_in + 3) / 4;
  if (k >= (size_t)B * nq) return;
  const int b = (int)(k / nq);
  const int i = 4 * (int)(k - (size_t)b * nq);
  const size_t step = (size_t)B * N_in;
  float* dst0 = trace + (size_t)b * N_in + i;
  float tr[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (i + q < N_in) dst0[q] = 0.0f;
  const uint8_t* src0 = s_in + (size_t)b * N_in;
  for (int t0 = 0; t0 < T - 1; t0 += kScanAhead) {
    const int np = min(kScanAhead, T - 1 - t0);
    uint32_t x[kScanAhead];
#pragma unroll
    for (int p = 0; p < kScanAhead; ++p) x[p] = load4<ALIGNED>(src0 + (size_t)(t0 + min(p, np - 1)) * step, i, N_in);
#pragma unroll
    for (int p = 0; p < kScanAhead; ++p) {
      if (p < np) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          tr[q] = __fadd_rn(__fmul_rn(alpha, tr[q]), ((x[p] >> (8 * q)) & 0xffu) ? 1.0f : 0.0f);
        float* dst = dst0 + (size_t)(t0 + p + 1) * step;
        if (ALIGNED) {
          *reinterpret_cast<float4*>(dst) = make_float4(tr[0], tr[1], tr[2], tr[3]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (i + q < N_in) dst[q] = tr[q];
        }
      }
    }
  }
}

// Blocks [0, nv) run the membrane recurrence of B * N_out neurons; blocks [nv, nv + nt) run the
// trace of B * N_in inputs.
// With bits != NULL the recurrence also marks the active set of Definition 1: bit (t, k) of the
// bitset, k = b * N_out + j, is |V[t,b,j] - theta| < b_th in float32, word t * W64 + k / 64,
// W64 = ceil(B * N_out / 64); one ballot per wavefront and step (its 64 k are one word).
__device__ __forceinline__ void mark_active(uint64_t* bits, size_t word, bool valid, float v, float theta,
                                            float b_th) {
  const uint64_t m = __ballot(valid && fabsf(v - theta) < b_th);
  if (lane_id() == 0) bits[word] = m;
}

__global__ __launch_bounds__(kScanThreads) void lif_scan(const uint8_t* __restrict__ s_in, int T, int B, int N_in,
                                                         int N_out, float alpha, float theta, float b_th,
                                                         float* __restrict__ V, uint8_t* __restrict__ s_out,
                                                         float* __restrict__ trace, float* __restrict__ trace_out,
                                                         float alpha_next, uint64_t* __restrict__ bits, int nv) {
  if ((int)blockIdx.x < nv) {
    const size_t k0 = (size_t)blockIdx.x * kScanThreads + (threadIdx.x & ~(kWave - 1));
    if (k0 >= (size_t)B * N_out) return;  // whole wavefront past the end
    const size_t k = (size_t)blockIdx.x * kScanThreads + threadIdx.x;  // b * N_out + j
    const bool valid = k < (size_t)B * N_out;
    const size_t kc = valid ? k : k0;  // lanes past the end compute on a valid column, store nothing
    const size_t step = (size_t)B * N_out;
    const size_t W64 = (step + kWave - 1) / kWave;
    const size_t wword = k0 / kWave;
    float v = 0.0f, to = 0.0f;
    if (valid) V[k] = 0.0f;
    if (trace_out && valid) trace_out[k] = 0.0f;
    if (bits) mark_active(bits, wword, valid, v, theta, b_th);
    // Two groups of kScanAhead steps in flight: a group's loads are issued before the previous
    // group's stores, so waiting for them (the memory counter retires in order) does not wait
    // for those stores as well. A group's loads read slots no earlier store writes.
    auto load = [&](float (&in)[kScanAhead], int t0) {
      const int np = min(kScanAhead, T - 1 - t0);
#pragma unroll
      for (int p = 0; p < kScanAhead; ++p) in[p] = V[(size_t)(t0 + min(p, np - 1) + 1) * step + kc];
    };
    auto walk = [&](const float (&in)[kScanAhead], int t0) {
      const int np = min(kScanAhead, T - 1 - t0);
#pragma unroll
      for (int p = 0; p < kScanAhead; ++p) {
        if (p < np) {
          const int t = t0 + p;
          const bool sp = v > theta;
          if (valid) s_out[(size_t)t * step + k] = (uint8_t)sp;
          v = __fadd_rn(__fadd_rn(__fmul_rn(alpha, v), in[p]), sp ? -1.0f : -0.0f);
          if (valid) __builtin_nontemporal_store(v, V + (size_t)(t + 1) * step + k);
          if (trace_out) {
            to = __fadd_rn(__fmul_rn(alpha_next, to), sp ? 1.0f : 0.0f);
            if (valid) trace_out[(size_t)(t + 1) * step + k] = to;
          }
          if (bits) mark_active(bits, (size_t)(t + 1) * W64 + wword, valid, v, theta, b_th);
        }
      }
    };
    float ina[kScanAhead], inb[kScanAhead];
    if (T > 1) load(ina, 0);
    for (int t0 = 0; t0 < T - 1; t0 += 2 * kScanAhead) {
      const int t1 = t0 + kScanAhead;
      if (t1 < T - 1) load(inb, t1);
      walk(ina, t0);
      if (t1 < T - 1) {
        if (t1 + kScanAhead < T - 1) load(ina, t1 + kScanAhead);
        walk(inb, t1);
      }
    }
    if (valid) s_out[(size_t)(T - 1) * step + k] = (uint8_t)(v > theta);
  } else {
    trace_walk((size_t)(blockIdx.x - nv) * kScanThreads + threadIdx.x, s_in, T, B, N_in, alpha, trace);
  }
}

// The weighted inputs of two rows at once (the sums and order of row_input_sums for each): the
// rows' spike lists are formed segment by segment and their W rows summed together, KB of each
// row in flight. x0 / x1 hold the first segment's spike bytes (loaded by the caller ahead of
// time); a null row has no spikes.
template <bool ALIGNED, int NQ, int KB>
__device__ __forceinline__ void row_pair_sums(const uint8_t* r0, const uint8_t* r1, const uint32_t (&x0)[kSegPieces],
                                              const uint32_t (&x1)[kSegPieces], const float* __restrict__ W,
                                              int N_in, int N_out, int col0, uint8_t* lst0, uint8_t* lst1,
                                              float (&acc0)[NQ][4], float (&acc1)[NQ][4]) {
  const int l = lane_id();
  const int jn = N_out - col0;  // columns of a W row from col0 on (a multiple of 4)
#pragma unroll
  for (int m = 0; m < NQ; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc0[m][q] = acc1[m][q] = 0.0f;
  for (int s0 = 0; s0 < N_in; s0 += kSegPieces * kPiece) {
    uint32_t y0[kSegPieces], y1[kSegPieces];
#pragma unroll
    for (int c = 0; c < kSegPieces; ++c) y0[c] = y1[c] = 0u;
    if (s0 == 0) {
#pragma unroll
      for (int c = 0; c < kSegPieces; ++c) {
        y0[c] = x0[c];
        y1[c] = x1[c];
      }
    } else {
      if (r0) load_segment<ALIGNED>(r0, s0, N_in, y0);
      if (r1) load_segment<ALIGNED>(r1, s0, N_in, y1);
    }
    int st0[kSegPieces], st1[kSegPieces];
    const int n0 = segment_list8(y0, lst0, st0);
    const int n1 = segment_list8(y1, lst1, st1);
    __builtin_amdgcn_wave_barrier();
    const int n = max(n0, n1);
    for (int k = 0; k < n; k += KB) {
      float4 wa[KB][NQ], wb[KB][NQ];
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int i0 = n0 > 0 ? list8_input(lst0, st0, min(k + u, n0 - 1), s0) : s0;
        const int i1 = n1 > 0 ? list8_input(lst1, st1, min(k + u, n1 - 1), s0) : s0;
        const float* w0 = W + (size_t)i0 * N_out + col0;
        const float* w1 = W + (size_t)i1 * N_out + col0;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          const int j = 4 * (l + kWave * m);
          wa[u][m] = j < jn ? *reinterpret_cast<const float4*>(w0 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
          wb[u][m] = j < jn ? *reinterpret_cast<const float4*>(w1 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const bool t0 = k + u < n0, t1 = k + u < n1;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          acc0[m][0] = t0 ? __fadd_rn(acc0[m][0], wa[u][m].x) : acc0[m][0];
          acc0[m][1] = t0 ? __fadd_rn(acc0[m][1], wa[u][m].y) : acc0[m][1];
          acc0[m][2] = t0 ? __fadd_rn(acc0[m][2], wa[u][m].z) : acc0[m][2];
          acc0[m][3] = t0 ? __fadd_rn(acc0[m][3], wa[u][m].w) : acc0[m][3];
          acc1[m][0] = t1 ? __fadd_rn(acc1[m][0], wb[u][m].x) : acc1[m][0];
          acc1[m][1] = t1 ? __fadd_rn(acc1[m][1], wb[u][m].y) : acc1[m][1];
          acc1[m][2] = t1 ? __fadd_rn(acc1[m][2], wb[u][m].z) : acc1[m][2];
          acc1[m][3] = t1 ? __fadd_rn(acc1[m][3], wb[u][m].w) : acc1[m][3];
        }
      }
    }
    __builtin_amdgcn_wave_barrier();  // the lists are rewritten by the next segment
  }
}

// Fused forward. Blocks [0, nfb): one per (sample b, column group cg of JW = 256 NQ columns),
// walking the time axis in tiles of kFuseP = 2 kFuseWaves steps. In a tile each wavefront forms the
// weighted inputs of two of the tile's rows (row_pair_sums) in an LDS tile; after a barrier each
// thread runs the membrane recurrence of its column over the tile's steps from the LDS tile, so
// V, S_out and the active bitset are written once and the weighted inputs never reach HBM; the
// spike bytes of the next tile's rows are requested before the recurrence. Blocks [nfb, ...):
// the input trace, one thread per input quad (trace_walk4), beside them. Bit-identical to
// lif_gather + lif_scan. With a bitset each wavefront's 64 columns must be one bitset word
// (N_out % 64 == 0, checked by the caller).
constexpr int kFuseThreads = 512;
constexpr int kFuseWaves = kFuseThreads / kWave;
constexpr int kFuseP = 2 * kFuseWaves;  // steps per tile: two rows per wavefront

template <bool ALIGNED, int NQ, bool STASH, bool TOUT>
__global__ __launch_bounds__(kFuseThreads) __attribute__((amdgpu_waves_per_eu(4))) void lif_fused(
    const uint8_t* __restrict__ s_in, const float* __restrict__ W, int T, int B, int N_in, int N_out, int G, int nfb,
    float alpha, float theta, float b_th, float* __restrict__ V, uint8_t* __restrict__ s_out,
    float* __restrict__ trace, float* __restrict__ trace_out, float alpha_next, uint64_t* __restrict__ bits) {
  constexpr int JW = 4 * kWave * NQ;  // columns of a group
  constexpr int KB = NQ >= 2 ? 4 : 8;
  static_assert(JW <= kFuseThreads, "one scan thread per column of the group");
  static_assert(!STASH || ALIGNED, "stashed spike bytes are whole input quads");
  if (!STASH && (int)blockIdx.x >= nfb) {
    trace_walk4<ALIGNED>((size_t)(blockIdx.x - nfb) * kFuseThreads + threadIdx.x, s_in, T, B, N_in, alpha, trace);
    return;
  }
  __shared__ __attribute__((aligned(16))) float tile[kFuseP][JW];
  __shared__ uint8_t lists[2 * kFuseWaves][kSegPieces * kPiece];
  // STASH (N_in <= one segment): the tile's spike bytes, input quad q of step p at [p][q], for the trace
  __shared__ uint32_t rowbytes[STASH ? kFuseP : 1][kSegPieces * kWave];
  const int w = threadIdx.x / kWave;
  const int l = lane_id();
  const int b = blockIdx.x / G;
  const int cg = blockIdx.x - b * G;
  const int c0 = cg * JW;
  const size_t vstep = (size_t)B * N_out;
  const size_t W64 = (vstep + kWave - 1) / kWave;
  const size_t istep = (size_t)B * N_in;
  // scan thread k: column c0 + k of sample b; wavefronts whose first column is past N_out skip
  const int k = threadIdx.x;
  const int kw = k - l;  // the wavefront's first column slot
  const bool scan_wave = kw < JW && c0 + kw < N_out;
  const bool valid = scan_wave && c0 + k < N_out;
  const size_t vk = (size_t)b * N_out + c0 + (valid ? k : kw);
  const size_t wword = ((size_t)b * N_out + c0 + kw) / kWave;
  // rows w and w + kFuseWaves of tile t0 (null past T - 2)
  auto row_of = [&](int t0, int p) -> const uint8_t* {
    const int t = t0 + p;
    return t < T - 1 ? s_in + (size_t)t * istep + (size_t)b * N_in : nullptr;
  };
  uint32_t x0[kSegPieces], x1[kSegPieces];
  auto prefetch = [&](int t0) {
    const uint8_t* r0 = row_of(t0, w);
    const uint8_t* r1 = row_of(t0, w + kFuseWaves);
#pragma unroll
    for (int c = 0; c < kSegPieces; ++c) x0[c] = x1[c] = 0u;
    if (r0) load_segment<ALIGNED>(r0, 0, N_in, x0);
    if (r1) load_segment<ALIGNED>(r1, 0, N_in, x1);
  };
  // STASH: the trace of the group's input quads, thread k taking quad q_lo + k
  const int nq = (N_in + 3) / 4;
  const int qpg = (nq + G - 1) / G;
  const int tq = (cg * qpg + k < nq && k < qpg) ? cg * qpg + k : -1;
  float tr[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (STASH && trace && tq >= 0)
    *reinterpret_cast<float4*>(trace + (size_t)b * N_in + 4 * tq) = make_float4(0.f, 0.f, 0.f, 0.f);
  float v = 0.0f, to = 0.0f;
  if (valid) V[vk] = 0.0f;
  if (TOUT && valid) trace_out[vk] = 0.0f;
  if (bits && scan_wave) mark_active(bits, wword, valid, v, theta, b_th);
  prefetch(0);
  for (int t0 = 0; t0 < T - 1; t0 += kFuseP) {
    const int np = min(kFuseP, T - 1 - t0);
    if (STASH) {
#pragma unroll
      for (int c = 0; c < kSegPieces; ++c) {
        rowbytes[w][c * kWave + l] = x0[c];
        rowbytes[w + kFuseWaves][c * kWave + l] = x1[c];
      }
    }
    {
      float acc0[NQ][4], acc1[NQ][4];
      row_pair_sums<ALIGNED, NQ, KB>(row_of(t0, w), row_of(t0, w + kFuseWaves), x0, x1, W, N_in, N_out, c0,
                                     lists[w], lists[w + kFuseWaves], acc0, acc1);
#pragma unroll
      for (int m = 0; m < NQ; ++m) {
        const int j = 4 * (l + kWave * m);
        *reinterpret_cast<float4*>(&tile[w][j]) = make_float4(acc0[m][0], acc0[m][1], acc0[m][2], acc0[m][3]);
        *reinterpret_cast<float4*>(&tile[w + kFuseWaves][j]) =
            make_float4(acc1[m][0], acc1[m][1], acc1[m][2], acc1[m][3]);
      }
    }
    __syncthreads();
    prefetch(t0 + kFuseP);  // in flight during the recurrence
    if (scan_wave) {
#pragma unroll
      for (int p = 0; p < kFuseP; ++p) {
        if (p < np) {
          const int t = t0 + p;
          const bool sp = v > theta;
          if (valid) s_out[(size_t)t * vstep + vk] = (uint8_t)sp;
          v = __fadd_rn(__fadd_rn(__fmul_rn(alpha, v), tile[p][k]), sp ? -1.0f : -0.0f);
          if (valid) __builtin_nontemporal_store(v, V + (size_t)(t + 1) * vstep + vk);
          if (TOUT) {
            to = __fadd_rn(__fmul_rn(alpha_next, to), sp ? 1.0f : 0.0f);
            if (valid) __builtin_nontemporal_store(to, trace_out + (size_t)(t + 1) * vstep + vk);
          }
          if (bits) mark_active(bits, (size_t)(t + 1) * W64 + wword, valid, v, theta, b_th);
        }
      }
    }
    if (STASH && trace && tq >= 0) {
      float* dst0 = trace + (size_t)b * N_in + 4 * tq;
#pragma unroll
      for (int p = 0; p < kFuseP; ++p) {
        if (p < np) {
          const uint32_t x = rowbytes[p][tq];
#pragma unroll
          for (int q = 0; q < 4; ++q) tr[q] = __fadd_rn(__fmul_rn(alpha, tr[q]), ((x >> (8 * q)) & 0xffu) ? 1.0f : 0.0f);
          __builtin_nontemporal_store((Quad{tr[0], tr[1], tr[2], tr[3]}), reinterpret_cast<Quad*>(dst0 + (size_t)(t0 + p + 1) * istep));
        }
      }
    }
    __syncthreads();  // the tile is rewritten by the next tile's sums
  }
  if (valid) s_out[(size_t)(T - 1) * vstep + vk] = (uint8_t)(v > theta);
}

template <bool ALIGNED, bool VEC>
void launch_gather(int NQ, dim3 grid, hipStream_t s, const uint8_t* s_in, const float* W, int T, int B, int N_in,
                   int N_out, float* V) {
#define SNN_G(Q)                                                                                              \
  hipLaunchKernelGGL((lif_gather<ALIGNED, VEC, Q>), grid, dim3(kGatherWaves * kWave), 0, s, s_in, W, T, B, N_in, \
                     N_out, V)
  if (NQ <= 1) SNN_G(1);
  else if (NQ <= 2) SNN_G(2);
  else if (NQ <= 4) SNN_G(4);
  else if (NQ <= 8) SNN_G(8);
  else SNN_G(16);
#undef SNN_G
}

}  // namespace
}  // namespace snn

using namespace snn;

namespace {

// Convolutional LIF layer (3x3 filters, stride 1, zero padding 1, channels last): neuron
// k = b * N + n, n = (y * W + x) * F + f, N = H * W * F. Its weighted input at step t is the
// filter applied to the input spikes of the 3x3 patch, added in ascending input index
// (y', x', c) from +0.0 in separately rounded float32 adds (the order of the layer's Toeplitz
// matrix in the fully connected form), then the same recurrence and marking as lif_scan.
// WAVE_PIXEL (F a multiple of 64): a wavefront's 64 neurons share one pixel, so its lanes load
// the patch bytes of several steps at once (lane = (step, tap)), one ballot gives the spiking
// taps of those steps, and each lane adds its filter's weights for the set taps in tap order.
// Otherwise each lane forms its own patch sums, kConvAhead steps at a time.
constexpr int kConvAhead = 8;

template <bool WAVE_PIXEL>
__global__ __launch_bounds__(kScanThreads) void conv_scan(const uint8_t* __restrict__ s_in, const float* __restrict__ Wc,
                                                          int T, int B, int H, int W, int C, int F, float alpha,
                                                          float theta, float b_th, float* __restrict__ V,
                                                          uint8_t* __restrict__ s_out, uint64_t* __restrict__ bits) {
  const size_t N = (size_t)H * W * F;
  const size_t step = (size_t)B * N;
  const size_t k0 = (size_t)blockIdx.x * kScanThreads + (threadIdx.x & ~(kWave - 1));
  if (k0 >= step) return;  // whole wavefront past the end
  const size_t k = (size_t)blockIdx.x * kScanThreads + threadIdx.x;
  const bool valid = k < step;
  const size_t kc = valid ? k : k0;  // lanes past the end compute on a valid neuron, store nothing
  const int b = (int)(kc / N);
  const int n = (int)(kc - (size_t)b * N);
  const int f = n % F;
  const int pix = n / F;
  const int y = pix / W;
  const int x = pix - y * W;
  const size_t W64 = (step + kWave - 1) / kWave;
  const size_t wword = k0 / kWave;
  const size_t in_step = (size_t)B * H * W * C;
  const uint8_t* xb = s_in + (size_t)b * H * W * C;
  const int ntap = 9 * C;
  // WAVE_PIXEL: lane l < q * ntap loads tap (l % ntap) of step (l / ntap) of the group
  const int q = WAVE_PIXEL ? min(kConvAhead, kWave / ntap) : kConvAhead;
  const int l = lane_id();
  const int lp = l / ntap;
  const int ltap = l - lp * ntap;
  const int lky = ltap / (3 * C);
  const int lkx = (ltap / C) % 3;
  const int lc = ltap % C;
  const int lyy = y + lky - 1;
  const int lxx = x + lkx - 1;
  const bool lin = lp < q && lyy >= 0 && lyy < H && lxx >= 0 && lxx < W;
  const size_t loff = ((size_t)(lin ? lyy : 0) * W + (lin ? lxx : 0)) * C + lc;
  const uint64_t tapmask = ntap >= 64 ? ~0ull : ((1ull << ntap) - 1ull);
  float v = 0.0f;
  if (valid) V[k] = 0.0f;
  if (bits) mark_active(bits, wword, valid, v, theta, b_th);
  for (int t0 = 0; t0 < T - 1; t0 += q) {
    const int np = min(q, T - 1 - t0);
    float in[kConvAhead];
    if (WAVE_PIXEL) {
      const bool ld = lin && lp < np;
      const uint64_t m = __ballot(ld && xb[(size_t)(t0 + lp) * in_step + loff] != 0);
#pragma unroll
      for (int p = 0; p < kConvAhead; ++p) {
        float acc = 0.0f;
        if (p < np) {
          uint64_t taps = (m >> (p * ntap)) & tapmask;
          while (taps) {
            const int tap = __builtin_ctzll(taps);
            acc = __fadd_rn(acc, Wc[tap * F + f]);
            taps &= taps - 1ull;
          }
        }
        in[p] = acc;
      }
    } else {
#pragma unroll
      for (int p = 0; p < kConvAhead; ++p) {
        const uint8_t* xt = xb + (size_t)(t0 + min(p, np - 1)) * in_step;
        float acc = 0.0f;
        for (int ky = 0; ky < 3; ++ky) {
          const int yy = y + ky - 1;
          if (yy < 0 || yy >= H) continue;
          for (int kx = 0; kx < 3; ++kx) {
            const int xx = x + kx - 1;
            if (xx < 0 || xx >= W) continue;
            const uint8_t* px = xt + ((size_t)yy * W + xx) * C;
            for (int c = 0; c < C; ++c)
              if (px[c]) acc = __fadd_rn(acc, Wc[((ky * 3 + kx) * C + c) * F + f]);
          }
        }
        in[p] = acc;
      }
    }
#pragma unroll
    for (int p = 0; p < kConvAhead; ++p) {
      if (p < np) {
        const int t = t0 + p;
        const bool sp = v > theta;
        if (valid) s_out[(size_t)t * step + k] = (uint8_t)sp;
        v = __fadd_rn(__fadd_rn(__fmul_rn(alpha, v), in[p]), sp ? -1.0f : -0.0f);
        if (valid) V[(size_t)(t + 1) * step + k] = v;
        if (bits) mark_active(bits, (size_t)(t + 1) * W64 + wword, valid, v, theta, b_th);
      }
    }
  }
  if (valid) s_out[(size_t)(T - 1) * step + k] = (uint8_t)(v > theta);
}

// The convolutional layer a 2x2 pooling window at a time, for F a multiple of 64, C in {1, 2, 4} and even H, W: a
// wavefront owns a window's four pixels x 64 filters, lane = (pixel column dx, filter pair), the two pixel rows in
// registers. Same operations in the same order as conv_scan. A step's 4 x 4 x C patch serves all four pixels (one
// ballot per 64 bytes, the next kPoolSteps steps' bytes in flight), the filters are read from LDS, V leaves in
// 512-byte and the spikes in 128-byte runs. With P != NULL the window's pooled spikes, picks and (with trace_pool)
// the pooled spikes' trace with leak alpha_next are written from the spikes in registers, so that pooling and
// trace read nothing back: the ballot of (row dy, filter parity q) holds the spikes of both pixel columns, and
// lane l takes pooled filter l. Bound: HBM stores (28 x 28 x 64, T = 100, B = 256: 8.4 GB).
// Whole forward there 3.43 -> 1.88 ms: conv_scan 2.18, pooling 0.39 and the pooled trace 0.33 ms before, this
// kernel 1.72 (2.33 with blocks in launch order and plain stores, 1.97 with the XCD order, 1.78 with V and the
// trace streamed past L2).
constexpr int kPoolSteps = 8;
typedef float Pair __attribute__((ext_vector_type(2)));
constexpr size_t kPoolLds = 32 * 1024;

// Every bit of a uniform word twice: bit i goes to bits 2 i and 2 i + 1.
__device__ __forceinline__ uint64_t twice(uint32_t x) {
  uint64_t r;
  asm("s_bitreplicate_b64_b32 %0, %1" : "=s"(r) : "s"(x));
  return r;
}

template <int C>
__global__ __launch_bounds__(kScanThreads) void conv_pool_scan(
    const uint8_t* __restrict__ s_in, const float* __restrict__ Wc, int T, int B, int H, int W, int F, int n_waves,
    float alpha, float theta, float b_th, float* __restrict__ V, uint8_t* __restrict__ s_out,
    uint64_t* __restrict__ bits, uint8_t* __restrict__ P, uint8_t* __restrict__ arg, float* __restrict__ trace_pool,
    float alpha_next) {
  extern __shared__ __attribute__((aligned(16))) float wl[];  // [9 C][F]
  for (int k = threadIdx.x; k < 9 * C * F; k += kScanThreads) wl[k] = Wc[k];
  __syncthreads();
  constexpr int kPatch = 16 * C;                         // bytes of a step's patch
  constexpr int kWords = kPoolSteps * kPatch / kWave;    // ballots per group of steps
  // Blocks are dealt to the 8 XCDs in turn: each XCD takes one contiguous eighth of the windows, so that lines
  // shared by neighbouring windows (bitset words, pooled spikes) fill up in one L2.
  const int nb = gridDim.x;
  const int block = nb % 8 == 0 ? (int)(blockIdx.x & 7) * (nb / 8) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(block * (kScanThreads / kWave) + threadIdx.x / kWave);
  if (wave >= n_waves) return;
  const int l = lane_id();
  const int fgs = F / kWave, hw = W / 2;
  const int fg = wave % fgs;
  const int win = wave / fgs;  // (b * H/2 + py) * W/2 + px
  const int px = win % hw;
  const int py = (win / hw) % (H / 2);
  const int b = win / (hw * (H / 2));
  const int dx = l >> 5, pair = l & 31;
  const int f0 = fg * kWave + 2 * pair;
  const size_t N = (size_t)H * W * F, step = (size_t)B * N, pstep = step / 4;
  const size_t W64 = step / kWave;  // F is a multiple of 64: whole words per pixel
  // offsets inside a step: the lane's neurons of row dy, its pooled neuron, the word of pixel (l >> 1, l & 1)
  const size_t pix0 = (size_t)b * H * W + (size_t)(2 * py) * W + 2 * px;
  const size_t base = pix0 * F;
  const int off0 = dx * F + f0, off1 = off0 + W * F;
  const size_t pbase = (size_t)win * F + fg * kWave;
  const size_t word0 = pix0 * fgs + fg;
  const int woff = ((l >> 1) & 1) * W * fgs + (l & 1) * fgs;
  const size_t in_step = (size_t)B * H * W * C;
  const uint8_t* xb = s_in + (size_t)b * H * W * C;
  // byte of word i that this lane loads: step and place in the patch
  int lstep[kWords], loff[kWords];
  bool lin[kWords];
#pragma unroll
  for (int i = 0; i < kWords; ++i) {
    const int id = i * kWave + l;
    lstep[i] = id / kPatch;
    const int q = id % kPatch;
    const int yy = 2 * py - 1 + q / (4 * C), xx = 2 * px - 1 + (q / C) % 4;
    lin[i] = yy >= 0 && yy < H && xx >= 0 && xx < W;
    loff[i] = lin[i] ? (yy * W + xx) * C + q % C : 0;
  }
  auto load = [&](uint32_t (&x)[kWords], int t0) {
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const int t = t0 + lstep[i];
      x[i] = (lin[i] && t < T - 1) ? xb[(size_t)t * in_step + loff[i]] : 0u;
    }
  };
  float v[2][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};
  float tr = 0.0f;
  auto put_v = [&](int t) {
    float* Vt = V + (size_t)t * step + base;
    // V and the trace are not read again soon and need not take the place of the other lines in L2
    __builtin_nontemporal_store(Pair{v[0][0], v[0][1]}, reinterpret_cast<Pair*>(Vt + off0));
    __builtin_nontemporal_store(Pair{v[1][0], v[1][1]}, reinterpret_cast<Pair*>(Vt + off1));
    if (bits) {
      uint64_t word[4];  // pixel (dy, dx): bit 2 pair + q from lane (dx, pair) of ballot (dy, q)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy) {
        const uint64_t a0 = __ballot(fabsf(v[dy][0] - theta) < b_th), a1 = __ballot(fabsf(v[dy][1] - theta) < b_th);
#pragma unroll
        for (int x = 0; x < 2; ++x)
          word[2 * dy + x] =
              (twice((uint32_t)(a0 >> (32 * x))) & 0x5555555555555555ull) |
              (twice((uint32_t)(a1 >> (32 * x))) & 0xAAAAAAAAAAAAAAAAull);
      }
      const uint64_t mine = l == 0 ? word[0] : (l == 1 ? word[1] : (l == 2 ? word[2] : word[3]));
      if (l < 4) bits[(size_t)t * W64 + word0 + woff] = mine;
    }
  };
  // spikes of step t (and what pooling makes of them); returns them for the recurrence
  auto put_spikes = [&](int t, bool (&sp)[2][2]) {
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int q = 0; q < 2; ++q) sp[dy][q] = v[dy][q] > theta;
    uint8_t* St = s_out + (size_t)t * step + base;
    __builtin_nontemporal_store((uint16_t)((sp[0][0] ? 1 : 0) | (sp[0][1] ? 256 : 0)), reinterpret_cast<uint16_t*>(St + off0));
    __builtin_nontemporal_store((uint16_t)((sp[1][0] ? 1 : 0) | (sp[1][1] ? 256 : 0)), reinterpret_cast<uint16_t*>(St + off1));
    if (P) {
      const uint64_t m00 = __ballot(sp[0][0]), m01 = __ballot(sp[0][1]);
      const uint64_t m10 = __ballot(sp[1][0]), m11 = __ballot(sp[1][1]);
      const uint64_t r0 = l & 1 ? m01 : m00, r1 = l & 1 ? m11 : m10;
      const int k = l >> 1;  // pooled filter l: parity l % 2, pair l / 2
      const bool s0 = ((uint32_t)r0 >> k) & 1u, s1 = ((uint32_t)(r0 >> 32) >> k) & 1u;
      const bool s2 = ((uint32_t)r1 >> k) & 1u, s3 = ((uint32_t)(r1 >> 32) >> k) & 1u;
      const bool any = s0 || s1 || s2 || s3;
      P[(size_t)t * pstep + pbase + l] = (uint8_t)any;
      arg[(size_t)t * pstep + pbase + l] = (uint8_t)(s0 ? 0 : (s1 ? 1 : (s2 ? 2 : (s3 ? 3 : 0))));
      if (trace_pool && t + 1 < T) {
        tr = __fadd_rn(__fmul_rn(alpha_next, tr), any ? 1.0f : 0.0f);
        __builtin_nontemporal_store(tr, trace_pool + (size_t)(t + 1) * pstep + pbase + l);
      }
    }
  };
  put_v(0);
  if (P && trace_pool) trace_pool[pbase + l] = 0.0f;
  uint32_t cur[kWords], nxt[kWords];
  load(cur, 0);
  for (int t0 = 0; t0 < T - 1; t0 += kPoolSteps) {
    load(nxt, t0 + kPoolSteps);
    uint64_t m[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) m[i] = __ballot(cur[i] != 0);
#pragma unroll
    for (int s = 0; s < kPoolSteps; ++s) {
      const int t = t0 + s;
      if (t < T - 1) {
        const uint64_t patch = kPatch == 64 ? m[s * kPatch / kWave]
                                            : (m[s * kPatch / kWave] >> (s * kPatch % kWave)) & ((1ull << (kPatch % 64)) - 1ull);
        float in[2][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};
        if (patch) {  // uniform: most steps of a window see no spike
          uint64_t taps[2];
#pragma unroll
          for (int dy = 0; dy < 2; ++dy) {
            taps[dy] = 0;
#pragma unroll
            for (int r = 0; r < 3; ++r)
              taps[dy] |= ((patch >> (((dy + r) * 4 + dx) * C)) & ((1ull << (3 * C)) - 1ull)) << (3 * C * r);
          }
          while (__ballot((taps[0] | taps[1]) != 0)) {
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
              if (taps[dy]) {
                const float2 wv = *reinterpret_cast<const float2*>(wl + (int)__builtin_ctzll(taps[dy]) * F + f0);
                in[dy][0] = __fadd_rn(in[dy][0], wv.x);
                in[dy][1] = __fadd_rn(in[dy][1], wv.y);
                taps[dy] &= taps[dy] - 1ull;
              }
            }
          }
        }
        bool sp[2][2];
        put_spikes(t, sp);
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            v[dy][q] = __fadd_rn(__fadd_rn(__fmul_rn(alpha, v[dy][q]), in[dy][q]), sp[dy][q] ? -1.0f : -0.0f);
        put_v(t + 1);
      }
    }
#pragma unroll
    for (int i = 0; i < kWords; ++i) cur[i] = nxt[i];
  }
  bool sp[2][2];
  put_spikes(T - 1, sp);
}

// Whether conv_pool_scan takes the layer: shapes and alignments it is written for (its V and spike stores are 8 and
// 2 bytes wide), and enough wavefronts. It has a quarter of conv_scan's, each step's work is in one of them, and
// below one per SIMD that step's latency sets the pace: 200 wavefronts, 100 steps 38 us conv_scan, 57 this one, 800
// 54 and 59, 1156 74 and 67. With the pooling it saves two launches, which outweighs that from half as many on or
// up to 50 steps (200 wavefronts: 20 steps 34 us in three passes, 27 so; 100 steps 63 and 88; 800: 92 and 94).
bool conv_pool_ok(int T, int B, int H, int W, int C, int F, bool pool, const float* V, const uint8_t* s_out) {
  const int64_t waves = (int64_t)B * (H / 2) * (W / 2) * (F / kWave);
  if (waves < (pool ? 2 : 4) * cu_count() && !(pool && T <= 50)) return false;
  return F % kWave == 0 && (C == 1 || C == 2 || C == 4) && H % 2 == 0 && W % 2 == 0 &&
         (size_t)9 * C * F * sizeof(float) <= kPoolLds && reinterpret_cast<uintptr_t>(V) % 8 == 0 &&
         reinterpret_cast<uintptr_t>(s_out) % 2 == 0;
}

void launch_conv_pool(const uint8_t* s_in, const float* Wc, int T, int B, int H, int W, int C, int F, float alpha,
                      float theta, float b_th, float* V, uint8_t* s_out, uint64_t* bits, uint8_t* P, uint8_t* arg,
                      float* trace_pool, float alpha_next, hipStream_t s) {
  const int waves = B * (H / 2) * (W / 2) * (F / kWave);
  const int blocks = (waves + kScanThreads / kWave - 1) / (kScanThreads / kWave);
  const dim3 g((unsigned)(blocks >= 64 ? (blocks + 7) / 8 * 8 : blocks));  // whole eighths (see the kernel)
  const size_t lds = (size_t)9 * C * F * sizeof(float);
#define SNN_CP(C_)                                                                                                \
  hipLaunchKernelGGL(conv_pool_scan<C_>, g, dim3(kScanThreads), lds, s, s_in, Wc, T, B, H, W, F, waves, alpha, theta, \
                     b_th, V, s_out, bits, P, arg, trace_pool, alpha_next)
  if (C == 1) SNN_CP(1);
  else if (C == 2) SNN_CP(2);
  else SNN_CP(4);
#undef SNN_CP
}

// The trace of spikes [T,B,N] alone (lif_scan's trace blocks).
void launch_trace(const uint8_t* s_in, int T, int B, int N, float alpha, float* trace, hipStream_t s) {
  const int nt = (int)(((size_t)B * N + kScanThreads - 1) / kScanThreads);
  hipLaunchKernelGGL(lif_scan, dim3((unsigned)nt), dim3(kScanThreads), 0, s, s_in, T, B, N, 1, alpha, 0.0f, 0.0f,
                     nullptr, nullptr, trace, nullptr, 1.0f, nullptr, 0);
}

snn_status lif_forward_impl(const uint8_t* s_in, const float* W, int T, int B, int N_in, int N_out, float alpha,
                            float theta, float b_th, float* V, uint8_t* s_out, float* trace_in, float* trace_out,
                            float alpha_next, uint64_t* bits, void* stream) {
  if (!s_in || !W || !V || !s_out) return SNN_ERR_INVALID_ARG;
  if (bad_dim(T) || bad_dim(B) || bad_dim(N_in) || bad_dim(N_out)) return SNN_ERR_INVALID_ARG;
  if (too_big(T, B, N_in) || too_big(T, B, N_out)) return SNN_ERR_INVALID_ARG;
  if (bad_alpha(alpha) || isnan(theta)) return SNN_ERR_INVALID_ARG;
  if (bits && (isnan(b_th) || b_th < 0.0f)) return SNN_ERR_INVALID_ARG;
  if (trace_out && bad_alpha(alpha_next)) return SNN_ERR_INVALID_ARG;
  if (N_out > 16 * 4 * kWave) return SNN_ERR_UNSUPPORTED;

  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool al = (N_in % 4) == 0 && (reinterpret_cast<uintptr_t>(s_in) % 4) == 0;
  {  // the fused kernel: whole float4 W columns, whole bitset words per wavefront, a 16-byte aligned trace,
     // and at least two blocks per CU (with fewer, its time walk is latency-bound and the two-kernel
     // form is faster: a 1024 -> 100 readout at T = 500, B = 256, 5% input spikes, takes 0.61 against
     // 0.46 ms)
    const int fq = N_out > 4 * kWave ? 2 : 1;
    const int G = (N_out + 4 * kWave * fq - 1) / (4 * kWave * fq);
    if ((N_out % 4) == 0 && (reinterpret_cast<uintptr_t>(W) % 16) == 0 && (!bits || N_out % kWave == 0) &&
        (!trace_in || !al || (reinterpret_cast<uintptr_t>(trace_in) % 16) == 0) &&
        (int64_t)B * G >= 2 * (int64_t)cu_count()) {
      // the trace from the tile's stashed spike bytes when a row is one segment and the group's input
      // quads fit one per thread; otherwise trace blocks beside the fused blocks
      const bool stash = al && N_in <= kSegPieces * kPiece && ((N_in + 3) / 4 + G - 1) / G <= kFuseThreads;
      const int nfb = B * G;
      const int ntb = (trace_in && !stash) ? (int)(((size_t)B * ((N_in + 3) / 4) + kFuseThreads - 1) / kFuseThreads) : 0;
      const dim3 g((unsigned)(nfb + ntb));
#define SNN_F(A, Q, ST)                                                                                              \
  do {                                                                                                               \
    if (trace_out)                                                                                                   \
      hipLaunchKernelGGL((lif_fused<A, Q, ST, true>), g, dim3(kFuseThreads), 0, s, s_in, W, T, B, N_in, N_out, G,     \
                         nfb, alpha, theta, b_th, V, s_out, trace_in, trace_out, alpha_next, bits);                  \
    else                                                                                                             \
      hipLaunchKernelGGL((lif_fused<A, Q, ST, false>), g, dim3(kFuseThreads), 0, s, s_in, W, T, B, N_in, N_out, G,    \
                         nfb, alpha, theta, b_th, V, s_out, trace_in, nullptr, 1.0f, bits);                          \
  } while (0)
      if (stash && fq == 2) SNN_F(true, 2, true);
      else if (stash) SNN_F(true, 1, true);
      else if (al && fq == 2) SNN_F(true, 2, false);
      else if (al) SNN_F(true, 1, false);
      else if (fq == 2) SNN_F(false, 2, false);
      else SNN_F(false, 1, false);
#undef SNN_F
      return launch_status();
    }
  }
  const bool vec = (N_out % 4) == 0 && (reinterpret_cast<uintptr_t>(W) % 16) == 0 &&
                   (reinterpret_cast<uintptr_t>(V) % 16) == 0;
  const int NQ = (N_out + 4 * kWave - 1) / (4 * kWave);
  const long rows = (long)(T - 1) * B;
  const auto multiple = [&](int b) { return N_in % b == 0 && reinterpret_cast<uintptr_t>(s_in) % b == 0; };
  if (rows > 0 && N_out <= kNarrowCols && multiple(4) && N_in <= 65536) {
    const int lanes = N_out <= 16 ? 16 : 32;
    const int per_block = kGatherWaves * (kWave / lanes);
    const dim3 g((unsigned)((rows + per_block - 1) / per_block));
#define SNN_GN(LB, L)                                                                                             \
  hipLaunchKernelGGL((lif_gather_narrow<LB, L>), g, dim3(kGatherWaves * kWave), 0, s, s_in, W, T, B, N_in, N_out, V)
    if (multiple(16)) {
      if (lanes == 16) SNN_GN(16, 16); else SNN_GN(16, 32);
    } else if (multiple(8)) {
      if (lanes == 16) SNN_GN(8, 16); else SNN_GN(8, 32);
    } else {
      if (lanes == 16) SNN_GN(4, 16); else SNN_GN(4, 32);
    }
#undef SNN_GN
  } else if (rows > 0) {
    const dim3 g((unsigned)((rows + kGatherWaves - 1) / kGatherWaves));
    if (al && vec) launch_gather<true, true>(NQ, g, s, s_in, W, T, B, N_in, N_out, V);
    else if (al) launch_gather<true, false>(NQ, g, s, s_in, W, T, B, N_in, N_out, V);
    else if (vec) launch_gather<false, true>(NQ, g, s, s_in, W, T, B, N_in, N_out, V);
    else launch_gather<false, false>(NQ, g, s, s_in, W, T, B, N_in, N_out, V);
  }
  const int nv = (int)(((size_t)B * N_out + kScanThreads - 1) / kScanThreads);
  const int nt = trace_in ? (int)(((size_t)B * N_in + kScanThreads - 1) / kScanThreads) : 0;
  hipLaunchKernelGGL(lif_scan, dim3((unsigned)(nv + nt)), dim3(kScanThreads), 0, s, s_in, T, B, N_in, N_out, alpha,
                     theta, b_th, V, s_out, trace_in, trace_out, alpha_next, bits, nv);
  return launch_status();
}

}  // namespace

extern "C" snn_status snn_lif_forward(const uint8_t* s_in, const float* W, int T, int B, int N_in, int N_out,
                                      float alpha, float theta, float* V, uint8_t* s_out, float* trace_in,
                                      void* stream) {
  return lif_forward_impl(s_in, W, T, B, N_in, N_out, alpha, theta, 0.0f, V, s_out, trace_in, nullptr, 1.0f,
                          nullptr, stream);
}

extern "C" size_t snn_active_bits_words(int T, int B, int N) {
  if (bad_dim(T) || bad_dim(B) || bad_dim(N) || too_big(T, B, N)) return 0;
  return (size_t)T * (((size_t)B * N + kWave - 1) / kWave);
}

extern "C" snn_status snn_lif_forward_active(const uint8_t* s_in, const float* W, int T, int B, int N_in, int N_out,
                                             float alpha, float theta, float b_th, float* V, uint8_t* s_out,
                                             float* trace_in, uint64_t* active_bits, void* stream) {
  if (!active_bits) return SNN_ERR_INVALID_ARG;
  return lif_forward_impl(s_in, W, T, B, N_in, N_out, alpha, theta, b_th, V, s_out, trace_in, nullptr, 1.0f,
                          active_bits, stream);
}

extern "C" snn_status snn_lif_forward_traces(const uint8_t* s_in, const float* W, int T, int B, int N_in,
                                             int N_out, float alpha, float theta, float b_th, float* V,
                                             uint8_t* s_out, float* trace_in, float* trace_out,
                                             float alpha_next, uint64_t* active_bits, void* stream) {
  return lif_forward_impl(s_in, W, T, B, N_in, N_out, alpha, theta, b_th, V, s_out, trace_in, trace_out, alpha_next,
                          active_bits, stream);
}

namespace {

// snn_conv_lif_forward, and with P the pooling and the pooled trace.
snn_status conv_forward_impl(const uint8_t* s_in, const float* Wc, int T, int B, int H, int W, int C, int F, float alpha,
                             float theta, float b_th, float* V, uint8_t* s_out, float* trace_in, uint64_t* active_bits,
                             uint8_t* P, uint8_t* arg, float* trace_pool, float alpha_next, void* stream) {
  if (!s_in || !Wc || !V || !s_out) return SNN_ERR_INVALID_ARG;
  if (bad_dim(T) || bad_dim(B) || bad_dim(H) || bad_dim(W) || bad_dim(C) || bad_dim(F)) return SNN_ERR_INVALID_ARG;
  if ((int64_t)H * W * F >= ((int64_t)1 << 31) || (int64_t)H * W * C >= ((int64_t)1 << 31)) return SNN_ERR_INVALID_ARG;
  if (too_big(T, B, H * W * F) || too_big(T, B, H * W * C)) return SNN_ERR_INVALID_ARG;
  if (bad_alpha(alpha) || isnan(theta)) return SNN_ERR_INVALID_ARG;
  if (active_bits && (isnan(b_th) || b_th < 0.0f)) return SNN_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool fused = conv_pool_ok(T, B, H, W, C, F, P != nullptr, V, s_out);
  if (fused) {
    launch_conv_pool(s_in, Wc, T, B, H, W, C, F, alpha, theta, b_th, V, s_out, active_bits, P, arg, trace_pool,
                     alpha_next, s);
  } else {
    const int nv = (int)(((size_t)B * H * W * F + kScanThreads - 1) / kScanThreads);
    if (F % kWave == 0 && 9 * C <= kWave)  // a wavefront's lanes are the filters of one pixel
      hipLaunchKernelGGL(conv_scan<true>, dim3((unsigned)nv), dim3(kScanThreads), 0, s, s_in, Wc, T, B, H, W, C, F,
                         alpha, theta, b_th, V, s_out, active_bits);
    else
      hipLaunchKernelGGL(conv_scan<false>, dim3((unsigned)nv), dim3(kScanThreads), 0, s, s_in, Wc, T, B, H, W, C, F,
                         alpha, theta, b_th, V, s_out, active_bits);
  }
  if (trace_in) launch_trace(s_in, T, B, H * W * C, alpha, trace_in, s);
  if (P && !fused) {
    const snn_status st = snn_maxpool_spikes(s_out, T, B, H, W, F, P, arg, stream);
    if (st != SNN_OK) return st;
    if (trace_pool) launch_trace(P, T, B, (H / 2) * (W / 2) * F, alpha_next, trace_pool, s);
  }
  return launch_status();
}

}  // namespace

extern "C" snn_status snn_conv_lif_forward(const uint8_t* s_in, const float* Wc, int T, int B, int H, int W, int C,
                                           int F, float alpha, float theta, float b_th, float* V, uint8_t* s_out,
                                           float* trace_in, uint64_t* active_bits, void* stream) {
  return conv_forward_impl(s_in, Wc, T, B, H, W, C, F, alpha, theta, b_th, V, s_out, trace_in, active_bits, nullptr,
                           nullptr, nullptr, 1.0f, stream);
}

extern "C" int snn_conv_forward_pools(int T, int B, int H, int W, int C, int F) {
  if (bad_dim(T) || bad_dim(B) || bad_dim(H) || bad_dim(W) || bad_dim(C) || bad_dim(F)) return 0;
  return conv_pool_ok(T, B, H, W, C, F, true, nullptr, nullptr) ? 1 : 0;
}

extern "C" snn_status snn_conv_lif_forward_pool(const uint8_t* s_in, const float* Wc, int T, int B, int H, int W,
                                                int C, int F, float alpha, float theta, float b_th, float* V,
                                                uint8_t* s_out, float* trace_in, uint64_t* active_bits, uint8_t* P,
                                                uint8_t* arg, float* trace_pool, float alpha_next, void* stream) {
  if (!P || !arg || H % 2 != 0 || W % 2 != 0) return SNN_ERR_INVALID_ARG;
  if (trace_pool && bad_alpha(alpha_next)) return SNN_ERR_INVALID_ARG;
  return conv_forward_impl(s_in, Wc, T, B, H, W, C, F, alpha, theta, b_th, V, s_out, trace_in, active_bits, P, arg,
                           trace_pool, alpha_next, stream);
}

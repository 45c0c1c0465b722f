// Dense float32 matrix products on the bf16 matrix cores, each operand split into three bf16 parts.
//
// x = h + m + l with h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), all rounded to nearest: three
// times 8 significant bits hold a float32's 24. A product takes the six terms down to 2^-16 of the
// leading one (hh, hm, mh, mm, hl, lh; what is left out is below 2^-24 of |x||y|), and the matrix cores
// form 16-bit products exactly and sum them in float32. hh goes to one accumulator and the five small
// terms to another, so the leading sum is rounded once per 8 products of K (a float32 MFMA chain: once
// per 1 or 2). The operands are scaled by 2^24, so that the parts of every float32 value are normal bf16
// values; a sum that comes out infinite or NaN (an operand of 2^104 and more, an infinity or a NaN, a sum of 2^80
// and more) makes its block form the tile again on the float32 matrix cores.
//
// Bound: the matrix cores, six bf16 products per float32 one (2.5 PFLOP/s / 6 = 417 TFLOP/s of useful
// work at the nominal rate; the float32 MFMA's nominal rate is 157). A block of four wavefronts owns
// 128 x 128 of C, a wavefront 64 x 64 (4 x 4 tiles of v_mfma_f32_16x16x32_bf16). A stage of 32 k is
// loaded into registers while the previous one is multiplied, split there and stored to LDS as
// [part][k / 8][row] pieces of 16 bytes, which the fragment reads (lane = row, 8 consecutive k) take
// without bank conflicts; two blocks per CU overlap one's split with the other's products. Measured at
// 128000 x 1024 x 1024: 1.55 (k down the rows) and 1.46 ms, 173 and 184 TFLOP/s (1040 and 1100 in bf16
// terms; a large bf16 product of the library reaches 1290 on this card), 1.75 ms with the six terms of
// a tile issued one after another; tiles of 32 x 32 x 16 are 1% slower. Error against 64 bits with 16000
// products of random sign per sum: 0.8e-6 of the result, float32 MFMA 3.3e-6.
#include "common.h"

namespace snn {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBM = 128, kBN = 128, kBK = 32;
constexpr int kThreads = 256;
constexpr int kKC = kBK / 8;      // pieces of 8 k per row and stage
// Operands are taken times 2^24: the parts of every float32, down to the last bit of the smallest subnormal, are
// then normal bf16 values (unscaled, values below 2^-109 lose bits of the third part, below 2^-117 of the second).
// Sums come out times 2^48. A value that scaled rounds past bf16's range (2^104 and half a bf16 step below it) has an
// infinite or NaN part, and every sum it enters is infinite or NaN (infinity times 0 included).
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;

// Eight values into their three parts, 16 bytes each.
__device__ __forceinline__ void split8(const float (&x)[8], uint4& h, uint4& m, uint4& l) {
  uint32_t hp[4], mp[4], lp[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float a = x[2 * q], b = x[2 * q + 1];
    hp[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
    const float ra = a - __uint_as_float(hp[q] << 16), rb = b - __uint_as_float(hp[q] & 0xffff0000u);
    mp[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{ra, rb}), bf16x2));
    const float sa = ra - __uint_as_float(mp[q] << 16), sb = rb - __uint_as_float(mp[q] & 0xffff0000u);
    lp[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{sa, sb}), bf16x2));
  }
  h = make_uint4(hp[0], hp[1], hp[2], hp[3]);
  m = make_uint4(mp[0], mp[1], mp[2], mp[3]);
  l = make_uint4(lp[0], lp[1], lp[2], lp[3]);
}

// One operand's share of a stage of ROWS (128 or 64) rows: two pieces or one (8 k of one row each) per thread.
//   KM: element (r, k) at p[k * ld + r] (rows contiguous): a piece is eight loads, each 256 contiguous
//       bytes over a wavefront.
//   else p[r * ld + k] (k contiguous): a piece is 32 contiguous bytes.
// Rows past the end read the last row (their results are not stored); k past k_hi reads as 0.
template <bool KM, int ROWS>
__device__ __forceinline__ void piece_of(int q, int& row, int& kc) {
  const int idx = threadIdx.x + kThreads * q;
  row = KM ? idx % ROWS : idx / kKC;
  kc = KM ? idx / ROWS : idx % kKC;
}

template <bool KM, bool VEC, int ROWS>
__device__ __forceinline__ void load_stage(const float* __restrict__ p, int ld, int r0, int R, int k0, int k_hi,
                                           float (&x)[ROWS / 64][8]) {
#pragma unroll
  for (int q = 0; q < ROWS / 64; ++q) {
    int row, kc;
    piece_of<KM, ROWS>(q, row, kc);
    const int r = min(r0 + row, R - 1);
    const int k = k0 + 8 * kc;
    if (KM) {
      if (k + 8 <= k_hi) {
#pragma unroll
        for (int u = 0; u < 8; ++u) x[q][u] = p[(size_t)(k + u) * ld + r];
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) x[q][u] = k + u < k_hi ? p[(size_t)(k + u) * ld + r] : 0.0f;
      }
    } else {
      const float* s = p + (size_t)r * ld + k;
      if (VEC && k + 8 <= k_hi) {
        const float4 a = *reinterpret_cast<const float4*>(s), b = *reinterpret_cast<const float4*>(s + 4);
        x[q][0] = a.x; x[q][1] = a.y; x[q][2] = a.z; x[q][3] = a.w;
        x[q][4] = b.x; x[q][5] = b.y; x[q][6] = b.z; x[q][7] = b.w;
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) x[q][u] = k + u < k_hi ? s[u] : 0.0f;
      }
    }
  }
}

// [part][k / 8][row] pieces; a line holds two more than its rows (the lines' stores spread over the banks).
template <int ROWS>
struct Stage {
  uint4 x[3][kKC][ROWS + 2];
};

template <bool KM, int ROWS>
__device__ __forceinline__ void store_stage(Stage<ROWS>& S, const float (&x)[ROWS / 64][8], float up) {
#pragma unroll
  for (int q = 0; q < ROWS / 64; ++q) {
    int row, kc;
    piece_of<KM, ROWS>(q, row, kc);
    float y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) y[u] = x[q][u] * up;
    split8(y, S.x[0][kc][row], S.x[1][kc][row], S.x[2][kc][row]);
  }
}

// The same stage as float32 lines [k][row], for a tile with a value out of the split's range.
template <int ROWS>
struct WideStage {
  float x[kBK][ROWS + 4];
};
static_assert(sizeof(WideStage<128>) <= sizeof(Stage<128>) && sizeof(WideStage<64>) <= sizeof(Stage<64>),
              "the float32 stage fits the split one's LDS");

template <bool KM, int ROWS>
__device__ __forceinline__ void store_wide(WideStage<ROWS>& S, const float (&x)[ROWS / 64][8]) {
#pragma unroll
  for (int q = 0; q < ROWS / 64; ++q) {
    int row, kc;
    piece_of<KM, ROWS>(q, row, kc);
#pragma unroll
    for (int u = 0; u < 8; ++u) S.x[8 * kc + u][row] = x[q][u];
  }
}

// A block's tile of C and its K slice z. Blocks are dealt to the 8 XCDs in turn. Short M and N, long K:
// the tiles of one slice run on one XCD and share its rows in that L2 (slices a multiple of 8: the XCDs
// get equally many). Long M: the N tiles of one M tile run on one XCD (32 M tiles and more, so that the
// last round of eight does not decide).
struct BlockTile {
  int tm, tn, z;
  bool ok;
};

__device__ __forceinline__ BlockTile slice_tile(int tiles_m, int tiles_n, int splits) {
  const int tiles = tiles_m * tiles_n;
  const int j = splits % 8 == 0 ? (int)blockIdx.x >> 3 : (int)blockIdx.x;
  const int z = splits % 8 == 0 ? (int)(blockIdx.x & 7) + 8 * (j / tiles) : j / tiles;
  const int t = j % tiles;
  return {t / tiles_n, t % tiles_n, z, z < splits};
}

__device__ __forceinline__ BlockTile row_tile(int tiles_m, int tiles_n) {
  const int j = tiles_m >= 32 ? (int)blockIdx.x >> 3 : (int)blockIdx.x;
  const int tm = tiles_m >= 32 ? (int)(blockIdx.x & 7) + 8 * (j / tiles_n) : j / tiles_n;
  return {tm, j % tiles_n, 0, tm < tiles_m};
}

// C[M x N] = sum over this block's K slice of A(m, k) B(k, n); slice z goes to C + z * c_split.
// GATHER: only the elements (r, col_idx[e]) of a CSR's entries e are wanted (row r = m of its T*B rows,
// columns ascending in a row) and go to out[e]. The block finds its rows' entries in its columns by
// bisection, passes its tile through LDS 64 rows at a time and reads the entries' elements there. Its tile
// is 128 x 64, and every 64 k its sums are moved to float64 registers (the matrix cores round the running
// sum every 8 k): the error stays below that of a wavefront's float32 dot product (1024 terms of a trained-like
// layer: 0.7e-7 of the result against 0.9e-7; 1.2e-7 with float32 totals per 256 k). The matrix cores round
// downwards, whatever the sign: a mean error of -4.6e-9 of the result's root mean square, which dW of the layer
// below (a sum over all rows of positive traces) adds up coherently. A's sign turns from one fold and one tile of
// rows to the next, so that it cancels (dW of the first of three 1024 x 1024 layers, 27% active: 1.89e-7 -> 1.51e-7
// of the result from 64 bits; 1.80e-7 entry by entry).
template <bool KM, bool VEC, bool GATHER>
__global__ __launch_bounds__(kThreads, 2) void gemm_split3(int M, int N, int K, const float* __restrict__ A, int lda,
                                                           const float* __restrict__ B, int ldb,
                                                           float* __restrict__ C, int ldc, int k_per_split,
                                                           size_t c_split, int tiles_m, int tiles_n, int splits,
                                                           GatherOut to, Gate gate) {
  if (!gate_open(gate)) return;
  constexpr int TN = GATHER ? 2 : 4;  // 16-wide column tiles of a wavefront
  constexpr int BN = 32 * TN;
  constexpr int kFold = 2;  // GATHER: stages between two moves to the float64 sums
  __shared__ __attribute__((aligned(16))) char lds[sizeof(Stage<kBM>) + sizeof(Stage<BN>)];
  __shared__ int range[GATHER ? 2 * kBM : 1];  // entries of the tile's rows in its columns: [range[r], range[kBM + r])
  Stage<kBM>& As = *reinterpret_cast<Stage<kBM>*>(lds);
  Stage<BN>& Bs = *reinterpret_cast<Stage<BN>*>(lds + sizeof(Stage<kBM>));
  const int w = threadIdx.x / kWave;
  const int l = threadIdx.x % kWave;
  const BlockTile bt = KM ? slice_tile(tiles_m, tiles_n, splits) : row_tile(tiles_m, tiles_n);
  if (!bt.ok) return;
  const int m0 = bt.tm * kBM, n0 = bt.tn * BN;
  const int wm = (w / 2) * 64, wn = (w % 2) * (BN / 2);
  const int lr = l % 16, lk = l / 16;

  if (GATHER) {  // one bound of one row per thread; the first and last tile also take columns outside [0, N)
    const int r = m0 + (int)threadIdx.x % kBM;
    const bool upper = threadIdx.x >= kBM;
    int lo = 0;
    if (r < M) {
      const auto clamped = [&](int v) { return (int)(v < 0 ? 0 : (v > to.cap ? to.cap : v)); };
      const int a = clamped(to.row_ptr[r]);
      const int z = max(a, clamped(to.row_ptr[r + 1]));
      const int want = upper ? n0 + BN : n0;
      int hi = z;
      lo = a;
      if (upper && bt.tn == tiles_n - 1) lo = z;
      if (!upper && bt.tn == 0) hi = a;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (to.col_idx[mid] < want) lo = mid + 1; else hi = mid;
      }
    }
    range[threadIdx.x] = lo;
  }

  const int k_lo = bt.z * k_per_split;
  const int k_hi = min(K, k_lo + k_per_split);
  f32x4 lead[4][TN], rest[4][TN];
  const auto clear = [&]() {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b) lead[a][b] = rest[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  clear();
  double total[4][GATHER ? TN : 1][4];
  float up = GATHER && (bt.tm & 1) ? -kUp : kUp;  // A's scale; GATHER: its sign turns with every fold
  const auto fold = [&](double down) {  // the sums times down into the float64 totals
    if constexpr (GATHER) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            total[a][b][v] = fma((double)lead[a][b][v] + (double)rest[a][b][v], down, total[a][b][v]);
      clear();
    }
  };
  const auto fold_scaled = [&]() {
    fold(up < 0.0f ? -(double)kDown : (double)kDown);
    if (GATHER) up = -up;
  };
  const auto clear_total = [&]() {
    if constexpr (GATHER) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) total[a][b][v] = 0.0;
    }
  };
  clear_total();

  float xa[2][8], xb[BN / 64][8];
  if (k_lo < k_hi) {
    load_stage<KM, VEC, kBM>(A, lda, m0, M, k_lo, k_hi, xa);
    load_stage<KM, VEC, BN>(B, ldb, n0, N, k_lo, k_hi, xb);
  }
  int stage = 0;
  for (int k0 = k_lo; k0 < k_hi; k0 += kBK) {
    store_stage<KM, kBM>(As, xa, up);
    store_stage<KM, BN>(Bs, xb, kUp);
    __syncthreads();
    if (k0 + kBK < k_hi) {
      load_stage<KM, VEC, kBM>(A, lda, m0, M, k0 + kBK, k_hi, xa);
      load_stage<KM, VEC, BN>(B, ldb, n0, N, k0 + kBK, k_hi, xb);
    }
    bf16x8 fa[3][4];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int a = 0; a < 4; ++a) fa[p][a] = __builtin_bit_cast(bf16x8, As.x[p][lk][wm + 16 * a + lr]);
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      bf16x8 fb[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) fb[p] = __builtin_bit_cast(bf16x8, Bs.x[p][lk][wn + 16 * b + lr]);
      // smallest terms first; neighbours in the issue order go to different accumulators
      constexpr int kTerm[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          f32x4& acc = t == 5 ? lead[a][b] : rest[a][b];
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[kTerm[t][0]][a], fb[kTerm[t][1]], acc, 0, 0, 0);
        }
    }
    if (GATHER && ++stage % kFold == 0) fold_scaled();
    __syncthreads();
  }
  fold_scaled();
  float down = kDown;
  // a sum that is not finite (a value or products out of the split's range, in several terms perhaps as opposite
  // infinities; or a NaN of the operands): the same sums in float32
  bool again = false;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (GATHER) again |= !(fabs(total[a][b][v]) < INFINITY);
        else again |= !(fabsf(lead[a][b][v] + rest[a][b][v]) < INFINITY);
      }
  if (__syncthreads_or(again)) {
    WideStage<kBM>& Aw = *reinterpret_cast<WideStage<kBM>*>(&As);
    WideStage<BN>& Bw = *reinterpret_cast<WideStage<BN>*>(&Bs);
    clear();
    clear_total();
    down = 1.0f;
    for (int k0 = k_lo; k0 < k_hi; k0 += kBK) {
      load_stage<KM, VEC, kBM>(A, lda, m0, M, k0, k_hi, xa);
      load_stage<KM, VEC, BN>(B, ldb, n0, N, k0, k_hi, xb);
      store_wide<KM, kBM>(Aw, xa);
      store_wide<KM, BN>(Bw, xb);
      __syncthreads();
      for (int k = 0; k < kBK; k += 4)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            lead[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(Aw.x[k + lk][wm + 16 * a + lr],
                                                             Bw.x[k + lk][wn + 16 * b + lr], lead[a][b], 0, 0, 0);
      fold(1.0);  // after every stage: float32 products are rounded into the running sum one by one
      __syncthreads();
    }
  }

  // accumulator layout of 16x16: register v of lane l holds row 4 (l / 16) + v, column l % 16
  if constexpr (!GATHER) {
    float* Cz = C + (size_t)bt.z * c_split;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = m0 + wm + 16 * a + 4 * lk + v;
          const int n = n0 + wn + 16 * b + lr;
          if (m < M && n < N) Cz[(size_t)m * ldc + n] = (lead[a][b][v] + rest[a][b][v]) * down;
        }
  } else {
    float(*tile)[BN + 4] = reinterpret_cast<float(*)[BN + 4]>(lds);
    static_assert(64 * (BN + 4) * sizeof(float) <= sizeof(lds), "half a tile of C fits the stages' LDS");
    for (int half = 0; half < 2; ++half) {
      if (w / 2 == half) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) tile[16 * a + 4 * lk + v][wn + 16 * b + lr] = (float)total[a][b][v];
      }
      __syncthreads();
      constexpr int kRows = 4;  // rows of a wavefront in flight
      for (int r0 = 16 * w; r0 < 16 * w + 16; r0 += kRows) {
        int lo[kRows], hi[kRows], n = 0;
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          lo[u] = range[64 * half + r0 + u];
          hi[u] = range[kBM + 64 * half + r0 + u];
          n = max(n, hi[u] - lo[u]);
        }
        for (int x = l; x - l < n; x += kWave) {
          int c[kRows];
#pragma unroll
          for (int u = 0; u < kRows; ++u) c[u] = lo[u] + x < hi[u] ? to.col_idx[lo[u] + x] : -1;
#pragma unroll
          for (int u = 0; u < kRows; ++u) {
            const int k = c[u] - n0;
            const float v = ((unsigned)k < (unsigned)BN && c[u] < N) ? tile[r0 + u][k] : 0.0f;
            if (lo[u] + x < hi[u]) to.out[lo[u] + x] = v;
          }
        }
      }
      __syncthreads();  // the tile is rewritten by the other half
    }
  }
}

// C[M x N] = sum over this block's K slice of A(k, m) B(k, n), float32 operands with their products and
// sums in float64 (v_mfma_f64_16x16x4_f64), each slice rounded to float32 once. Bound: the float64 matrix
// cores (78.6 TFLOP/s nominal; 1024 x 1024 x 128000 takes 4.23 ms, 63 TFLOP/s, the library's 4096^3 product
// 68); converting the operands costs one instruction per 16 x 4 fragment.
// Block 128 x 128, wavefront 64 x 64 (4 x 4 tiles), stages of 16 k double buffered in LDS; lines of 144
// floats put the four k of a fragment on different banks.
constexpr int kDK = 16;
constexpr int kDLd = kBM + 16;
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <bool VEC>
__global__ __launch_bounds__(kThreads, 2) void gemm_f64(int M, int N, int K, const float* __restrict__ A, int lda,
                                                        const float* __restrict__ B, int ldb, float* __restrict__ C,
                                                        int ldc, int k_per_split, size_t c_split, int tiles_m,
                                                        int tiles_n, int splits, Gate gate) {
  if (!gate_open(gate)) return;
  __shared__ __attribute__((aligned(16))) float As[2][kDK][kDLd], Bs[2][kDK][kDLd];
  const int w = threadIdx.x / kWave;
  const int l = threadIdx.x % kWave;
  const BlockTile bt = slice_tile(tiles_m, tiles_n, splits);
  if (!bt.ok) return;
  const int m0 = bt.tm * kBM, n0 = bt.tn * kBN, z = bt.z;
  const int k_lo = z * k_per_split;
  const int k_hi = min(K, k_lo + k_per_split);
  const int wm = (w / 2) * 64, wn = (w % 2) * 64;
  const int lr = l % 16, lk = l / 16;
  f64x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // a thread's part of a stage: lines tid / 32 and 8 + tid / 32, four columns
  const int c4 = 4 * (threadIdx.x % 32), ln = threadIdx.x / 32;
  float4 xa[2], xb[2];
  auto load = [&](const float* __restrict__ p, int ld, int c0, int R, int k0, float4 (&x)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = k0 + ln + 8 * q;
      const float* row = p + (size_t)min(k, k_hi - 1) * ld;
      const int c = c0 + c4;
      if (VEC && c + 4 <= R) {
        x[q] = *reinterpret_cast<const float4*>(row + c);
      } else {  // columns past the end read the last one (their results are not stored)
        x[q] = make_float4(row[min(c, R - 1)], row[min(c + 1, R - 1)], row[min(c + 2, R - 1)], row[min(c + 3, R - 1)]);
      }
      if (k >= k_hi) x[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  };
  if (k_lo < k_hi) {
    load(A, lda, m0, M, k_lo, xa);
    load(B, ldb, n0, N, k_lo, xb);
  }
  int cur = 0;
  for (int k0 = k_lo; k0 < k_hi; k0 += kDK, cur ^= 1) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<float4*>(&As[cur][ln + 8 * q][c4]) = xa[q];
      *reinterpret_cast<float4*>(&Bs[cur][ln + 8 * q][c4]) = xb[q];
    }
    __syncthreads();  // one barrier per stage: the next stage is stored to the other buffer
    if (k0 + kDK < k_hi) {
      load(A, lda, m0, M, k0 + kDK, xa);
      load(B, ldb, n0, N, k0 + kDK, xb);
    }
#pragma unroll
    for (int ks = 0; ks < kDK; ks += 4) {
      double fa[4], fb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        fa[q] = (double)As[cur][ks + lk][wm + 16 * q + lr];
        fb[q] = (double)Bs[cur][ks + lk][wn + 16 * q + lr];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
  }
  // register v of lane l holds row 4 v + l / 16, column l % 16 of its 16 x 16 tile
  float* Cz = C + (size_t)z * c_split;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + wm + 16 * a + 4 * v + lk;
        const int n = n0 + wn + 16 * b + lr;
        if (m < M && n < N) Cz[(size_t)m * ldc + n] = (float)acc[a][b][v];
      }
}

}  // namespace

// Two blocks of 128 x 128 fit a CU, and the product takes as long as the CU with the most blocks: the splits are
// those with the least time by that count (a block alone on its CU keeps the matrix cores about three quarters
// busy). Splits that are no multiple of 8 lose slice_tile's L2 sharing (5%). Against "about two blocks per CU,
// rounded to a multiple of 8", a sparse dW on the float64 product (with writing G): 76800 x 2312 x 200 3.12 ->
// 1.82 ms (304 blocks before), 25600 x 1500 x 900 2.08 -> 1.54 (576), 25600 x 784 x 1300 1.71 -> 1.22 (539); a
// dense backward of these layers 1.43 -> 1.26, 1.09 -> 1.03 and 0.96 -> 0.86 ms.
SplitPlan plan_splits(int M, int N, int K, double mac_rate) {
  const int tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN);
  const int cus = cu_count();
  SplitPlan best{1, 0.0};
  for (int s = 1; s <= 64 && (s == 1 || s <= K / 256); ++s) {
    const int64_t blocks = (int64_t)s * tiles;
    const double per_cu = blocks <= cus ? 1.35 : (double)((blocks + cus - 1) / cus);
    const double product = per_cu * ((K + s - 1) / s) * kBM * kBN * cus / mac_rate;
    const double t = product * (s % 8 ? 1.05 : 1.0) + (s > 1 ? 5e-6 + (double)s * M * N * 8.0 / 4e12 : 0.0);
    if (s == 1 || t < best.seconds) best = {s, t};
  }
  return best;
}

void gemm_split_km(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc, int splits,
                   size_t c_split, hipStream_t s) {
  const int tm = (M + kBM - 1) / kBM, tn = (N + kBN - 1) / kBN;
  int kps = (K + splits - 1) / splits;
  kps = (kps + kBK - 1) / kBK * kBK;
  hipLaunchKernelGGL((gemm_split3<true, false, false>), dim3((unsigned)(splits * tm * tn)), dim3(kThreads), 0, s, M, N,
                     K, A, lda, B, ldb, C, ldc, kps, c_split, tm, tn, splits, GatherOut{}, Gate{});
}

namespace {

template <bool GATHER>
void launch_kc(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc,
               const GatherOut& to, const Gate& gate, hipStream_t s) {
  const int bn = GATHER ? kBN / 2 : kBN;
  const int tm = (M + kBM - 1) / kBM, tn = (N + bn - 1) / bn;
  const bool vec = lda % 4 == 0 && ldb % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(B) % 16 == 0;
  const int kps = (K + kBK - 1) / kBK * kBK;
  const dim3 g((unsigned)((tm >= 32 ? (tm + 7) / 8 * 8 : tm) * tn));
  if (vec)
    hipLaunchKernelGGL((gemm_split3<false, true, GATHER>), g, dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc,
                       kps, 0, tm, tn, 1, to, gate);
  else
    hipLaunchKernelGGL((gemm_split3<false, false, GATHER>), g, dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc,
                       kps, 0, tm, tn, 1, to, gate);
}

}  // namespace

void gemm_split_kc(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc,
                   hipStream_t s) {
  launch_kc<false>(M, N, K, A, lda, B, ldb, C, ldc, GatherOut{}, Gate{}, s);
}

void gemm_split_kc_gather(int M, int N, int K, const float* A, int lda, const float* B, int ldb, const GatherOut& to,
                          const Gate& gate, hipStream_t s) {
  launch_kc<true>(M, N, K, A, lda, B, ldb, nullptr, 0, to, gate, s);
}

void gemm_f64_km(int M, int N, int K, const float* A, int lda, const float* B, int ldb, float* C, int ldc, int splits,
                 size_t c_split, const Gate& gate, hipStream_t s) {
  const int tm = (M + kBM - 1) / kBM, tn = (N + kBN - 1) / kBN;
  int kps = (K + splits - 1) / splits;
  kps = (kps + kDK - 1) / kDK * kDK;
  const bool vec = lda % 4 == 0 && ldb % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(B) % 16 == 0;
  const dim3 g((unsigned)(splits * tm * tn));
  if (vec)
    hipLaunchKernelGGL(gemm_f64<true>, g, dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc, kps, c_split, tm, tn,
                       splits, gate);
  else
    hipLaunchKernelGGL(gemm_f64<false>, g, dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc, kps, c_split, tm, tn,
                       splits, gate);
}

}  // namespace snn

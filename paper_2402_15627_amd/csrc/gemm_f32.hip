// fp32 projection GEMMs with the fused epilogues of the block (the bf16 ones
// are in gemm.hip).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_common.h"
#include "kernels.h"

namespace pb {
namespace {

// --------------------------------------------------------- fp32 MFMA GEMM
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).  As in the bf16 kernels
// the N tile is the MFMA's "A" operand: lane l holds columns 16 n + 4 g .. + 3
// (g = l >> 4, n = 0..3) of row l & 15, and a wave's 64 columns are one column
// group of the LayerNorm backward's row terms.  Within a 16-k step MFMA j
// contracts over k = 4 g + j, so a lane's operand values for the four MFMAs
// of a step are four consecutive k of one row.
//
// Measured against the vector-ALU kernel this replaced (64 x 64 tiles, scalar
// loads, two barriers per 16 k): dh of a block of 666 tokens, hidden 1024 and
// 7168 in-projection columns 836 -> 107 us (12 -> 91 TFLOP/s, split 7 ways
// along K), its in-projection 181 -> 107 us, its weight gradients 466 -> 164
// us; dh at 128 x 256 x 1792 207 -> 13 us.  A 2048 cube runs at 117 TFLOP/s,
// where a large library fp32 product reaches 137 on this chip.
constexpr int kFN = 64;  // tile columns
constexpr int kFThreads = 256;

// ---- 64 x 64 tiles
// Four waves, 16 x 64 each, K-tile 32, two LDS stages.  Matrix-core bound: a
// 16-k step costs a wave 16 MFMAs (512 cycles) against 5 LDS reads, so plain
// register-staged loads do, as long as two tiles of loads are in flight (one
// in registers for the next stage, one behind it).
//
// LDS: a K-contiguous operand is stored [row][k], 16-byte chunks XOR-ed by
// the row, read four k at a time.  An MN-contiguous operand is stored
// [k][row] as it lies in memory, rows padded to 4 mod 16 floats so that the
// four lane groups (k = 4 g + j) read distinct banks: no transpose.
constexpr int kFM = 64, kFK = 32;
template <bool KC>
struct F32Tile {
  static constexpr int kLd = kFM + 4;
  static constexpr int kFloats = KC ? kFM * kFK : kFK * kLd;
  static constexpr int kVec = kFM * kFK / 4 / kFThreads;  // float4 per thread
  // distinct 16-byte bank groups for 16 rows (of 128 bytes) at one chunk
  static PB_DEV int swz(int row, int c) { return c ^ ((row >> 1) & 7); }

  const float* p[kVec];  // this thread's float4 of the next K-tile
  size_t step;
  // Row (KC) or k (MN) and, in float4, k or column of this thread's vector i.
  static PB_DEV int major(int i) {
    return KC ? threadIdx.x / (kFK / 4) + i * (kFThreads / (kFK / 4))
              : threadIdx.x / (kFM / 4) + i * (kFThreads / (kFM / 4));
  }
  static PB_DEV int minor() { return 4 * (int)(threadIdx.x % ((KC ? kFK : kFM) / 4)); }
  PB_DEV void init(const float* __restrict__ X, int ld, int R0, int Rmax) {
    // rows (columns) past the end read the last ones: their results are not
    // stored
#pragma unroll
    for (int i = 0; i < kVec; ++i)
      p[i] = KC ? X + (size_t)min(R0 + major(i), Rmax - 1) * ld + minor()
                : X + (size_t)major(i) * ld + min(R0 + minor(), Rmax - 4);
    step = KC ? kFK : (size_t)kFK * ld;
  }
  PB_DEV void skip(int tiles) {
#pragma unroll
    for (int i = 0; i < kVec; ++i) p[i] += (size_t)tiles * step;
  }
  // The next K-tile, of which `left` k remain (from this tile's first); k
  // past the end read zero.
  PB_DEV void load(f32x4 (&r)[kVec], int left) {
    if (left >= kFK) {
#pragma unroll
      for (int i = 0; i < kVec; ++i) {
        r[i] = *reinterpret_cast<const f32x4*>(p[i]);
        p[i] += step;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kVec; ++i)
        r[i] = (KC ? minor() : major(i)) < left ? *reinterpret_cast<const f32x4*>(p[i])
                                                : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  static PB_DEV void store(float* __restrict__ lds, const f32x4 (&r)[kVec]) {
#pragma unroll
    for (int i = 0; i < kVec; ++i) {
      if constexpr (KC)
        *reinterpret_cast<f32x4*>(lds + major(i) * kFK + swz(major(i), minor() / 4) * 4) = r[i];
      else
        *reinterpret_cast<f32x4*>(lds + major(i) * kLd + minor()) = r[i];
    }
  }
  // Values k = 16 s + 4 g + 0..3 of tile row `row` (g the lane group).
  static PB_DEV f32x4 frag(const float* __restrict__ lds, int row, int s, int g) {
    if constexpr (KC) {
      return *reinterpret_cast<const f32x4*>(lds + row * kFK + swz(row, 4 * s + g) * 4);
    } else {
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = lds[(16 * s + 4 * g + j) * kLd + row];
      return v;
    }
  }
};

template <bool AK, bool BK, Epi EPI, bool GT>
__global__ __launch_bounds__(kFThreads) void gemm_f32_kernel(const float* __restrict__ A, int lda,
                                                             const float* __restrict__ B, int ldb,
                                                             int M, int N, int K, EpiArgs ep,
                                                             int splits, float* __restrict__ part) {
  typedef F32Tile<AK> TA;
  typedef F32Tile<BK> TB;
  constexpr int kStage = TA::kFloats + TB::kFloats;
  __shared__ __attribute__((aligned(16))) float smem[2 * kStage];

  const int tiles_m = (M + kFM - 1) / kFM, tiles_n = (N + kFN - 1) / kFN;
  int tm, tn;
  const int tiles = tiles_m * tiles_n;
  const int lid = xcd_remap(blockIdx.x, tiles * splits);
  const int slice = lid / tiles;  // a run of work items walks the tiles of one K-slice
  tile_of<8>(lid - slice * tiles, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * kFM, n0 = tn * kFN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, g = lane >> 4;
  const int wm = 16 * wave;

  f32x4 acc[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the row sums of A, when asked for, from the first tile column: this lane's
  // share of row wm + fr
  const bool rows = EPI == Epi::StoreF32 && ep.rowsum && tn == 0;
  float rsum = 0.f;
  TA ta;
  TB tb;
  ta.init(A, lda, m0, M);
  tb.init(B, ldb, n0, N);
  const int nk_all = (K + kFK - 1) / kFK, chunk = (nk_all + splits - 1) / splits;
  const int kt0 = slice * chunk, nk = min(chunk, nk_all - kt0);
  K -= kt0 * kFK;  // k from the slice's first; its end counts for the last slice only
  ta.skip(kt0);
  tb.skip(kt0);
  f32x4 ra[2][TA::kVec], rb[2][TB::kVec];
  auto load = [&](int t, auto S) {
    constexpr int s = decltype(S)::value;
    ta.load(ra[s], K - t * kFK);
    tb.load(rb[s], K - t * kFK);
  };
  auto store = [&](int t, auto S) {
    constexpr int s = decltype(S)::value;
    float* st = smem + (t & 1) * kStage;
    TA::store(st, ra[s]);
    TB::store(st + TA::kFloats, rb[s]);
  };
  // tile t from its stage; tile t + 1 (register set s) to the other stage at
  // the end, tile t + 2 requested (set 1 - s, tile t's) at the start
  auto step = [&](int t, auto S) {
    constexpr int s = decltype(S)::value;
    if (t + 2 < nk) load(t + 2, std::integral_constant<int, 1 - s>{});
    const float* la = smem + (t & 1) * kStage;
    const float* lb = la + TA::kFloats;
    f32x4 a[2], b[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      a[ks] = TA::frag(la, wm + fr, ks, g);
      if constexpr (EPI == Epi::StoreF32)
        if (rows) rsum += (a[ks][0] + a[ks][1]) + (a[ks][2] + a[ks][3]);
#pragma unroll
      for (int n = 0; n < 4; ++n) b[ks][n] = TB::frag(lb, 16 * n + fr, ks, g);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[ks][n][j], a[ks][j], acc[n], 0, 0, 0);
    if (t + 1 < nk) store(t + 1, S);
    __syncthreads();
  };
  constexpr std::integral_constant<int, 0> c0;
  constexpr std::integral_constant<int, 1> c1;
  load(0, c0);
  if (nk > 1) load(1, c1);
  store(0, c0);
  __syncthreads();
  for (int t = 0; t < nk; t += 2) {
    step(t, c1);
    if (t + 1 < nk) step(t + 1, c0);
  }

  const int m = m0 + wm + fr;
  const bool mok = m < M;
  if (splits > 1) {  // this slice's partial result, for f32_splitk_reduce
    float* row = part + ((size_t)slice * M + m) * N;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int c = n0 + 16 * n + 4 * g;
      if (mok && c < N) *reinterpret_cast<f32x4*>(row + c) = acc[n];
    }
    return;
  }
  if (rows) {
    rsum += __shfl_xor(rsum, 16, 64);
    rsum += __shfl_xor(rsum, 32, 64);
    if (g == 0 && mok) ep.rowsum[m] = rsum;
  }
  float s1 = 0.f, s2 = 0.f, mu = 0.f, rs = 0.f;
  if (EPI == Epi::LnGrad && mok) mu = ep.mean[m], rs = ep.rstd[m];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int c = n0 + 16 * n + 4 * g;
    if (mok && c < N) {
      const float v[4] = {acc[n][0], acc[n][1], acc[n][2], acc[n][3]};
      epi_store4<float, EPI, GT>(ep, m, c, v);
      if constexpr (EPI == Epi::LnGrad) ln_terms4<float>(ep, m, c, v, mu, rs, s1, s2);
    }
  }
  if constexpr (EPI == Epi::LnGrad) {
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      s1 += __shfl_xor(s1, off, 64);
      s2 += __shfl_xor(s2, off, 64);
    }
    if (g == 0 && mok) ep.rowpart[(size_t)m * ep.rowpart_ld + n0 / 64] = make_float2(s1, s2);
  }
}

// ---- 16 x 64 tiles, K split over the waves
// For the smallest grids.  Every wave computes the whole tile over its own
// slices of 32 k (wave w takes slices w, w + kSW, ...), so no operand value is
// shared between waves: fragments go straight from global memory to registers,
// with no LDS stage and no barrier in the loop, and the waves hide each
// other's latency.  The accumulators are added through LDS in wave order at
// the end.
constexpr int kSW = 8;  // waves per workgroup
constexpr int kSThreads = 64 * kSW;
constexpr int kSK = 32;  // k per slice

template <bool KC, int NB>
struct F32Frags {
  const float* p[KC ? NB : 1];
  int roff[KC ? 1 : NB];  // MN: column offset of each block
  size_t ld, step;
  PB_DEV void init(const float* __restrict__ X, int ld_, int R0, int Rmax, int wave, int fr,
                   int g) {
    ld = ld_;
    if constexpr (KC) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
        p[n] = X + (size_t)min(R0 + 16 * n + fr, Rmax - 1) * ld + kSK * wave + 4 * g;
      step = kSK * kSW;
    } else {
      p[0] = X + (size_t)(kSK * wave + 4 * g) * ld;
#pragma unroll
      for (int n = 0; n < NB; ++n) roff[n] = min(R0 + 16 * n + fr, Rmax - 1);
      step = (size_t)kSK * kSW * ld;
    }
  }
  // k = 16 s + 4 g + j of the slice at v[s][n][j]; `left` k remain from the
  // slice's first; k past the end read zero.
  PB_DEV void load(f32x4 (&v)[2][NB], int left, int g) {
    if (left >= kSK) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          if constexpr (KC) {
            v[s][n] = *reinterpret_cast<const f32x4*>(p[n] + 16 * s);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[s][n][j] = p[0][(16 * s + j) * ld + roff[n]];
          }
        }
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const int k = 16 * s + 4 * g;
          if constexpr (KC) {
            v[s][n] = k < left ? *reinterpret_cast<const f32x4*>(p[n] + 16 * s)
                               : f32x4{0.f, 0.f, 0.f, 0.f};
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              v[s][n][j] = k + j < left ? p[0][(16 * s + j) * ld + roff[n]] : 0.f;
          }
        }
    }
#pragma unroll
    for (int n = 0; n < (KC ? NB : 1); ++n) p[n] += step;
  }
};

template <bool AK, bool BK, Epi EPI, bool GT>
__global__ __launch_bounds__(kSThreads) void gemm_f32_waves_kernel(
    const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb, int M, int N,
    int K, EpiArgs ep) {
  __shared__ __attribute__((aligned(16))) float smem[kSW * 16 * kFN];
  __shared__ float rbuf[EPI == Epi::StoreF32 ? kSW * 16 : 1];
  const int tiles_m = (M + 15) / 16, tiles_n = (N + kFN - 1) / kFN;
  int tm, tn;
  tile_of<32>(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 16, n0 = tn * kFN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, g = lane >> 4;

  f32x4 acc[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool rows = EPI == Epi::StoreF32 && ep.rowsum && tn == 0;
  float rsum = 0.f;
  F32Frags<AK, 1> fa;
  F32Frags<BK, 4> fb;
  fa.init(A, lda, m0, M, wave, fr, g);
  fb.init(B, ldb, n0, N, wave, fr, g);
  f32x4 a[2][2][1], b[2][2][4];  // two slices: one multiplied, one in flight
  auto load = [&](int k0, auto S) {
    constexpr int s = decltype(S)::value;
    fa.load(a[s], K - k0, g);
    fb.load(b[s], K - k0, g);
  };
  auto mma = [&](auto S) {
    constexpr int s = decltype(S)::value;
    if constexpr (EPI == Epi::StoreF32) {
      if (rows) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          rsum += (a[s][ks][0][0] + a[s][ks][0][1]) + (a[s][ks][0][2] + a[s][ks][0][3]);
      }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[s][ks][n][j], a[s][ks][0][j], acc[n], 0,
                                                        0, 0);
  };
  constexpr std::integral_constant<int, 0> c0;
  constexpr std::integral_constant<int, 1> c1;
  constexpr int kHop = kSK * kSW;
  int k0 = kSK * wave;
  if (k0 < K) load(k0, c0);
  for (; k0 < K; k0 += 2 * kHop) {
    if (k0 + kHop < K) load(k0 + kHop, c1);
    mma(c0);
    if (k0 + 2 * kHop < K) load(k0 + 2 * kHop, c0);
    if (k0 + kHop < K) mma(c1);
  }

  // waves 0 .. 3 fold the eight partial tiles in wave order, 16 lanes to a row
#pragma unroll
  for (int n = 0; n < 4; ++n)
    *reinterpret_cast<f32x4*>(smem + (wave * 16 + fr) * kFN + 16 * n + 4 * g) = acc[n];
  if constexpr (EPI == Epi::StoreF32) {
    if (rows) {
      rsum += __shfl_xor(rsum, 16, 64);
      rsum += __shfl_xor(rsum, 32, 64);
      if (g == 0) rbuf[wave * 16 + fr] = rsum;
    }
  }
  __syncthreads();
  if (threadIdx.x >= 256) return;
  if constexpr (EPI == Epi::StoreF32) {
    if (rows && threadIdx.x < 16 && m0 + (int)threadIdx.x < M) {
      float v = 0.f;
      for (int w = 0; w < kSW; ++w) v += rbuf[w * 16 + threadIdx.x];
      ep.rowsum[m0 + threadIdx.x] = v;
    }
  }
  const int row = threadIdx.x >> 4, c4 = 4 * (threadIdx.x & 15);
  f32x4 sum = *reinterpret_cast<const f32x4*>(smem + row * kFN + c4);
#pragma unroll
  for (int w = 1; w < kSW; ++w)
    sum += *reinterpret_cast<const f32x4*>(smem + (w * 16 + row) * kFN + c4);
  const int m = m0 + row, c = n0 + c4;
  const bool ok = m < M && c < N;
  const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
  if (ok) epi_store4<float, EPI, GT>(ep, m, c, v);
  if constexpr (EPI == Epi::LnGrad) {
    float s1 = 0.f, s2 = 0.f;
    if (ok) ln_terms4<float>(ep, m, c, v, ep.mean[m], ep.rstd[m], s1, s2);
    s1 = row16_sum(s1);
    s2 = row16_sum(s2);
    if (c4 == 0 && m < M) ep.rowpart[(size_t)m * ep.rowpart_ld + n0 / 64] = make_float2(s1, s2);
  }
}

// Sum of `splits` partial results of four columns, `stride` floats apart, in
// slice order.  Four loads are in flight at a time: with one, each slice costs
// the whole memory latency (the tiny block's step 86.5 -> 82.7 us; the bf16
// GEMMs' reduction, far larger and bound by the partial tiles' bytes, gains
// nothing).
PB_DEV f32x4 sum_slices(const float* __restrict__ p, size_t stride, int splits) {
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; s += 4) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u < splits) v[u] = *reinterpret_cast<const f32x4*>(p + (size_t)(s + u) * stride);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u < splits) sum += v[u];
  }
  return sum;
}

// Sum of the K-slices' partial results [splits][M][N] in slice order, then
// the epilogue: 16 lanes to a row's 64-column group, four columns each.
template <Epi EPI, bool GT>
__global__ __launch_bounds__(256) void f32_splitk_reduce(const float* __restrict__ part, int M,
                                                         int N, int splits, EpiArgs ep) {
  const int groups = (N + kFN - 1) / kFN;
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) >> 4;  // (row, group)
  if (i >= (long long)M * groups) return;
  const int m = (int)(i / groups), grp = (int)(i - (long long)m * groups);
  const int c = grp * kFN + 4 * (threadIdx.x & 15);
  const bool ok = c < N;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (ok) {
    const float* p = part + (size_t)m * N + c;
    const f32x4 sum = sum_slices(p, (size_t)M * N, splits);
    v[0] = sum[0], v[1] = sum[1], v[2] = sum[2], v[3] = sum[3];
    epi_store4<float, EPI, GT>(ep, m, c, v);
  }
  if constexpr (EPI == Epi::LnGrad) {
    float s1 = 0.f, s2 = 0.f;
    if (ok) ln_terms4<float>(ep, m, c, v, ep.mean[m], ep.rstd[m], s1, s2);
    s1 = row16_sum(s1);
    s2 = row16_sum(s2);
    if ((threadIdx.x & 15) == 0) ep.rowpart[(size_t)m * ep.rowpart_ld + grp] = make_float2(s1, s2);
  }
}

// The launch of an fp32 GEMM: 64 x 64 tiles, whole or split along K, or 16 x
// 64 ones, whichever is estimated fastest.  The estimates (us) are fits to
// times measured on shapes from 128 x 256 x 1792 to 2048 x 2048 x 2048:
//  - 64 x 64 tiles: a K-tile of 32 costs a CU 0.88 us with one workgroup on it
//    (76 TFLOP/s over the chip), 0.70 with two, 0.57 with four (117): with one
//    wave per SIMD each K-tile's barrier and LDS reads are exposed;
//  - split along K: the same for the shorter K, plus the launch that sums the
//    slices (5 us, and the partial results at 4 TB/s);
//  - 16 x 64: 0.28 us per 32 k and tile, tiles taken a CU at a time (60
//    TFLOP/s: bound by the CU's load path), for the smallest grids.
struct F32Plan {
  int rows, splits;
};
F32Plan f32_plan(int M, int N, int K, bool may_split) {
  const long long tn = (N + kFN - 1) / kFN, t64 = (M + kFM - 1) / kFM * tn;
  const long long t16 = (M + 15) / 16 * tn;
  const int nk = (K + kFK - 1) / kFK;
  auto waves = [](long long wgs) { return (double)((wgs + kCUs - 1) / kCUs); };
  auto t64_us = [&](long long wgs, int steps) {
    const double w = waves(wgs);
    return w * steps * (w < 2 ? 0.88 : w < 3 ? 0.70 : w < 4 ? 0.63 : 0.57);
  };
  F32Plan best{64, 1};
  double us = t64_us(t64, nk);
  const double t16_us = waves(t16) * nk * 0.28;
  if (t16_us < us) best = F32Plan{16, 1}, us = t16_us;
  if (may_split)
    for (int s = 2; s <= std::min(16, nk); ++s) {
      const int chunk = (nk + s - 1) / s;
      if ((nk + chunk - 1) / chunk != s) continue;  // the last slices would be empty
      const double c = t64_us(t64 * s, chunk) + 5.0 + 8.0 * M * N * s / 4e6;
      if (c < us) best = F32Plan{64, s}, us = c;
    }
  return best;
}
GemmLaunch launch_of(const F32Plan& p, int M, int N) {
  GemmLaunch g;
  g.tiles = ((M + p.rows - 1) / p.rows) * ((N + kFN - 1) / kFN);
  // a split is reported, and its workspace sized, in 256 x 256 blocks of the
  // output, as for bf16
  const int blocks = ((M + 255) / 256) * ((N + 255) / 256);
  g.plan = p.splits > 1 ? SplitPlan{0, blocks, p.splits} : SplitPlan{g.tiles, 0, 1};
  g.workgroups = g.tiles * p.splits;
  g.threads = p.rows == 64 ? kFThreads : kSThreads;
  return g;
}

// The plan of a launch that has ws_floats of space for slices.
F32Plan launched_plan(int M, int N, int K, size_t ws_floats) {
  const F32Plan p = f32_plan(M, N, K, true);
  return p.splits > 1 && ws_floats < gemm_split_floats(Dt::F32, M, N, K) ? f32_plan(M, N, K, false)
                                                                         : p;
}

template <bool AK, bool BK, Epi EPI, bool GT>
void launch_layout(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                   const EpiArgs& ep, float* ws, size_t ws_floats, hipStream_t s) {
  const F32Plan p = launched_plan(M, N, K, ws ? ws_floats : 0);
  const GemmLaunch g = launch_of(p, M, N);
  if (p.rows == 16) {
    gemm_f32_waves_kernel<AK, BK, EPI, GT>
        <<<g.workgroups, g.threads, 0, s>>>(A, lda, B, ldb, M, N, K, ep);
    return;
  }
  gemm_f32_kernel<AK, BK, EPI, GT>
      <<<g.workgroups, g.threads, 0, s>>>(A, lda, B, ldb, M, N, K, ep, p.splits, ws);
  if (p.splits > 1) {
    const long long lanes = 16LL * M * ((N + kFN - 1) / kFN);
    f32_splitk_reduce<EPI, GT><<<(unsigned)((lanes + 255) / 256), 256, 0, s>>>(ws, M, N, p.splits,
                                                                               ep);
  }
}

}  // namespace

bool gemm_f32_rowsum_supported(int M, int N, int K, size_t ws_floats) {
  return launched_plan(M, N, K, ws_floats).splits == 1;
}

GemmLaunch gemm_f32_launch_of(int M, int N, int K) {
  return launch_of(f32_plan(M, N, K, true), M, N);
}

void launch_gemm_f32(Epi epi, bool a_kcontig, bool b_kcontig, const float* A, int lda,
                     const float* B, int ldb, int M, int N, int K, const EpiArgs& ep, float* ws,
                     size_t ws_floats, hipStream_t s) {
  auto run = [&](auto launch) { launch(A, lda, B, ldb, M, N, K, ep, ws, ws_floats, s); };
  const bool gt = ep.gelu_tanh != 0;
  switch (epi) {
    case Epi::StoreF32: run(launch_layout<false, false, Epi::StoreF32, true>); break;
    case Epi::BiasGelu:
      if (gt) run(launch_layout<true, true, Epi::BiasGelu, true>);
      else run(launch_layout<true, true, Epi::BiasGelu, false>);
      break;
    case Epi::BiasResid: run(launch_layout<true, true, Epi::BiasResid, true>); break;
    case Epi::DgeluSplit:
      if (b_kcontig) run(launch_layout<true, true, Epi::DgeluSplit, true>);  // plain stores
      else if (gt) run(launch_layout<true, false, Epi::DgeluSplit, true>);
      else run(launch_layout<true, false, Epi::DgeluSplit, false>);
      break;
    case Epi::LnGrad: run(launch_layout<true, false, Epi::LnGrad, true>); break;
  }
}

}  // namespace pb

// bf16 projection GEMMs for small grids: 64 x 64 tiles, K split over the waves
// of a workgroup.
//
// With few tokens the 256 x 256 tiles of gemm.hip are too few for the chip:
// split along K they cost a second launch, and either way a tile's long
// prologue and epilogue run once, in code that is fetched cold.  Here a
// workgroup of eight waves computes a 64 x 64 tile; wave w takes the slices of
// 32 k number w, w + 8, ..., so the waves share no operand values and the loop
// has no barrier: a K-contiguous operand's fragments go from global memory
// straight to registers, an MN-contiguous one's 32 x 64 slice passes through 4
// KB of LDS of the wave's own, whose rows are read back transposed.  The
// accumulators are added through LDS in wave order and the epilogue of four
// columns per thread follows.  Bound by latency (a slice is 16 MFMAs behind its
// loads) and, with a workgroup on every CU, by the CU's load path.  Measured,
// 256 x 256 tiles and these: 128 x 256 x 512 12 and 6.5 us, 256 x 2560 x 512
// 16.6 and 7, 512 x 4096 x 1024 27 and 16 to 20; step of a block of 256 tokens,
// hidden 512 119 -> 92 us, 333 tokens, hidden 256 140 -> 80, 2 x 56, hidden 256
// 102 -> 56.  gemm_small_wins has the rule that chooses between the two.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_common.h"
#include "kernels.h"

namespace pb {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
#define PB_LDS __attribute__((address_space(3)))

constexpr int kT = 64;            // tile rows and columns
constexpr int kW = 8;             // waves
constexpr int kThreads = 64 * kW;
constexpr int kSl = 32;           // k per slice
constexpr int kSliceBytes = kSl * kT * 2;
constexpr int kMergeRows = 32;    // rows merged at a time
constexpr int kLdsBytes = kW * kMergeRows * kT * 4;
static_assert(2 * kW * kSliceBytes <= kLdsBytes, "both operands' slices fit");

// 16-byte chunk c (8 of 64 columns) of row k of an MN-contiguous slice (128-byte
// rows): the four rows of a transposing read lie in distinct 64-byte quarters
// of the bank period, and row groups 8 apart in distinct halves of a quarter.
PB_DEV int swz_k(int k, int c) { return c ^ (4 * ((k >> 1) & 1)) ^ (2 * ((k >> 3) & 1)); }

// One operand of this wave: loads of a slice, and its fragments.
template <bool KC>
struct Side {
  const bf16* p[4];  // KC: row 16 n + (l & 15), k 8 (l >> 4); else k (l >> 3) + 8 n
  size_t step;       // elements per hop of kW slices
  PB_DEV void init(const bf16* __restrict__ X, int ld, int R0, int Rmax, int wave, int lane) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      // rows (columns) past the end read the last: their results are not stored
      if constexpr (KC)
        p[n] = X + (size_t)min(R0 + 16 * n + (lane & 15), Rmax - 1) * ld + kSl * wave +
               8 * (lane >> 4);
      else
        p[n] = X + (size_t)(kSl * wave + (lane >> 3) + 8 * n) * ld +
               min(R0 + 8 * (lane & 7), Rmax - 8);
    }
    step = KC ? (size_t)kSl * kW : (size_t)kSl * kW * ld;
  }
  // `left` k remain from the slice's first; k past the end read zero (a
  // K-contiguous operand's K is a multiple of 8).
  PB_DEV void load(u32x4 (&r)[4], int left, int lane) {
    if (left >= kSl) {
#pragma unroll
      for (int n = 0; n < 4; ++n) r[n] = *reinterpret_cast<const u32x4*>(p[n]);
    } else {
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const bool ok = (KC ? 8 * (lane >> 4) : (lane >> 3) + 8 * n) < left;
        r[n] = ok ? *reinterpret_cast<const u32x4*>(p[n]) : u32x4{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) p[n] += step;
  }
  // The slice's MFMA operands: block n's row 16 n + (l & 15), k 8 (l >> 4) .. + 7.
  static PB_DEV void frags(const u32x4 (&r)[4], unsigned char* __restrict__ lds, int lane,
                           bf16x8 (&f)[4]) {
    if constexpr (KC) {
#pragma unroll
      for (int n = 0; n < 4; ++n) f[n] = __builtin_bit_cast(bf16x8, r[n]);
    } else {
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int k = (lane >> 3) + 8 * n;
        *reinterpret_cast<u32x4*>(lds + k * 128 + swz_k(k, lane & 7) * 16) = r[n];
      }
      // (one wave's LDS accesses are served in order; keep the compiler's too)
      asm volatile("" ::: "memory");
      // lane 4 j + q of a 16-lane group addresses k-row kb + j, columns 4 q .. + 3,
      // and receives its own column's four k
      const int i = lane & 15, j = i >> 2, q = i & 3, k1 = 8 * (lane >> 4) + j, k2 = k1 + 4;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int mn = 16 * n + 4 * q, c = mn >> 3, off = (mn & 7) * 2;
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (PB_LDS s16x4*)(lds + k1 * 128 + swz_k(k1, c) * 16 + off));
        const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (PB_LDS s16x4*)(lds + k2 * 128 + swz_k(k2, c) * 16 + off));
        const bf16x4 a4 = __builtin_bit_cast(bf16x4, a), b4 = __builtin_bit_cast(bf16x4, b);
        f[n] = bf16x8{a4[0], a4[1], a4[2], a4[3], b4[0], b4[1], b4[2], b4[3]};
      }
      asm volatile("" ::: "memory");
    }
  }
};

struct SmallGemm {
  const bf16* A;
  int lda;
  const bf16* B;
  int ldb;
  int M, N, K;
  EpiArgs ep;
};

// Tile lid of the GEMM.  With ep.rowsum (weight gradients), the first tile
// column also sums the rows of A.
template <bool AK, bool BK, Epi EPI, bool GT>
PB_DEV void small_tile(const SmallGemm& G, int lid, unsigned char* __restrict__ smem) {
  const EpiArgs& ep = G.ep;
  const int M = G.M, N = G.N, K = G.K;
  int tm, tn;
  tile_of<8>(lid, (M + kT - 1) / kT, (N + kT - 1) / kT, tm, tn);
  const int m0 = tm * kT, n0 = tn * kT;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char* la = smem + 2 * wave * kSliceBytes;
  unsigned char* lb = la + kSliceBytes;

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rsum[4] = {0.f, 0.f, 0.f, 0.f};
  const bool rows = EPI == Epi::StoreF32 && ep.rowsum && tn == 0;

  Side<AK> sa;
  Side<BK> sb;
  sa.init(G.A, G.lda, m0, M, wave, lane);
  sb.init(G.B, G.ldb, n0, N, wave, lane);
  u32x4 ra[2][4], rb[2][4];  // one slice multiplied, one in flight
  auto load = [&](int k0, auto S) {
    constexpr int s = decltype(S)::value;
    sa.load(ra[s], K - k0, lane);
    sb.load(rb[s], K - k0, lane);
  };
  auto mma = [&](auto S) {
    constexpr int s = decltype(S)::value;
    bf16x8 fa[4], fb[4];
    Side<AK>::frags(ra[s], la, lane, fa);
    Side<BK>::frags(rb[s], lb, lane, fb);
    if constexpr (EPI == Epi::StoreF32) {
      if (rows) {
#pragma unroll
        for (int i = 0; i < 4; ++i) rsum[i] = sum_bf16x8(fa[i], rsum[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int n = 0; n < 4; ++n)
        acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[n], fa[i], acc[i][n], 0, 0, 0);
  };
  constexpr std::integral_constant<int, 0> c0;
  constexpr std::integral_constant<int, 1> c1;
  constexpr int kHop = kSl * kW;
  int k0 = kSl * wave;
  if (k0 < K) load(k0, c0);
  for (; k0 < K; k0 += 2 * kHop) {
    if (k0 + kHop < K) load(k0 + kHop, c1);
    mma(c0);
    if (k0 + 2 * kHop < K) load(k0 + 2 * kHop, c0);
    if (k0 + kHop < K) mma(c1);
  }

  // 32 rows at a time: every wave's partial rows to LDS (16-byte chunks XOR-ed
  // by the row), then 16 lanes to a row add the eight in wave order
  f32x4* buf = reinterpret_cast<f32x4*>(smem);
  const int row = threadIdx.x >> 4, c = threadIdx.x & 15;
  const int col = n0 + 4 * c;
#pragma unroll
  for (int h = 0; h < kT / kMergeRows; ++h) {
    __syncthreads();  // the slices' (or the previous rows') space is free
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int r = 16 * i + (lane & 15);
        buf[(wave * kMergeRows + r) * 16 + ((4 * n + (lane >> 4)) ^ (r & 15))] = acc[2 * h + i][n];
      }
    __syncthreads();
    f32x4 sum = buf[row * 16 + (c ^ (row & 15))];
#pragma unroll
    for (int w = 1; w < kW; ++w) sum += buf[(w * kMergeRows + row) * 16 + (c ^ (row & 15))];
    const int m = m0 + kMergeRows * h + row;
    const bool ok = m < M && col < N;
    const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
    if (ok) epi_store4<bf16, EPI, GT>(ep, m, col, v);
    if constexpr (EPI == Epi::LnGrad) {
      float s1 = 0.f, s2 = 0.f;
      if (ok) ln_terms4<bf16>(ep, m, col, v, ep.mean[m], ep.rstd[m], s1, s2);
      s1 = row16_sum(s1);
      s2 = row16_sum(s2);
      if (c == 0 && m < M) ep.rowpart[(size_t)m * ep.rowpart_ld + n0 / 64] = make_float2(s1, s2);
    }
  }
  if constexpr (EPI == Epi::StoreF32) {
    if (rows) {  // uniform over the workgroup
      __syncthreads();
      float* rbuf = reinterpret_cast<float*>(smem);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = rsum[i];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lane < 16) rbuf[wave * kT + 16 * i + lane] = v;
      }
      __syncthreads();
      const int m = m0 + (int)threadIdx.x;
      if (threadIdx.x < kT && m < M) {
        float v = 0.f;
        for (int w = 0; w < kW; ++w) v += rbuf[w * kT + threadIdx.x];
        ep.rowsum[m] = v;
      }
    }
  }
}

template <bool AK, bool BK, Epi EPI, bool GT>
__global__ __launch_bounds__(kThreads) void gemm_bf16_small_kernel(SmallGemm G) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsBytes];
  small_tile<AK, BK, EPI, GT>(G, xcd_remap(blockIdx.x, gridDim.x), smem);
}

// The backward's shared launches: dC or dh, then the weight gradient.
template <Epi E1, bool GT>
__global__ __launch_bounds__(kThreads) void gemm_bf16_small_pair(SmallGemm g1, int tiles1,
                                                                 SmallGemm g2, int tiles2) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsBytes];
  const int b = (int)blockIdx.x;
  if (b < tiles1)
    small_tile<true, false, E1, GT>(g1, xcd_remap(b, tiles1), smem);
  else
    small_tile<false, false, Epi::StoreF32, true>(g2, xcd_remap(b - tiles1, tiles2), smem);
}

SmallGemm desc(const GemmSpec& g) {
  return SmallGemm{(const bf16*)g.A, g.lda, (const bf16*)g.B, g.ldb, g.M, g.N, g.K, g.ep};
}

}  // namespace

int gemm_small_tiles(int M, int N) { return ((M + kT - 1) / kT) * ((N + kT - 1) / kT); }
int gemm_small_threads() { return kThreads; }

void launch_gemm_small(const GemmSpec& g, hipStream_t s) {
  auto run = [&](auto kernel) {
    kernel<<<gemm_small_tiles(g.M, g.N), kThreads, 0, s>>>(desc(g));
  };
  const bool gt = g.ep.gelu_tanh != 0;
  switch (g.epi) {
    case Epi::StoreF32: run(gemm_bf16_small_kernel<false, false, Epi::StoreF32, true>); break;
    case Epi::BiasGelu:
      if (gt) run(gemm_bf16_small_kernel<true, true, Epi::BiasGelu, true>);
      else run(gemm_bf16_small_kernel<true, true, Epi::BiasGelu, false>);
      break;
    case Epi::BiasResid: run(gemm_bf16_small_kernel<true, true, Epi::BiasResid, true>); break;
    case Epi::DgeluSplit:
      if (g.b_kcontig) run(gemm_bf16_small_kernel<true, true, Epi::DgeluSplit, true>);
      else if (gt) run(gemm_bf16_small_kernel<true, false, Epi::DgeluSplit, true>);
      else run(gemm_bf16_small_kernel<true, false, Epi::DgeluSplit, false>);
      break;
    case Epi::LnGrad: run(gemm_bf16_small_kernel<true, false, Epi::LnGrad, true>); break;
  }
}

void launch_gemm_small_pair(const GemmSpec& g1, const GemmSpec& g2, hipStream_t s) {
  const int t1 = gemm_small_tiles(g1.M, g1.N), t2 = gemm_small_tiles(g2.M, g2.N);
  auto run = [&](auto kernel) {
    kernel<<<t1 + t2, kThreads, 0, s>>>(desc(g1), t1, desc(g2), t2);
  };
  if (g1.epi == Epi::LnGrad) run(gemm_bf16_small_pair<Epi::LnGrad, true>);
  else if (g1.ep.gelu_tanh) run(gemm_bf16_small_pair<Epi::DgeluSplit, true>);
  else run(gemm_bf16_small_pair<Epi::DgeluSplit, false>);
}

}  // namespace pb

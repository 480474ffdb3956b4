// fp32 causal sliding-window attention, forward and backward, on
// v_mfma_f32_16x16x4_f32 (the bf16 kernels are in attn.hip).
//
// One workgroup of four waves owns 16 rows (queries, or keys in the dK/dV
// role) of one head and walks tiles of 16 rows of the other side, tile t on
// wave t mod 4; the waves' partial results are merged through LDS at the end.
// Splitting a block's tiles over the waves (rather than giving each wave its
// own rows) keeps the chip busy at the sizes the fp32 path runs at, where the
// blocks are few: bound by latency there, by the matrix cores in longer ones.
//
// As in the bf16 kernels everything is computed transposed, so that a lane
// owns one of the block's 16 rows (column l & 15 of every product) and the
// probabilities leave the score accumulators in the order in which the next
// MFMA contracts them: lane group g = l >> 4 holds other-side rows 4 g + e at
// element e, and MFMA j of that product contracts over rows 4 g + j.  Operand
// fragments go straight from global memory to registers: row fragments as
// float4 (four consecutive features), transposed ones as one float per lane
// over 16 consecutive features; no value is shared between waves, so LDS
// would add a pass and nothing else.
//
// Rows outside the window meet probability zero, and 0 x Inf is NaN in a
// product that takes a whole tile.  A workgroup with any non-finite result
// recomputes its rows from the definition (*_row below), each row reading the
// rows of its own window only, so that a non-finite value reaches exactly the
// rows that see it.
//
// Measured (2 x 333 tokens, 16 heads of 64, window 150): forward 343 -> 12.7
// us, backward 614 -> 34 us against one thread per row looping over its
// window; 128 tokens, 4 heads of 64, window 64: 150 -> 7.2 and 267 -> 8.4 us.
#include "common.h"
#include "kernels.h"

namespace pb {
namespace {

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kAW = 4;  // waves per workgroup
constexpr int kAR = 16;  // rows per block and tile

struct F32Attn {
  const float *Q, *K, *V;
  int ld;
  const float* O;
  int ld_o;
  const float* dO;
  int ld_do;
  int S, H, W;
  float scale;
};

PB_DEV float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
// Exponentials of scores in base 2.  In fp32 the products with log2 e lose up to
// 2^-24 of a logit, an error of the probability itself where logits are large,
// and a rounded scale log2 e in the forward alone would leave lse at another
// temperature than the backward's; so what these roundings leave over is added
// back.  dV against float64 with logits of 64 rms: 2 x 333 tokens, 16 heads of
// 64 5.1e-6 -> 2.9e-6, 1024 tokens, 4 heads of 128 7.8e-6 -> 5.0e-6 (natural
// exponentials of scores summed serially: 3.2e-6 and 6.0e-6); a block of 666
// tokens, hidden 1024 579 us with and without, of 128 tokens 71.1 and 70.8.
constexpr float kLog2eRest = 1.9259630e-8f;  // log2 e - kLog2e
struct Base2 {
  float c, rest;  // scale log2 e
  PB_DEV Base2(float scale) {
    c = scale * kLog2e;
    rest = fmaf(scale, kLog2eRest, fmaf(scale, kLog2e, -c));
  }
  // 2^(score - ref), ref a base-2 reference, s finite
  PB_DEV float exp(float s, float ref) const { return exp2_hw(fmaf(s, rest, fmaf(s, c, -ref))); }
  // e^(score - L)
  PB_DEV float prob(float s, float L) const {
    const float L2 = L * kLog2e, left = fmaf(L, kLog2eRest, fmaf(L, kLog2e, -L2));
    return exp2_hw(fmaf(s, rest, fmaf(s, c, -L2) - left));
  }
};
PB_DEV f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
PB_DEV bool finite4(const f32x4& v) {
  // an infinity or NaN in any element makes the sum of v - v NaN
  const float z = (v[0] - v[0]) + (v[1] - v[1]) + (v[2] - v[2]) + (v[3] - v[3]);
  return z == 0.f;
}
// Sum over the four lane groups (lanes l, l ^ 16, l ^ 32, l ^ 48).
PB_DEV float sum_groups(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
PB_DEV float max_groups(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

// Features 16 s + 4 g .. + 3 of one row, s = 0 .. D/16 - 1.
template <int D>
PB_DEV void row_frag(const float* __restrict__ row, int g, f32x4 (&v)[D / 16]) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s) v[s] = *reinterpret_cast<const f32x4*>(row + 16 * s + 4 * g);
}
// acc(row, column) += sum over features of a(row) b(column), two chains.
template <int D>
PB_DEV f32x4 dot_rows(const f32x4 (&a)[D / 16], const f32x4 (&b)[D / 16]) {
  f32x4 acc[2] = {zero4(), zero4()};
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][j], b[s][j], acc[s & 1], 0, 0, 0);
  return acc[0] + acc[1];
}
// out[db](feature 16 db + 4 g + e, column) += sum over the tile's rows of
// X(row, feature) p(row, column); x[j] points to feature i of row 4 g + j.
template <int D>
PB_DEV void add_rows(const float* const (&x)[4], const f32x4& p, f32x4 (&out)[D / 16]) {
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      out[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][16 * db], p[j], out[db], 0, 0, 0);
}

// Sum of the waves' [16][D] partial results: each thread's float4 number n is
// row (threadIdx.x + 256 n) / (D / 4).  buf: kAW * 16 * (D + 4) floats, free
// on entry; the caller's next barrier must come before it is written again.
template <int D>
struct Merge {
  static constexpr int kVec = (kAR * D / 4 + 255) / 256;
  static constexpr int kFloats = kAW * kAR * (D + 4);
  static PB_DEV bool has(int n) { return (int)threadIdx.x + 256 * n < kAR * D / 4; }
  static PB_DEV int row(int n) { return ((int)threadIdx.x + 256 * n) / (D / 4); }
  static PB_DEV int col(int n) { return 4 * (((int)threadIdx.x + 256 * n) % (D / 4)); }
  static PB_DEV void run(float* __restrict__ buf, const f32x4 (&part)[D / 16], float f, int wave,
                         int i, int g, f32x4 (&sum)[kVec]) {
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
      *reinterpret_cast<f32x4*>(buf + (wave * kAR + i) * (D + 4) + 16 * db + 4 * g) = part[db] * f;
    __syncthreads();
#pragma unroll
    for (int n = 0; n < kVec; ++n) {
      sum[n] = zero4();
      if (!has(n)) continue;
#pragma unroll
      for (int w = 0; w < kAW; ++w)
        sum[n] += *reinterpret_cast<const f32x4*>(buf + (w * kAR + row(n)) * (D + 4) + col(n));
    }
  }
};

// ------------------------------------------------- rows by the definition
// One wave per row, features e = lane + 64 n.
template <int D>
PB_DEV float row_dot(const float* __restrict__ a, const float* __restrict__ b, int lane) {
  float s = 0.f;
  for (int e = lane; e < D; e += 64) s = fmaf(a[e], b[e], s);
  return wave_sum(s);
}
template <int D>
PB_DEV void fwd_row(const F32Attn& p, size_t tok0, int c0, int q, float* __restrict__ out,
                    float* __restrict__ lse, int lane) {
  constexpr int NE = (D + 63) / 64;
  const float* qr = p.Q + (tok0 + q) * p.ld + c0;
  float acc[NE] = {}, m = kNegInf, l = 0.f;
  for (int j = max(0, q - p.W + 1); j <= q; ++j) {
    const float s = row_dot<D>(qr, p.K + (tok0 + j) * p.ld + c0, lane) * p.scale;
    const float* vr = p.V + (tok0 + j) * p.ld + c0;
    const float mn = fmaxf(m, s), a = expf(m - mn), pr = expf(s - mn);
    l = l * a + pr;
#pragma unroll
    for (int n = 0; n < NE; ++n)
      if (lane + 64 * n < D) acc[n] = acc[n] * a + pr * vr[lane + 64 * n];
    m = mn;
  }
#pragma unroll
  for (int n = 0; n < NE; ++n)
    if (lane + 64 * n < D) out[lane + 64 * n] = acc[n] / l;
  if (lane == 0) *lse = m + logf(l);
}
template <int D>
PB_DEV void dq_row(const F32Attn& p, size_t tok0, int c0, int q, float L, float delta,
                   float* __restrict__ out, int lane) {
  constexpr int NE = (D + 63) / 64;
  const float* qr = p.Q + (tok0 + q) * p.ld + c0;
  const float* gr = p.dO + (tok0 + q) * p.ld_do + c0;
  float acc[NE] = {};
  for (int j = max(0, q - p.W + 1); j <= q; ++j) {
    const float* kr = p.K + (tok0 + j) * p.ld + c0;
    const float s = row_dot<D>(qr, kr, lane);
    const float dp = row_dot<D>(gr, p.V + (tok0 + j) * p.ld + c0, lane);
    const float ds = expf(s * p.scale - L) * (dp - delta);
#pragma unroll
    for (int n = 0; n < NE; ++n)
      if (lane + 64 * n < D) acc[n] = fmaf(ds, kr[lane + 64 * n], acc[n]);
  }
#pragma unroll
  for (int n = 0; n < NE; ++n)
    if (lane + 64 * n < D) out[lane + 64 * n] = acc[n] * p.scale;
}
template <int D>
PB_DEV void dkdv_row(const F32Attn& p, size_t tok0, int c0, int j, const float* __restrict__ lse,
                     float* __restrict__ dk, float* __restrict__ dv, int lane) {
  constexpr int NE = (D + 63) / 64;
  const float* kr = p.K + (tok0 + j) * p.ld + c0;
  const float* vr = p.V + (tok0 + j) * p.ld + c0;
  float ak[NE] = {}, av[NE] = {};
  const int last = min(p.S - 1, j + p.W - 1);
  for (int i = j; i <= last; ++i) {
    const float* qr = p.Q + (tok0 + i) * p.ld + c0;
    const float* gr = p.dO + (tok0 + i) * p.ld_do + c0;
    const float delta = row_dot<D>(gr, p.O + (tok0 + i) * p.ld_o + c0, lane);
    const float pr = expf(row_dot<D>(qr, kr, lane) * p.scale - lse[i]);
    const float ds = pr * (row_dot<D>(gr, vr, lane) - delta);
#pragma unroll
    for (int n = 0; n < NE; ++n)
      if (lane + 64 * n < D) {
        av[n] = fmaf(pr, gr[lane + 64 * n], av[n]);
        ak[n] = fmaf(ds, qr[lane + 64 * n], ak[n]);
      }
  }
#pragma unroll
  for (int n = 0; n < NE; ++n)
    if (lane + 64 * n < D) {
      dk[lane + 64 * n] = ak[n] * p.scale;
      dv[lane + 64 * n] = av[n];
    }
}

// Linear workgroup id with the block index slowest, so that every head's
// longest blocks start first.
struct WorkItem {
  int bx, head, b;
};
PB_DEV WorkItem work_item() {
  const int hb_n = (int)(gridDim.y * gridDim.z);
  const int L = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
  const int hb = L % hb_n;
  return WorkItem{L / hb_n, hb % (int)gridDim.y, hb / (int)gridDim.y};
}

// ---------------------------------------------------------------- forward
template <int D>
__global__ __launch_bounds__(64 * kAW) void attn_fwd_f32(F32Attn p, float* __restrict__ O,
                                                         int ld_o, float* __restrict__ lse) {
  __shared__ __attribute__((aligned(16))) float buf[Merge<D>::kFloats];
  __shared__ float ml[2][kAW][kAR];
  const WorkItem wi = work_item();
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = p.S, W = p.W, c0 = wi.head * D;
  const int q0 = ((int)gridDim.x - 1 - wi.bx) * kAR, q = q0 + i;
  const size_t tok0 = (size_t)wi.b * S;
  const Base2 base(p.scale);
  f32x4 qf[D / 16], acc[D / 16];
  row_frag<D>(p.Q + (tok0 + min(q, S - 1)) * p.ld + c0, g, qf);
#pragma unroll
  for (int db = 0; db < D / 16; ++db) acc[db] = zero4();
  float m = kNegInf, l = 0.f;  // base-2 reference of this wave's keys; this lane's share of the sum
  const int last = min(q0 + kAR - 1, S - 1);
  for (int k0 = (max(0, q0 - W + 1) & ~(kAR - 1)) + kAR * wave; k0 <= last; k0 += kAR * kAW) {
    f32x4 kf[D / 16];
    row_frag<D>(p.K + (tok0 + min(k0 + i, S - 1)) * p.ld + c0, g, kf);
    const float* vr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      vr[j] = p.V + (tok0 + min(k0 + 4 * g + j, S - 1)) * p.ld + c0 + i;
    f32x4 s = dot_rows<D>(kf, qf);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int key = k0 + 4 * g + e;
      s[e] = (unsigned)(q - key) < (unsigned)W && key < S ? s[e] : kNegInf;
    }
    const float mt = max_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * base.c;
    const float mn = fmaxf(m, mt), mu = mn == kNegInf ? 0.f : mn, a = exp2_hw(m - mu);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = s[e] == kNegInf ? 0.f : base.exp(s[e], mu);
    l = l * a + ((s[0] + s[1]) + (s[2] + s[3]));
    m = mn;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) acc[db] *= a;
    add_rows<D>(vr, s, acc);
  }
  // merge the waves' keys: a common reference per query, then the quotient
  l = sum_groups(l);
  if (g == 0) ml[0][wave][i] = m, ml[1][wave][i] = l;
  __syncthreads();
  float M = kNegInf, L = 0.f;
#pragma unroll
  for (int w = 0; w < kAW; ++w) M = fmaxf(M, ml[0][w][i]);
  const float mu = M == kNegInf ? 0.f : M;
#pragma unroll
  for (int w = 0; w < kAW; ++w) L += ml[1][w][i] * exp2_hw(ml[0][w][i] - mu);
  f32x4 o[Merge<D>::kVec];
  Merge<D>::run(buf, acc, exp2_hw(m - mu) / L, wave, i, g, o);
  const float ls = fmaf(M, kLn2, logf(L));
  bool bad = wave == 0 && g == 0 && q < S && !(ls - ls == 0.f);
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    bad |= Merge<D>::has(n) && q0 + Merge<D>::row(n) < S && !finite4(o[n]);
  float* lrow = lse + ((size_t)wi.b * p.H + wi.head) * S;
  if (__syncthreads_or(bad)) {
    for (int r = q0 + wave; r < min(q0 + kAR, S); r += kAW)
      fwd_row<D>(p, tok0, c0, r, O + (tok0 + r) * ld_o + c0, lrow + r, lane);
    return;
  }
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    if (Merge<D>::has(n) && q0 + Merge<D>::row(n) < S)
      *reinterpret_cast<f32x4*>(O + (tok0 + q0 + Merge<D>::row(n)) * ld_o + c0 +
                                Merge<D>::col(n)) = o[n];
  if (wave == 0 && g == 0 && q < S) lrow[q] = ls;
}

// --------------------------------------------------------------- backward
// dQ of one block of queries, and their row terms delta = rowsum(dO O).
template <int D>
PB_DEV void dq_block(const F32Attn& p, const float* __restrict__ lse, float* __restrict__ delta,
                     float* __restrict__ dQ, int ld_d, int q0, int head, int b,
                     float* __restrict__ buf) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = p.S, W = p.W, c0 = head * D, q = q0 + i, qc = min(q, S - 1);
  const size_t tok0 = (size_t)b * S, ro = ((size_t)b * p.H + head) * S;
  const Base2 base(p.scale);
  const float L = lse[ro + qc];
  f32x4 qf[D / 16], gf[D / 16], dq[D / 16];
  row_frag<D>(p.Q + (tok0 + qc) * p.ld + c0, g, qf);
  row_frag<D>(p.dO + (tok0 + qc) * p.ld_do + c0, g, gf);
  f32x4 t = zero4();
  row_frag<D>(p.O + (tok0 + qc) * p.ld_o + c0, g, dq);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    t += dq[s] * gf[s];
    dq[s] = zero4();
  }
  const float dl = sum_groups((t[0] + t[1]) + (t[2] + t[3]));
  if (wave == 0 && g == 0 && q < S) delta[ro + q] = dl;
  const int last = min(q0 + kAR - 1, S - 1);
  for (int k0 = (max(0, q0 - W + 1) & ~(kAR - 1)) + kAR * wave; k0 <= last; k0 += kAR * kAW) {
    f32x4 kf[D / 16], vf[D / 16];
    const size_t row = (tok0 + min(k0 + i, S - 1)) * p.ld + c0;
    row_frag<D>(p.K + row, g, kf);
    row_frag<D>(p.V + row, g, vf);
    const float* kr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      kr[j] = p.K + (tok0 + min(k0 + 4 * g + j, S - 1)) * p.ld + c0 + i;
    const f32x4 s = dot_rows<D>(kf, qf);
    f32x4 ds = dot_rows<D>(vf, gf);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int key = k0 + 4 * g + e;
      const bool ok = (unsigned)(q - key) < (unsigned)W && key < S;
      ds[e] = ok ? base.prob(s[e], L) * (ds[e] - dl) : 0.f;
    }
    add_rows<D>(kr, ds, dq);
  }
  f32x4 o[Merge<D>::kVec];
  Merge<D>::run(buf, dq, p.scale, wave, i, g, o);
  bool bad = false;
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    bad |= Merge<D>::has(n) && q0 + Merge<D>::row(n) < S && !finite4(o[n]);
  if (__syncthreads_or(bad)) {
    for (int r = wave; r < kAR && q0 + r < S; r += kAW)
      dq_row<D>(p, tok0, c0, q0 + r, __shfl(L, r, 64), __shfl(dl, r, 64),
                dQ + (tok0 + q0 + r) * ld_d + c0, lane);
    return;
  }
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    if (Merge<D>::has(n) && q0 + Merge<D>::row(n) < S)
      *reinterpret_cast<f32x4*>(dQ + (tok0 + q0 + Merge<D>::row(n)) * ld_d + c0 +
                                Merge<D>::col(n)) = o[n];
}

// dK and dV of one block of keys.  The row terms of the queries it walks are
// formed here too (one more row fragment per tile), so that the backward is
// one launch.
template <int D>
PB_DEV void dkdv_block(const F32Attn& p, const float* __restrict__ lse, float* __restrict__ dK,
                       float* __restrict__ dV, int ld_d, int j0, int head, int b,
                       float* __restrict__ buf) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = p.S, W = p.W, c0 = head * D, key = j0 + i;
  const size_t tok0 = (size_t)b * S, ro = ((size_t)b * p.H + head) * S;
  const Base2 base(p.scale);
  f32x4 kf[D / 16], vf[D / 16], dk[D / 16], dv[D / 16];
  const size_t own = (tok0 + min(key, S - 1)) * p.ld + c0;
  row_frag<D>(p.K + own, g, kf);
  row_frag<D>(p.V + own, g, vf);
#pragma unroll
  for (int db = 0; db < D / 16; ++db) dk[db] = dv[db] = zero4();
  const int last = (int)min((long long)S - 1, (long long)j0 + kAR - 1 + W - 1);
  for (int q0 = j0 + kAR * wave; q0 <= last; q0 += kAR * kAW) {
    const int qi = min(q0 + i, S - 1);
    f32x4 qf[D / 16], gf[D / 16], t = zero4();
    row_frag<D>(p.dO + (tok0 + qi) * p.ld_do + c0, g, gf);
    row_frag<D>(p.O + (tok0 + qi) * p.ld_o + c0, g, qf);
#pragma unroll
    for (int s = 0; s < D / 16; ++s) t += qf[s] * gf[s];
    // row i's terms in every lane with l & 15 = i; a lane needs rows 4 g + e
    const float dli = sum_groups((t[0] + t[1]) + (t[2] + t[3]));
    const float Li = lse[ro + qi];
    row_frag<D>(p.Q + (tok0 + qi) * p.ld + c0, g, qf);
    const float *qr[4], *gr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const size_t row = tok0 + min(q0 + 4 * g + j, S - 1);
      qr[j] = p.Q + row * p.ld + c0 + i;
      gr[j] = p.dO + row * p.ld_do + c0 + i;
    }
    f32x4 pr = dot_rows<D>(qf, kf);
    f32x4 ds = dot_rows<D>(gf, vf);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = q0 + 4 * g + e;
      const bool ok = (unsigned)(q - key) < (unsigned)W && q < S;
      const float L = __shfl(Li, 4 * g + e, 64), dl = __shfl(dli, 4 * g + e, 64);
      pr[e] = ok ? base.prob(pr[e], L) : 0.f;
      ds[e] = ok ? pr[e] * (ds[e] - dl) : 0.f;
    }
    add_rows<D>(gr, pr, dv);
    add_rows<D>(qr, ds, dk);
  }
  f32x4 ov[Merge<D>::kVec], ok[Merge<D>::kVec];
  Merge<D>::run(buf, dv, 1.f, wave, i, g, ov);
  __syncthreads();
  Merge<D>::run(buf, dk, p.scale, wave, i, g, ok);
  bool bad = false;
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    bad |= Merge<D>::has(n) && j0 + Merge<D>::row(n) < S && !(finite4(ov[n]) && finite4(ok[n]));
  if (__syncthreads_or(bad)) {
    for (int r = j0 + wave; r < min(j0 + kAR, S); r += kAW)
      dkdv_row<D>(p, tok0, c0, r, lse + ro, dK + (tok0 + r) * ld_d + c0,
                  dV + (tok0 + r) * ld_d + c0, lane);
    return;
  }
#pragma unroll
  for (int n = 0; n < Merge<D>::kVec; ++n)
    if (Merge<D>::has(n) && j0 + Merge<D>::row(n) < S) {
      const size_t at = (tok0 + j0 + Merge<D>::row(n)) * ld_d + c0 + Merge<D>::col(n);
      *reinterpret_cast<f32x4*>(dK + at) = ok[n];
      *reinterpret_cast<f32x4*>(dV + at) = ov[n];
    }
}

// Both roles in one launch, alternating, each longest first.
template <int D>
__global__ __launch_bounds__(64 * kAW) void attn_bwd_f32(F32Attn p, const float* __restrict__ lse,
                                                         float* __restrict__ delta,
                                                         float* __restrict__ dQ,
                                                         float* __restrict__ dK,
                                                         float* __restrict__ dV, int ld_d) {
  __shared__ __attribute__((aligned(16))) float buf[Merge<D>::kFloats];
  const WorkItem wi = work_item();
  const int nb = (int)gridDim.x / 2, r = wi.bx >> 1;
  if (wi.bx & 1)
    dq_block<D>(p, lse, delta, dQ, ld_d, (nb - 1 - r) * kAR, wi.head, wi.b, buf);
  else
    dkdv_block<D>(p, lse, dK, dV, ld_d, r * kAR, wi.head, wi.b, buf);
}

F32Attn args_of(const AttnShape& a, const float* q, const float* k, const float* v, int ld) {
  F32Attn p{};
  p.Q = q, p.K = k, p.V = v, p.ld = ld;
  p.S = a.seq, p.H = a.heads, p.W = a.window;
  p.scale = 1.0f / sqrtf((float)a.head_dim);
  return p;
}
unsigned blocks_of(const AttnShape& a) { return (unsigned)((a.seq + kAR - 1) / kAR); }

}  // namespace

void launch_attn_forward_f32(const AttnShape& a, const float* q, const float* k, const float* v,
                             int ld_qkv, float* o, int ld_o, float* lse, hipStream_t s) {
  const F32Attn p = args_of(a, q, k, v, ld_qkv);
  const dim3 g(blocks_of(a), a.heads, a.batch);
  if (a.head_dim == 64) attn_fwd_f32<64><<<g, 64 * kAW, 0, s>>>(p, o, ld_o, lse);
  else if (a.head_dim == 96) attn_fwd_f32<96><<<g, 64 * kAW, 0, s>>>(p, o, ld_o, lse);
  else attn_fwd_f32<128><<<g, 64 * kAW, 0, s>>>(p, o, ld_o, lse);
}

void launch_attn_backward_f32(const AttnShape& a, const float* q, const float* k, const float* v,
                              int ld_qkv, const float* o, int ld_o, const float* d_o, int ld_do,
                              const float* lse, float* delta, float* dq, float* dk, float* dv,
                              int ld_d, hipStream_t s) {
  F32Attn p = args_of(a, q, k, v, ld_qkv);
  p.O = o, p.ld_o = ld_o, p.dO = d_o, p.ld_do = ld_do;
  const dim3 g(2 * blocks_of(a), a.heads, a.batch);
  if (a.head_dim == 64)
    attn_bwd_f32<64><<<g, 64 * kAW, 0, s>>>(p, lse, delta, dq, dk, dv, ld_d);
  else if (a.head_dim == 96)
    attn_bwd_f32<96><<<g, 64 * kAW, 0, s>>>(p, lse, delta, dq, dk, dv, ld_d);
  else
    attn_bwd_f32<128><<<g, 64 * kAW, 0, s>>>(p, lse, delta, dq, dk, dv, ld_d);
}

}  // namespace pb

// Device code shared by the projection GEMMs: the epilogues of four consecutive
// output columns, a fragment's row sum and the order in which tiles are walked.
#pragma once

#include "common.h"
#include "kernels.h"

namespace pb {

// CUs of MI355X.
constexpr int kCUs = 256;

// ------------------------------------------------------------- epilogues
// Four consecutive output columns n..n+3 of row m.  GT: tanh form of GeLU.
template <typename T, Epi EPI, bool GT>
PB_DEV void epi_store4(const EpiArgs& ep, int m, int n, const float* v) {
  if constexpr (EPI == Epi::StoreF32) {
    store4((float*)ep.out + (size_t)m * ep.ld_out + n, v);
  } else if constexpr (EPI == Epi::LnGrad) {
    store4((T*)ep.out + (size_t)m * ep.ld_out + n, v);
  } else if constexpr (EPI == Epi::BiasGelu) {
    float b[4], z[4];
    load4((const T*)ep.bias + n, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = v[e] + b[e];
    store4((T*)ep.out + (size_t)m * ep.ld_out + n, z);
    if (n >= ep.split) {
      float g[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = gelu<T, GT>(z[e]);
      store4((T*)ep.out2 + (size_t)m * ep.ld_out2 + (n - ep.split) + ep.col2, g);
    }
  } else if constexpr (EPI == Epi::BiasResid) {
    float b[4], r[4], o[4];
    load4((const T*)ep.bias + n, b);
    load4((const T*)ep.resid + (size_t)m * ep.ld_out + n, r);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = v[e] + b[e] + r[e];
    store4((T*)ep.out + (size_t)m * ep.ld_out + n, o);
  } else {  // DgeluSplit
    if (n < ep.split) {
      store4((T*)ep.out + (size_t)m * ep.ld_out + n, v);
    } else {
      const size_t off = (size_t)m * ep.ld_out2 + (n - ep.split) + ep.col2;
      float u[4], o[4];
      load4((const T*)ep.aux + off, u);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = v[e] * gelu_grad<T, GT>(u[e]);
      store4((T*)ep.out2 + off, o);
    }
  }
}

// LnGrad: the LayerNorm backward's row terms of four columns n..n+3 of row m,
// added to s1 (sum g) and s2 (sum g xhat), g = gamma dh.
template <typename T>
PB_DEV void ln_terms4(const EpiArgs& ep, int m, int n, const float* v, float mu, float rs,
                      float& s1, float& s2) {
  float gm[4], xv[4];
  load4((const T*)ep.bias + n, gm);
  load4((const T*)ep.aux + (size_t)m * ep.ld_out + n, xv);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float g = gm[e] * v[e];
    s1 += g;
    s2 += g * ((xv[e] - mu) * rs);
  }
}

// Sum of a fragment's eight bf16 values, added to acc in fp32.
PB_DEV float sum_bf16x8(const bf16x8& p, float acc) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 8; i += 2)
    acc = __builtin_amdgcn_fdot2_f32_bf16(bf16x2_t{p[i], p[i + 1]}, one, acc, false);
  return acc;
}

// Tile order.  Workgroup b runs on XCD b % 8; xcd_remap gives each XCD a
// contiguous run of logical ids, and tile_of walks logical ids in groups of G
// tile-rows, so concurrently running workgroups on one XCD share operand
// strips in its L2.  The LDS-DMA GEMMs take G = tile_group(epilogue): groups
// of 4 rows (a 32-workgroup XCD share spans 4 x 8 tiles) measured faster for
// the backward's GEMMs and the in-projection, groups of 8 for the
// out-projection (BiasResid); groups of 2 or 16 were slower for all.
PB_DEV int xcd_remap(int bid, int n) {
  const int q = n / 8, r = n % 8, x = bid % 8;
  return x * q + min(x, r) + bid / 8;
}
constexpr int tile_group(Epi e) { return e == Epi::BiasResid ? 8 : 4; }
template <int G = 8>
PB_DEV void tile_of(int lid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int per_group = G * tiles_n;
  const int group = lid / per_group;
  const int first_m = group * G;
  const int gsize = min(tiles_m - first_m, G);
  const int in_group = lid - group * per_group;
  tm = first_m + in_group % gsize;
  tn = in_group / gsize;
}
PB_DEV void tile_coords(int tiles_m, int tiles_n, int& tm, int& tn) {
  tile_of(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

}  // namespace pb

// Which GEMM a merge call takes: a rule on sizes and alignment (host code
// that needs no HIP, so that a test can compile it by itself).
#pragma once

#include <stdint.h>

namespace sm {

struct GemmShape {
  int bm, bn;  // output tile of a workgroup
};

// gemm_ksplit_nt_gelu's tiles, then the other kernels
constexpr GemmShape kGemmShapes[] = {{32, 32},  {32, 64},  {64, 64},   {96, 64},   {128, 64}, {160, 64},
                                     {192, 64}, {256, 128}, {256, 256}, {128, 128}, {64, 16}};
constexpr int kKtShapeCount = 7;
constexpr int kGemmWide = 7;    // gemm_wide_bf16_nt_gelu
constexpr int kGemm256 = 8;     // gemm256_bf16_nt_gelu
constexpr int kGemmPlain = 9;   // gemm_bf16_nt_gelu, or for fp32 gemm_f32_nt_gelu (64 x 64)
constexpr int kGemmSkinny = 10;  // gemm_skinny_bf16_gelu
constexpr int kGemmKinds = 9;   // those that the cost rule chooses from
constexpr int kGemmCus = 256;
constexpr int kSkinnyMaxM = 64;  // rows that the 16-column kernel takes

// Times in microseconds at K = 64 nk (bf16), fitted
// to sweeps over M = 1..30,000 at N = K = 512..8192 on the box (each within
// about 10%): a grid of t tiles runs as waves of one workgroup per compute
// unit; a k-tile of a wave takes a time that grows with the bytes each
// workgroup loads for it (BM + BN rows) and, for the large tiles, with the
// part f of the compute units that are busy (the matrix clock falls); each
// wave adds its prologue and epilogue.  Measured at K = N = 4096:
//   M = 64      32x32 9.6    64x64 16.7
//   M = 609     160x64 31    128x64 47    256x128 58    256x256 86
//   M = 1700    160x64 95    256x128 67   256x256 94
//   M = 2400    256x128 119  256x256 95
//   M = 4200    256x256 195, of which the 17th row of tiles alone about 78
// The last line is why a call may be cut in two by rows: whole waves of the
// large tile, and the rows that remain by whatever is fastest for them.

inline float gemm_cost(int kind, int M, int N, int K, bool f32) {
  const int bm = kGemmShapes[kind].bm, bn = kGemmShapes[kind].bn;
  if (N % bn || (f32 && kind >= kKtShapeCount)) return 3.0e38f;
  const int64_t tiles = (int64_t)((M + bm - 1) / bm) * (N / bn);
  const int64_t full = tiles / kGemmCus;
  const float f = (float)(tiles % kGemmCus) / kGemmCus, nk = (float)(K / (f32 ? 32 : 64));
  if (kind == kGemm256) return 7.f + full * (nk * 1.53f + 14.f) + (f > 0.f ? nk * (0.88f + 0.65f * f) + 14.f : 0.f);
  if (kind == kGemmWide) return 6.f + full * (nk * 0.88f + 8.f) + (f > 0.f ? nk * (0.55f + 0.33f * f) + 8.f : 0.f);
  const float kt = f32 ? 0.04f + 0.16f * (bm / 32) * (bn / 32) : 0.0021f * (bm + bn) - 0.04f;
  return 3.f + (full + (f > 0.f ? 1 : 0)) * (nk * kt + 0.8f * (bm / 32));
}

struct GemmPlan {
  int kind, rows;        // rows [0, rows) with `kind`
  int kind2;             // and the rest with kind2 (rows < M)
};

// Direct-to-LDS loads want operands that are 16-byte aligned; others take the
// kernels with plain loads.
inline GemmPlan plan_gemm(int M, int N, int K, bool f32, bool aligned) {
  if (!aligned) return GemmPlan{!f32 && M <= kSkinnyMaxM ? kGemmSkinny : kGemmPlain, M, 0};
  auto best = [&](int m, float *cost) {
    int b = 0;
    for (int k = 0; k < kGemmKinds; ++k) {
      const float c = gemm_cost(k, m, N, K, f32);
      if (k == 0 || c < *cost) {
        *cost = c;
        b = k;
      }
    }
    return b;
  };
  GemmPlan p{0, M, 0};
  float cost = 0.f;
  p.kind = best(M, &cost);
  if (f32) return p;
  for (int kind = kGemmWide; kind <= kGemm256; ++kind) {
    const int bm = kGemmShapes[kind].bm, tiles_n = N / kGemmShapes[kind].bn;
    const int64_t row_tiles = (M + bm - 1) / bm;
    const int64_t waves = row_tiles * tiles_n / kGemmCus;
    if (tiles_n > kGemmCus || waves < 1 || waves > 4) continue;  // (beyond a few waves the last one weighs little)
    const int64_t m1 = waves * kGemmCus / tiles_n * bm;
    if (m1 <= 0 || m1 >= M) continue;
    float rest = 0.f;
    const int k2 = best((int)(M - m1), &rest);
    const float c = gemm_cost(kind, (int)m1, N, K, f32) + rest;
    if (c < 0.95f * cost) {
      cost = c;
      p = GemmPlan{kind, (int)m1, k2};
    }
  }
  return p;
}

}  // namespace sm

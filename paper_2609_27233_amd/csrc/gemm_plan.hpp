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
constexpr int kGemmKinds = 10;  // those that the cost rule chooses from
constexpr int kGemmCus = 256;
constexpr int kSkinnyMaxM = 64;  // rows that the 16-column kernel takes

// Time of a GEMM with N = K in microseconds: a grid runs as waves of one
// workgroup per slot (one per compute unit; two of the 128 x 128 tile, eight
// of the vector-ALU one, whose LDS is small), and
//   t = c0 + full (c1 + c2 nk) + [part > 0] (c3 + c4 nk + (c5 nk + c6) part)
// with `full` whole waves, a last one that fills `part` of the slots, and nk
// k-tiles.  The numbers are least-squares fits to 1551 pairs of M = 16..70,000
// and d = 256..8192, each kernel weighted where it is near the best
// (profiles/merge_gemm_tile-sweep.md).  Two things they do not show have a
// term of their own: below d = 2048 a last wave of 256 x 128 tiles over more
// than 192 units takes longer (d = 1024: 168 tiles 23 us, 216 tiles 31), and
// the K-split tiles lose once they run in three waves.  Over those pairs the
// pick is 0.15% slower than the best kernel on average, 10% at most.  At d =
// 4096, us:
//   M = 64      32x32 9.6    64x64 16.7
//   M = 609     160x64 31    128x64 47    256x128 58    256x256 86
//   M = 1700    160x64 95    256x128 67   256x256 94
//   M = 2400    256x128 119  256x256 95
//   M = 4200    256x256 195, of which the 17th row of tiles alone about 78
// The last line is why a call may be cut in two by rows: whole waves of the
// large tile, and the rows that remain by whatever is fastest for them.
// At d = 256 and M = 19,972: 128x128 14, 160x64 21, 256x256 25.

constexpr float kGemmCost[kGemmKinds][7] = {
    {2.399f, 0.753f, 0.083f, 0.000f, 0.079f, 0.029f, 0.000f},  // 32 x 32
    {1.247f, 2.047f, 0.152f, 1.665f, 0.131f, 0.020f, 0.268f},  // 32 x 64
    {0.808f, 3.805f, 0.205f, 3.058f, 0.171f, 0.033f, 0.635f},  // 64 x 64
    {0.000f, 5.855f, 0.245f, 4.670f, 0.192f, 0.041f, 1.298f},  // 96 x 64
    {0.000f, 7.959f, 0.288f, 5.316f, 0.225f, 0.052f, 2.067f},  // 128 x 64
    {0.000f, 9.665f, 0.345f, 5.888f, 0.272f, 0.052f, 3.262f},  // 160 x 64
    {0.000f, 11.764f, 0.381f, 6.697f, 0.279f, 0.090f, 4.006f},  // 192 x 64
    {0.000f, 15.303f, 0.912f, 9.187f, 0.538f, 0.278f, 5.967f},  // 256 x 128
    {3.642f, 18.459f, 1.563f, 15.833f, 0.833f, 0.559f, 4.868f},  // 256 x 256
    {6.845f, 8.233f, 1.127f, 0.000f, 0.547f, 0.740f, 5.142f},  // 128 x 128
};
constexpr float kGemmCostF32[kKtShapeCount + 1][7] = {
    {2.431f, 1.058f, 0.148f, 0.000f, 0.165f, 0.029f, 0.017f},  // 32 x 32
    {0.000f, 2.475f, 0.334f, 3.163f, 0.313f, 0.035f, 0.470f},  // 32 x 64
    {2.560f, 4.352f, 0.581f, 1.845f, 0.568f, 0.061f, 0.990f},  // 64 x 64
    {5.511f, 6.211f, 0.783f, 0.000f, 0.766f, 0.067f, 1.674f},  // 96 x 64
    {2.807f, 7.974f, 1.021f, 3.832f, 0.988f, 0.050f, 2.600f},  // 128 x 64
    {2.420f, 9.490f, 1.250f, 4.587f, 1.226f, 0.000f, 5.094f},  // 160 x 64
    {2.663f, 10.657f, 1.467f, 5.732f, 1.447f, 0.021f, 4.642f},  // 192 x 64
    {0.000f, 2.936f, 6.811f, 2.772f, 1.068f, 6.012f, 6.426f},  // the vector ALU, 64 x 64
};

inline float gemm_cost(int kind, int M, int N, int K, bool f32) {
  const bool valu = f32 && kind == kGemmPlain;
  const int bm = valu ? 64 : kGemmShapes[kind].bm, bn = valu ? 64 : kGemmShapes[kind].bn;
  if (N % bn || (f32 && kind >= kKtShapeCount && !valu)) return 3.0e38f;
  const int slots = kGemmCus * (valu ? 8 : kind == kGemmPlain ? 2 : 1);
  const int64_t tiles = (int64_t)((M + bm - 1) / bm) * (N / bn);
  const int64_t full = tiles / slots;
  const int last = (int)(tiles % slots);
  const float part = (float)last / slots, nk = (float)(K / (f32 ? 32 : 64));
  const float *c = f32 ? kGemmCostF32[valu ? kKtShapeCount : kind] : kGemmCost[kind];
  float t = c[0] + full * (c[1] + c[2] * nk);
  if (last > 0) t += c[3] + c[4] * nk + (c[5] * nk + c[6]) * part;
  if (!f32 && kind == kGemmWide && K < 2048 && last > 192) t += 4.f;
  if (!f32 && kind < kKtShapeCount && full + (last > 0) >= 3) t *= 1.1f;
  return t;
}

struct GemmPlan {
  int kind, rows;        // rows [0, rows) with `kind`
  int kind2;             // and the rest with kind2 (rows < M)
};

// Direct-to-LDS loads want operands that are 16-byte aligned; others take the
// kernels with plain loads.
inline GemmPlan plan_gemm(int M, int N, int K, bool f32, bool aligned) {
  if (!aligned) return GemmPlan{!f32 && M <= kSkinnyMaxM ? kGemmSkinny : kGemmPlain, M, 0};
  // (a few rows of narrow tables: 2.4 us against 2.6 with 32 x 32 tiles at d = 256, 3.2 and 3.3 at 768, 3.8 both at 1024)
  if (!f32 && M <= 8 && K <= 768) return GemmPlan{kGemmSkinny, M, 0};
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
    if (k2 != kind && c < 0.98f * cost) {
      cost = c;
      p = GemmPlan{kind, (int)m1, k2};
    }
  }
  return p;
}

}  // namespace sm

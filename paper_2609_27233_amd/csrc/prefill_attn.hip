// Prefill attention over the paged cache (gfx950).
//
// The prefill pass that prompt compression shortens ("Efficiency Analysis":
// every layer of the prefill runs over the compressed sequence).  Request i
// brings the m_i query rows of the last m_i cached positions of sequence
// s = seq_ids[i]; the row at position p attends causally to entries 0..p:
//   out[row, h] = sum_{j <= p} softmax_j(scale q . K[s, j, g]) V[s, j, g],
//   g = h / G (grouped query).
//
// One workgroup of eight waves per (request, kv head, block of positions).
// It holds 256 / KS query vectors: BQ = 256 / KS / G positions x the G query
// heads of kv head g, so every K/V tile it loads serves all of them; with
// KS > 1 (calls too small to fill the chip, see prefill_plan.hpp) the waves
// form KS groups that hold the same vectors and take every KS-th tile of
// keys, and their softmax states are merged through LDS at the end.  A wave owns 32
// vectors, the columns of the transposed score blocks
//   S^T (32 keys x 32 queries) = K (32 x D) . Q^T        (v_mfma_f32_32x32x16_bf16)
// and accumulates
//   O^T (D x 32 queries) += V^T (D x 32 keys) . P^T.
// At about 220 registers a wave, two waves share each SIMD, so one wave's
// softmax runs while the other's products occupy the matrix unit.
// In S^T a lane holds 16 keys of one query column, so the softmax row
// statistics need one lane swap per tile.  The K rows of a block are read in
// a permuted order so that the 16 scores a lane holds are exactly the keys
// its PV operand needs (8 contiguous tokens per 16-key step): no shuffle
// between the two products.  K/V tiles of 64 keys (32 with KS = 4) go through LDS, the next
// tile's global loads in flight while the current one is multiplied.
//
// Softmax: exp2 of (score x scale log2 e - reference), with the reference
// (a running maximum) moved only when a tile's maximum exceeds it by more
// than 2^8.  Any reference gives the same ratios; keeping it mostly fixed
// skips the rescale of the accumulators on almost every tile.
#include "common.hpp"
#include "prefill_plan.hpp"

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// round-to-nearest-even pair conversion (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t cvt_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

namespace sm {

constexpr int kPfWaves = 8;
constexpr int kPfThreads = 64 * kPfWaves;
static_assert(kPfVec == 32 * kPfWaves, "32 query vectors per wave");
constexpr int kPfMaxPages = 4096;
constexpr float kPfLog2e = 1.4426950408889634f;

struct PrefillArgs {
  const uint16_t *k_pool;
  const uint16_t *v_pool;
  const int32_t *block_table;
  const int32_t *lengths;
  const int32_t *seq_ids;
  const int32_t *q_offsets;
  const uint16_t *q;
  uint16_t *out;
  int32_t *err;
  int n, total_rows, max_rows, Hkv, Hq, G, BQ, nqb, bs_log2, num_blocks, max_seqs, max_blocks;
  uint32_t page_bytes;  // bytes of one page over all kv heads
  float scale_log2e;    // |scale| log2(e), at least 1e-30
  uint32_t q_sign;      // 0x80008000 when scale < 0: q enters with its sign flipped
};

// Score-block row rho (0..31) holds token tau(rho) of the block: within each
// 16 rows the middle two groups of four swap places, so that the rows a lane
// holds after S^T = K . Q^T ({8 g + 4 h + e}) are tokens 8 h .. 8 h + 7 of
// each 16-key step, in register order.
__device__ __forceinline__ int pf_token_of_row(int rho) {
  const int q = (rho >> 2) & 3;
  const int q2 = q == 1 ? 2 : q == 2 ? 1 : q;
  return (rho & ~15) | (q2 << 2) | (rho & 3);
}

// What a workgroup works on: kv head g and block qb of a request's rows; the
// request's first row, row count, sequence and length, and whether they are valid.
struct PfBlock {
  int g, qb, r0, m, s, L;
  bool ok;
};

__device__ __forceinline__ PfBlock pf_block(const PrefillArgs &a) {
  // Workgroup -> (request i, kv head g, block qb).  Workgroups are dealt to
  // the eight XCDs in turn; here the blocks of one (request, head) pair all
  // land on one XCD, so its L2 fetches the pair's K/V once, and eight pairs
  // run side by side.  Within a pair the longest blocks go first.
  const int nqb = a.nqb, P = a.n * a.Hkv, Pfull = P & ~7;
  const int b = blockIdx.x;
  int pair, j;
  if (b < Pfull * nqb) {
    const int k = b >> 3;
    pair = (k / nqb) * 8 + (b & 7);
    j = k - (k / nqb) * nqb;
  } else {
    const int b2 = b - Pfull * nqb;
    pair = Pfull + b2 / nqb;
    j = b2 - (b2 / nqb) * nqb;
  }
  const int qb = nqb - 1 - j, g = pair % a.Hkv, i = pair / a.Hkv;
  // ---- request checks (uniform) ----
  const int r0 = a.q_offsets[i], r1 = a.q_offsets[i + 1];
  const bool rows_ok = r0 >= 0 && r1 >= r0 && r1 <= a.total_rows;  // before any row is addressed
  const int m = rows_ok ? r1 - r0 : 0;
  const int s = a.seq_ids[i];
  int L = 0;
  bool ok = rows_ok && m <= a.max_rows && s >= 0 && s < a.max_seqs;
  if (ok) {
    L = a.lengths[s];
    ok = L >= 0 && L <= (a.max_blocks << a.bs_log2) && m <= L;
  }
  return PfBlock{g, qb, r0, m, s, L, ok};
}

// LDS of a workgroup: the ring of K and V buffers, which the merge of the wave
// groups uses again, then the page ids and a flag.
template <int DH, int KS>
constexpr int pf_lds_bytes() {
  const int keys = KS == 4 ? 32 : 64, vp = keys == 32 ? 32 : keys + 8;
  const int ring = 4 * (KS * keys * (DH + 8) + KS * DH * vp);
  const int merge = KS > 1 ? (kPfWaves * 32 * (DH + 4) + kPfWaves * 64) * 4 : 0;
  return (ring > merge ? ring : merge) + kPfMaxPages * 4 + 16;
}

template <int DH, int KS>
__device__ __forceinline__ void prefill_body(const PrefillArgs &a, const PfBlock &wg, uint8_t *lds) {
  constexpr int KEYS = KS == 4 ? 32 : 64;  // keys per tile
  constexpr int SUB = KEYS / 32;           // 32-key score blocks per tile
  constexpr int SPAN = KS * KEYS;          // keys per pass: one tile for each of the KS wave groups
  constexpr int VG = kPfWaves / KS;        // waves per group: 32 VG query vectors per workgroup
  constexpr bool RAISE = KS > 1 || DH == 128;  // priority around the score products (measured below)
  constexpr int KP = DH + 8;        // K tile row pitch (bf16)
  // V tile rows: 72 elements for 64 keys; 32 keys have no room for padding,
  // so chunk c of row r sits at c ^ (r / 4 % 4) (16 rows of one chunk hit
  // all 64 banks once)
  constexpr int VP = KEYS == 32 ? 32 : KEYS + 8;
  auto v_at = [](int row, int chunk) { return row * VP + 8 * (KEYS == 32 ? chunk ^ ((row >> 2) & 3) : chunk); };
  constexpr int NKS = DH / 16;      // k steps of S^T
  constexpr int NRB = DH / 32;      // 32-dim row blocks of O^T
  constexpr int KCH = DH / 8;       // 16-byte chunks of a K row
  constexpr int VCH = KEYS / 8;     // 16-byte chunks of a V row (one dim) in a tile
  constexpr int KTOT = SPAN * KCH, VTOT = KS * DH * VCH;  // 16-byte chunks per pass
  constexpr int KU = (KTOT + kPfThreads - 1) / kPfThreads;  // K chunks per thread and tile
  constexpr int VU = (VTOT + kPfThreads - 1) / kPfThreads;  // V chunks per thread and tile
  constexpr int KBUF = SPAN * KP, VBUF = KS * DH * VP;  // elements of one buffer
  constexpr int RING = 2 * (KBUF + VBUF) * 2;
  constexpr int OPITCH = DH + 4;                        // floats of one vector's outputs in the merge of the groups
  constexpr int MERGE = KS > 1 ? (kPfWaves * 32 * OPITCH + kPfWaves * 64) * 4 : 0;
  constexpr int PAGES = RING > MERGE ? RING : MERGE;
  static_assert(PAGES + kPfMaxPages * 4 + 16 == pf_lds_bytes<DH, KS>(), "LDS of the workgroup");
  int *pages = (int *)(lds + PAGES), *bad_flag = pages + kPfMaxPages;
  uint16_t *k_lds = (uint16_t *)lds, *v_lds = k_lds + 2 * KBUF;  // [2][KBUF], [2][KS][DH * VP]

  const int g = wg.g, qb = wg.qb, r0 = wg.r0, m = wg.m, s = wg.s, L = wg.L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c32 = lane & 31, h2 = lane >> 5;
  const int vg = w % VG, kg = w / VG;  // this wave's vectors and its group's share of the keys
  const int bs_log2 = a.bs_log2, bs = 1 << bs_log2;

  if (!wg.ok) {  // block 0 reports the request and zeroes its rows
    if (qb != 0) return;
    if (tid == 0) set_err(a.err, SM_ERR_EINVAL);
    const int per_row = a.G * DH;  // this kv head's query heads
    for (int64_t e = tid; e < (int64_t)m * per_row; e += kPfThreads) {
      const int rr = (int)(e / per_row), k = (int)(e - (int64_t)rr * per_row);
      a.out[((int64_t)(r0 + rr) * a.Hq + g * a.G) * DH + k] = 0;
    }
    return;
  }
  const int q_lo = qb * a.BQ;  // first row of this block within the request
  if (q_lo >= m) return;
  const int nq = min(a.BQ, m - q_lo);
  const int pos0 = L - m + q_lo;  // position of row q_lo
  const int kend = pos0 + nq;     // keys [0, kend) are needed

  // ---- page ids of keys [0, kend) into LDS, range-checked ----
  if (tid == 0) *bad_flag = 0;
  __syncthreads();
  const int npg = (kend + bs - 1) >> bs_log2;
  for (int p = tid; p < npg; p += kPfThreads) {
    int blk = a.block_table[(int64_t)s * a.max_blocks + p];
    if (blk < 0 || blk >= a.num_blocks) {
      *bad_flag = 1;
      blk = 0;
    }
    pages[p] = blk;
  }
  __syncthreads();
  if (*bad_flag) {  // a corrupt block table: this block's rows are zero
    if (tid == 0) set_err(a.err, SM_ERR_EINVAL);
    const int per_row = a.G * DH;
    for (int e = tid; e < nq * per_row; e += kPfThreads) {
      const int rr = e / per_row, k = e - rr * per_row;
      a.out[((int64_t)(r0 + q_lo + rr) * a.Hq + g * a.G) * DH + k] = 0;
    }
    return;
  }

  // ---- this wave's 32 query vectors: v = 32 vg + c32 -> query head g G + v / BQ, row q_lo + v % BQ ----
  const int v = 32 * vg + c32;
  const int hh = v / a.BQ, rr = v - hh * a.BQ;
  const bool vok = hh < a.G && rr < nq;
  const int vhead = g * a.G + (vok ? hh : 0);
  const int vrow = r0 + q_lo + (vok ? rr : 0);
  const int vpos = vok ? pos0 + rr : -1;  // an idle vector sees no key
  u32x4_t qf[NKS];
  {
    const uint16_t *qp = a.q + ((int64_t)vrow * a.Hq + vhead) * DH + 8 * h2;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      qf[ks] = vok ? *(const u32x4_t *)(qp + 16 * ks) ^ a.q_sign : u32x4_t{0u, 0u, 0u, 0u};
  }
  // wave-wide position range of the valid vectors: tiles past all of them
  // are skipped, tiles before all of them need no mask
  int wave_lo = vok ? vpos : 0x7fffffff, wave_hi = vpos;
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) {
    wave_lo = min(wave_lo, __shfl_xor(wave_lo, sh));
    wave_hi = max(wave_hi, __shfl_xor(wave_hi, sh));
  }
  wave_lo = __builtin_amdgcn_readfirstlane(wave_lo);
  wave_hi = __builtin_amdgcn_readfirstlane(wave_hi);

  // ---- tile loader: 16-byte chunks, K as rows of tokens, V as dim-major runs of 8 tokens ----
  // A chunk's offset within its page is fixed per thread; a tile adds a
  // uniform (t0 mod bs) and its page id.  Tokens past kend re-read page 0.
  const uint64_t page_bytes = a.page_bytes;
  const char *kbase = (const char *)a.k_pool + (int64_t)g * bs * DH * 2;
  const char *vbase = (const char *)a.v_pool + (int64_t)g * bs * DH * 2;
  int ktk[KU], koff[KU], vtk[VU], voff[VU];
#pragma unroll
  for (int u = 0; u < KU; ++u) {
    const int id = min(tid + kPfThreads * u, KTOT - 1);
    ktk[u] = id / KCH;
    koff[u] = ((ktk[u] & (bs - 1)) * DH + (id % KCH) * 8) * 2;
  }
#pragma unroll
  for (int u = 0; u < VU; ++u) {
    const int id = min(tid + kPfThreads * u, VTOT - 1);
    vtk[u] = id / (DH * VCH) * KEYS + 8 * (id % VCH);
    voff[u] = (id / VCH % DH * bs + (vtk[u] & (bs - 1))) * 2;
  }
  auto fetch = [&](int t0, u32x4_t (&kv)[KU + VU]) {
    const int tin = t0 & (bs - 1);  // 0 when a page is no longer than a pass
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int tok = t0 + ktk[u];
      const uint32_t blk = pages[tok < kend ? tok >> bs_log2 : 0];
      kv[u] = *(const u32x4_t *)(kbase + blk * page_bytes + (koff[u] + tin * DH * 2));
    }
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int tok = t0 + vtk[u];
      const uint32_t blk = pages[tok < kend ? tok >> bs_log2 : 0];
      kv[KU + u] = *(const u32x4_t *)(vbase + blk * page_bytes + (voff[u] + tin * 2));
    }
    if (t0 + SPAN > L) {  // the last tile: V entries past the length may hold anything
#pragma unroll
      for (int u = 0; u < VU; ++u) {
        const int nvalid = L - (t0 + vtk[u]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (2 * e >= nvalid) kv[KU + u][e] = 0u;
          else if (2 * e + 1 >= nvalid) kv[KU + u][e] &= 0xffffu;
        }
      }
    }
  };
  auto stash = [&](int buf, const u32x4_t (&kv)[KU + VU]) {
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int id = tid + kPfThreads * u;
      if (KTOT % kPfThreads == 0 || id < KTOT) *(u32x4_t *)(&k_lds[buf * KBUF + (id / KCH) * KP + (id % KCH) * 8]) = kv[u];
    }
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int id = tid + kPfThreads * u;
      if (VTOT % kPfThreads == 0 || id < VTOT) *(u32x4_t *)(&v_lds[buf * VBUF + v_at(id / VCH, id % VCH)]) = kv[KU + u];
    }
  };

  f32x16_t o[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[rb][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sl2 = a.scale_log2e;
  const int krow = pf_token_of_row(c32);  // this lane's K row in the S^T operand

  const int ntiles = (kend + SPAN - 1) / SPAN;
  u32x4_t stage[KU + VU];
  fetch(0, stage);
  stash(0, stage);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int buf = t & 1, t0 = t * SPAN + kg * KEYS;  // this group's tile
    if (t + 1 < ntiles) fetch((t + 1) * SPAN, stage);  // in flight during this pass

    if (t0 <= wave_hi) {
      // S^T = K . Q^T, one 32-key block at a time: its fragment reads first,
      // then its products.  Raised priority until the V reads are issued: the
      // wave that feeds the matrix unit goes before the SIMD's other wave's
      // softmax, so the two fall out of step.  Kernel alone, us without and
      // with, D = 128: KS = 4, 512 rows after 16384 231, 211; 256 after 4096 at
      // 28/4 heads 63, 57; KS = 2, 1024 after 8192 180, 178; KS = 1 next to
      // nothing (16 x 2458 945, 942; 16 x 4096 2371, 2364; 2 x 2048 after 8192
      // 609, 606).  D = 64: KS = 4 and 2 the same, KS = 1 1.5% slower with it
      // (8 x 4096 373, 378).  Around the second product instead KS = 4 lost.
      if constexpr (RAISE) __builtin_amdgcn_s_setprio(1);
      f32x16_t sc[SUB];
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[sb][e] = 0.f;
        const uint16_t *kl = &k_lds[buf * KBUF + (kg * KEYS + 32 * sb + krow) * KP + 8 * h2];
        u32x4_t kf[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) kf[ks] = *(const u32x4_t *)(kl + 16 * ks);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
          sc[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(qf[ks]), sc[sb], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, NKS, 0);  // LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, NKS, 0);  // MFMA
      }
      // V fragments of the first block: lane (d, h2) feeds dims 32 rb + d, tokens 16 kst + 8 h2 .. +7
      u32x4_t vf[NRB][2];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int kst = 0; kst < 2; ++kst)
          vf[rb][kst] = *(const u32x4_t *)(&v_lds[buf * VBUF + v_at(kg * DH + 32 * rb + c32, 2 * kst + h2)]);

      if constexpr (RAISE) __builtin_amdgcn_s_setprio(0);

      // online softmax per query column; register r of block sb holds token
      // t0 + 32 sb + tau(8 (r >> 2) + 4 h2 + (r & 3)).  Masked scores become
      // -inf in place: exp2 of -inf is 0 (the multiplier is positive).
      if (t0 + KEYS - 1 > wave_lo) {
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int tok = t0 + 32 * sb + pf_token_of_row(8 * (r >> 2) + 4 * h2 + (r & 3));
            sc[sb][r] = tok <= vpos ? sc[sb][r] : -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[sb][r]);
      float a0, b0;
      swap32(mx, a0, b0);
      mx = fmaxf(a0, b0);
      const float ms = mx == -INFINITY ? -INFINITY : mx * sl2;  // in log2 units
      const bool move = ms > m_run + 8.0f;
      const float m_new = move ? ms : m_run;
      const float mb = m_new == -INFINITY ? 0.f : m_new;  // a column with no key yet
      if (__ballot(move) != 0) {  // rare: rescale before this tile's products are added
        const float alpha = move ? __builtin_amdgcn_exp2f(m_run - mb) : 1.f;
        l_run *= alpha;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) o[rb] *= alpha;
      }
      m_run = m_new;
      float ps = 0.f;
      u32x4_t pf[SUB][2];
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[sb][r] = __builtin_amdgcn_exp2f(fmaf(sc[sb][r], sl2, -mb));
          ps += sc[sb][r];
        }
        const f32x16_t &x = sc[sb];
#pragma unroll
        for (int kst = 0; kst < 2; ++kst)
          pf[sb][kst] = u32x4_t{cvt_bf16x2(x[8 * kst + 0], x[8 * kst + 1]), cvt_bf16x2(x[8 * kst + 2], x[8 * kst + 3]),
                                cvt_bf16x2(x[8 * kst + 4], x[8 * kst + 5]), cvt_bf16x2(x[8 * kst + 6], x[8 * kst + 7])};
      }
      l_run += ps;

      // O^T += V^T . P^T
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb) {
        if (sb > 0) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int kst = 0; kst < 2; ++kst)
              vf[rb][kst] = *(const u32x4_t *)(&v_lds[buf * VBUF + v_at(kg * DH + 32 * rb + c32, 4 * sb + 2 * kst + h2)]);
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int kst = 0; kst < 2; ++kst)
            o[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[rb][kst]), as_bf16x8(pf[sb][kst]), o[rb], 0, 0, 0);
      }
    }

    if (t + 1 < ntiles) stash(buf ^ 1, stage);
    __syncthreads();
  }

  // ---- normalize and store: register 4 gg + e of block rb = dim 32 rb + 8 gg + 4 h2 + e ----
  float a0, b0;
  swap32(l_run, a0, b0);
  float l_tot = a0 + b0;
  if constexpr (KS > 1) {
    // The groups' softmax states, merged through LDS (the ring is free: the
    // loop ends on a barrier).  Every wave leaves its reference and sum and,
    // scaled to the common reference, its output columns; then wave kg of a
    // group's KS waves adds the KS partials of its DH / KS dims.
    float *ml = (float *)lds, *po = ml + kPfWaves * 64;  // [wave][32 m, 32 l], [wave][32][OPITCH]
    const int live = min(KS, (kend + KEYS - 1) / KEYS);   // groups that had a tile at all
    if (h2 == 0) {
      ml[w * 64 + c32] = m_run;
      ml[w * 64 + 32 + c32] = l_tot;
    }
    __syncthreads();
    float m_all = -INFINITY;
    for (int k = 0; k < live; ++k) m_all = fmaxf(m_all, ml[(k * VG + vg) * 64 + c32]);
    const float mb = m_all == -INFINITY ? 0.f : m_all;  // an idle column
    l_tot = 0.f;
    for (int k = 0; k < live; ++k)
      l_tot += ml[(k * VG + vg) * 64 + 32 + c32] * __builtin_amdgcn_exp2f(ml[(k * VG + vg) * 64 + c32] - mb);
    const float mine = __builtin_amdgcn_exp2f(m_run - mb);
    if (kg < live)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
          *(f32x4_t *)&po[(w * 32 + c32) * OPITCH + 32 * rb + 8 * gg + 4 * h2] =
              f32x4_t{o[rb][4 * gg] * mine, o[rb][4 * gg + 1] * mine, o[rb][4 * gg + 2] * mine, o[rb][4 * gg + 3] * mine};
    __syncthreads();
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (!vok) return;
    // lane (c32, h2) takes dims d0 .. d0 + DH / KS / 2 - 1 of its column
    constexpr int DW = DH / KS / 2;
    const int d0 = kg * (DH / KS) + h2 * DW;
    f32x4_t y[DW / 4];
#pragma unroll
    for (int c = 0; c < DW / 4; ++c) y[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < live; ++k)
#pragma unroll
      for (int c = 0; c < DW / 4; ++c) y[c] += *(const f32x4_t *)&po[((k * VG + vg) * 32 + c32) * OPITCH + d0 + 4 * c];
    uint16_t *op = a.out + ((int64_t)vrow * a.Hq + vhead) * DH + d0;
#pragma unroll
    for (int c = 0; c < DW / 4; ++c)
      *(uint2 *)(op + 4 * c) = make_uint2(cvt_bf16x2(y[c][0] * inv, y[c][1] * inv), cvt_bf16x2(y[c][2] * inv, y[c][3] * inv));
    return;
  }
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  if (!vok) return;
  uint16_t *op = a.out + ((int64_t)vrow * a.Hq + vhead) * DH + 4 * h2;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int gg = 0; gg < 4; ++gg)
      *(uint2 *)(op + 32 * rb + 8 * gg) = make_uint2(cvt_bf16x2(o[rb][4 * gg + 0] * inv, o[rb][4 * gg + 1] * inv),
                                                     cvt_bf16x2(o[rb][4 * gg + 2] * inv, o[rb][4 * gg + 3] * inv));
}

template <int DH, int KS>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_bf16(PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[pf_lds_bytes<DH, KS>()];
  prefill_body<DH, KS>(a, pf_block(a), lds);
}

// For calls of few rows: blocks of KS = 4, but a request of up to kPfFewKeys
// keys is done sooner by the waves of its vectors alone than by four groups
// and their merge.  The length is known here only, so the choice is too.  Us
// alone and split, D = 128: one row of 32/8 heads 1 key 5.6, 6.7; 201 9.2,
// 9.5; 401 12.5, 12.0; 4097 78, 53; 64 rows of 8/8 heads 64 keys 6.1, 8.3; 264
// 11.3, 12.0; 364 12.5, 12.4; 564 16.0, 15.1.  D = 64, one row of 16/4: 201
// 6.9, 7.1; 301 7.6, 7.7; 401 9.3, 8.8.
constexpr int kPfFewKeys = 320;

template <int DH>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_few_bf16(PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[pf_lds_bytes<DH, 4>()];
  static_assert(pf_lds_bytes<DH, 1>() <= pf_lds_bytes<DH, 4>(), "one LDS for both");
  const PfBlock wg = pf_block(a);
  if (wg.L <= kPfFewKeys) prefill_body<DH, 1>(a, wg, lds);
  else prefill_body<DH, 4>(a, wg, lds);
}

}  // namespace sm

using namespace sm;

SM_API sm_status sm_prefill_attention(const sm_paged_cache *c, const int32_t *seq_ids, int n,
                                      const int32_t *q_offsets, int total_rows, const void *q, int num_q_heads,
                                      float scale, int max_rows, void *out, hipStream_t stream) {
  if (!c || n < 0 || max_rows < 0 || total_rows < 0) return SM_EINVAL;
  if (n == 0) return SM_OK;
  if (!seq_ids || !q_offsets || !q || !out || !c->k_pool || !c->v_pool || !c->block_table || !c->lengths ||
      !c->err)
    return SM_EINVAL;
  if (c->dtype != SM_BF16 || !(fabsf(scale) <= 3.0e38f)) return SM_EINVAL;  // a finite scale
  const int H = c->num_kv_heads, D = c->head_dim, bs = c->block_size;
  if (H <= 0 || num_q_heads <= 0 || num_q_heads % H != 0) return SM_EINVAL;
  const int G = num_q_heads / H;
  if (G > 16 || (D != 64 && D != 128)) return SM_EINVAL;
  if (bs < 16 || (bs & (bs - 1)) != 0 || c->max_blocks_per_seq <= 0 || c->max_blocks_per_seq > kPfMaxPages ||
      c->num_blocks <= 0 || c->max_seqs <= 0)
    return SM_EINVAL;
  if (n > 65535 || (uint64_t)H * bs * D * 2 > 0xffffffffull) return SM_EINVAL;
  PrefillArgs a;
  a.k_pool = (const uint16_t *)c->k_pool;
  a.v_pool = (const uint16_t *)c->v_pool;
  a.block_table = c->block_table;
  a.lengths = c->lengths;
  a.seq_ids = seq_ids;
  a.q_offsets = q_offsets;
  a.q = (const uint16_t *)q;
  a.out = (uint16_t *)out;
  a.err = c->err;
  a.n = n;
  a.total_rows = total_rows;
  a.max_rows = max_rows;
  a.Hkv = H;
  a.Hq = num_q_heads;
  a.G = G;
  const PrefillPlan plan = plan_prefill(n, H, G, total_rows, max_rows, (int64_t)c->max_blocks_per_seq * bs);
  const int ks = plan.splits;
  a.BQ = kPfVec / ks / G;
  int bl = 0;
  while ((1 << bl) < bs) ++bl;
  a.bs_log2 = bl;
  a.num_blocks = c->num_blocks;
  a.max_seqs = c->max_seqs;
  a.max_blocks = c->max_blocks_per_seq;
  a.page_bytes = (uint32_t)((uint64_t)H * bs * D * 2);
  // A positive multiplier keeps exp2(-inf) = 0 for masked keys.  Below 1e-30
  // every weight rounds to 1 in fp32 either way (|q . k| stays far below 1e30).
  a.scale_log2e = fmaxf(fabsf(scale) * kPfLog2e, 1e-30f);
  a.q_sign = scale < 0.f ? 0x80008000u : 0u;
  const int nqb = max_rows > 0 ? (max_rows + a.BQ - 1) / a.BQ : 1;  // block 0 reports bad requests
  if ((int64_t)nqb * n * H > 0x7fffffff) return SM_EINVAL;
  a.nqb = nqb;
  const dim3 grid(nqb * n * H);
  const auto kernel = D == 128 ? (plan.few ? prefill_few_bf16<128> : ks == 4 ? prefill_bf16<128, 4>
                                  : ks == 2 ? prefill_bf16<128, 2> : prefill_bf16<128, 1>)
                               : (plan.few ? prefill_few_bf16<64> : ks == 4 ? prefill_bf16<64, 4>
                                  : ks == 2 ? prefill_bf16<64, 2> : prefill_bf16<64, 1>);
  hipLaunchKernelGGL(kernel, grid, dim3(kPfThreads), 0, stream, a);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

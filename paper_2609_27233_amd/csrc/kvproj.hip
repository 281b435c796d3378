// The K/V state of one input row per request at its compressed position
// (gfx950).
//
// After a decode-time merge the frozen backbone takes the surrogate z_s as
// one input embedding and produces one K/V state per layer for the span
// (appendix "Decoding-time Integration").  For the first attention layer
// that state is
//   K = RoPE_p(W_k RMSNorm(x)),  V = W_v RMSNorm(x),
// with x the step's input row (a surrogate or a plain token embedding), p
// the slot it takes in the cache (the sequence's length after the crop),
// and the norm's gain folded into W_k and W_v.
//
// The projection is a skinny product: a handful of rows against 2 Hkv D x d
// weights (16 MB at d = 4096, Hkv D = 1024), so it is bound by streaming
// the weights once.  RMSNorm is a per-row scalar and commutes with the
// product, so the product runs on the raw rows:
//  1. split-K MFMA partials: a workgroup takes 64 output features x 256 of
//     the d inputs for up to 64 rows (v_mfma_f32_16x16x32_bf16, the rows'
//     slice staged in LDS, the weight fragments loaded straight into the
//     operand registers), 256 x d/256 workgroups for d = 4096;
//  2. one workgroup per (row, 256 output features) sums the partials in a
//     fixed order (the result does not depend on scheduling), scales by
//     1/rms, rotates K by the position (the angle formed and reduced in
//     double precision, then fp32 sin/cos) and writes bf16 rows.
// sm_kv_append_projected runs all checks and the block allocation of
// sm_kv_append in one more workgroup of the first launch, beside the product,
// which leaves each row's position and page in the workspace, and the second
// launch writes the rows straight into the pages (a third launch that
// appended them took 15 us for 16 rows, 29 for 128).
#include "cache_meta.hpp"

namespace sm {

constexpr int kPjThreads = 256;
constexpr int kPjRows = 64;   // rows per workgroup
constexpr int kPjFeat = 64;   // output features per workgroup, 16 per wave
constexpr int kPjK = 256;     // inputs per workgroup
constexpr int kPjMaxChunks = 64;  // d <= 64 x 256

struct ProjArgs {
  const uint16_t *x;   // [n][d]
  const uint16_t *Wk;  // [HD][d]
  const uint16_t *Wv;  // [HD][d]
  float *part;         // [d / kPjK][n][2 HD]
  int n, d, HD;
};

// Where a row goes: its position (the sequence's length before the call) and
// the page that takes it, -1 when it is not appended.
struct RowSlot {
  int pos, blk;
};

// The metadata of kv_append for one row per request, by one workgroup of
// kPjThreads threads (thread t holds requests 4 t .. 4 t + 3): the same
// checks in the same order, the same block order; all applied or nothing.
__device__ void append_rows_meta(const CacheArgs &c, const int32_t *seq_ids, int n, RowSlot *slots) {
  constexpr int RPT = SM_MAX_REQUESTS / kPjThreads;
  __shared__ __attribute__((aligned(16))) int ids[SM_MAX_REQUESTS];
  __shared__ int red[16];
  __shared__ int fl_inval, fl_range, fl_stack;
  const int t = threadIdx.x, r0 = RPT * t;
  const int err0 = *c.err, top = *c.free_top;
  const int cap = c.max_blocks << c.bs_log2, bs = 1 << c.bs_log2;
  int s[RPT], L[RPT], need[RPT], blk[RPT], mine = 0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) s[k] = r0 + k < n ? seq_ids[r0 + k] : -1;
#pragma unroll
  for (int k = 0; k < RPT; ++k) L[k] = s[k] >= 0 && s[k] < c.max_seqs ? c.lengths[s[k]] : 0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    ids[r0 + k] = s[k];
    if (r0 + k < n) slots[r0 + k] = RowSlot{L[k], -1};
  }
  if (t == 0) fl_inval = fl_range = fl_stack = 0;
  __syncthreads();
  if (err0 != 0) return;  // sticky: the cache is frozen
  bool bad = false, range = false;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    if (r0 + k < n) {
      bad |= !id_ok(ids, r0 + k, s[k], c.max_seqs);
      range |= L[k] < 0 || L[k] >= cap;  // (no L + 1: a corrupt length may be the largest int)
      need[k] = (L[k] & (bs - 1)) == 0;
    } else {
      need[k] = 0;
    }
    mine += need[k];
  }
  if (bad) fl_inval = 1;
  if (range) fl_range = 1;
  int total;
  int pop = block_inclusive_scan(mine, red, &total) - mine;  // (its barriers order the flags)
  if (fl_inval || fl_range || top < 0 || top > c.num_blocks || total > top) {
    if (t == 0) set_err(c.err, fl_inval ? SM_ERR_EINVAL : fl_range ? SM_ERR_ERANGE : SM_ERR_ENOMEM);
    return;
  }
  // popped ids must name real blocks; a row in a partly filled page takes
  // that page, which is checked for itself
  bool bad_pop = false;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    blk[k] = -1;
    if (r0 + k < n) {
      if (need[k]) {
        blk[k] = c.free_stack[top - 1 - pop];
        ++pop;
      } else {
        blk[k] = c.block_table[(int64_t)s[k] * c.max_blocks + (L[k] >> c.bs_log2)];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k) bad_pop |= need[k] && (blk[k] < 0 || blk[k] >= c.num_blocks);
  if (bad_pop) fl_stack = 1;
  __syncthreads();
  if (fl_stack) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return;
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k)
    if (r0 + k < n) {
      if (need[k]) c.block_table[(int64_t)s[k] * c.max_blocks + (L[k] >> c.bs_log2)] = blk[k];
      else if (blk[k] < 0 || blk[k] >= c.num_blocks) {
        set_err(c.err, SM_ERR_EINVAL);  // corrupt block table: the row is not written
        blk[k] = -1;
      }
      c.lengths[s[k]] = L[k] + 1;
      slots[r0 + k].blk = blk[k];
    }
  if (t == 0) *c.free_top = top - total;
}

// The appending form has one workgroup more, so a flat grid, whose index
// arithmetic would take the 128 registers of four waves per SIMD to 136 and
// leave three: hence its bound.  The other form keeps the grid of three
// dimensions, with which it needs 128 as it is.  1024 rows, d = 4096, HD =
// 1024, both kernels: 153 us, on a flat grid with three waves 170; 128 rows 28.6
// and 29.4; appended (with a rollback) 183 and 194, 33.8 and 34.9.
template <bool APPEND>
__global__ __launch_bounds__(kPjThreads, APPEND ? 4 : 1) void kv_proj_partial_kernel(ProjArgs a, CacheArgs c, const int32_t *seq_ids,
                                                                     RowSlot *slots) {
  __shared__ __attribute__((aligned(16))) uint16_t xs[kPjRows][kPjK + 8];
  if (APPEND && blockIdx.x == 0) {  // dispatched first: it runs beside the product
    append_rows_meta(c, seq_ids, a.n, slots);
    return;
  }
  int fb = blockIdx.x, kc = blockIdx.y, rg = blockIdx.z;
  if constexpr (APPEND) {
    const int id = blockIdx.x - 1, nfb = 2 * a.HD / kPjFeat, nkc = a.d / kPjK;
    fb = id % nfb, kc = id / nfb % nkc, rg = id / (nfb * nkc);
  }
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r = lane & 15, q4 = lane >> 4;
  const int f0 = fb * kPjFeat + 16 * w;  // this wave's 16 features: all K (f0 < HD) or all V
  const uint16_t *W = f0 < a.HD ? a.Wk + (int64_t)f0 * a.d : a.Wv + (int64_t)(f0 - a.HD) * a.d;
  const int k0 = kc * kPjK, r0 = rg * kPjRows;
  const int nr = min(kPjRows, a.n - r0);
  // weight fragments: lane (r, q4) holds W[f0 + r][k0 + 32 s + 8 q4 .. +7]
  u32x4_t wf[kPjK / 32];
#pragma unroll
  for (int s = 0; s < kPjK / 32; ++s)
    wf[s] = __builtin_nontemporal_load((const u32x4_t *)(W + (int64_t)r * a.d + k0 + 32 * s + 8 * q4));
  // the rows' slice k0 .. k0 + 255 into LDS (rows past n are zero)
  const int rows16 = (nr + 15) & ~15;  // whole 16-row tiles
  for (int c = tid; c < rows16 * (kPjK / 8); c += kPjThreads) {
    const int row = c / (kPjK / 8), ch = c % (kPjK / 8);
    u32x4_t v = u32x4_t{0u, 0u, 0u, 0u};
    if (row < nr) v = *(const u32x4_t *)(a.x + (int64_t)(r0 + row) * a.d + k0 + 8 * ch);
    *(u32x4_t *)&xs[row][8 * ch] = v;
  }
  __syncthreads();
  const int ntile = (nr + 15) >> 4;
  f32x4_t acc[kPjRows / 16];
#pragma unroll
  for (int t = 0; t < kPjRows / 16; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < kPjK / 32; ++s)
#pragma unroll
    for (int t = 0; t < kPjRows / 16; ++t)
      if (t < ntile) {
        // x operand: lane (r, q4) holds row 16 t + r, inputs 32 s + 8 q4 .. +7
        const u32x4_t xf = *(const u32x4_t *)&xs[16 * t + r][32 * s + 8 * q4];
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xf), as_bf16x8(wf[s]), acc[t], 0, 0, 0);
      }
  // lane (r, q4), register e: row 16 t + 4 q4 + e, feature f0 + r
#pragma unroll
  for (int t = 0; t < kPjRows / 16; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * t + 4 * q4 + e;
      if (row < nr) a.part[((int64_t)kc * a.n + r0 + row) * (2 * a.HD) + f0 + r] = acc[t][e];
    }
}

struct ProjEpiArgs {
  const uint16_t *x;
  const float *part;
  const int32_t *seq_ids;
  const int32_t *lengths;
  uint16_t *K, *V;        // [n][HD] bf16, or the pools
  const RowSlot *slots;   // rows go into the pools
  int n, d, HD, D, nkc, max_seqs;
  float rms_eps;
  double inv_freq[64];    // theta^(-2j/D), j < D/2, computed on the host
};

constexpr double kTwoPi = 6.283185307179586476925286766559;

// One workgroup per (block of 256 output features, row): a block covers
// whole heads, so both halves of every rotary pair are at hand.
template <bool APPEND>
__global__ __launch_bounds__(kPjThreads) void kv_proj_epilogue_kernel(ProjEpiArgs a, int Hkv, int bs_log2) {
  __shared__ float ys[kPjThreads];
  __shared__ float red[16];
  const int fb = blockIdx.x, i = blockIdx.y, tid = threadIdx.x;
  const int f = fb * kPjThreads + tid;  // K features first, then V
  double pos;
  RowSlot rs = {0, -1};
  if constexpr (APPEND) {
    rs = a.slots[i];
    if (rs.blk < 0) return;  // the append failed, or the row's page is not usable (uniform: one row per workgroup)
    pos = (double)rs.pos;
  } else {
    const int s = a.seq_ids[i];
    pos = (s >= 0 && s < a.max_seqs) ? (double)a.lengths[s] : 0.0;
  }
  // the split-K partials, summed in a fixed order once all are loaded; their
  // loads are in flight while the row's RMSNorm scale is reduced
  float pv[kPjMaxChunks];
#pragma unroll
  for (int kc = 0; kc < kPjMaxChunks; ++kc)
    pv[kc] = kc < a.nkc ? a.part[((int64_t)kc * a.n + i) * (2 * a.HD) + f] : 0.f;
  float ss = 0.f;
  for (int k = 8 * tid; k < a.d; k += 8 * kPjThreads) {
    const u32x4_t v = *(const u32x4_t *)(a.x + (int64_t)i * a.d + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __uint_as_float(v[e] << 16), hi = __uint_as_float(v[e] & 0xffff0000u);
      ss += lo * lo + hi * hi;
    }
  }
  ss = block_sum(ss, red);
  const float inv = rsqrtf(ss / a.d + a.rms_eps);
  float y = 0.f;
#pragma unroll
  for (int kc = 0; kc < kPjMaxChunks; ++kc) y += pv[kc];
  y *= inv;
  ys[tid] = y;
  __syncthreads();
  // this feature's place: its row, or its slot in the page
  const int fk = f < a.HD ? f : f - a.HD;
  const int64_t kat = APPEND ? (((int64_t)rs.blk * Hkv + fk / a.D) << bs_log2) * a.D +
                                   (int64_t)(rs.pos & ((1 << bs_log2) - 1)) * a.D + fk % a.D
                             : (int64_t)i * a.HD + fk;
  if (f < a.HD) {
    // rotate-half RoPE: pair (j, j + D/2) turned by pos theta^(-2j/D); the
    // angle is formed and reduced to [-pi, pi] in double precision
    const int half = a.D / 2, jd = f % a.D, j = jd % half;
    const double ang = pos * a.inv_freq[j];
    const float r = (float)(ang - kTwoPi * rint(ang / kTwoPi));
    const float c = cosf(r), sn = sinf(r);
    const float other = ys[jd < half ? tid + half : tid - half];
    const float out = jd < half ? y * c - other * sn : y * c + other * sn;
    a.K[kat] = f32_to_bf16(out);
  } else {
    const int64_t vat = APPEND ? ((((int64_t)rs.blk * Hkv + fk / a.D) * a.D + fk % a.D) << bs_log2) +
                                     (rs.pos & ((1 << bs_log2) - 1))
                               : kat;
    a.V[vat] = f32_to_bf16(y);
  }
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

static size_t part_bytes(int n, int d, int HD) { return align256((size_t)(d / kPjK) * n * 2 * HD * sizeof(float)); }

}  // namespace sm

using namespace sm;

static bool proj_ok(const sm_paged_cache *c, int n, const void *x, const sm_kv_proj_params *p) {
  if (!c || !p || n < 0 || n > SM_MAX_REQUESTS || n > c->max_seqs) return false;
  if (c->dtype != SM_BF16 || (c->head_dim != 64 && c->head_dim != 128) || c->num_kv_heads <= 0) return false;
  const int HD = c->num_kv_heads * c->head_dim;
  if (HD > 2048 || (2 * HD) % kPjThreads != 0) return false;
  if (p->d <= 0 || p->d % kPjK != 0 || p->d > kPjK * kPjMaxChunks || !(p->rope_theta > 0.f) ||
      !(p->rms_eps >= 0.f))
    return false;
  return n == 0 || (x && p->W_k && p->W_v && c->lengths);
}

SM_API size_t sm_kv_project_workspace_bytes(int n, int d, int num_kv_heads, int head_dim) {
  if (n < 0 || d <= 0 || d % kPjK != 0 || d > kPjK * kPjMaxChunks || num_kv_heads <= 0 || head_dim <= 0)
    return 0;
  const int HD = num_kv_heads * head_dim;
  return part_bytes(n, d, HD) + 2 * align256((size_t)n * HD * 2) + align256((size_t)(n + 1) * 4);
}

// K, V: [n][HD] rows, or with `slots` the pools of `ca` (the append).
static sm_status launch_project(const sm_paged_cache *c, const int32_t *seq_ids, int n, const void *x,
                                const sm_kv_proj_params *p, void *K, void *V, const CacheArgs &ca, RowSlot *slots,
                                float *part, hipStream_t stream) {
  const int HD = c->num_kv_heads * c->head_dim;
  ProjArgs a{(const uint16_t *)x, (const uint16_t *)p->W_k, (const uint16_t *)p->W_v, part, n, p->d, HD};
  const dim3 grid(2 * HD / kPjFeat, p->d / kPjK, (n + kPjRows - 1) / kPjRows);
  ProjEpiArgs e{(const uint16_t *)x, part, seq_ids, c->lengths, (uint16_t *)K, (uint16_t *)V, slots,
                n, p->d, HD, c->head_dim, p->d / kPjK, c->max_seqs, p->rms_eps, {}};
  for (int j = 0; j < c->head_dim / 2; ++j) e.inv_freq[j] = pow((double)p->rope_theta, -2.0 * j / c->head_dim);
  const dim3 egrid(2 * HD / kPjThreads, n);
  if (slots) {
    hipLaunchKernelGGL(kv_proj_partial_kernel<true>, dim3(grid.x * grid.y * grid.z + 1), dim3(kPjThreads), 0,
                       stream, a, ca, seq_ids, slots);
    hipLaunchKernelGGL(kv_proj_epilogue_kernel<true>, egrid, dim3(kPjThreads), 0, stream, e, ca.Hkv, ca.bs_log2);
  } else {
    hipLaunchKernelGGL(kv_proj_partial_kernel<false>, grid, dim3(kPjThreads), 0, stream, a, ca, seq_ids, slots);
    hipLaunchKernelGGL(kv_proj_epilogue_kernel<false>, egrid, dim3(kPjThreads), 0, stream, e, 0, 0);
  }
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

SM_API sm_status sm_kv_project(const sm_paged_cache *c, const int32_t *seq_ids, int n, const void *x,
                               const sm_kv_proj_params *p, void *K, void *V, void *ws, size_t ws_bytes,
                               hipStream_t stream) {
  if (!proj_ok(c, n, x, p)) return SM_EINVAL;
  if (n == 0) return SM_OK;
  if (!seq_ids || !K || !V || !ws ||
      ws_bytes < sm_kv_project_workspace_bytes(n, p->d, c->num_kv_heads, c->head_dim))
    return SM_EINVAL;
  return launch_project(c, seq_ids, n, x, p, K, V, CacheArgs{}, nullptr, (float *)ws, stream);
}

SM_API sm_status sm_kv_append_projected(const sm_paged_cache *c, const int32_t *seq_ids, int n, const void *x,
                                        const sm_kv_proj_params *p, void *ws, size_t ws_bytes,
                                        hipStream_t stream) {
  if (!proj_ok(c, n, x, p)) return SM_EINVAL;
  CacheArgs ca;
  if (!cache_ok(c, ca)) return SM_EINVAL;  // (as sm_kv_append)
  if (n == 0) return SM_OK;
  if (!seq_ids || !ws || ws_bytes < sm_kv_project_workspace_bytes(n, p->d, c->num_kv_heads, c->head_dim))
    return SM_EINVAL;
  float *part = (float *)ws;
  RowSlot *slots = (RowSlot *)((char *)ws + part_bytes(n, p->d, c->num_kv_heads * c->head_dim));
  return launch_project(c, seq_ids, n, x, p, c->k_pool, c->v_pool, ca, slots, part, stream);
}

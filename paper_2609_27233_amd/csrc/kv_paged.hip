// Paged KV-cache bookkeeping for span merging (gfx950):
//   kv_rollback  crop k entries per sequence (decoding-time merge, the paper's
//                "crop the n-1 cached entries" step); metadata only
//   kv_append    append K/V rows (the surrogate's single state, a decode
//                token, or a whole compressed prompt)
//   pack_spans   keep mask -> compressed positions -> packed rows (prompt
//                merging, "Prompt-time Integration")
//
// Metadata kernels run as ONE workgroup of 1024 threads: every request is
// validated first (all-or-nothing), then block ids move between the block
// table and the LIFO free stack at positions fixed by prefix sums, so the
// result is deterministic and identical to the sequential definition
// (rollback pushes in reverse request order, highest logical block first;
// append pops in request order, lowest logical block first).
#include "cache_meta.hpp"

namespace sm {

__global__ __launch_bounds__(kMetaThreads) void rollback_kernel(CacheArgs c, const int32_t *seq_ids,
                                                                 const int32_t *ks, int n) {
  const int t = threadIdx.x;
  const int s = t < n ? seq_ids[t] : -1, k = t < n ? ks[t] : 0;
  rollback_body(c, rollback_reads(c, s), s, k, n);
}

// Validation and block allocation of kv_append, run by one workgroup of
// kMetaThreads threads (thread t owns request t).  Returns true, uniformly
// across the workgroup, when the call was applied; on return *L_old holds
// request t's length before the call.
struct AppendShared {
  int red[16];
  int fl_inval, fl_range, fl_stack, s_err, s_top;
  int incl[kMetaThreads];   // inclusive prefix of the blocks each request pops
  int first[kMetaThreads];  // its first new logical block
  int sid[kMetaThreads];    // its sequence
};

__device__ bool append_meta_body(const CacheArgs &c, const int32_t *seq_ids, const int32_t *row_offsets, int n,
                                 int total_rows, AppendShared &sh, int &s_out, int &L_old) {
  const int t = threadIdx.x;
  if (t == 0) {
    sh.fl_inval = 0;
    sh.fl_range = 0;
    sh.fl_stack = 0;
    sh.s_err = *c.err;
    sh.s_top = *c.free_top;
    if (row_offsets[0] != 0 || row_offsets[n] != total_rows) sh.fl_inval = 1;
  }
  __syncthreads();
  if (sh.s_err != 0) return false;  // sticky: the cache is frozen

  const bool active = t < n;
  int s = 0, m = 0;
  if (active) {
    s = seq_ids[t];
    m = row_offsets[t + 1] - row_offsets[t];
    sh.sid[t] = s;
  }
  __syncthreads();
  if (active && (m < 0 || !id_ok(sh.sid, t, s, c.max_seqs))) sh.fl_inval = 1;
  __syncthreads();
  if (sh.fl_inval) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return false;
  }
  const int cap = c.max_blocks << c.bs_log2;
  int L = 0, need = 0;
  if (active) {
    L = c.lengths[s];
    if (L < 0 || (int64_t)L + m > cap) sh.fl_range = 1;
    else need = blocks_for(L + m, c.bs_log2) - blocks_for(L, c.bs_log2);
  }
  __syncthreads();
  if (sh.fl_range) {
    if (t == 0) set_err(c.err, SM_ERR_ERANGE);
    return false;
  }
  int total;
  const int incl = block_inclusive_scan(need, sh.red, &total);
  const int top = sh.s_top;
  if (top < 0 || top > c.num_blocks || total > top) {
    if (t == 0) set_err(c.err, SM_ERR_ENOMEM);
    return false;
  }
  // every id about to be popped must name a real block
  // (the first kPopCache ids of each thread stay in registers for the pops)
  constexpr int kPopCache = 4;
  int popv[kPopCache];
#pragma unroll
  for (int k = 0; k < kPopCache; ++k) {
    const int j = t + k * (int)blockDim.x;
    popv[k] = j < total ? c.free_stack[top - 1 - j] : 0;
  }
#pragma unroll
  for (int k = 0; k < kPopCache; ++k)
    if (t + k * (int)blockDim.x < total && (popv[k] < 0 || popv[k] >= c.num_blocks)) sh.fl_stack = 1;
  for (int j = t + kPopCache * (int)blockDim.x; j < total; j += blockDim.x) {
    const int blk = c.free_stack[top - 1 - j];
    if (blk < 0 || blk >= c.num_blocks) sh.fl_stack = 1;
  }
  __syncthreads();
  if (sh.fl_stack) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return false;
  }
  if (active) {
    sh.incl[t] = incl;
    sh.first[t] = blocks_for(L, c.bs_log2);
    sh.sid[t] = s;
    c.lengths[s] = L + m;
  }
  __syncthreads();
  // pop p goes to the request whose range [incl - need, incl) holds it:
  // free_stack[top - 1 - p] -> block_table[s][first + p - (incl - need)];
  // all threads share the pops (a prompt batch takes thousands of blocks)
  auto pop = [&](int p, int blk) {
    int lo = 0, hi = n - 1;  // first request with incl > p
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sh.incl[mid] > p) hi = mid;
      else lo = mid + 1;
    }
    const int before = lo ? sh.incl[lo - 1] : 0;
    c.block_table[(int64_t)sh.sid[lo] * c.max_blocks + sh.first[lo] + (p - before)] = blk;
  };
#pragma unroll
  for (int k = 0; k < kPopCache; ++k) {
    const int p = t + k * (int)blockDim.x;
    if (p < total) pop(p, popv[k]);
  }
  for (int p = t + kPopCache * (int)blockDim.x; p < total; p += blockDim.x) pop(p, c.free_stack[top - 1 - p]);
  if (t == 0) *c.free_top = top - total;
  s_out = s;
  L_old = L;
  return true;
}

__global__ __launch_bounds__(kMetaThreads) void append_meta_kernel(CacheArgs c, const int32_t *seq_ids,
                                                                    const int32_t *row_offsets, int n,
                                                                    int total_rows) {
  __shared__ AppendShared sh;
  int s, L;
  append_meta_body(c, seq_ids, row_offsets, n, total_rows, sh, s, L);
}

// Copy rows [r_begin, r_end) of K and V into their slots; row_blk/row_slot
// (LDS) give the destination of row r - r_begin (block -1: skip).  One unit
// = one 16-byte group of one row (VEC elements of one head); `upr` divides
// by the units per row.  Threads `lane0`, lane0 + stride, ... share the
// units; each unit's K and V loads are issued before its stores.
template <typename T>
__device__ __forceinline__ void copy_rows(const CacheArgs &c, const T *__restrict__ K, const T *__restrict__ V,
                                          int r_begin, int r_end, const FastDiv &upr, const int *row_blk,
                                          const int *row_slot, int lane0, int stride) {
  constexpr int VEC = 16 / sizeof(T);
  const int bs = 1 << c.bs_log2;
  const int gpl2 = c.dh_log2 - (sizeof(T) == 2 ? 3 : 2);  // log2(groups per head)
  const int row_elems = c.Hkv << c.dh_log2;
  const int units = (r_end - r_begin) * (int)upr.d;
  T *kp = (T *)c.k_pool;
  T *vp = (T *)c.v_pool;
  for (int u = lane0; u < units; u += stride) {
    const int rr = (int)fdiv((uint32_t)u, upr);
    const int gi = u - rr * (int)upr.d;           // group within the row
    const int g = gi >> gpl2, d0 = (gi & ((1 << gpl2) - 1)) * VEC;
    const int64_t src = (int64_t)(r_begin + rr) * row_elems + (int64_t)gi * VEC;
    const u32x4_t kv = *(const u32x4_t *)(K + src);
    const u32x4_t vv = *(const u32x4_t *)(V + src);
    const int blk = row_blk[rr];
    if (blk < 0) continue;
    const int slot = row_slot[rr];
    *(u32x4_t *)(kp + (((int64_t)blk * c.Hkv + g) * bs + slot) * c.DH + d0) = kv;
    T *vdst = vp + (((int64_t)blk * c.Hkv + g) * c.DH + d0) * bs + slot;
    const T *ve = (const T *)&vv;
#pragma unroll
    for (int e = 0; e < VEC; ++e) vdst[e * bs] = ve[e];
  }
}

// Small appends (a decode step: one row per sequence) in ONE workgroup,
// metadata and copy together.  The sequence of dependent global accesses is
// kept short: (1) ids / offsets / error word, (2) lengths, (3) the tail
// block of each sequence and the popped free-stack entries, (4) the row
// copies.  Same validation order and block order as the two-kernel path.
constexpr int kSmallBytes = 64 * 1024;  // of K (and of V) per call
constexpr int kSmallRows = 1024;

template <typename T>
__global__ __launch_bounds__(kMetaThreads) void append_small_kernel(CacheArgs c, const int32_t *seq_ids,
                                                                     const int32_t *row_offsets, int n,
                                                                     int total_rows, const T *__restrict__ K,
                                                                     const T *__restrict__ V, FastDiv upr) {
  __shared__ int red[16];
  __shared__ int ids[kMetaThreads];
  __shared__ int fl_inval, fl_range, fl_stack, s_err, s_top;
  __shared__ int row_blk[kSmallRows], row_slot[kSmallRows];
  const int t = threadIdx.x;
  const bool active = t < n;
  // (1)
  int s = -1, r0 = 0, r1 = 0;
  if (active) {
    s = seq_ids[t];
    r0 = row_offsets[t];
    r1 = row_offsets[t + 1];
    ids[t] = s;
  }
  if (t == 0) {
    fl_range = 0;
    fl_stack = 0;
    s_err = *c.err;
    s_top = *c.free_top;
    fl_inval = (row_offsets[0] != 0 || row_offsets[n] != total_rows);
  }
  __syncthreads();
  if (s_err != 0) return;  // sticky: the cache is frozen
  if (active) {
    bool ok = r1 >= r0 && s >= 0 && s < c.max_seqs;
    for (int j = 0; j < t && ok; ++j) ok = ids[j] != s;
    if (!ok) fl_inval = 1;
  }
  __syncthreads();
  if (fl_inval) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return;
  }
  // (2)
  const int m = r1 - r0;
  const int cap = c.max_blocks << c.bs_log2;
  int L = 0, need = 0;
  if (active) {
    L = c.lengths[s];
    if (L < 0 || (int64_t)L + m > cap) fl_range = 1;
    else need = blocks_for(L + m, c.bs_log2) - blocks_for(L, c.bs_log2);
  }
  __syncthreads();
  if (fl_range) {
    if (t == 0) set_err(c.err, SM_ERR_ERANGE);
    return;
  }
  int total;
  const int incl = block_inclusive_scan(need, red, &total);
  const int top = s_top;
  if (top < 0 || top > c.num_blocks || total > top) {
    if (t == 0) set_err(c.err, SM_ERR_ENOMEM);
    return;
  }
  // (3) every popped id must name a real block; the partially filled tail
  // block (if a new row lands in it) is read once
  for (int j = t; j < total; j += kMetaThreads) {
    const int blk = c.free_stack[top - 1 - j];
    if (blk < 0 || blk >= c.num_blocks) fl_stack = 1;
  }
  int32_t *brow = c.block_table + (int64_t)(active ? s : 0) * c.max_blocks;
  const int first = blocks_for(L, c.bs_log2);  // first logical block to allocate
  const int lp_tail = L >> c.bs_log2;           // page of the first new row
  const int tail_blk = (active && m > 0 && lp_tail < first) ? brow[lp_tail] : -1;
  __syncthreads();
  if (fl_stack) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return;
  }
  const int bs = 1 << c.bs_log2;
  if (active) {
    const int pop0 = incl - need;  // pops already taken by earlier requests
    for (int q = 0; q < need; ++q) brow[first + q] = c.free_stack[top - 1 - (pop0 + q)];
    c.lengths[s] = L + m;
    for (int r = r0; r < r1; ++r) {
      const int pos = L + (r - r0);
      const int lp = pos >> c.bs_log2;
      const int b = (lp < first) ? tail_blk : c.free_stack[top - 1 - (pop0 + lp - first)];
      const bool ok = b >= 0 && b < c.num_blocks;
      if (!ok) set_err(c.err, SM_ERR_EINVAL);  // corrupt block table
      row_blk[r] = ok ? b : -1;
      row_slot[r] = pos & (bs - 1);
    }
  }
  if (t == 0) *c.free_top = top - total;
  __syncthreads();
  // (4) the copy, in units of one 16-byte group of one row: the K group
  // goes to its token-major page with one 16-byte store, the V group's
  // elements go to the dim-major page one slot at a time
  copy_rows<T>(c, K, V, 0, total_rows, upr, row_blk, row_slot, t, kMetaThreads);
}

// Copy phase of kv_append, run after append_meta_kernel has validated the
// call, taken the blocks and advanced the lengths.  The unit of work is a
// 16-slot segment (16-aligned positions) of a destination page that the
// call writes: request i writes positions [L_old, L_new) of its sequence,
// which touch segments L_old / 16 .. (L_new - 1) / 16.  The grid is
// persistent (at most the resident workgroups): each workgroup forms the
// prefix sum of the segment counts over the requests once, then takes
// kSegPerWg consecutive segments at a time, one per group of kSegThreads
// threads, stepping by the grid (measured 7% faster for a 39k-row prompt
// batch than one launch-wide wave of two-segment workgroups, which paid
// the prefix sum's chain of dependent reads for every 256 KB they moved).
// Slots outside [L_old, L_new) are never written.
//  * K pages are token-major ([head][slot][dim]): every 16-byte group of a
//    row is a 16-byte load and a 16-byte store.
//  * V pages are dim-major ([head][dim][slot]): a thread loads VEC rows x
//    VEC dims (VEC 16-byte loads: VEC consecutive positions, VEC dims of
//    one head), transposes them in registers and stores VEC 16-byte
//    groups (VEC consecutive slots of one dim); partly covered groups fall
//    back to one store per element.
// Every load of a thread is issued before its stores.  The error word is
// read beside the first index loads; nothing is written if it is set.
constexpr int kSegSlots = 16;
constexpr int kSegThreads = 256;
constexpr int kSegPerWg = 1;
constexpr int kSegWgThreads = kSegThreads * kSegPerWg;
constexpr int kMaxRowElems = 2048;  // num_kv_heads * head_dim

// out[i] = element i of in[0..VEC-1] (a VEC x VEC transpose of 16-byte rows)
__device__ __forceinline__ void transpose_rows(const u32x4_t (&in)[8], u32x4_t (&out)[8]) {  // bf16
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t x = in[2 * w][i >> 1], y = in[2 * w + 1][i >> 1];
      out[i][w] = (i & 1) ? ((x >> 16) | (y & 0xffff0000u)) : ((x & 0xffffu) | (y << 16));
    }
}
__device__ __forceinline__ void transpose_rows(const u32x4_t (&in)[4], u32x4_t (&out)[4]) {  // fp32
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) out[i][j] = in[j][i];
}

struct SegDesc {
  int row0, lold, lnew, seg, blk;  // blk -1: nothing to write
};

template <typename T>
__global__ __launch_bounds__(kSegWgThreads) void append_segments_kernel(CacheArgs c, const int32_t *seq_ids,
                                                                        const int32_t *row_offsets, int n,
                                                                        const T *__restrict__ K,
                                                                        const T *__restrict__ V) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int RPT = (SM_MAX_REQUESTS + kSegWgThreads - 1) / kSegWgThreads;  // requests per thread
  __shared__ int red[16];
  __shared__ SegDesc sd[kSegPerWg];
  const int t = threadIdx.x;
  // segments per request, requests RPT t .. RPT t + RPT - 1, and the error word
  const int err0 = *c.err;
  int cnt[RPT], sq[RPT], ro[RPT], mm[RPT], ln[RPT], mine = 0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int j = RPT * t + k;
    sq[k] = j < n ? seq_ids[j] : 0;
    ro[k] = j < n ? row_offsets[j] : 0;
    mm[k] = j < n ? row_offsets[j + 1] - ro[k] : 0;
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int j = RPT * t + k;
    // advanced by the metadata pass (ids are checked: this read precedes
    // the error word's, which tells whether that pass failed)
    ln[k] = (j < n && sq[k] >= 0 && sq[k] < c.max_seqs) ? c.lengths[sq[k]] : 0;
    cnt[k] = (j < n && mm[k] > 0) ? ((ln[k] - 1) >> 4) - ((ln[k] - mm[k]) >> 4) + 1 : 0;
    mine += cnt[k];
  }
  if (t < kSegPerWg) sd[t].blk = -1;
  int total;
  const int incl = block_inclusive_scan(mine, red, &total);  // (its barriers order the sd writes)
  if (__syncthreads_or(err0 != 0)) return;  // uniform
  for (int b0 = blockIdx.x * kSegPerWg; b0 < total; b0 += gridDim.x * kSegPerWg) {
    if (b0 != (int)blockIdx.x * kSegPerWg) {
      __syncthreads();  // every thread holds the previous segments' descriptors
      if (t < kSegPerWg) sd[t].blk = -1;
      __syncthreads();
    }
    {
      int before = incl - mine;
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
#pragma unroll
        for (int q = 0; q < kSegPerWg; ++q) {
          const int b = b0 + q;
          if (b < total && b >= before && b < before + cnt[k]) {
            const int seg = ((ln[k] - mm[k]) >> 4) + (b - before);
            SegDesc d;
            d.row0 = ro[k];
            d.lold = ln[k] - mm[k];
            d.lnew = ln[k];
            d.seg = seg;
            d.blk = c.block_table[(int64_t)sq[k] * c.max_blocks + ((seg << 4) >> c.bs_log2)];
            if (d.blk < 0 || d.blk >= c.num_blocks) {
              set_err(c.err, SM_ERR_EINVAL);  // corrupt block table: the segment is not written
              d.blk = -1;
            }
            sd[q] = d;
          }
        }
        before += cnt[k];
      }
    }
    __syncthreads();
    const int q = t / kSegThreads, tt = t - q * kSegThreads;
    const SegDesc d = sd[q];
    if (d.blk < 0) continue;  // (no barrier in the copy: the next one is the next iteration's)
    const int bs = 1 << c.bs_log2;
    const int p0 = d.seg << 4;                       // first position of the segment
    const int lo = max(p0, d.lold) - p0, hi = min(p0 + kSegSlots, d.lnew) - p0;  // valid slots [lo, hi)
    const int slot0 = p0 & (bs - 1);
    const int64_t row_elems = (int64_t)c.Hkv << c.dh_log2;
    const int64_t rbase = (int64_t)(d.row0 + p0 - d.lold) * row_elems;  // input offset of slot 0's row
    T *kp = (T *)c.k_pool + (int64_t)d.blk * row_elems * bs;
    T *vp = (T *)c.v_pool + (int64_t)d.blk * row_elems * bs;
    const int vpr = (int)(row_elems / VEC);        // 16-byte groups per row
    const int gshift = c.dh_log2;                  // element index -> head

    // V: sub-unit = (head, VEC dims, VEC slots)
    const int dgs = (1 << c.dh_log2) / VEC;        // dim groups per head
    const int sub_units = c.Hkv * dgs * (kSegSlots / VEC);
    // K: unit = one 16-byte group of one slot's row
    const int k_units = kSegSlots * vpr;
    for (int base_v = 0, base_k = 0; base_v < sub_units || base_k < k_units;
         base_v += kSegThreads, base_k += 8 * kSegThreads) {
      // loads
      u32x4_t va[VEC];
      const int su = base_v + tt;
      int sg = 0, g = 0, dg = 0;
      if (su < sub_units) {
        sg = su % (kSegSlots / VEC);
        const int hd = su / (kSegSlots / VEC);
        g = hd / dgs;
        dg = hd - g * dgs;
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
          const int sl = sg * VEC + j;
          va[j] = (sl >= lo && sl < hi)
                      ? *(const u32x4_t *)(V + rbase + (int64_t)sl * row_elems + ((int64_t)g << gshift) + dg * VEC)
                      : u32x4_t{0u, 0u, 0u, 0u};
        }
      }
      u32x4_t ka[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = base_k + u * kSegThreads + tt;
        const int sl = e / vpr;
        ka[u] = (e < k_units && sl >= lo && sl < hi)
                    ? *(const u32x4_t *)(K + rbase + (int64_t)sl * row_elems + (int64_t)(e - sl * vpr) * VEC)
                    : u32x4_t{0u, 0u, 0u, 0u};
      }
      // stores
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = base_k + u * kSegThreads + tt;
        const int sl = e / vpr;
        if (e < k_units && sl >= lo && sl < hi) {
          const int el = (e - sl * vpr) * VEC;      // element within the row
          const int gg = el >> gshift, dd = el & ((1 << gshift) - 1);
          // streaming stores: whole 256-byte runs of a token-major page
          // (measured 1.2x faster for the call than plain stores; the V
          // pages' 32-byte pieces are faster as plain stores that L2 merges)
          __builtin_nontemporal_store(ka[u], (u32x4_t *)(kp + (((int64_t)gg * bs + slot0 + sl) << gshift) + dd));
        }
      }
      if (su < sub_units) {
        u32x4_t vt[VEC];
        transpose_rows(va, vt);
        const int s_first = sg * VEC;
        T *vd = vp + (((int64_t)g << gshift) + dg * VEC) * bs + slot0 + s_first;
        if (s_first >= lo && s_first + VEC <= hi) {
#pragma unroll
          for (int i = 0; i < VEC; ++i) *(u32x4_t *)(vd + (int64_t)i * bs) = vt[i];
        } else {
#pragma unroll
          for (int i = 0; i < VEC; ++i) {
            const T *e = (const T *)&vt[i];
#pragma unroll
            for (int j = 0; j < VEC; ++j)
              if (s_first + j >= lo && s_first + j < hi) vd[(int64_t)i * bs + j] = e[j];
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// pack_spans

constexpr int kPackThreads = 1024;
constexpr int kPackMaxPer = 4;    // tokens per thread of an index workgroup
constexpr int kRemoved = INT32_MIN;

struct PackArgs {
  int B, total_tokens, num_spans;
  const int32_t *seq_offsets, *span_start, *span_len, *seq_span_offsets;
  int32_t *pi, *packed_offsets, *packed_src;
  const int32_t *token_ids;
  const void *emb;
  int64_t emb_rows;
  const void *surrogates;
  int d;
  void *packed;
  int32_t *err;
};

// Index pass of pack_spans.  With R(t) the positions removed before t in the
// whole batch, a kept token t goes to packed row t - R(t), and its compressed
// position is that less the row of its sequence's first token.  So the
// batch is cut into pieces of kPackThreads x PER tokens whatever its
// sequences' lengths (one workgroup per sequence took 38 us for one sequence
// of 32,768 tokens, 17 for 16 of 4,096), and each workgroup needs only the
// span list: one pass over it validates all of it (so that no workgroup
// writes with offsets computed from invalid input), counts the positions
// removed before its piece, before the sequence that the piece begins in and
// in all, and marks the spans that fall into its piece in LDS.  The span ->
// sequence search and the bounds it checks read LDS copies of the offsets
// when they fit (kPackSsoLds entries; IN_LDS), else global memory; each thread
// loads its spans kPackBatch at a time, so that their loads share one round
// trip, and searches again only when a span is past the sequence of the one
// before (a search per span: 586 us, not 422, for 128 x 32,768 tokens).
// PER is 1 up to kPackWgs workgroups, then 4.  Each repeats the pass over the
// spans, so there are no more of them: a larger batch (MANY) gives each
// several consecutive pieces, and from its second piece on a workgroup reads
// the spans that start there only.  Index pass in us with a workgroup per
// piece, and so: 64 x 32,768 tokens, 262,144 spans: 418, 191; 128 x 32,768:
// 1652, 422 (a workgroup per sequence took 258 and 557).
constexpr int kPackWgs = 256;
constexpr int kPackSsoLds = 4096;

// last b in [0, n) with at(b) <= x (at(0) <= x)
template <class F>
__device__ __forceinline__ int last_le(F at, int n, int x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (at(mid) <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int PER, bool MANY, bool IN_LDS>
__global__ __launch_bounds__(kPackThreads) void pack_index_kernel(PackArgs a, int pieces) {
  constexpr int CHUNK = kPackThreads * PER;
  __shared__ int src[CHUNK];         // packed source of each token, then its packed row
  __shared__ int sso[IN_LDS ? kPackSsoLds : 1], so[IN_LDS ? kPackSsoLds : 1];
  __shared__ int red[16];
  __shared__ int flag, s_err, sums[4];
  const int t = threadIdx.x;
  int c0 = blockIdx.x * CHUNK * (MANY ? pieces : 1), cn = min(CHUNK, a.total_tokens - c0);  // (cn = 0: no tokens at all)
  if (t == 0) {
    s_err = *a.err;
    flag = a.seq_offsets[0] != 0 || a.seq_offsets[a.B] != a.total_tokens || a.seq_span_offsets[0] != 0 ||
           a.seq_span_offsets[a.B] != a.num_spans;
  }
  if (t < 4) sums[t] = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) src[t + u * kPackThreads] = c0 + t + u * kPackThreads;
  bool bad = false;
  for (int b = t; b <= a.B; b += kPackThreads) {
    const int s1 = a.seq_span_offsets[b], o1 = a.seq_offsets[b];
    if constexpr (IN_LDS) {
      sso[b] = s1;
      so[b] = o1;
    }
    if (b < a.B) bad |= a.seq_offsets[b + 1] < o1 || a.seq_span_offsets[b + 1] < s1;
  }
  __syncthreads();
  if (s_err != 0) return;
  if (bad) flag = 1;
  __syncthreads();
  if (flag) {
    if (blockIdx.x == 0 && t == 0) set_err(a.err, SM_ERR_EINVAL);
    return;
  }
  auto sso_at = [&](int b) { return IN_LDS ? sso[b] : a.seq_span_offsets[b]; };
  auto so_at = [&](int b) { return IN_LDS ? so[b] : a.seq_offsets[b]; };
  const int q0 = so_at(last_le(so_at, a.B, c0));  // start of the sequence that holds c0
  int rem_q0 = 0, rem_c0 = 0, rem_all = 0, before_end = 0;  // (this thread's spans)
  constexpr int kPackBatch = 4;
  int b = last_le(sso_at, a.B, t);  // sequence b with sso[b] <= s < sso[b + 1]
  for (int s0 = t; s0 < a.num_spans; s0 += kPackBatch * kPackThreads) {
    int st[kPackBatch], ln[kPackBatch], pe[kPackBatch];
#pragma unroll
    for (int k = 0; k < kPackBatch; ++k) {
      const int s = s0 + k * kPackThreads;
      const bool in = s < a.num_spans;
      st[k] = in ? a.span_start[s] : 0;
      ln[k] = in ? a.span_len[s] : 1;
      pe[k] = (in && s > 0) ? a.span_start[s - 1] + a.span_len[s - 1] : 0;  // end of the previous span
    }
#pragma unroll
    for (int k = 0; k < kPackBatch; ++k) {
      const int s = s0 + k * kPackThreads;
      if (s >= a.num_spans) break;
      if (s >= sso_at(b + 1)) b = last_le(sso_at, a.B, s);
      bool ok = ln[k] >= 1 && st[k] >= so_at(b) && (int64_t)st[k] + ln[k] <= so_at(b + 1);
      if (ok && s > sso_at(b)) ok = st[k] >= pe[k];
      if (!ok) {
        bad = true;
        continue;
      }
      rem_all += ln[k] - 1;
      if (st[k] < q0) rem_q0 += ln[k] - 1;
      if (st[k] < c0) rem_c0 += min(ln[k] - 1, c0 - st[k]);
      const int end = st[k] + ln[k] - 1;  // its last token keeps the surrogate
      if (MANY) before_end += st[k] < c0 + cn;
      if (end >= c0 && st[k] < c0 + cn) {
        for (int u = max(st[k], c0); u < min(end, c0 + cn); ++u) src[u - c0] = kRemoved;
        if (end < c0 + cn) src[end - c0] = -1 - s;
      }
    }
  }
  if (bad) flag = 1;
  // the sums by a wave reduction and one LDS add per wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    rem_q0 += __shfl_xor(rem_q0, off, kWave);
    rem_c0 += __shfl_xor(rem_c0, off, kWave);
    rem_all += __shfl_xor(rem_all, off, kWave);
    if (MANY) before_end += __shfl_xor(before_end, off, kWave);
  }
  if ((t & 63) == 0) {
    atomicAdd(&sums[0], rem_q0);
    atomicAdd(&sums[1], rem_c0);
    atomicAdd(&sums[2], rem_all);
    if (MANY) atomicAdd(&sums[3], before_end);
  }
  __syncthreads();
  if (flag) {
    if (blockIdx.x == 0 && t == 0) set_err(a.err, SM_ERR_EINVAL);
    return;
  }
  int removed = sums[1], row_q0 = q0 - sums[0];  // positions removed before c0; the row of the token at q0
  int next_span = sums[3];                      // the first span that starts past the piece
  for (int piece = 1;; ++piece) {
    // packed rows of the piece's tokens: each thread owns PER consecutive ones
    int v[PER], cnt = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      v[u] = PER * t + u < cn ? src[PER * t + u] : kRemoved;
      cnt += v[u] != kRemoved;
    }
    int tot;
    int g = c0 - removed + block_inclusive_scan(cnt, red, &tot) - cnt;  // (its barriers: every src entry is read)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (PER * t + u < cn) {
        src[PER * t + u] = g;
        if (v[u] != kRemoved) a.packed_src[g++] = v[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = t + u * kPackThreads;
      if (e < cn) {
        const int first = so_at(last_le(so_at, a.B, c0 + e));  // its sequence's first token
        a.pi[c0 + e] = src[e] - (first >= c0 ? src[first - c0] : row_q0);
      }
    }
    const bool last = c0 + cn >= a.total_tokens;
    for (int b = t; b <= a.B; b += kPackThreads) {
      const int o = so_at(b);
      if (o >= c0 && o < c0 + cn) a.packed_offsets[b] = src[o - c0];
      else if (last && o == a.total_tokens) a.packed_offsets[b] = o - sums[2];
    }
    if (!MANY || last || piece == pieces) return;
    // The next piece: positions removed before it, the row of the first token
    // of the sequence that it begins in, and the spans in it (the list is
    // valid, so its starts ascend), from the one that may reach into it.
    removed += cn - tot;
    const int next0 = c0 + CHUNK, first = so_at(last_le(so_at, a.B, next0));
    if (first >= c0 && first < next0) row_q0 = src[first - c0];
    __syncthreads();  // src is read
    c0 = next0;
    cn = min(CHUNK, a.total_tokens - c0);
#pragma unroll
    for (int u = 0; u < PER; ++u) src[t + u * kPackThreads] = c0 + t + u * kPackThreads;
    __syncthreads();
    for (int s0 = max(next_span - 1, 0), got = kPackBatch * kPackThreads; got == kPackBatch * kPackThreads;
         s0 += kPackBatch * kPackThreads) {
      int mine = 0;
#pragma unroll
      for (int k = 0; k < kPackBatch; ++k) {
        const int s = s0 + t + k * kPackThreads;
        if (s >= a.num_spans) continue;
        const int st = a.span_start[s], end = st + a.span_len[s] - 1;
        mine += st < c0 + cn;
        if (end >= c0 && st < c0 + cn) {
          for (int u = max(st, c0); u < min(end, c0 + cn); ++u) src[u - c0] = kRemoved;
          if (end < c0 + cn) src[end - c0] = -1 - s;
        }
      }
      block_inclusive_scan(mine, red, &got);  // (its barriers: the marks are there)
      next_span = s0 + got;
    }
  }
}

// Copy phase of pack_spans: packed[r] = emb[token_ids[src]] (src >= 0) or
// surrogates[-1 - src], src = packed_src[r].  One wave per packed row, the
// waves striding over the rows; no barriers.  The next row's source index
// is loaded before the current row's data and its token id right after, so
// the two dependent index loads ride along the data round trip.
constexpr int kPackRowThreads = 256;
constexpr int kPackLaneGroups = 16;  // 16-byte groups per lane and pass (1024 per wave)

template <typename T>
__device__ __forceinline__ const T *pack_source(const PackArgs &a, int src, int tok) {
  if (src < 0) return (const T *)a.surrogates + (int64_t)(-1 - src) * a.d;
  if (tok < 0 || tok >= a.emb_rows) return nullptr;
  return (const T *)a.emb + (int64_t)tok * a.d;
}

template <typename T>
__global__ __launch_bounds__(kPackRowThreads) void pack_rows_kernel(PackArgs a) {
  const int lane = threadIdx.x & 63;
  const int nwaves = gridDim.x * (kPackRowThreads / 64);
  int r = blockIdx.x * (kPackRowThreads / 64) + (threadIdx.x >> 6);
  const int err0 = *a.err;
  const int nrows = a.packed_offsets[a.B];
  if (err0 != 0 || r >= nrows) return;
  constexpr int VEC = 16 / sizeof(T);
  const int vpr = a.d / VEC;
  int src = a.packed_src[r];
  const T *row = pack_source<T>(a, src, src >= 0 ? a.token_ids[src] : 0);
  for (; r < nrows; r += nwaves) {
    const int rn = r + nwaves;
    const int src_n = rn < nrows ? a.packed_src[rn] : -1;
    if (!row && lane == 0) set_err(a.err, SM_ERR_EINVAL);  // token id out of range: row skipped
    T *dst = (T *)a.packed + (int64_t)r * a.d;
    int tok_n = 0;
    for (int v0 = 0; v0 < vpr; v0 += 64 * kPackLaneGroups) {
      u32x4_t v[kPackLaneGroups];
#pragma unroll
      for (int u = 0; u < kPackLaneGroups; ++u) {
        const int idx = v0 + 64 * u + lane;
        if (row && idx < vpr) v[u] = *(const u32x4_t *)(row + (int64_t)idx * VEC);
      }
      if (v0 == 0 && rn < nrows && src_n >= 0) tok_n = a.token_ids[src_n];
#pragma unroll
      for (int u = 0; u < kPackLaneGroups; ++u) {
        const int idx = v0 + 64 * u + lane;
        // streaming stores: the packed rows are read back by the backbone's
        // prefill, not by this pass (measured 1.3x faster than plain stores)
        if (row && idx < vpr) __builtin_nontemporal_store(v[u], (u32x4_t *)(dst + (int64_t)idx * VEC));
      }
    }
    row = rn < nrows ? pack_source<T>(a, src_n, tok_n) : nullptr;
  }
}

}  // namespace sm

using namespace sm;

SM_API sm_status sm_kv_rollback(const sm_paged_cache *c, const int32_t *seq_ids, const int32_t *k, int n,
                                hipStream_t stream) {
  CacheArgs a;
  if (!cache_ok(c, a) || n < 0 || n > SM_MAX_REQUESTS || n > c->max_seqs) return SM_EINVAL;
  if (n == 0) return SM_OK;
  if (!seq_ids || !k) return SM_EINVAL;
  hipLaunchKernelGGL(rollback_kernel, dim3(1), dim3(kMetaThreads), 0, stream, a, seq_ids, k, n);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

// Resident copy workgroups over the whole device (looked up once per
// element type): the persistent grid of append_segments_kernel.
template <typename T>
static int seg_resident() {
  static const int nb = [] {
    int dev = 0, cus = 0, occ = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, append_segments_kernel<T>, kSegWgThreads, 0) !=
            hipSuccess ||
        occ <= 0)
      occ = 1;
    return cus * occ;
  }();
  return nb;
}

SM_API sm_status sm_kv_append(const sm_paged_cache *c, const int32_t *seq_ids, const int32_t *row_offsets,
                              int n, int total_rows, const void *K, const void *V, hipStream_t stream) {
  CacheArgs a;
  if (!cache_ok(c, a) || n < 0 || n > SM_MAX_REQUESTS || n > c->max_seqs || total_rows < 0)
    return SM_EINVAL;
  if (n == 0) return total_rows == 0 ? SM_OK : SM_EINVAL;
  if (!seq_ids || !row_offsets || (total_rows > 0 && (!K || !V))) return SM_EINVAL;
  const size_t es = c->dtype == SM_BF16 ? 2 : 4;
  if (c->num_kv_heads * c->head_dim > kMaxRowElems) return SM_EINVAL;
  const size_t tensor_bytes = (size_t)total_rows * c->num_kv_heads * c->head_dim * es;
  const FastDiv upr = make_fastdiv((uint32_t)(c->num_kv_heads * c->head_dim * es / 16));
  if (total_rows > 0 && total_rows <= kSmallRows && tensor_bytes <= (size_t)kSmallBytes) {
    if (c->dtype == SM_BF16)
      hipLaunchKernelGGL(append_small_kernel<uint16_t>, dim3(1), dim3(kMetaThreads), 0, stream, a, seq_ids,
                         row_offsets, n, total_rows, (const uint16_t *)K, (const uint16_t *)V, upr);
    else
      hipLaunchKernelGGL(append_small_kernel<float>, dim3(1), dim3(kMetaThreads), 0, stream, a, seq_ids,
                         row_offsets, n, total_rows, (const float *)K, (const float *)V, upr);
    return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
  }
  hipLaunchKernelGGL(append_meta_kernel, dim3(1), dim3(kMetaThreads), 0, stream, a, seq_ids, row_offsets, n,
                     total_rows);
  if (hipGetLastError() != hipSuccess) return SM_EHIP;
  if (total_rows == 0) return SM_OK;
  // segments touched: at most ceil(m / 16) + 1 per request
  const int64_t segs = (int64_t)(total_rows + kSegSlots - 1) / kSegSlots + 2 * (int64_t)n;
  const int64_t wgs = (segs + kSegPerWg - 1) / kSegPerWg;
  const int resident = c->dtype == SM_BF16 ? seg_resident<uint16_t>() : seg_resident<float>();
  const dim3 grid((unsigned)(wgs < resident ? wgs : resident));
  if (c->dtype == SM_BF16)
    hipLaunchKernelGGL(append_segments_kernel<uint16_t>, grid, dim3(kSegWgThreads), 0, stream, a, seq_ids,
                       row_offsets, n, (const uint16_t *)K, (const uint16_t *)V);
  else
    hipLaunchKernelGGL(append_segments_kernel<float>, grid, dim3(kSegWgThreads), 0, stream, a, seq_ids,
                       row_offsets, n, (const float *)K, (const float *)V);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

SM_API sm_status sm_pack_spans(int B, const int32_t *seq_offsets, int total_tokens, int num_spans,
                               const int32_t *span_start, const int32_t *span_len,
                               const int32_t *seq_span_offsets, int32_t *pi, int32_t *packed_offsets,
                               int32_t *packed_src, const int32_t *token_ids, const void *emb,
                               int64_t emb_rows, const void *surrogates, int d, sm_dtype dt, void *packed,
                               int32_t *err, hipStream_t stream) {
  if (B < 0 || total_tokens < 0 || num_spans < 0 || B > 65535) return SM_EINVAL;
  if (B == 0) return SM_OK;
  if (!seq_offsets || !seq_span_offsets || !packed_offsets || !err) return SM_EINVAL;
  if (total_tokens > 0 && (!pi || !packed_src)) return SM_EINVAL;
  if (num_spans > 0 && (!span_start || !span_len)) return SM_EINVAL;
  if (packed) {
    if (dt != SM_F32 && dt != SM_BF16) return SM_EINVAL;
    if (!token_ids || !emb || (num_spans > 0 && !surrogates) || d <= 0 || d % 8 || emb_rows <= 0)
      return SM_EINVAL;
  }
  PackArgs a;
  a.B = B;
  a.total_tokens = total_tokens;
  a.num_spans = num_spans;
  a.seq_offsets = seq_offsets;
  a.span_start = span_start;
  a.span_len = span_len;
  a.seq_span_offsets = seq_span_offsets;
  a.pi = pi;
  a.packed_offsets = packed_offsets;
  a.packed_src = packed_src;
  a.token_ids = token_ids;
  a.emb = emb;
  a.emb_rows = emb_rows;
  a.surrogates = surrogates;
  a.d = d;
  a.packed = packed;
  a.err = err;
  const int64_t n1 = ((int64_t)total_tokens + kPackThreads - 1) / kPackThreads;  // pieces of PER = 1
  const int64_t n4 = (n1 + kPackMaxPer - 1) / kPackMaxPer;
  const int many = (int)((n4 + kPackWgs - 1) / kPackWgs);
  const bool in_lds = B + 1 <= kPackSsoLds;
  const int64_t grid = n1 <= kPackWgs ? (n1 > 0 ? n1 : 1) : (n4 + many - 1) / many;
  const auto index = n1 <= kPackWgs ? (in_lds ? pack_index_kernel<1, false, true> : pack_index_kernel<1, false, false>)
                     : many <= 1    ? (in_lds ? pack_index_kernel<kPackMaxPer, false, true>
                                              : pack_index_kernel<kPackMaxPer, false, false>)
                                    : (in_lds ? pack_index_kernel<kPackMaxPer, true, true>
                                              : pack_index_kernel<kPackMaxPer, true, false>);
  hipLaunchKernelGGL(index, dim3((unsigned)grid), dim3(kPackThreads), 0, stream, a, many);
  if (hipGetLastError() != hipSuccess) return SM_EHIP;
  if (packed && total_tokens > 0) {
    // one wave per packed row, striding: up to 4 waves per compute unit's
    // worth of workgroups (the packed rows are at most total_tokens)
    const int64_t wgs = ((int64_t)total_tokens + 3) / 4;
    const dim3 grid((unsigned)(wgs < 2048 ? wgs : 2048));
    if (dt == SM_BF16)
      hipLaunchKernelGGL(pack_rows_kernel<uint16_t>, grid, dim3(kPackRowThreads), 0, stream, a);
    else
      hipLaunchKernelGGL(pack_rows_kernel<float>, grid, dim3(kPackRowThreads), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return SM_EHIP;
  }
  return SM_OK;
}

// Paged-cache descriptor and the metadata steps that more than one source
// uses (gfx950).
#pragma once

#include "common.hpp"

namespace sm {

struct CacheArgs {
  void *k_pool;
  void *v_pool;
  int32_t *block_table;
  int32_t *lengths;
  int32_t *free_stack;
  int32_t *free_top;
  int32_t *err;
  int Hkv, DH, dh_log2, bs_log2, num_blocks, max_seqs, max_blocks;
};

constexpr int kMetaThreads = 1024;

__device__ __forceinline__ int blocks_for(int len, int bs_log2) {
  return (len + (1 << bs_log2) - 1) >> bs_log2;
}

// Distinct, in-range sequence ids; thread t checks request t against all
// earlier requests.
// request t's sequence id is in range and no earlier request of the call
// names it (ids: the call's ids, staged in LDS; no early exit, so the
// reads issue back to back)
__device__ __forceinline__ bool id_ok(const int *ids, int t, int s, int max_seqs) {
  bool dup = false;
  for (int j = 0; j < t; ++j) dup |= ids[j] == s;
  return s >= 0 && s < max_seqs && !dup;
}

// What kv_rollback reads of the cache's state, requested as soon as the ids
// are there: the error word, the top of the free stack and the length of
// this thread's sequence (its id may be out of range: checked before use).
struct RollbackReads {
  int err, top, len;
};

__device__ __forceinline__ RollbackReads rollback_reads(const CacheArgs &c, int s) {
  return RollbackReads{*c.err, *c.free_top, s >= 0 && s < c.max_seqs ? c.lengths[s] : 0};
}

// kv_rollback by one workgroup of kMetaThreads threads, thread t with request
// t's sequence s and count k (t < n).  Returns with all of it applied or, an
// error bit set, nothing.
__device__ __forceinline__ void rollback_body(const CacheArgs &c, const RollbackReads &rd, int s, int k, int n) {
  __shared__ int red[16];
  __shared__ int fl_inval, fl_range, fl_many;
  __shared__ int ids[kMetaThreads];
  const int t = threadIdx.x;
  if (rd.err != 0) return;  // sticky: the cache is frozen until the caller clears err
  const bool active = t < n;
  if (t == 0) {
    fl_inval = 0;
    fl_range = 0;
    fl_many = 0;
  }
  if (active) ids[t] = s;
  __syncthreads();
  if (active && (k < 0 || !id_ok(ids, t, s, c.max_seqs))) fl_inval = 1;
  __syncthreads();
  if (fl_inval) {
    if (t == 0) set_err(c.err, SM_ERR_EINVAL);
    return;
  }
  const int cap = c.max_blocks << c.bs_log2;
  int L = 0, freed = 0;
  if (active) {
    L = rd.len;
    if (L < 0 || L > cap || k > L) fl_range = 1;
    else freed = blocks_for(L, c.bs_log2) - blocks_for(L - k, c.bs_log2);
    // up to two blocks a request (a decode step's crop) the search costs more than it saves
    if (freed > 2) fl_many = 1;
  }
  __syncthreads();
  if (fl_range) {
    if (t == 0) set_err(c.err, SM_ERR_ERANGE);
    return;
  }
  int total;
  const int incl = block_inclusive_scan(freed, red, &total);
  const int top = rd.top;
  if (top < 0 || (int64_t)top + total > c.num_blocks) {  // stack cannot take the blocks
    if (t == 0) set_err(c.err, SM_ERR_ERANGE);
    return;
  }
  // Requests are served in reverse order: request t's first push lands above
  // the blocks of every later request, its highest logical block first.
  if (fl_many) {
    // The freed blocks of all requests as one list, a thread per block: a
    // thread alone with its request's blocks waits out a table read per block
    // (16 requests of 154 blocks: 32.6 us; as one list 6.6 us).
    __shared__ int ends[kMetaThreads], lens[kMetaThreads];
    ends[t] = incl;  // threads past n repeat the total
    lens[t] = L;
    __syncthreads();
    for (int e = t; e < total; e += kMetaThreads) {
      int r = 0;  // the first request whose blocks end past e
#pragma unroll
      for (int step = kMetaThreads / 2; step > 0; step >>= 1) r += ends[r + step - 1] <= e ? step : 0;
      int32_t *cell = c.block_table + (int64_t)ids[r] * c.max_blocks + blocks_for(lens[r], c.bs_log2) -
                      1 - (e - (r > 0 ? ends[r - 1] : 0));
      c.free_stack[top + total - ends[r] + (e - (r > 0 ? ends[r - 1] : 0))] = *cell;
      *cell = -1;
    }
  } else if (active) {
    int pos = top + (total - incl);
    int32_t *row = c.block_table + (int64_t)s * c.max_blocks;
    const int nb_old = blocks_for(L, c.bs_log2);
    for (int j = nb_old - 1; j >= nb_old - freed; --j) {
      c.free_stack[pos++] = row[j];
      row[j] = -1;
    }
  }
  if (active) c.lengths[s] = L - k;
  if (t == 0) *c.free_top = top + total;
}

}  // namespace sm

static inline int ilog2_pow2(int v) {
  if (v <= 0 || (v & (v - 1))) return -1;
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

static inline bool cache_ok(const sm_paged_cache *c, sm::CacheArgs &a) {
  if (!c) return false;
  if (c->dtype != SM_F32 && c->dtype != SM_BF16) return false;
  if (c->head_dim != 64 && c->head_dim != 128) return false;
  const int l = ilog2_pow2(c->block_size);
  if (l < 4 || l > 9) return false;
  if (c->num_kv_heads <= 0 || c->num_blocks <= 0 || c->max_seqs <= 0 || c->max_blocks_per_seq <= 0)
    return false;
  if ((int64_t)c->max_blocks_per_seq * c->block_size > INT32_MAX / 2) return false;
  if (!c->k_pool || !c->v_pool || !c->block_table || !c->lengths || !c->free_stack || !c->free_top ||
      !c->err)
    return false;
  a.k_pool = c->k_pool;
  a.v_pool = c->v_pool;
  a.block_table = c->block_table;
  a.lengths = c->lengths;
  a.free_stack = c->free_stack;
  a.free_top = c->free_top;
  a.err = c->err;
  a.Hkv = c->num_kv_heads;
  a.DH = c->head_dim;
  a.dh_log2 = c->head_dim == 128 ? 7 : 6;
  a.bs_log2 = l;
  a.num_blocks = c->num_blocks;
  a.max_seqs = c->max_seqs;
  a.max_blocks = c->max_blocks_per_seq;
  return true;
}

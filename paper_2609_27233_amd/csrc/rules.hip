// Merge-rule matching on the GPU (gfx950).
//
// The rule set R (appendix "Non-overlapping Assignment in a Sequence": the
// 2- to 4-grams kept after the frequency filter, about 2.17M for the
// Llama-3 tokenizer) lives in an open-addressing hash table in HBM.  Each
// slot holds one rule as four int32 token ids (tail -1) and its index in
// the rule list; linear probing, load at most 3/4.
//
//  * Build: one thread per rule claims a slot with a 64-bit compare-and-swap
//    of (fingerprint, rule index + 1).  A thread that meets its own key
//    (same fingerprint, equal tokens read from the immutable rule list)
//    keeps the smaller index with a 64-bit atomic min, so a rule listed
//    twice resolves to its first index.  A second pass copies the keys into
//    the slots.  No thread ever waits on another.
//  * Prompt matching ("Rule Matching": left to right, 4-, 3-, then 2-grams,
//    take the longest match and jump past it, else step one token).  The
//    greedy chain is a composition of maps: a stretch of positions maps the
//    chain's entry offset (0..3 past its start) to its exit offset, and to
//    the number of spans taken on the way.  No window crosses a sequence's
//    end, so the chain lands on every sequence start by itself and the whole
//    batch is one chain, cut into blocks of 256 positions whatever the
//    sequences' lengths:
//      1. every position looks up its longest rule (independent lookups) and
//         every block folds its maps into one;
//      2. every block folds the maps of the blocks before it (its true entry
//         and the spans before it; one scan gives them to all in a large
//         batch) and emits its spans at their final place, and the CSR offset
//         of every sequence that starts in it.
//    The result is exactly the sequential scan's.
//  * Decode matching ("Decoding-time Integration"): per sequence a 16-byte
//    state (number of raw tokens since the last merge, capped at 3, and
//    those tokens) is enough for suffixes of at most 4.  The new token
//    completes the longest rule suffix (4, 3, 2 in turn) or joins the raw
//    tail.  On a match, n - 1 cached entries are to be cropped; the call can
//    run the cache rollback right after.
#include "cache_meta.hpp"

typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

namespace sm {

// MurmurHash3's 64-bit finalizer (Appleby, MurmurHash3, public domain).
__device__ __forceinline__ uint64_t fmix64(uint64_t k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  return k;
}

__device__ __forceinline__ uint64_t rule_hash(i32x4_t k) {
  const uint64_t lo = (uint64_t)(uint32_t)k.x | ((uint64_t)(uint32_t)k.y << 32);
  const uint64_t hi = (uint64_t)(uint32_t)k.z | ((uint64_t)(uint32_t)k.w << 32);
  return fmix64(lo ^ fmix64(hi + 0x9e3779b97f4a7c15ull));
}

__device__ __forceinline__ bool key_eq(i32x4_t a, i32x4_t b) {
  return a.x == b.x && a.y == b.y && a.z == b.z && a.w == b.w;
}

// n of a well-formed rule (n >= 2 leading ids >= 0, then -1), else 0
__device__ __forceinline__ int key_len(i32x4_t k) {
  const int n = k.x < 0 ? 0 : k.y < 0 ? 1 : k.z < 0 ? 2 : k.w < 0 ? 3 : 4;
  const bool tail = (n > 0 || k.x == -1) && (n > 1 || k.y == -1) && (n > 2 || k.z == -1) && (n > 3 || k.w == -1);
  return tail && n >= 2 ? n : 0;
}

// the rule id of key k, or -1; the probe ends at the first empty slot
__device__ __forceinline__ int rule_find(const i32x4_t *keys, const int32_t *ids, uint32_t mask, i32x4_t k) {
  const uint64_t h = rule_hash(k);
  for (uint32_t p = 0; p <= mask; ++p) {
    const uint32_t s = (uint32_t)(h + p) & mask;
    const i32x4_t e = keys[s];
    if (e.x == -1) return -1;
    if (key_eq(e, k)) return ids[s];
  }
  return -1;
}

// The longest of up to three candidate keys (cand[0] the longest) that is a
// rule: the three probe chains advance together, kProbe slots of each at a
// time, so their memory latencies overlap instead of adding up (a wave waits
// for the longest of its 192 chains; the slots of a round mostly share a
// 128-byte line).  want[c] = false skips a candidate.  Returns the index of
// the winning candidate (or -1) and its rule id in *id.
constexpr int kProbe = 4;

__device__ __forceinline__ int rule_find_longest(const i32x4_t *keys, const int32_t *ids, uint32_t mask,
                                                 const i32x4_t (&cand)[3], const bool (&want)[3], int *id) {
  uint32_t slot[3];
  int state[3];  // -2 probing, -1 absent, else the slot that holds it
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    slot[c] = (uint32_t)rule_hash(cand[c]) & mask;
    state[c] = want[c] ? -2 : -1;
  }
  for (uint32_t p = 0; p <= mask; p += kProbe) {  // (the capacity is a multiple of kProbe)
    i32x4_t e[3][kProbe];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (state[c] == -2)
#pragma unroll
        for (int k = 0; k < kProbe; ++k) e[c][k] = keys[(slot[c] + k) & mask];
    bool busy = false;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (state[c] != -2) continue;
#pragma unroll
      for (int k = 0; k < kProbe; ++k) {
        if (state[c] != -2) continue;
        if (e[c][k].x == -1) state[c] = -1;
        else if (key_eq(e[c][k], cand[c])) state[c] = (int)((slot[c] + k) & mask);
      }
      slot[c] = (slot[c] + kProbe) & mask;
      busy |= state[c] == -2;
    }
    if (!busy) break;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (state[c] >= 0) {
      *id = ids[state[c]];
      return c;
    }
  *id = -1;
  return -1;
}

// ---- build ----------------------------------------------------------------

__global__ void rules_clear_kernel(uint64_t *claim, int cap) {
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < cap; s += gridDim.x * blockDim.x) claim[s] = 0;
}

__global__ void rules_claim_kernel(const i32x4_t *rules, int count, uint64_t *claim, uint32_t mask,
                                   int32_t *err) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= count) return;
  const i32x4_t k = rules[r];
  if (!key_len(k)) {
    set_err(err, SM_ERR_EINVAL);
    return;
  }
  const uint64_t h = rule_hash(k);
  const uint64_t fp = (h >> 32) | 1ull;  // non-zero: an empty slot reads 0
  const uint64_t word = (fp << 32) | (uint32_t)(r + 1);
  for (uint32_t p = 0; p <= mask; ++p) {
    const uint32_t s = (uint32_t)(h + p) & mask;
    const uint64_t old = atomicCAS((unsigned long long *)&claim[s], 0ull, (unsigned long long)word);
    if (old == 0) return;  // claimed
    if ((old >> 32) == fp && key_eq(rules[(uint32_t)old - 1], k)) {
      atomicMin((unsigned long long *)&claim[s], (unsigned long long)word);  // same key: smallest index
      return;
    }
  }
  set_err(err, SM_ERR_ERANGE);  // no free slot (the host keeps the load at most 3/4)
}

__global__ void rules_fill_kernel(const i32x4_t *rules, const uint64_t *claim, int cap, i32x4_t *keys,
                                  int32_t *ids) {
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < cap; s += gridDim.x * blockDim.x) {
    const uint64_t w = claim[s];
    if (w == 0) {
      keys[s] = i32x4_t{-1, -1, -1, -1};
      ids[s] = -1;
    } else {
      const int id = (int)(uint32_t)w - 1;
      keys[s] = rules[id];
      ids[s] = id;
    }
  }
}

__global__ void rules_lookup_kernel(const i32x4_t *keys, const int32_t *ids, uint32_t mask, const i32x4_t *grams,
                                    int m, int32_t *out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const i32x4_t k = grams[i];
  out[i] = key_len(k) ? rule_find(keys, ids, mask, k) : -1;
}

// ---- prompt matching --------------------------------------------------------

constexpr int kMatchBlock = 256;                  // positions per block, folded by one wave
constexpr int kMatchLane = kMatchBlock / 64;      // positions per lane of that wave
// The lookups want many compute units: each lane's probe is a line of its own,
// one lane per cycle and unit, so workgroups of 256.  The emit pass takes four
// of their blocks per workgroup: each workgroup reads all sequence offsets and
// its share of the folds before it.  Call in us with one, two, four and eight
// blocks: 1 x 4096 tokens 11.8, 12.3, 12.4, 13.1; 16 x 32,768 30.7, 30.5,
// 28.2, 28.0; 60,000 x 16 257, 160, 99, 75.
constexpr int kEmitBlocks = 4;
constexpr int kEmitThreads = 64 * kEmitBlocks;
constexpr int kShareRead = 4;                     // folds a thread of the emit pass reads at a time
// Emit workgroups up to which each forms its own entry from the folds before
// it (524,288 positions).  That is one launch less but work that grows with
// the square of the batch: 128 x 32,768 tokens, 50,000 rules: 194 us a call,
// 153 with the scan (17 of them); 256 x 32,768: 547 and 293.
constexpr int kScanEmit = 512;
constexpr int kMatchLds = 2048;                   // sequence offsets held in LDS
constexpr uint32_t kMapIdentity = 0x03020100u;    // e -> e, a byte per entry

// What a stretch of at most 256 positions does to the chain, a byte per entry
// offset e: it leaves at offset map_e past the stretch's end, after cnt_e
// spans (at most 128: a span takes two positions).
struct ChainFold {
  uint32_t map, cnt;
};

__device__ __forceinline__ uint32_t byte_at(uint32_t v, uint32_t e) { return (v >> (8 * e)) & 255u; }
// byte e of the result is v's byte f_e: one v_perm_b32, whose selectors 0 to
// 3 pick from its second operand.  With v a map this is f, then v; with v
// counts it is what a stretch entered through f counts.  (With two bits per
// entry, shifts, and a sum per entry the lookup pass of 16 x 4096 tokens over
// 50,000 rules took 22 us instead of 11, the emit pass 10 instead of 4.4.)
__device__ __forceinline__ uint32_t through(uint32_t f, uint32_t v) { return __builtin_amdgcn_perm(v, v, f); }

// the fold of a lane's kMatchLane positions, match lengths (0 = none) in
// 4-bit fields of L: from the last position back
__device__ __forceinline__ ChainFold lane_fold(uint32_t L) {
  ChainFold f{0u, 0u};
#pragma unroll
  for (int p = kMatchLane - 1; p >= 0; --p) {
    const uint32_t len = (L >> (4 * p)) & 15u, next = p + max(len, 1u);
    const bool out = next >= (uint32_t)kMatchLane;  // past the lane's positions: offset at most 3
    f.map |= (out ? next - kMatchLane : byte_at(f.map, next)) << (8 * p);
    f.cnt |= ((len ? 1u : 0u) + (out ? 0u : byte_at(f.cnt, next))) << (8 * p);
  }
  return f;
}

// Inclusive scan of the lanes' maps.  Only the maps are scanned: with a
// lane's entry known, the spans before it are an ordinary prefix sum.
__device__ __forceinline__ uint32_t wave_map_scan(uint32_t f) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t g = __shfl_up(f, off, kWave);
    if (lane >= off) f = through(g, f);
  }
  return f;
}
// the map before lane l, from the inclusive scan
__device__ __forceinline__ uint32_t map_before(uint32_t incl) {
  const uint32_t g = __shfl_up(incl, 1, kWave);
  return (threadIdx.x & 63) ? g : kMapIdentity;
}

// match lengths of the four positions of a lane, bytes -> 4-bit fields
__device__ __forceinline__ uint32_t pack_lens(uint32_t v) {
  return (v & 15u) | ((v >> 4) & 0xf0u) | ((v >> 8) & 0xf00u) | ((v >> 12) & 0xf000u);
}

// 1. longest rule starting at every position (0 = none) and its id; the
// block's fold.  Positions before the first sequence have theirs in the high
// four bits, which only match_bad_offsets reads.  IN_LDS: the sequence offsets fit kMatchLds (decided by the
// host: a pointer to one or the other would make every read a flat one).
template <bool IN_LDS>
__global__ __launch_bounds__(kMatchBlock) void match_len_kernel(const i32x4_t *keys, const int32_t *ids, uint32_t mask,
                                                                const int32_t *tokens, const int32_t *seq_offsets,
                                                                int B, int total, int8_t *mlen, int32_t *rid,
                                                                ChainFold *folds) {
  __shared__ int so[IN_LDS ? kMatchLds : 1];
  __shared__ uint32_t lens[kMatchBlock / 4];
  const int tid = threadIdx.x, t = blockIdx.x * kMatchBlock + tid;
  int x[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = t + j < total ? tokens[t + j] : -1;
  if constexpr (IN_LDS) {
    for (int b = tid; b <= B; b += kMatchBlock) so[b] = seq_offsets[b];
    __syncthreads();
  }
  auto off = [&](int b) { return IN_LDS ? so[b] : seq_offsets[b]; };
  // the sequence holding t: the last b with seq_offsets[b] <= t
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off(mid) <= t) lo = mid;
    else hi = mid - 1;
  }
  const int end = min(off(lo + 1), total);
  // before the first sequence: no part of the chain (a sequence may hold the
  // position all the same if the offsets are out of order)
  const bool gap = t < off(0) && lo == 0 && off(0) <= off(1) && off(1) <= total;
  i32x4_t cand[3];
  bool want[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {  // candidate c: the (4 - c)-gram at t
    const int n = 4 - c;
    bool ok = t + n <= end;
#pragma unroll
    for (int j = 0; j < 4; ++j) ok = ok && (j >= n || x[j] >= 0);
    want[c] = ok;
    cand[c] = i32x4_t{x[0], x[1], n > 2 ? x[2] : -1, n > 3 ? x[3] : -1};
  }
  int id;
  const int c = rule_find_longest(keys, ids, mask, cand, want, &id);
  const int len = c >= 0 ? 4 - c : 0;
  if (t < total) {
    mlen[t] = (int8_t)(gap ? len << 4 : len);
    rid[t] = id;
  }
  ((uint8_t *)lens)[tid] = (uint8_t)(gap ? 0 : len);
  __syncthreads();
  if (tid < 64) {
    const ChainFold f = lane_fold(pack_lens(lens[tid]));
    const uint32_t incl = wave_map_scan(f.map);
    uint32_t c = through(map_before(incl), f.cnt);  // this lane's spans, by the block's entry
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) c += __shfl_xor(c, o, kWave);  // (no byte passes 128)
    if (tid == 63) folds[blockIdx.x] = ChainFold{incl, c};
  }
}

// Inclusive scan over the workgroup of sums that stop at cap (at most 2^30 - 1,
// so that no addition overflows).
__device__ __forceinline__ int capped_scan(int v, int cap, int *red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = min(v, cap);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(v, off, kWave);
    if (lane >= off) v = min(v + u, cap);
  }
  __syncthreads();
  if (lane == 63) red[w] = v;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < w; ++k) before = min(before + red[k], cap);
  return min(before + v, cap);
}

// Offsets out of order or range (an error path: such a batch is not one
// chain): their sequences get no spans, the others theirs.  Every workgroup
// counts the spans of all sequences, a thread per sequence, whole blocks
// through their folds; so each knows the places of those it writes, every
// gridDim.x-th.  Overlapping sequences may hold more spans than the outputs
// (total / 2): those past the end are dropped.
__device__ void match_bad_offsets(const int8_t *mlen, const int32_t *rid, const ChainFold *folds,
                                  const int32_t *seq_offsets, int B, int total, int32_t *span_start, int32_t *span_len,
                                  int32_t *span_rule, int32_t *seq_span_offsets, int32_t *err) {
  __shared__ uint32_t wmap[kEmitBlocks];
  __shared__ int red[16], sums[kEmitThreads];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int cap = total / 2, grid = (int)gridDim.x;
  const int first = seq_offsets[0], second = seq_offsets[1];
  const int gap = first >= 0 && first <= second && second <= total ? first : 0;  // the folds leave out what is before it
  auto len_of = [&](int p) { return (mlen[p] & 15) | (mlen[p] >> 4); };
  int base = 0;
  for (int b0 = 0; b0 < B; b0 += kEmitThreads) {
    const int b = b0 + tid;
    int lo = 0, hi = 0;
    if (b < B) {
      lo = seq_offsets[b];
      hi = seq_offsets[b + 1];
      if (!(lo >= 0 && lo <= hi && hi <= total)) {
        if (blockIdx.x == 0) set_err(err, SM_ERR_EINVAL);
        lo = hi = 0;
      }
    }
    int n = 0;
    for (int p = lo; p < hi;) {
      const uint32_t e = p & (kMatchBlock - 1);
      if (e < 4 && (p | (kMatchBlock - 1)) < hi && (p & -kMatchBlock) >= gap) {  // the block to its end, entered at e
        const ChainFold f = folds[p / kMatchBlock];
        n += (int)byte_at(f.cnt, e);
        p = (p | (kMatchBlock - 1)) + 1 + (int)byte_at(f.map, e);
      } else {
        const int len = len_of(p);
        n += len ? 1 : 0;
        p += max(len, 1);
      }
    }
    const int end = min(base + capped_scan(n, cap, red), cap);
    sums[tid] = end;
    if (blockIdx.x == 0 && b < B) seq_span_offsets[b + 1] = end;
    __syncthreads();
    for (int s = b0 + (((int)blockIdx.x - b0) % grid + grid) % grid; s < min(b0 + kEmitThreads, B); s += grid) {
      const int slo = seq_offsets[s], shi = seq_offsets[s + 1];
      if (!(slo >= 0 && slo <= shi && shi <= total)) continue;
      int o = s > b0 ? sums[s - b0 - 1] : base;
      uint32_t entry = 0;
      for (int q = slo; q < shi; q += kMatchLane * kEmitThreads) {
        const int t0 = q + kMatchLane * tid;
        uint32_t L = 0;
#pragma unroll
        for (int j = 0; j < kMatchLane; ++j)
          if (t0 + j < shi) L |= (uint32_t)len_of(t0 + j) << (4 * j);
        const ChainFold f = lane_fold(L);
        const uint32_t incl = wave_map_scan(f.map);
        if (lane == 63) wmap[w] = incl;
        __syncthreads();
        uint32_t e = entry;
#pragma unroll
        for (int k = 0; k < kEmitBlocks; ++k) {
          if (k < w) e = byte_at(wmap[k], e);
          entry = byte_at(wmap[k], entry);
        }
        e = byte_at(map_before(incl), e);
        const int mine = (int)byte_at(f.cnt, e);
        int all;
        int at = o + block_inclusive_scan(mine, red, &all) - mine;  // (its barriers: wmap is read)
#pragma unroll
        for (int p = 0; p < kMatchLane; ++p)
          if (e == (uint32_t)p) {
            const uint32_t len = (L >> (4 * p)) & 15u;
            if (len) {
              if (at < cap) {
                span_start[at] = t0 + p;
                span_len[at] = (int)len;
                span_rule[at] = rid[t0 + p];
              }
              ++at;
            }
            e += max(len, 1u);
          }
        o += all;
      }
    }
    base = sums[kEmitThreads - 1];
    __syncthreads();
  }
  if (blockIdx.x == 0 && tid == 0) seq_span_offsets[0] = 0;
}

// Where the chain enters an emit workgroup's positions (offset past their
// first) and the spans taken before.
struct ChainEntry {
  uint32_t entry;
  int spans;
};

// 1b. those of all emit workgroups by one workgroup, a contiguous share per
// thread: the shares' maps and their scan give every share's entry, walking
// the share from there its spans, and walking it again every place in it
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void match_scan_kernel(const ChainFold *folds, int nwg, ChainEntry *at) {
  __shared__ uint32_t wmap[kScanThreads / 64];
  __shared__ int red[16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int per = (nwg + kScanThreads - 1) / kScanThreads, g0 = min(tid * per, nwg), g1 = min(g0 + per, nwg);
  uint32_t map = kMapIdentity;
#pragma unroll 4
  for (int k = kEmitBlocks * g0; k < kEmitBlocks * g1; ++k) map = through(map, folds[k].map);
  const uint32_t incl = wave_map_scan(map);
  if (lane == 63) wmap[w] = incl;
  __syncthreads();
  uint32_t entry = 0;
  for (int k = 0; k < w; ++k) entry = byte_at(wmap[k], entry);
  entry = byte_at(map_before(incl), entry);
  int spans = 0;
  uint32_t e = entry;
#pragma unroll 4
  for (int k = kEmitBlocks * g0; k < kEmitBlocks * g1; ++k) {
    spans += (int)byte_at(folds[k].cnt, e);
    e = byte_at(folds[k].map, e);
  }
  int total;
  int before = block_inclusive_scan(spans, red, &total) - spans;
  for (int g = g0; g < g1; ++g) {
    at[g] = ChainEntry{entry, before};
#pragma unroll
    for (int k = 0; k < kEmitBlocks; ++k) {
      const ChainFold f = folds[kEmitBlocks * g + k];
      before += (int)byte_at(f.cnt, entry);
      entry = byte_at(f.map, entry);
    }
  }
}

// 2. the spans of a workgroup's blocks (one per wave) at their final place,
// and the CSR offsets of the sequences that start in them.  SCANNED: `at` is
// there.
template <bool IN_LDS, bool SCANNED>
__global__ __launch_bounds__(kEmitThreads) void match_emit_kernel(const int8_t *mlen, const int32_t *rid,
                                                                  const ChainFold *folds, const ChainEntry *at,
                                                                  const int32_t *seq_offsets,
                                                                  int B, int total, int nwg, int32_t *span_start,
                                                                  int32_t *span_len, int32_t *span_rule,
                                                                  int32_t *seq_span_offsets, int32_t *err) {
  __shared__ uint32_t wmap[kEmitBlocks];
  __shared__ int wsum[kEmitBlocks], spans_end;
  __shared__ int so[IN_LDS ? kMatchLds : 1];
  __shared__ int lane_entry[kEmitThreads], lane_before[kEmitThreads];
  __shared__ uint32_t lane_len[kEmitThreads];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int blk0 = blockIdx.x * kEmitBlocks;  // this workgroup's first block
  const int c0 = blk0 * kMatchBlock, c1 = min(c0 + kEmitBlocks * kMatchBlock, total);
  const bool last = (int)blockIdx.x == nwg - 1;
  if (B == 0) {
    if (tid == 0) seq_span_offsets[0] = 0;
    return;
  }
  // Four positions' match lengths and ids per lane, the folds of its own
  // blocks, and the offsets: all requested before any is used (lanes past the
  // batch's end read its last four and mask them)
  const int t0 = c0 + kMatchLane * tid;
  const int tc = min(t0, max(total - 1, 0) & ~(kMatchLane - 1));
  const uint32_t lens4 = *(const uint32_t *)(mlen + tc);
  const i32x4_t id4 = *(const i32x4_t *)(rid + tc);
  const int per = SCANNED ? 0 : (blk0 + kEmitThreads - 1) / kEmitThreads;  // blocks before, a contiguous share per thread
  ChainEntry mine_at = {0u, 0};
  if constexpr (SCANNED) mine_at = at[blockIdx.x];
  ChainFold own[kEmitBlocks];
#pragma unroll
  for (int k = 0; k < kEmitBlocks; ++k) own[k] = folds[blk0 + k];
  int o_lo = seq_offsets[min(tid, B)], o_hi = seq_offsets[min(tid + 1, B)];
  uint32_t map = kMapIdentity;  // of this thread's share
  int cnt0 = 0, cnt1 = 0, cnt2 = 0, cnt3 = 0;
  const int share_end = min((tid + 1) * per, blk0);
  for (int k = tid * per; k < share_end; k += kShareRead) {
    ChainFold fold[kShareRead];
#pragma unroll
    for (int j = 0; j < kShareRead; ++j) fold[j] = folds[min(k + j, blk0)];
#pragma unroll
    for (int j = 0; j < kShareRead; ++j)
      if (k + j < share_end) {
        const uint32_t c = through(map, fold[j].cnt);
        cnt0 += byte_at(c, 0);
        cnt1 += byte_at(c, 1);
        cnt2 += byte_at(c, 2);
        cnt3 += byte_at(c, 3);
        map = through(map, fold[j].map);
      }
  }
  // offsets in order and range?
  bool bad = false;
  for (int b = tid; b <= B; b += kEmitThreads) {
    if (b > tid) {
      o_lo = seq_offsets[b];
      o_hi = seq_offsets[min(b + 1, B)];
    }
    if constexpr (IN_LDS) so[b] = o_lo;
    if (b < B) bad |= !(o_lo >= 0 && o_lo <= o_hi && o_hi <= total);
  }
  const uint32_t incl = wave_map_scan(map);
  if (lane == 63) wmap[w] = incl;
  if (__syncthreads_or(bad)) {
    match_bad_offsets(mlen, rid, folds, seq_offsets, B, total, span_start, span_len, span_rule, seq_span_offsets, err);
    return;
  }
  // the chain enters the batch at offset 0: the entry of this thread's
  // share, and the spans of all shares
  uint32_t entry = 0;
  for (int k = 0; k < w; ++k) entry = byte_at(wmap[k], entry);
  const uint32_t se = byte_at(map_before(incl), entry);
  int c = se < 2 ? (se == 0 ? cnt0 : cnt1) : (se == 2 ? cnt2 : cnt3);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) c += __shfl_xor(c, off, kWave);
  if (lane == 0) wsum[w] = c;
  __syncthreads();
  int before = mine_at.spans;  // spans before, and entry of, this wave's block
  entry = mine_at.entry;
  if constexpr (!SCANNED)
#pragma unroll
    for (int k = 0; k < kEmitBlocks; ++k) {
      before += wsum[k];
      entry = byte_at(wmap[k], entry);
    }
#pragma unroll
  for (int k = 0; k < kEmitBlocks; ++k)
    if (k < w && total > 0) {  // (no tokens: no folds were written)
      before += byte_at(own[k].cnt, entry);
      entry = byte_at(own[k].map, entry);
    }
  uint32_t L = pack_lens(lens4);
#pragma unroll
  for (int j = 0; j < kMatchLane; ++j)
    if (t0 + j >= total) L &= ~(15u << (4 * j));
  const ChainFold x = lane_fold(L);
  const uint32_t e0 = byte_at(map_before(wave_map_scan(x.map)), entry);
  const int mine = (int)byte_at(x.cnt, e0);
  int k0 = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(k0, off, kWave);
    if (lane >= off) k0 += u;
  }
  if (tid == kEmitThreads - 1) spans_end = before + k0;  // spans up to the workgroup's end
  k0 += before - mine;
  int o = k0;
  uint32_t next = e0;  // the chain's next position among this lane's
#pragma unroll
  for (int p = 0; p < kMatchLane; ++p)
    if (next == (uint32_t)p) {
      const uint32_t len = (L >> (4 * p)) & 15u;
      if (len) {
        span_start[o] = t0 + p;
        span_len[o] = (int)len;
        span_rule[o] = id4[p];
        ++o;
      }
      next += max(len, 1u);
    }
  lane_entry[tid] = (int)e0;
  lane_before[tid] = k0;
  lane_len[tid] = L;
  __syncthreads();
  // a sequence starting at t: the spans whose start is before t
  auto off = [&](int b) { return IN_LDS ? so[b] : seq_offsets[b]; };
  int b0 = 0, hi = B + 1;  // first b with off(b) >= c0
  while (b0 < hi) {
    const int mid = (b0 + hi) >> 1;
    if (off(mid) >= c0) hi = mid;
    else b0 = mid + 1;
  }
  for (int b = b0 + tid; b <= B; b += kEmitThreads) {
    const int t = off(b);
    if (t >= c1 && !last) break;
    int k = spans_end;
    if (t < c1) {
      const int l = (t - c0) / kMatchLane, pe = (t - c0) % kMatchLane;
      const uint32_t Lt = lane_len[l];
      k = lane_before[l];
      for (int p = lane_entry[l]; p < pe;) {
        const int len = (int)((Lt >> (4 * p)) & 15u);
        k += len ? 1 : 0;
        p += max(len, 1);
      }
    }
    seq_span_offsets[b] = k;
  }
}

// ---- decode matching --------------------------------------------------------

constexpr int kDecThreads = 1024;  // one request per thread, one workgroup

static_assert(kDecThreads == kMetaThreads, "the crop runs on the threads that matched");

// CROP: the rollback that the matches imply follows in the same launch (as a
// launch of its own it took 3.9 us and the gap before it).
template <bool CROP>
__global__ __launch_bounds__(kDecThreads) void match_decode_kernel(const i32x4_t *keys, const int32_t *ids,
                                                                   uint32_t mask, i32x4_t *state, int max_seqs,
                                                                   const int32_t *seq_ids,
                                                                   const int32_t *new_tokens, int n,
                                                                   int32_t *k_out, int32_t *rule_out,
                                                                   int32_t *err, CacheArgs cache) {
  __shared__ int sid[kDecThreads];
  __shared__ int bad;
  const int i = threadIdx.x;
  const int s = i < n ? seq_ids[i] : -1;
  RollbackReads rd = {};
  if constexpr (CROP) rd = rollback_reads(cache, s);
  sid[i] = s;
  if (i == 0) bad = 0;
  __syncthreads();
  if (i < n) {
    bool ok = s >= 0 && s < max_seqs;
    for (int j = 0; j < i && ok; ++j) ok = sid[j] != s;
    if (!ok) bad = 1;
  }
  __syncthreads();
  int crop = 0;
  if (i < n) {
    if (bad) {  // nothing changes: no state update, no crop
      if (i == 0) set_err(err, SM_ERR_EINVAL);
      k_out[i] = 0;
      rule_out[i] = -1;
    } else {
      const i32x4_t st = state[s];
      const int r = min(max(st.x, 0), 3);  // raw tokens since the last merge, at most 3 kept
      const int w[4] = {st.y, st.z, st.w, new_tokens[i]};
      i32x4_t cand[3];
      bool want[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {  // candidate c: the suffix of m = 4 - c tokens
        const int m = 4 - c;
        bool ok = m <= r + 1;
#pragma unroll
        for (int j = 0; j < 4; ++j) ok = ok && (j < 4 - m || w[j] >= 0);
        want[c] = ok;
        cand[c] = i32x4_t{w[4 - m], w[5 - m], m > 2 ? w[6 - m] : -1, m > 3 ? w[3] : -1};
      }
      int id;
      const int c = rule_find_longest(keys, ids, mask, cand, want, &id);
      crop = c >= 0 ? 3 - c : 0;  // n - 1 entries to crop
      state[s] = id >= 0 ? i32x4_t{0, -1, -1, -1} : i32x4_t{min(r + 1, 3), w[1], w[2], w[3]};
      k_out[i] = crop;
      rule_out[i] = id;
    }
  }
  if constexpr (CROP) rollback_body(cache, rd, s, crop, n);
}

static bool table_ok(const sm_rule_table *t) {
  return t && t->keys && t->ids && t->err && t->capacity >= 16 && (t->capacity & (t->capacity - 1)) == 0;
}

}  // namespace sm

using namespace sm;

SM_API size_t sm_rules_build_workspace_bytes(int capacity) {
  return capacity > 0 ? (size_t)capacity * sizeof(uint64_t) : 0;
}

SM_API sm_status sm_rules_build(const int32_t *rules, int count, const sm_rule_table *t, void *ws, size_t ws_bytes,
                                hipStream_t stream) {
  if (!table_ok(t) || count < 0 || (int64_t)count * 4 > (int64_t)t->capacity * 3) return SM_EINVAL;
  if (!ws || ws_bytes < sm_rules_build_workspace_bytes(t->capacity) || (count > 0 && !rules)) return SM_EINVAL;
  uint64_t *claim = (uint64_t *)ws;
  const int cap = t->capacity;
  const int grid = min((cap + 255) / 256, 4096);
  hipLaunchKernelGGL(rules_clear_kernel, dim3(grid), dim3(256), 0, stream, claim, cap);
  if (count > 0)
    hipLaunchKernelGGL(rules_claim_kernel, dim3((count + 255) / 256), dim3(256), 0, stream, (const i32x4_t *)rules,
                       count, claim, (uint32_t)(cap - 1), t->err);
  hipLaunchKernelGGL(rules_fill_kernel, dim3(grid), dim3(256), 0, stream, (const i32x4_t *)rules, claim, cap,
                     (i32x4_t *)t->keys, t->ids);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

SM_API sm_status sm_rules_lookup(const sm_rule_table *t, const int32_t *grams, int m, int32_t *ids,
                                 hipStream_t stream) {
  if (!table_ok(t) || m < 0) return SM_EINVAL;
  if (m == 0) return SM_OK;
  if (!grams || !ids) return SM_EINVAL;
  hipLaunchKernelGGL(rules_lookup_kernel, dim3((m + 255) / 256), dim3(256), 0, stream, (const i32x4_t *)t->keys,
                     t->ids, (uint32_t)(t->capacity - 1), (const i32x4_t *)grams, m, ids);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// What callers have always been asked for.  The call uses its first part: the
// lengths (1 B a token), the ids (4 B) and the folds (8 B per 256 and per 1024
// positions).
SM_API size_t sm_match_prompt_workspace_bytes(int B, int total_tokens) {
  if (B < 0 || total_tokens < 0) return 0;
  const size_t T = (size_t)total_tokens;
  return align256(T) + 4 * align256(4 * T) + align256(4 * (size_t)B + 4);
}

SM_API sm_status sm_match_prompt(const sm_rule_table *t, const int32_t *token_ids, const int32_t *seq_offsets,
                                 int B, int total_tokens, int32_t *span_start, int32_t *span_len,
                                 int32_t *span_rule, int32_t *seq_span_offsets, void *ws, size_t ws_bytes,
                                 hipStream_t stream) {
  if (!table_ok(t) || B < 0 || total_tokens < 0 || B > 65535) return SM_EINVAL;
  if (!seq_offsets || !seq_span_offsets || (total_tokens > 0 && (!token_ids || !span_start || !span_len ||
                                                                  !span_rule)))
    return SM_EINVAL;
  if (!ws || ws_bytes < sm_match_prompt_workspace_bytes(B, total_tokens)) return SM_EINVAL;
  const size_t T = (size_t)total_tokens;
  char *p = (char *)ws;
  int8_t *mlen = (int8_t *)p;
  p += align256(T);
  int32_t *rid = (int32_t *)p;
  p += align256(4 * T);
  ChainFold *folds = (ChainFold *)p;  // 8 bytes per 256 positions
  const uint32_t mask = (uint32_t)(t->capacity - 1);
  // (whole emit workgroups: blocks past the last token fold to nothing)
  const int nemit = (total_tokens + kEmitBlocks * kMatchBlock - 1) / (kEmitBlocks * kMatchBlock);
  const bool any = B > 0 && nemit > 0, in_lds = B + 1 <= kMatchLds;
  if (any)
    hipLaunchKernelGGL(in_lds ? match_len_kernel<true> : match_len_kernel<false>, dim3(nemit * kEmitBlocks),
                       dim3(kMatchBlock), 0, stream, (const i32x4_t *)t->keys, t->ids, mask, token_ids, seq_offsets, B,
                       total_tokens, mlen, rid, folds);
  const bool scanned = any && nemit > kScanEmit;
  ChainEntry *at = (ChainEntry *)(folds + (size_t)nemit * kEmitBlocks);  // 8 bytes per 1024 positions
  if (scanned)
    hipLaunchKernelGGL(match_scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, folds, nemit, at);
  // (no sequences, or no tokens: only the offsets, all zero)
  const auto emit = scanned ? (in_lds ? match_emit_kernel<true, true> : match_emit_kernel<false, true>)
                            : (in_lds ? match_emit_kernel<true, false> : match_emit_kernel<false, false>);
  hipLaunchKernelGGL(emit, dim3(any ? nemit : 1), dim3(kEmitThreads), 0, stream, mlen, rid, folds, at, seq_offsets, B,
                     B > 0 ? total_tokens : 0, any ? nemit : 1, span_start, span_len, span_rule, seq_span_offsets,
                     t->err);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

SM_API sm_status sm_match_decode(const sm_rule_table *t, int32_t *state, int max_seqs, const int32_t *seq_ids,
                                 const int32_t *new_tokens, int n, int32_t *k_out, int32_t *rule_out,
                                 const sm_paged_cache *cache, hipStream_t stream) {
  if (!table_ok(t) || n < 0 || n > kDecThreads || max_seqs <= 0) return SM_EINVAL;
  if (cache) {  // the rollback's own synchronous checks, before anything is enqueued
    if (sm_kv_rollback(cache, seq_ids, k_out, 0, stream) != SM_OK || n > cache->max_seqs || n > SM_MAX_REQUESTS)
      return SM_EINVAL;
  }
  if (n == 0) return SM_OK;
  if (!state || !seq_ids || !new_tokens || !k_out || !rule_out) return SM_EINVAL;
  CacheArgs ca = {};
  if (cache && cache_ok(cache, ca))  // (checked above)
    hipLaunchKernelGGL(match_decode_kernel<true>, dim3(1), dim3(kDecThreads), 0, stream, (const i32x4_t *)t->keys,
                       t->ids, (uint32_t)(t->capacity - 1), (i32x4_t *)state, max_seqs, seq_ids, new_tokens, n, k_out,
                       rule_out, t->err, ca);
  else
    hipLaunchKernelGGL(match_decode_kernel<false>, dim3(1), dim3(kDecThreads), 0, stream, (const i32x4_t *)t->keys,
                       t->ids, (uint32_t)(t->capacity - 1), (i32x4_t *)state, max_seqs, seq_ids, new_tokens, n, k_out,
                       rule_out, t->err, ca);
  return hipGetLastError() == hipSuccess ? SM_OK : SM_EHIP;
}

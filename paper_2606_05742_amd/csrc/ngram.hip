// Incremental device-resident n-gram index: the lexical match of Sec. 3.3
// (the longest-suffix generalisation of the exact-match set) answered from an
// index that is updated with each iteration's new tokens, instead of a scan
// of the whole context.
//
// Per sequence and n-gram length n (1 .. n_max) the index holds an
// open-addressing table of the distinct n-grams that end at a candidate
// position j in [n-1, L-2] (a slot keeps one such end position as its key,
// so keys are compared token by token against the context, never by hash
// alone), and for each n-gram an ascending array of all its end positions in
// a per-level pool.  Positions only grow, so arrays are append-only: a full
// array moves to one of twice the capacity (the pool never needs more than
// 12 ints per context token; see ngram_pool_ints).
//
// build kernel: one workgroup per region of a level's table (see its comment).
//
// update kernel (appends with more levels than one workgroup has waves, and
// builds of levels with an overfull region): one workgroup per (level,
// sequence).  The positions that became candidates since the last update (all
// of them when the level starts from scratch) are inserted in
// batches of 256 in ascending order: each batch is sorted by n-gram hash,
// equal n-grams form contiguous groups (checked token by token; a hash
// collision inside a batch falls back to inserting that batch one position at
// a time), each group's first thread finds or creates its slot and reserves
// room, arrays that overflow are copied by the whole workgroup, and every
// thread writes its position at its rank inside its group, so every array
// stays ascending.
//
// append kernel: one workgroup per sequence, one wave per level, each wave
// inserting its level's new positions 64 at a time (a register bitonic sort
// of hash bits and index forms the groups; a batch holding two different
// n-grams with equal bits falls back to one position at a time); a level that
// was never built, or whose context shrank or pool overflowed, is rebuilt
// from scratch by its wave.  With the match fused in, every wave looks the
// last n tokens up in its own level beside its insertions, so an iteration
// costs one launch.
//
// match kernel: one workgroup per sequence; lane n-1 of the first wave looks
// up the last n tokens at level n, the longest level with a hit gives n*,
// and its array is copied out as C_lex: one contiguous read.
#include <algorithm>

#include "adapld_internal.h"
#include "device_utils.h"

namespace adapld {
namespace {

constexpr int kNgThreads = 256;

struct NgSlot {
  int key_end;   // an end position of the slot's n-gram; -1: empty
  int off;       // its position array in the pool
  int count;
  int cap;
};

struct NgHeader {
  int pool_top;      // ints of the pool in use
  int indexed_len;   // context length the level reflects
  int overflow;      // nonzero: the pool overflowed (the level is unusable)
  int magic;         // kNgMagic once a build has initialised the level
};

constexpr int kNgMagic = 0x6e677232;   // of this hash and probing; an index laid out otherwise counts as never built
constexpr size_t kNgRegion = 8192;   // slots per region (a smaller table is one region)

struct NgLevel {
  NgSlot* tab;
  int32_t* pool;
  NgHeader* hdr;
  size_t mask;
  int pool_ints;
};

__device__ __forceinline__ NgLevel ng_level(void* index, int b, int n, int n_max, int L_stride) {
  const size_t slots = ngram_slots(L_stride);
  const size_t lb = ngram_level_bytes(L_stride);
  char* base = static_cast<char*>(index) + ((size_t)b * n_max + (n - 1)) * lb;
  NgLevel l;
  l.tab = reinterpret_cast<NgSlot*>(base);
  l.pool = reinterpret_cast<int32_t*>(base + slots * sizeof(NgSlot));
  l.hdr = reinterpret_cast<NgHeader*>(base + slots * sizeof(NgSlot) + ngram_pool_ints(L_stride) * 4);
  l.mask = slots - 1;
  l.pool_ints = (int)ngram_pool_ints(L_stride);
  return l;
}

// Hash of the n tokens ending at j, newest first: two multiplicative 32-bit
// chains (the low one places the n-gram in the table; a 64-bit product costs
// several quarter-rate multiplies), each finished by murmur3's avalanche step.
// The loops over tokens stay short: the append kernels run once per launch on
// cold code, and their tokens share a cache line or two (with four tokens per
// step here and in ng_equal and a 64-bit probe, us a call: 16 x 8192 tokens, 4
// appended, 4 levels 8.7 -> 8.5, 16 levels 14.5 -> 13.4, 20 levels 23.6 -> 21.8).
__device__ __forceinline__ uint32_t ng_mix(uint32_t h, uint32_t t) {
  h = (h ^ t) * 0x9E3779B1u;
  return h ^ (h >> 15);
}
__device__ __forceinline__ uint32_t ng_finish(uint32_t h) {
  h = (h ^ (h >> 16)) * 0x85EBCA6Bu;
  h = (h ^ (h >> 13)) * 0xC2B2AE35u;
  return h ^ (h >> 16);
}
__device__ __forceinline__ uint64_t ng_hash(const int32_t* M, int j, int n) {
  uint32_t lo = (uint32_t)n, hi = ~(uint32_t)n;
#pragma unroll 2
  for (int i = 0; i < n; ++i) {
    const uint32_t t = (uint32_t)M[j - i];
    lo = ng_mix(lo, t);
    hi = ng_mix(hi, t * 0x85EBCA77u);
  }
  return ((uint64_t)ng_finish(hi) << 32) | ng_finish(lo);
}

__device__ __forceinline__ bool ng_equal(const int32_t* M, int j0, int j1, int n) {
  int differ = 0;
#pragma unroll 1
  for (int i = 0; i < n && differ == 0; ++i) differ = M[j0 - i] ^ M[j1 - i];
  return differ == 0;
}

// The slot of the n-gram ending at j (creating it when `insert`), or -1 when
// it is absent.  Probing is linear and wraps inside the slot's region of
// kNgRegion slots, so that a build can give each region to one workgroup; a
// region that is full goes on in the next one.  The table is at most half
// full, so an empty slot ends every probe; the loop is bounded by the table's
// size all the same.
//
// The result is one variable that is set on every path: with a return at each
// end of the search, the inlined result was undefined in the loop, and one
// build read an unset register for the lanes that had found their n-gram.
__device__ __forceinline__ int ng_probe(const NgLevel& lv, const int32_t* M, int j, int n, uint64_t h, bool insert,
                                        bool& created) {
  const uint32_t mask = (uint32_t)lv.mask;   // at most 2^25 slots
  const uint32_t rm = min(mask, (uint32_t)kNgRegion - 1u);
  uint32_t s = (uint32_t)h & mask;
  int at = -1;
  created = false;
  for (uint32_t left = mask + 1u; left != 0u; --left) {
    int k = __hip_atomic_load(&lv.tab[s].key_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (k < 0 && insert) {
      k = atomicCAS(&lv.tab[s].key_end, -1, j);
      created = k < 0;
    }
    if (k < 0 || ng_equal(M, k, j, n)) {   // empty (or claimed just now), or found
      at = k >= 0 || created ? (int)s : -1;
      break;
    }
    s = (s & ~rm) | ((s + 1u) & rm);
    if (((left - 1u) & rm) == 0u) s = (s + rm + 1u) & mask;   // the region is full
  }
  return at;
}

__device__ __forceinline__ int pow2_at_least(int v) {
  int c = 4;
  while (c < v) c <<= 1;
  return c;
}

// Reserve `ints` of the pool; -1 (and the overflow flag) when it is full.
__device__ __forceinline__ int ng_reserve(int* s_top, int* s_over, int pool_ints, int ints) {
  const int off = atomicAdd(s_top, ints);
  if (off + ints > pool_ints) {
    atomicOr(s_over, 1);
    return -1;
  }
  return off;
}

// Insert [j_lo, j_lo + cnt) one position at a time (one thread): the path
// taken when a batch holds two different n-grams with equal hash bits.
__device__ void ng_insert_serial(const NgLevel& lv, const int32_t* M, int n, int j_lo, int cnt, int* top, int* over) {
  for (int i = 0; i < cnt; ++i) {
    const int j = j_lo + i;
    bool created;
    const int s = ng_probe(lv, M, j, n, ng_hash(M, j, n), true, created);
    if (s < 0) {
      *over = 1;
      continue;
    }
    NgSlot& sl = lv.tab[s];
    int c0 = created ? 0 : sl.count, cap = created ? 0 : sl.cap, off = created ? -1 : sl.off;
    if (c0 + 1 > cap) {
      const int ncap = pow2_at_least(c0 + 1);
      const int noff = *top;
      if (noff + ncap > lv.pool_ints) {
        *over = 1;
        continue;
      }
      *top = noff + ncap;
      for (int e = 0; e < c0; ++e) lv.pool[noff + e] = lv.pool[off + e];
      off = noff;
      cap = ncap;
    }
    lv.pool[off + c0] = j;
    sl.off = off;
    sl.count = c0 + 1;
    sl.cap = cap;
  }
}

// Insert [j_lo, j_lo + cnt) (cnt <= 64) with one wave and no barriers: the
// groups of ng_insert_batch, formed by a register bitonic sort of (hash bits,
// index).  The sort key keeps the hash's top 32 bits and its low 26 bits (the
// table index of every table this index can have: at most 2^26 slots), then
// the index, so equal n-grams are contiguous and in position order.  *top is
// the level's pool top, owned by this wave.
//
// With jq >= 0 the last lane, free when cnt < 64, looks up the n-gram that ends
// at jq beside the insertions, in the same memory round trips.  True if that
// answered (*q_cnt positions from *q_off, in every lane); false if the lane was
// taken or the batch may hold that n-gram itself, whose array then changed.
__device__ bool ng_insert_wave(const NgLevel& lv, const int32_t* M, int n, int j_lo, int cnt, int* top, int* over,
                               int jq, int* q_cnt, int* q_off) {
  const int lane = lane_id();
  const bool valid = lane < cnt;
  const bool query = jq >= 0 && cnt < kWave && lane == kWave - 1;
  uint64_t key = 0;   // invalid lanes sort last
  uint64_t gq = 0;    // the query's group key
  if (valid || query) {
    const uint64_t h = ng_hash(M, query ? jq : j_lo + lane, n);
    const uint64_t bits = (h & 0xffffffff00000000ull) | ((h & 0x3ffffffull) << 6);
    gq = bits >> 6;
    if (valid) key = ~(bits | (uint64_t)lane);
  }
  gq = readlane_u64(gq, kWave - 1);
  // ascending (hash bits, index)
  const uint64_t v = ~(cnt <= 16 ? bitonic_sort_desc_first<16>(key) : bitonic_sort_desc(key));
  const int jt = j_lo + (int)(v & 63);
  const uint64_t gk = v >> 6;                    // the group key
  const uint64_t gprev = shfl_u64(gk, lane > 0 ? lane - 1 : 0);
  const int jprev = __shfl(jt, lane > 0 ? lane - 1 : 0, kWave);
  const bool head = valid && (lane == 0 || gprev != gk);
  const bool differs = valid && !head && !ng_equal(M, jprev, jt, n);
  if (__ballot(differs)) {
    if (lane == 0) ng_insert_serial(lv, M, n, j_lo, cnt, top, over);
    return false;
  }
  const uint64_t heads = __ballot(head);
  const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);   // lanes 0 .. lane
  const int hp = valid ? 63 - __builtin_clzll(heads & upto) : 0;      // this lane's group head
  const uint64_t after = heads & ~upto;
  const int gend = after ? __builtin_ctzll(after) : cnt;             // (head) end of its group
  int slot = -1, off = -1, c0 = 0, cap = 0, req = 0;
  if (head || query) {
    bool created;
    // the table index is the low bits of the hash (= key bits 6..31 here)
    slot = ng_probe(lv, M, query ? jq : jt, n, ((query ? gq : gk) & 0x3ffffffull), head, created);
    if (slot >= 0 && !created) {
      off = lv.tab[slot].off;
      c0 = lv.tab[slot].count;
      cap = lv.tab[slot].cap;
    }
    if (head && slot >= 0 && c0 + (gend - lane) > cap) req = pow2_at_least(c0 + (gend - lane));
  }
  const bool answered = jq >= 0 && cnt < kWave && __ballot(valid && gk == gq) == 0;
  *q_cnt = __builtin_amdgcn_readlane(slot >= 0 ? c0 : 0, kWave - 1);
  *q_off = __builtin_amdgcn_readlane(off, kWave - 1);
  // room for the groups that grow: a wave prefix sum of the requests
  const int incl = wave_incl_scan_i32(req);
  const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
  const int top0 = *top;
  const bool fits = top0 + total <= lv.pool_ints;
  int noff = -1;
  if (req > 0 && fits) noff = top0 + incl - req;
  uint64_t moves = __ballot(req > 0 && fits && c0 > 0);
  if (lane == 0) {
    if (fits) *top = top0 + total;
    else if (total > 0) *over = 1;
  }
  while (moves) {   // the whole wave copies each array that moves
    const int h = __builtin_ctzll(moves);
    moves &= moves - 1;
    const int from = __shfl(off, h, kWave), to = __shfl(noff, h, kWave), len = __shfl(c0, h, kWave);
    for (int e = lane; e < len; e += kWave) lv.pool[to + e] = lv.pool[from + e];
  }
  if (req > 0) {
    off = noff;   // -1 when the pool is full
    cap = req;
  }
  if (head && slot >= 0 && off >= 0) {
    lv.tab[slot].off = off;
    lv.tab[slot].count = c0 + (gend - lane);
    lv.tab[slot].cap = cap;
  } else if (head) {
    *over = 1;
  }
  const int goff = __shfl(head ? off : 0, hp, kWave), gc0 = __shfl(c0, hp, kWave);
  if (valid && goff >= 0) lv.pool[goff + gc0 + (lane - hp)] = jt;
  return answered;
}

// Insert candidate end positions [j_lo, j_lo + cnt) (cnt <= kNgThreads) of
// one level, keeping every position array ascending.
__device__ void ng_insert_batch(const NgLevel& lv, const int32_t* M, int n, int j_lo, int cnt, int* s_top,
                                int* s_over) {
  __shared__ uint64_t s_key[kNgThreads];
  __shared__ int s_idx[kNgThreads];
  __shared__ int s_hp[kNgThreads];     // group head of each sorted element
  __shared__ int s_gend[kNgThreads];   // (head) end of its group
  __shared__ int s_goff[kNgThreads];   // (head) array offset after any move
  __shared__ int s_gc0[kNgThreads];    // (head) array length before the batch
  __shared__ int s_rel[kNgThreads][3]; // moves: old offset, new offset, length
  __shared__ int s_nrel, s_collide;
  const int tid = threadIdx.x;
  // 1. hash, then sort (hash, index) ascending; entries past cnt hash to ~0
  //    and keep their larger indices, so the cnt valid ones come first.
  const bool valid_in = tid < cnt;
  s_key[tid] = valid_in ? ng_hash(M, j_lo + tid, n) : ~0ull;
  s_idx[tid] = tid;
  if (tid == 0) {
    s_nrel = 0;
    s_collide = 0;
  }
  __syncthreads();
  for (int k = 2; k <= kNgThreads; k <<= 1) {
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      const int p = tid ^ jj;
      if (p > tid) {
        const uint64_t a = s_key[tid], c = s_key[p];
        const int ia = s_idx[tid], ic = s_idx[p];
        const bool gt = a > c || (a == c && ia > ic);
        const bool up = (tid & k) == 0;
        if (gt == up) {
          s_key[tid] = c;
          s_key[p] = a;
          s_idx[tid] = ic;
          s_idx[p] = ia;
        }
      }
      __syncthreads();
    }
  }
  // 2. groups of equal hash, checked token by token against the predecessor
  const bool valid = tid < cnt;
  const int jt = j_lo + s_idx[tid];
  const bool head = valid && (tid == 0 || s_key[tid - 1] != s_key[tid]);
  if (valid && !head && !ng_equal(M, j_lo + s_idx[tid - 1], jt, n)) s_collide = 1;
  s_hp[tid] = head ? tid : 0;
  __syncthreads();
  for (int off = 1; off < kNgThreads; off <<= 1) {   // inclusive max-scan: the head of every element
    const int v = tid >= off ? s_hp[tid - off] : 0;
    __syncthreads();
    s_hp[tid] = max(s_hp[tid], v);
    __syncthreads();
  }
  if (valid && (tid + 1 == cnt || s_key[tid + 1] != s_key[tid])) s_gend[s_hp[tid]] = tid + 1;
  __syncthreads();
  if (s_collide) {
    // A hash collision inside the batch: insert one position at a time.
    if (tid == 0) ng_insert_serial(lv, M, n, j_lo, cnt, s_top, s_over);
    __syncthreads();
    return;
  }
  // 3. each group's head finds or creates its slot and reserves room
  if (head) {
    bool created;
    const int s = ng_probe(lv, M, jt, n, s_key[tid], true, created);
    int off = -1, c0 = 0, cap = 0;
    if (s >= 0) {
      NgSlot& sl = lv.tab[s];
      if (!created) {
        off = sl.off;
        c0 = sl.count;
        cap = sl.cap;
      }
      const int nc = c0 + (s_gend[tid] - tid);
      if (nc > cap) {
        const int ncap = pow2_at_least(nc);
        const int noff = ng_reserve(s_top, s_over, lv.pool_ints, ncap);
        if (noff >= 0) {
          if (c0 > 0) {
            const int r = atomicAdd(&s_nrel, 1);
            s_rel[r][0] = off;
            s_rel[r][1] = noff;
            s_rel[r][2] = c0;
          }
          off = noff;
          cap = ncap;
        } else {
          off = -1;   // overflow: the level is marked unusable
        }
      }
      if (off >= 0) {
        sl.off = off;
        sl.count = nc;
        sl.cap = cap;
      }
    } else {
      *s_over = 1;
    }
    s_goff[tid] = off;
    s_gc0[tid] = c0;
  }
  __syncthreads();
  // 4. moved arrays are copied by the whole workgroup; new positions go to
  //    their rank inside their group (disjoint from the copies)
  for (int r = 0; r < s_nrel; ++r) {
    const int from = s_rel[r][0], to = s_rel[r][1], len = s_rel[r][2];
    for (int e = tid; e < len; e += kNgThreads) lv.pool[to + e] = lv.pool[from + e];
  }
  if (valid) {
    const int h = s_hp[tid];
    if (s_goff[h] >= 0) lv.pool[s_goff[h] + s_gc0[h] + (tid - h)] = jt;
  }
  __syncthreads();
}

struct NgArgs {
  const int32_t* tokens;
  const int32_t* lens;
  void* index;
  int B, L_stride, n_max;
};

__global__ __launch_bounds__(kNgThreads) void ngram_update_kernel(const NgArgs a) {
  __shared__ int s_top, s_over, s_start;
  const int n = blockIdx.x + 1;
  const int b = blockIdx.y;
  const NgLevel lv = ng_level(a.index, b, n, a.n_max, a.L_stride);
  const int32_t* M = a.tokens + (size_t)b * a.L_stride;
  const int L = min(max(a.lens[b], 0), a.L_stride);
  if (threadIdx.x == 0) {
    const NgHeader h = *lv.hdr;
    // A level never built, a context that shrank or an unusable level starts from scratch.
    const bool fresh = h.magic != kNgMagic || L < h.indexed_len || h.indexed_len < 0 || h.overflow;
    s_top = fresh ? 0 : h.pool_top;
    s_over = 0;
    s_start = fresh ? -1 : max(n - 1, h.indexed_len - 1);
  }
  __syncthreads();
  int j0 = s_start;
  if (j0 < 0) {
    for (size_t s = threadIdx.x; s <= lv.mask; s += kNgThreads) lv.tab[s] = NgSlot{-1, 0, 0, 0};
    j0 = n - 1;
    __syncthreads();
  }
  // candidate end positions [j0, L-2], in batches, ascending
  for (int lo = j0; lo <= L - 2; lo += kNgThreads) ng_insert_batch(lv, M, n, lo, min(kNgThreads, L - 1 - lo), &s_top, &s_over);
  if (threadIdx.x == 0) *lv.hdr = NgHeader{s_top, L, s_over, kNgMagic};
}

// ------------------------------------------------------------------ build
// From scratch, a level is built by one workgroup per region of its table:
// the workgroup lists the positions whose n-gram falls into its region, in
// ascending order, groups them in a copy of the region's keys in LDS, sizes
// every group's array with one reservation of the pool, and writes the whole
// region, empty slots included, in one coalesced pass (so nothing has to be
// cleared first and no global atomic is taken per n-gram).  A position's rank
// in its array is the number of smaller list indices in its group: counted in
// LDS for a small group, by a bitmap of the list for a large one.  More
// positions than one list holds are counted list by list first, then listed
// again and placed.
//
// What bounds it: the latency of a dozen dependent phases and the writing of
// the table (16 bytes per slot, at least two slots per position of capacity).
// Build calls against one workgroup per level that sorts 256 positions at a
// time (the update kernel), us, Zipf tokens over 128 Ki ids, 4 levels: 1 x 512
// 34 / 12, 16 x 8192 486 / 78, 1 x 131072 7360 / 271, 64 x 32768 2055 / 767;
// contexts of 2 % of the capacity 16 x 8192 17.8 / 16.3, 64 x 8192 23.3 / 28.7.
// Threads beyond the context skip the hashes, and a position's probe starts
// where its listing hash says: 64 levels of 16 x 8192 at 2 % 175 -> 105, full
// 1231 -> 1075.  Many levels of short rows stay dearer than by level where the
// contexts are nearly empty or full (57 and 985 there), not between (at 30 %
// 149 against 280): a near-empty one costs its region's workgroup some 7 us.
constexpr int kBuildThreads = 1024;
constexpr int kBuildWaves = kBuildThreads / kWave;
constexpr int kBuildItems = 4096;            // listed positions
constexpr int kBuildRun = 8;                 // positions per thread and round
constexpr int kBuildSlots = (int)kNgRegion / kBuildThreads;   // table slots per thread
constexpr int kBuildSmall = 32;              // largest group ranked by counting

// Exclusive prefix of v over the workgroup in thread order; *sum gets the sum.
__device__ __forceinline__ int build_scan(int v, int* s_red, int* sum) {
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int incl = wave_incl_scan_i32(v);
  __syncthreads();   // earlier reads of s_red are done
  if (lane == kWave - 1) s_red[wave] = incl;
  __syncthreads();
  const int sums = wave_incl_scan_i32(lane < kBuildWaves ? s_red[lane & (kBuildWaves - 1)] : 0);
  *sum = __builtin_amdgcn_readlane(sums, kWave - 1);
  return incl - v + (wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0);
}

struct BuildShared {
  int key[kNgRegion];            // an end position of the slot's n-gram, -1: empty
  int cnt[kNgRegion];            // its positions; then the pool index of the next one to place (-1: no room)
  uint16_t num[kNgRegion];       // its positions in the current list
  uint16_t first[kNgRegion];     // its first place in grp, then one past its last
  int pos[kBuildItems];          // the list, ascending
  uint16_t slot[kBuildItems];    // where their probes start, then their slots
  uint16_t grp[kBuildItems];     // list indices, group by group
  uint16_t big[kBuildItems / kBuildSmall];
  uint32_t map[kBuildWaves][kBuildItems / 32];
  int red[kBuildWaves];
  int base, nbig, over;
};

// Finds (or claims) the slots of the listed positions s.pos[0, count), from
// the starts that the listing left there.
__device__ __forceinline__ void build_group(const int32_t* __restrict__ M, int n, int rm, int count, BuildShared& s) {
  for (int i = threadIdx.x; i < count; i += kBuildThreads) {
    const int j = s.pos[i];
    int at = s.slot[i];
    int step = 0;
    for (; step <= rm; ++step, at = (at + 1) & rm) {
      const int o = atomicCAS(&s.key[at], -1, j);
      if (o == -1 || ng_equal(M, o, j, n)) break;
    }
    if (step > rm) s.over = 1;   // more n-grams than the region has slots: the level is built by the update kernel
    s.slot[i] = (uint16_t)at;
  }
}

// Writes the listed positions to their groups' arrays, ascending.
__device__ __forceinline__ void build_place(const NgLevel& lv, int nslots, int count, BuildShared& s) {
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int i = tid; i < nslots / 2; i += kBuildThreads) reinterpret_cast<uint32_t*>(s.num)[i] = 0u;
  if (tid == 0) s.nbig = 0;
  __syncthreads();
  // 16-bit counters two to a word: a list has at most kBuildItems of either
  for (int i = tid; i < count; i += kBuildThreads) {
    const int sl = s.slot[i];
    atomicAdd(reinterpret_cast<uint32_t*>(s.num) + (sl >> 1), 1u << (16 * (sl & 1)));
  }
  __syncthreads();
  int c[kBuildSlots], sum = 0, total;
#pragma unroll
  for (int q = 0; q < kBuildSlots; ++q) {
    const int sl = tid + q * kBuildThreads;
    c[q] = sl < nslots ? s.num[sl] : 0;
    sum += c[q];
  }
  int at = build_scan(sum, s.red, &total);
#pragma unroll
  for (int q = 0; q < kBuildSlots; ++q) {
    const int sl = tid + q * kBuildThreads;
    if (c[q]) s.first[sl] = (uint16_t)at;
    if (c[q] > kBuildSmall) s.big[atomicAdd(&s.nbig, 1)] = (uint16_t)sl;
    at += c[q];
  }
  __syncthreads();
  // list indices group by group, in any order inside a group
  for (int i = tid; i < count; i += kBuildThreads) {
    const int sl = s.slot[i];
    const uint32_t old = atomicAdd(reinterpret_cast<uint32_t*>(s.first) + (sl >> 1), 1u << (16 * (sl & 1)));
    s.grp[(old >> (16 * (sl & 1))) & 0xffffu] = (uint16_t)i;
  }
  __syncthreads();
  for (int e = tid; e < count; e += kBuildThreads) {
    const int i = s.grp[e];
    const int sl = s.slot[i];
    const int cr = s.num[sl];
    const int dst = s.cnt[sl];
    if (cr > kBuildSmall || dst < 0) continue;
    const int g0 = s.first[sl] - cr;
    int rank = 0;
    for (int x = 0; x < cr; ++x) rank += s.grp[g0 + x] < i ? 1 : 0;
    lv.pool[dst + rank] = s.pos[i];
  }
  for (int g = wave; g < s.nbig; g += kBuildWaves) {
    const int sl = s.big[g];
    const int cr = s.num[sl];
    const int g0 = s.first[sl] - cr;
    int dst = s.cnt[sl];
    if (dst < 0) continue;
    uint32_t* map = s.map[wave];
    for (int w = lane; w < kBuildItems / 32; w += kWave) map[w] = 0u;
    __threadfence_block();
    for (int x = lane; x < cr; x += kWave) {
      const int i = s.grp[g0 + x];
      atomicOr(&map[i >> 5], 1u << (i & 31));
    }
    __threadfence_block();
    for (int w0 = 0; w0 < kBuildItems / 32; w0 += kWave) {
      uint32_t bits = map[w0 + lane];
      const int incl = wave_incl_scan_i32(__popc(bits));
      int to = dst + incl - __popc(bits);
      dst += __builtin_amdgcn_readlane(incl, kWave - 1);
      while (bits) {
        const int e = __builtin_ctz(bits);
        bits &= bits - 1;
        lv.pool[to++] = s.pos[32 * (w0 + lane) + e];
      }
    }
  }
  __syncthreads();   // the list and the cursors are read
  // the next list's positions follow this one's
#pragma unroll
  for (int q = 0; q < kBuildSlots; ++q) {
    const int sl = tid + q * kBuildThreads;
    if (c[q] && s.cnt[sl] >= 0) s.cnt[sl] += c[q];
  }
}

__global__ __launch_bounds__(kBuildThreads) void ngram_build_kernel(const NgArgs a) {
  __shared__ BuildShared s;
  const int tid = threadIdx.x;
  const int region = blockIdx.x;
  const int n = blockIdx.y + 1;
  const int b = blockIdx.z;
  const NgLevel lv = ng_level(a.index, b, n, a.n_max, a.L_stride);
  const int32_t* __restrict__ M = a.tokens + (size_t)b * a.L_stride;
  const int L = min(max(a.lens[b], 0), a.L_stride);
  const int nslots = (int)min(lv.mask + 1, kNgRegion);
  const int rm = nslots - 1;
  for (int i = tid; i < nslots; i += kBuildThreads) {
    s.key[i] = -1;
    s.cnt[i] = 0;
  }
  if (tid == 0) s.over = 0;

  // Lists the region's positions among kBuildRun consecutive ones per thread
  // and round, in order; use(count) gets every full list and the last one.
  auto each_list = [&](auto use) {
    int count = 0, lists = 0;
    for (int j0 = n - 1; j0 <= L - 2; j0 += kBuildThreads * kBuildRun) {
      const int j = j0 + tid * kBuildRun;
      uint32_t h[kBuildRun];
      uint32_t mine = 0;
      if (j <= L - 2) {   // the waves beyond the context skip the hashes
#pragma unroll
        for (int e = 0; e < kBuildRun; ++e) h[e] = (uint32_t)n;
        // token i of the hashes of the run: a window of tokens that moves back
        int t[kBuildRun];
#pragma unroll
        for (int e = 0; e < kBuildRun; ++e) t[e] = M[min(j + e, L - 1)];
        for (int i = 0; i < n; ++i) {
          const int older = M[max(j - i - 1, 0)];
#pragma unroll
          for (int e = 0; e < kBuildRun; ++e) h[e] = ng_mix(h[e], (uint32_t)t[e]);
#pragma unroll
          for (int e = kBuildRun - 1; e > 0; --e) t[e] = t[e - 1];
          t[0] = older;
        }
#pragma unroll
        for (int e = 0; e < kBuildRun; ++e) {
          h[e] = ng_finish(h[e]) & (uint32_t)lv.mask;
          if (j + e <= L - 2 && (int)(h[e] / kNgRegion) == region) mine |= 1u << e;
        }
      }
      int found;
      int at = count + build_scan(__popc(mine), s.red, &found);
      count += found;
      const bool last = j0 + kBuildThreads * kBuildRun > L - 2;
      for (;;) {
        int k = at;
#pragma unroll
        for (int e = 0; e < kBuildRun; ++e) {
          if ((mine >> e & 1u) == 0u) continue;
          if (k >= 0 && k < kBuildItems) {
            s.pos[k] = j + e;
            s.slot[k] = (uint16_t)(h[e] & rm);
          }
          ++k;
        }
        if (count < kBuildItems && !last) break;
        __syncthreads();   // the list (and, the first time, the empty region) is written
        use(min(count, kBuildItems));
        __syncthreads();   // ... and used
        ++lists;
        at -= kBuildItems;
        count -= min(count, kBuildItems);
        if (count == 0) break;
      }
    }
    return lists;
  };

  int held = 0;   // size of the last list
  const int lists = each_list([&](int count) {
    build_group(M, n, rm, count, s);
    __syncthreads();
    for (int i = tid; i < count; i += kBuildThreads) atomicAdd(&s.cnt[s.slot[i]], 1);
    held = count;
  });
  __syncthreads();
  // One reservation for all arrays of the region, then its slots.
  int need = 0, total;
#pragma unroll
  for (int q = 0; q < kBuildSlots; ++q) {
    const int sl = tid + q * kBuildThreads;
    if (sl < nslots && s.cnt[sl] > 0) need += pow2_at_least(s.cnt[sl]);
  }
  int off = build_scan(need, s.red, &total);
  if (tid == 0) s.base = total > 0 ? atomicAdd(&lv.hdr->pool_top, total) : 0;
  __syncthreads();
  off += s.base;
#pragma unroll
  for (int q = 0; q < kBuildSlots; ++q) {
    const int sl = tid + q * kBuildThreads;
    if (sl < nslots) {
      NgSlot v{-1, 0, 0, 0};
      const int c = s.cnt[sl];
      if (c > 0) {
        const int cap = pow2_at_least(c);
        const bool fits = off + cap <= lv.pool_ints;
        if (!fits) s.over = 1;
        v = NgSlot{s.key[sl], off, c, cap};
        s.cnt[sl] = fits ? off : -1;
        off += cap;
      }
      lv.tab[(size_t)region * kNgRegion + sl] = v;
    }
  }
  __syncthreads();
  if (tid == 0 && s.over) atomicOr(&lv.hdr->overflow, 1);
  if (lists == 1) build_place(lv, nslots, held, s);
  else if (lists > 1)
    each_list([&](int count) {
      build_group(M, n, rm, count, s);
      __syncthreads();
      build_place(lv, nslots, count, s);
    });
}

// The headers of a build: nothing in use, the length it will reflect, and
// whether the update kernel has the level to build (by the overflow mark).
__global__ void ngram_header_kernel(const NgArgs a, int unbuilt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.B * a.n_max) return;
  const int b = i / a.n_max;
  const NgLevel lv = ng_level(a.index, b, i - b * a.n_max + 1, a.n_max, a.L_stride);
  *lv.hdr = NgHeader{0, min(max(a.lens[b], 0), a.L_stride), unbuilt, kNgMagic};
}

// Appending, one wave per level (n_max <= kNgAppendWaves), each inserting its
// level's new positions 64 at a time; with MATCH every wave also looks up the
// last n tokens in its level, beside the last insertions, and the workgroup
// copies out the longest level that hit, so an iteration costs one launch.
// It is a chain of dependent memory round trips (header, tokens, slot, key's
// tokens, pool), with one workgroup per sequence; looking up after the
// insertions instead, in one wave, repeated the chain: 4 levels, 16 x 8192
// tokens, 4 appended, 10.3 -> 8.5 us per launch (host-paced from about 8).
constexpr int kNgAppendWaves = 16;

template <bool MATCH>
__global__ __launch_bounds__(kNgAppendWaves * kWave) void ngram_append_kernel(const NgArgs a, int32_t* __restrict__ cand_pos,
                                                                             int32_t* __restrict__ cand_count,
                                                                             int32_t* __restrict__ match_n) {
  __shared__ int s_top[kNgAppendWaves], s_over[kNgAppendWaves];
  __shared__ int s_cnt[kNgAppendWaves], s_off[kNgAppendWaves];
  const int b = blockIdx.x;
  const int wave = threadIdx.x / kWave;
  const int lane = lane_id();
  const int n = wave + 1;
  const int32_t* M = a.tokens + (size_t)b * a.L_stride;
  const int L = min(max(a.lens[b], 0), a.L_stride);
  if (n <= a.n_max) {
    const NgLevel lv = ng_level(a.index, b, n, a.n_max, a.L_stride);
    const NgHeader h = *lv.hdr;
    const bool fresh = h.magic != kNgMagic || L < h.indexed_len || h.indexed_len < 0 || h.overflow;
    int j0 = max(n - 1, h.indexed_len - 1);
    if (fresh) {   // a context that shrank, or a level never built: start from scratch
      for (size_t s = lane; s <= lv.mask; s += kWave) lv.tab[s] = NgSlot{-1, 0, 0, 0};
      j0 = n - 1;
    }
    if (lane == 0) {
      s_top[wave] = fresh ? 0 : h.pool_top;
      s_over[wave] = 0;
    }
    const int jq = MATCH && L >= n + 1 ? L - 1 : -1;   // the query of this level
    bool answered = false;
    int cnt = 0, off = 0;
    for (int lo = j0; lo <= L - 2; lo += kWave)
      answered = ng_insert_wave(lv, M, n, lo, min(kWave, L - 1 - lo), &s_top[wave], &s_over[wave],
                                lo + kWave > L - 2 ? jq : -1, &cnt, &off);
    if (lane == 0) *lv.hdr = NgHeader{s_top[wave], L, s_over[wave], kNgMagic};
    if constexpr (MATCH) {
      if (!answered) {
        cnt = off = 0;
        if (jq >= 0 && lane == 0) {
          bool created;
          const int s = ng_probe(lv, M, jq, n, ng_hash(M, jq, n), false, created);
          if (s >= 0) {
            cnt = lv.tab[s].count;
            off = lv.tab[s].off;
          }
        }
      }
      if (lane == 0) {
        s_cnt[wave] = cnt;
        s_off[wave] = off;
      }
    }
  }
  if constexpr (MATCH) {
    __syncthreads();   // every level of this sequence is up to date
    int nstar = 0;     // the longest level with a hit; -1: a level overflowed
    for (int w = 0; w < a.n_max; ++w) {
      if (s_cnt[w] > 0 && nstar >= 0) nstar = w + 1;
      if (s_over[w] != 0) nstar = -1;
    }
    const int cnt = nstar > 0 ? s_cnt[nstar - 1] : 0;
    if (cnt > 0) {
      const NgLevel lv = ng_level(a.index, b, nstar, a.n_max, a.L_stride);
      const int32_t* __restrict__ src = lv.pool + s_off[nstar - 1];
      int32_t* __restrict__ dst = cand_pos + (size_t)b * a.L_stride;
      for (int i = threadIdx.x; i < cnt; i += blockDim.x) dst[i] = src[i];
    }
    if (threadIdx.x == 0) {
      cand_count[b] = cnt;
      match_n[b] = nstar;
    }
  }
}

// The lexical match of sequence b from its (up-to-date) index, by the first
// wave of the workgroup: lane n-1 looks up level n; writes the outputs.
__device__ void ng_match_seq(const NgArgs& a, int b, int32_t* __restrict__ cand_pos, int32_t* __restrict__ cand_count,
                             int32_t* __restrict__ match_n, int* s_n, int* s_off, int* s_cnt) {
  const int lane = lane_id();
  const int32_t* M = a.tokens + (size_t)b * a.L_stride;
  const int L = min(max(a.lens[b], 0), a.L_stride);
  if (threadIdx.x < kWave) {
    // lane n-1 looks up level n
    const int n = lane + 1;
    int cnt = 0, off = 0;
    bool stale = false;
    if (n <= a.n_max) {
      const NgLevel lv = ng_level(a.index, b, n, a.n_max, a.L_stride);
      const NgHeader h = *lv.hdr;
      stale = h.magic != kNgMagic || h.indexed_len != L || h.overflow != 0;
      if (!stale && L >= n + 1) {
        bool created;
        const int s = ng_probe(lv, M, L - 1, n, ng_hash(M, L - 1, n), false, created);
        if (s >= 0) {
          cnt = lv.tab[s].count;
          off = lv.tab[s].off;
        }
      }
    }
    const uint64_t hit = __ballot(cnt > 0);
    const bool any_stale = __ballot(stale) != 0;
    const int top = hit ? 63 - __builtin_clzll(hit) : -1;   // the longest level with a hit
    if (lane == 0) {
      *s_n = any_stale ? -1 : top + 1;
      *s_cnt = 0;
      *s_off = 0;
    }
    if (!any_stale && lane == top) {
      *s_cnt = cnt;
      *s_off = off;
    }
  }
  __syncthreads();
  const int nstar = *s_n, cnt = *s_cnt;
  if (cnt > 0) {
    const NgLevel lv = ng_level(a.index, b, nstar, a.n_max, a.L_stride);
    const int32_t* __restrict__ src = lv.pool + *s_off;
    int32_t* __restrict__ dst = cand_pos + (size_t)b * a.L_stride;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) dst[i] = src[i];
  }
  if (threadIdx.x == 0) {
    cand_count[b] = cnt;
    match_n[b] = nstar;
  }
}

__global__ __launch_bounds__(kNgThreads) void ngram_match_kernel(const NgArgs a, int32_t* __restrict__ cand_pos,
                                                                 int32_t* __restrict__ cand_count,
                                                                 int32_t* __restrict__ match_n) {
  __shared__ int s_n, s_off, s_cnt;
  ng_match_seq(a, blockIdx.x, cand_pos, cand_count, match_n, &s_n, &s_off, &s_cnt);
}

}  // namespace

hipError_t launch_ngram_build(const int32_t* tokens, const int32_t* lens, int B, int L_stride, int n_max,
                              void* index, hipStream_t stream) {
  const NgArgs a{tokens, lens, index, B, L_stride, n_max};
  const size_t slots = ngram_slots(L_stride);
  const unsigned regions = (unsigned)((slots + kNgRegion - 1) / kNgRegion);
  // A region's workgroup hashes the whole row, one such workgroup fits a CU,
  // and a row has a region per 2048 to 4096 tokens of capacity: its time, about
  // (18 + levels) / 16 ns a position and round of 256 workgroups, grows with
  // the square of the row.  The update kernel takes 65 ns a position, more
  // beyond some 600 (sequence, level) pairs, whose workgroups share the CUs.
  // Full rows, us by region / by level: 64 x 131072 tokens, 4 levels (32
  // rounds) 6500 / 8540; 16 x 131072, 16 levels (32 rounds) 9080 / 8890; 2 x
  // 131072, 64 levels (16 rounds) 10700 / 10300; 256 x 32768, 4 levels (32
  // rounds, 1024 pairs) 2790 / 3560; 1 x 4194304, 4 levels (16 rounds) 70300 /
  // 260000.
  const long pairs = (long)B * n_max;
  const long rounds = (regions * pairs + 255) / 256;
  const bool by_region = rounds * (n_max + 18) <= 930 * std::max(pairs, 600L) / 600;
  hipLaunchKernelGGL(ngram_header_kernel, dim3((B * n_max + 255) / 256), dim3(256), 0, stream, a, by_region ? 0 : 1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (by_region) {
    hipLaunchKernelGGL(ngram_build_kernel, dim3(regions, n_max, B), dim3(kBuildThreads), 0, stream, a);
    // One region holds every n-gram of its context.  Of several, one can get
    // more than it has slots (chosen tokens; never seen in text); the update
    // kernel then builds that level anew, going on in the next region, and
    // finds nothing to do in the others.
    if ((e = hipGetLastError()) != hipSuccess || regions == 1) return e;
  }
  hipLaunchKernelGGL(ngram_update_kernel, dim3(n_max, B), dim3(kNgThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_ngram_append(const int32_t* tokens, const int32_t* lens, int B, int L_stride, int n_max, void* index,
                               int32_t* cand_pos, int32_t* cand_count, int32_t* match_n, hipStream_t stream) {
  const NgArgs a{tokens, lens, index, B, L_stride, n_max};
  if (n_max > kNgAppendWaves) {   // more levels than one workgroup's waves: one workgroup for each
    hipLaunchKernelGGL(ngram_update_kernel, dim3(n_max, B), dim3(kNgThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !cand_pos) return e;
    hipLaunchKernelGGL(ngram_match_kernel, dim3(B), dim3(kNgThreads), 0, stream, a, cand_pos, cand_count, match_n);
    return hipGetLastError();
  }
  const dim3 block(n_max * kWave);
  if (cand_pos)
    hipLaunchKernelGGL(ngram_append_kernel<true>, dim3(B), block, 0, stream, a, cand_pos, cand_count, match_n);
  else
    hipLaunchKernelGGL(ngram_append_kernel<false>, dim3(B), block, 0, stream, a, cand_pos, cand_count, match_n);
  return hipGetLastError();
}

hipError_t launch_ngram_match(const int32_t* tokens, const int32_t* lens, const void* index, int B, int L_stride,
                              int n_max, int32_t* cand_pos, int32_t* cand_count, int32_t* match_n,
                              hipStream_t stream) {
  const NgArgs a{tokens, lens, const_cast<void*>(index), B, L_stride, n_max};
  hipLaunchKernelGGL(ngram_match_kernel, dim3(B), dim3(kNgThreads), 0, stream, a, cand_pos, cand_count, match_n);
  return hipGetLastError();
}

}  // namespace adapld

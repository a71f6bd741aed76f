// Bulk writes grouped by bucket.
//
// One write operation by one tile (hw_ops.hpp) costs five to six requests to
// random lines: the lock's atomic, the tag bucket, the claim, the publish, the
// release.  When a call brings several operations per bucket, that is the same
// lines again and again, and in tables with fewer buckets than the chip holds
// tiles the tiles also wait for each other's locks.  A bulk call therefore moves
// its operations next to each other first:
//
//  1. k_bulk_split moves the (key, value) pairs to bins of consecutive home buckets,
//     in one or two levels, until a bin (a "part") covers at most bulk_slots() slots
//     and BULK_CAP operations.  `pos` keeps where each operation went.
//  2. k_bulk_write gives each part to one block: duplicates of a key merge in an LDS
//     hash table, the locks of the part's buckets are taken once, the buckets'
//     tags (or keys) are read into LDS once, every operation that its home bucket
//     decides is decided there by one lane, and claims and new slots are written
//     back in slot order, whole lines at a time.  Operations that need another
//     bucket run the per-tile code of hw_ops.hpp under the lock the block holds.
//  3. k_bulk_finish brings the statuses back to the operations' order (k_bulk_back
//     before it, for the second level) and runs what the parts did not take -- bins
//     that overflowed (skewed keys), buckets whose lock another call held -- one tile
//     per distinct key of 64 operations.
//
// Locks: a block tries each lock byte once and never waits for one, so it cannot
// deadlock with tiles that wait in the queues; it holds them for a bounded time.
// Everything written to the table, and every read that can race, is the same
// access as in the per-tile code (tag or key claimed first, then one publish, then
// the release after all writes completed), so queries and writers of other calls
// may run beside it.  The order of a call's operations is free, so any grouping of
// them is one serialisation.
//
// Measured, one tile per operation against grouped, microseconds, 64-bit keys: ICEBERG,
// half of 2^23 slots' keys inserted 665 / 219, all of them updated 1326 / 465, half erased
// 699 / 198; ICEBERG_M, 2^27 slots, 6288 / 3353, 12260 / 7928, 7073 / 3026; P2HT(M) erases
// of half the keys, 2^23 slots 700 / 216, 2^27 6336 / 3438.
#pragma once

#include "hw_ops.hpp"

namespace hw {

constexpr int BULK_THREADS = 256;
constexpr int BULK_CAP = 1024;        // most operations per part: 4 per thread
constexpr uint64_t BULK_MIN_OPS = 2048;  // smaller calls are not grouped: four launches cost more than they save
constexpr int BULK_BINS = 1024;       // most bins per level
constexpr int BULK_SPLIT_THREADS = 1024;
constexpr uint32_t BULK_WIDE_TILE = 1u << 22;  // operations from which a split tile takes 8192 of them, not 4096
constexpr uint32_t BULK_NONE = 0xFFFFFFFFu;  // pos of an operation its bin had no room for
constexpr uint32_t BULK_CSTRIDE = 32;        // first-level cursors: one per 128-byte line
// Most slots per part: what fits in LDS as 2-byte tags, or as keys, beside the
// operations.
template <class C>
constexpr int bulk_slots() {
  return C::TAGS ? 4096 : sizeof(typename C::K) == 8 ? 1024 : 2048;
}
// states of an operation while its part is worked on (final ones are ST_*)
constexpr uint8_t BULK_PENDING = 255;  // left to k_bulk_finish
constexpr uint8_t BULK_SLOW = 254;     // needs more than its home bucket
constexpr uint8_t BULK_NEW = 253;      // has a slot, not yet published
constexpr uint32_t BULK_NO_OP = 0xFFFFu;

// How a call's operations are split (host: bulk_plan in capi.hip).
struct BulkPlan {
  uint32_t levels;     // 1 or 2
  uint32_t shift;      // log2 of the buckets per part
  uint32_t parts;      // ceil(home buckets / 2^shift)
  uint32_t sub;        // two levels: log2 of the parts per first-level bin
  uint32_t bins;       // first-level bins (parts when levels == 1)
  uint32_t cap1, cap;  // room of a first-level bin / of a part, in operations
  uint32_t hash_n;     // entries of a part's merge table: a power of two, at least 3/2 of cap
  uint32_t slow_tiles; // tiles of a block that work on what the home bucket does not decide
  // byte offsets in the scratch buffer
  uint64_t off_cursor1, off_cursor, zero_bytes, off_pos1, off_pos, off_rec1, off_rec, off_stat1, off_stat, bytes;
};

// The home bucket of a key: the one whose lock its writers take.  nf != 0: iceberg's
// front yard and chaining (multiply-shift), else a power of two.
struct HomeMap {
  uint32_t mask, nf;
};
__device__ __forceinline__ uint32_t home_bucket(const HomeMap& m, uint64_t h) {
  return m.nf ? __umulhi((uint32_t)h, m.nf) : (uint32_t)h & m.mask;
}

template <typename K>
struct alignas(2 * sizeof(K)) BulkPair {
  K key, val;
};

// Moves operations to bins: bin = (home bucket >> shift) - first bin of the region,
// room `cap` per bin.  Level one reads the call's arrays (one region of n
// operations), level two (REC) the first level's bins, one region each.
//
// Bound by memory: each pair is read and written once.  A block counts its tile's
// operations per bin in LDS, reserves room with one atomic per bin, and writes
// each pair to its place; the runs of one bin are short (a tile's share), and the
// XCD's L2 merges them into lines.
template <typename K, bool VALS, bool REC, int PER>
__device__ __forceinline__ void
bulk_split(uint32_t block, const K* __restrict__ keys, const K* __restrict__ vals, uint32_t n, uint32_t region_cap,
             const uint32_t* __restrict__ region_count, HomeMap home, uint32_t shift, uint32_t bins_log2, uint32_t bins,
             uint32_t cap, uint32_t* __restrict__ cursor, uint32_t cstride, K* __restrict__ rec,
             uint32_t* __restrict__ pos) {
  constexpr uint32_t TILE = BULK_SPLIT_THREADS * PER;
  __shared__ uint32_t hist[BULK_BINS], base[BULK_BINS];
  const uint32_t tid = threadIdx.x;
  uint32_t region = 0, t0 = block * TILE, count = n;
  if constexpr (REC) {
    const uint32_t tiles = (region_cap + TILE - 1) / TILE;
    region = block / tiles;
    t0 = (block % tiles) * TILE;
    count = region_count[region * BULK_CSTRIDE];
    if (count > region_cap) count = region_cap;
    if (t0 >= count) return;
  }
  const uint32_t bin0 = REC ? region << bins_log2 : 0;
  const uint32_t in0 = region * region_cap;
  for (uint32_t b = tid; b < bins; b += BULK_SPLIT_THREADS) hist[b] = 0;
  __syncthreads();
  K key[PER], val[PER];
  uint32_t at[PER];  // bin << 16 | rank within the tile's share of the bin
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = t0 + r * BULK_SPLIT_THREADS + tid;
    if (i >= count) continue;
    if constexpr (REC && VALS) {
      const BulkPair<K> p = ((const BulkPair<K>*)keys)[in0 + i];
      key[r] = p.key;
      val[r] = p.val;
    } else {
      key[r] = keys[in0 + i];
      if constexpr (VALS) val[r] = vals[in0 + i];
    }
  }
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = t0 + r * BULK_SPLIT_THREADS + tid;
    if (i >= count) continue;
    const uint32_t bin = (home_bucket(home, fmix64((uint64_t)key[r] ^ HASH_SALT)) >> shift) - bin0;
    at[r] = bin << 16 | __hip_atomic_fetch_add(&hist[bin], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  for (uint32_t b = tid; b < bins; b += BULK_SPLIT_THREADS) {
    const uint32_t c = hist[b];
    base[b] = c ? __hip_atomic_fetch_add(cursor + (uint64_t)(bin0 + b) * cstride, c, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT)
                : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = t0 + r * BULK_SPLIT_THREADS + tid;
    if (i >= count) continue;
    const uint32_t bin = at[r] >> 16, o = base[bin] + (at[r] & 0xFFFFu);
    uint32_t dst = BULK_NONE;
    if (o < cap) {
      dst = (bin0 + bin) * cap + o;
      if constexpr (VALS) ((BulkPair<K>*)rec)[dst] = BulkPair<K>{key[r], val[r]};
      else rec[dst] = key[r];
    }
    pos[in0 + i] = dst;
  }
}

template <typename K, bool VALS, bool REC, int PER>
__global__ void __launch_bounds__(BULK_SPLIT_THREADS)
k_bulk_split(const K* __restrict__ keys, const K* __restrict__ vals, uint32_t n, uint32_t region_cap,
             const uint32_t* __restrict__ region_count, HomeMap home, uint32_t shift, uint32_t bins_log2, uint32_t bins,
             uint32_t cap, uint32_t* __restrict__ cursor, uint32_t cstride, K* __restrict__ rec,
             uint32_t* __restrict__ pos) {
  bulk_split<K, VALS, REC, PER>(blockIdx.x, keys, vals, n, region_cap, region_count, home, shift, bins_log2, bins, cap,
                                cursor, cstride, rec, pos);
}

// Clears the cursors; mark: the erase flag of a table whose erases mark it before
// anything is removed (hw_ops.hpp), else null.
template <typename K>
__global__ void __launch_bounds__(256)
k_bulk_zero(uint4* p, uint32_t n16, uint32_t* mark) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) p[i] = make_uint4(0, 0, 0, 0);
  if (i == 0 && mark && ld(mark) == 0) st(mark, 1u);
}

// What a part's block keeps in LDS, laid out for the call's own part size: a block's
// work is a chain of round trips (locks, tags, keys, claims, new slots), so what
// counts is how many blocks take turns on a CU, and a small part must not pay
// for a large one's arrays.
template <class C, bool ERASE>
struct BulkLds {
  using K = typename C::K;
  static constexpr int B = C::CHAIN ? 8 : C::B;  // slot units per bucket
  using Mask = typename std::conditional<(B > 32), uint64_t, uint32_t>::type;
  using Img = typename std::conditional<C::TAGS, uint16_t, K>::type;
  static constexpr bool SERIAL = !ERASE && C::CHAIN;  // one tile per bucket

  K* keys;
  K* vals;            // upserts: a key's values merge into its leader's
  uint32_t* hash;     // while duplicates merge: leader of each key (index + 1)
  Img* img;           // then, in the same place: tags or keys as read under the locks (img_at),
  uint16_t* op_of;    // and the operation that takes each slot
  Mask* free;         // free slots of each bucket
  uint32_t* taken;    // free slots handed out
  uint32_t* head;     // the bucket's slow operations, where one tile takes them all
  uint32_t* word;     // n_slow, flag
  uint16_t* list;     // operations that need more than their home bucket
  uint16_t* next;     // (see head)
  uint8_t* state;
  uint8_t* need;
  uint8_t* held;
  uint8_t* ends;      // an absent key's search ends in this bucket

  // Places the arrays at `base` (null to size them); returns their bytes.
  __host__ __device__ __forceinline__ uint32_t place(char* base, uint32_t cap, uint32_t hash_n, uint32_t buckets) {
    uint32_t at = 0;
    auto take = [&](uint32_t bytes) {
      char* p = base + at;
      at += (bytes + 15) & ~15u;
      return p;
    };
    const uint32_t slots = buckets * B;
    keys = (K*)take(cap * (uint32_t)sizeof(K));
    vals = (K*)take(ERASE ? 0 : cap * (uint32_t)sizeof(K));
    const uint32_t img_b = slots * (uint32_t)sizeof(Img), both = img_b + slots * 2, h = hash_n * 4;
    hash = (uint32_t*)take(h > both ? h : both);
    img = (Img*)hash;
    op_of = (uint16_t*)((char*)hash + img_b);
    free = (Mask*)take(buckets * (uint32_t)sizeof(Mask));
    taken = (uint32_t*)take(buckets * 4);
    head = (uint32_t*)take(SERIAL ? buckets * 4 : 0);
    word = (uint32_t*)take(8);
    list = (uint16_t*)take(cap * 2);
    next = (uint16_t*)take(SERIAL ? cap * 2 : 0);
    state = (uint8_t*)take(cap);
    need = (uint8_t*)take(buckets);
    held = (uint8_t*)take(buckets);
    ends = (uint8_t*)take(buckets);
    return at;
  }
  // Element j of bucket b.  Lanes look at the same j of different buckets, whose rows
  // would start in the same few banks: each row is permuted by its bucket.  Tags
  // keep their groups of four (8 bytes).
  __device__ __forceinline__ uint32_t img_at(uint32_t b, uint32_t j) const {
    if constexpr (C::TAGS) return b * B + ((((j >> 2) ^ b) & (B / 4 - 1)) << 2 | (j & 3));
    else return b * B + ((j ^ b) & (B - 1));
  }
};

template <typename Mask>
__device__ __forceinline__ uint32_t nth_bit(Mask m, uint32_t n) {
  for (uint32_t i = 0; i < n; ++i) m &= m - 1;
  return (uint32_t)__ffsll((unsigned long long)m) - 1;
}

// Merges an operation's value into the one (in LDS) of its key's first operation.
template <typename K>
__device__ __forceinline__ void merge_value(K* to, K v, int combine) {
  if (combine == C_SUM) __hip_atomic_fetch_add(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else if (combine == C_MIN) __hip_atomic_fetch_min(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else if (combine == C_MAX) __hip_atomic_fetch_max(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else if (combine == C_REPLACE) __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// An operation's status, given that of its key's first one.
template <bool ERASE>
__device__ __forceinline__ uint8_t follow(uint8_t s, bool first) {
  return first || s != ST_DONE ? s : ERASE ? (uint8_t)ST_MISS : (uint8_t)ST_EXISTED;
}

// Instrumented builds: an upsert that its home bucket decided (others are counted where
// they search).
__device__ __forceinline__ void count_home_write(const TableDev& tv) {
  probe_add(tv, PC_WRITE, 1);
  probe_add(tv, PC_VISIT, 1);
}

// Which elements of bucket b of the part's image equal x (a tag or a key; the first
// n of them are looked at where they are keys).
template <class Lds, typename X>
__device__ __forceinline__ typename Lds::Mask image_equal(const Lds& L, uint32_t b, X x, int n) {
  using Mask = typename Lds::Mask;
  Mask m = 0;
  if constexpr (sizeof(typename Lds::Img) == 2) {
#pragma unroll
    for (int q = 0; q < Lds::B / 4; ++q) {
      const uint64_t w = *(const uint64_t*)(L.img + L.img_at(b, 4 * q));
#pragma unroll
      for (int j = 0; j < 4; ++j) m |= (Mask)(((uint32_t)(w >> (16 * j)) & 0xFFFFu) == (uint32_t)x) << (4 * q + j);
    }
  } else {
#pragma unroll
    for (int j = 0; j < n; ++j) m |= (Mask)(L.img[L.img_at(b, j)] == x) << j;
  }
  return m;
}

// The slot of `key` among the candidates m (tag matches) of the bucket at slot s0,
// `first` being the key word of the first candidate; -1 if none holds it.
template <class C, typename Mask>
__device__ __forceinline__ int32_t match_key(const TableDev& tv, uint64_t s0, Mask m, typename C::K first,
                                             typename C::K key) {
  typename C::K k = first;
  while (m) {
    const uint32_t j = nth_bit(m, 0);
    if (k == key) return (int32_t)j;
    m &= m - 1;
    if (m) k = ld(Ops<C>::key_ptr(tv, s0 + nth_bit(m, 0)));
  }
  return -1;
}

// Erases of two-choice tables with tags: a lane per listed operation looks for its key
// in the alternate bucket.  The lanes of a group read each other's tag buckets
// together, 16 bytes a lane, so that a bucket is one request and all of a wave's
// buckets one round trip.
template <class C>
__device__ __forceinline__ void bulk_alternates(const TableDev& tv, const BulkLds<C, true>& L, uint32_t n) {
  using K = typename C::K;
  using O = Ops<C>;
  constexpr int B = C::B;
  constexpr int G = B / 8;  // lanes per group: 8 tags each
  const uint32_t lane = __lane_id(), g = lane % G, group = lane - g;
#pragma unroll 1
  for (uint32_t u0 = threadIdx.x - lane; u0 < n; u0 += BULK_THREADS) {
    const bool mine = u0 + lane < n;
    const uint32_t i = L.list[mine ? u0 + lane : u0];
    const K key = L.keys[i];
    const typename O::Home h = O::home_of(tv, key);
    const uint32_t b2 = h.h2 & tv.bucket_mask, tag = tag_of((uint64_t)key);
    uint64_t lo[G], hi[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const uint64_t* src = (const uint64_t*)tv.tagw + (uint64_t)__shfl(b2, (int)(group + j), 64) * (B / 4) + 2 * g;
      lo[j] = ld(src);
      hi[j] = ld(src + 1);
    }
    uint32_t cand = 0;  // of the lane's own operation
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const uint32_t tj = __shfl(tag, (int)(group + j), 64);
      uint32_t c = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) c |= (uint32_t)(((uint32_t)((k < 4 ? lo[j] : hi[j]) >> (16 * (k % 4))) & 0xFFFFu) == tj) << k;
      c <<= 8 * g;
#pragma unroll
      for (int o = 1; o < G; o <<= 1) c |= __shfl_xor(c, o, 64);
      if ((uint32_t)j == g) cand = c;
    }
    if (!mine) continue;
    uint8_t s = ST_MISS;
    if (b2 != h.b1 && cand) {  // else the key has one bucket, searched already
      const uint64_t s0 = (uint64_t)b2 * B;
      const int32_t j = match_key<C, uint32_t>(tv, s0, cand, ld(O::key_ptr(tv, s0 + nth_bit(cand, 0))), key);
      if (j >= 0) {
        st(O::key_ptr(tv, s0 + j), (K)O::EMPTY);
        wait_mem();  // the key is gone before its tag is
        st((uint16_t*)tv.tagw + s0 + j, (uint16_t)TAG_EMPTY);
        s = ST_DONE;
      }
    }
    L.state[i] = s;
  }
}

// Works on one part: operations rec[0, count) whose home buckets are [b0, b0 + nb),
// statuses (or BULK_PENDING) to stat[0, count).  rec has room for `cap` of them.
//
// Bound by requests to memory, far fewer than one tile per operation would send:
// per bucket one lock atomic, one read of its tags, one release; per four new tags
// one compare-and-swap; new slots in whole lines.
template <class C, bool ERASE>
__device__ __forceinline__ void bulk_part(const TableDev& tv, BulkLds<C, ERASE> L, const typename C::K* __restrict__ rec,
                                          const uint32_t* __restrict__ cursor, uint32_t cap, uint32_t hash_n, uint32_t b0,
                                          uint32_t nb, uint32_t slow_tiles, int combine, uint8_t* __restrict__ stat) {
  using K = typename C::K;
  using O = Ops<C>;
  using Lds = BulkLds<C, ERASE>;
  using Mask = typename Lds::Mask;
  constexpr int B = Lds::B;
  constexpr int PER = BULK_CAP / BULK_THREADS;
  constexpr bool ALTERNATE = ERASE && C::DESIGN == D_P2_M && B <= 32;  // its registers
  const uint32_t tid = threadIdx.x;
  const uint64_t slot0 = (uint64_t)b0 * B;
  const uint32_t slots = nb * B;
  uint32_t* const n_slow_lds = L.word;
  uint32_t* const flag_lds = L.word + 1;
  K key[PER];
  uint16_t lb[PER];    // the operation's bucket, within the part
  uint16_t lead[PER];  // the key's leader

  // ---- load, reset.  The pairs are fetched beside their count: room that holds
  // none is memory all the same.
  uint32_t count = *cursor;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= cap) continue;
    if constexpr (ERASE) {
      key[r] = rec[i];
    } else {
      const BulkPair<K> p = ((const BulkPair<K>*)rec)[i];
      key[r] = p.key;
      L.vals[i] = p.val;
    }
    L.keys[i] = key[r];
  }
  if (count > cap) count = cap;
  if (count == 0) return;
  for (uint32_t e = tid; e < hash_n; e += BULK_THREADS) L.hash[e] = 0;
  for (uint32_t b = tid; b < nb; b += BULK_THREADS) {
    L.need[b] = 0;
    L.held[b] = 0;
    L.taken[b] = 0;
    L.free[b] = 0;
    L.ends[b] = 0;
    if constexpr (Lds::SERIAL) L.head[b] = 0;
  }
  if (tid == 0) {
    *n_slow_lds = 0;
    *flag_lds = 0;
  }
  __syncthreads();
  uint32_t dh[PER];  // where the merge table starts looking
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= count) continue;
    const uint64_t h = fmix64((uint64_t)key[r] ^ HASH_SALT);
    lb[r] = (uint16_t)(O::home_of_hash(tv, h) - b0);
    dh[r] = (uint32_t)(h >> 32) & (hash_n - 1);
    if (key[r] < Keys<K>::FIRST_INVALID) L.need[lb[r]] = 1;
  }
  __syncthreads();

  // ---- locks: one try each; a held byte leaves the bucket's operations to k_bulk_finish
  // (a lane per 8 bytes of the lock array: atomics on one line are served one after another)
  {
    const uint32_t per = 8u >> tv.locks.shift;  // buckets per 8 bytes
    for (uint32_t g = tid; g * per < nb; g += BULK_THREADS) {
      uint64_t want = 0;
      for (uint32_t j = 0; j < per && g * per + j < nb; ++j)
        if (L.need[g * per + j]) want |= 1ull << (8 * (((b0 + g * per + j) << tv.locks.shift) & 7));
      if (!want) continue;
      const uint64_t old = try_locks(tv.locks, b0 + g * per, want);
      for (uint32_t j = 0; j < per && g * per + j < nb; ++j) {
        const uint64_t bit = 1ull << (8 * (((b0 + g * per + j) << tv.locks.shift) & 7));
        if ((want & bit) && !(old & bit)) L.held[g * per + j] = 1;
      }
    }
  }

  // ---- merge duplicates: the first operation to enter its key leads it
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= count) continue;
    lead[r] = (uint16_t)i;
    if (key[r] >= Keys<K>::FIRST_INVALID) continue;
    uint32_t e = dh[r];
    while (true) {
      uint32_t cur = 0;
      if (__hip_atomic_compare_exchange_strong(&L.hash[e], &cur, i + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP))
        break;
      if (L.keys[cur - 1] == key[r]) {
        lead[r] = (uint16_t)(cur - 1);
        break;
      }
      e = (e + 1) & (hash_n - 1);
    }
    if constexpr (!ERASE)
      if (lead[r] != i) merge_value(&L.vals[lead[r]], L.vals[i], combine);
  }
  __syncthreads();  // the locks' answers have arrived: reads below come after them; the merge table is done with

  // ---- the buckets' tags or keys, read once
  if constexpr (C::TAGS) {
    const uint64_t* src = (const uint64_t*)(tv.tagw + slot0 / 2);
    for (uint32_t q = tid; q < slots / 4; q += BULK_THREADS) {
      const uint64_t x = ld(src + q);
      const uint32_t b = q / (B / 4), j = q % (B / 4) * 4;
      *(uint64_t*)(L.img + L.img_at(b, j)) = x;
      uint32_t f = 0;
      bool e = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t t = (uint32_t)(x >> (16 * k)) & 0xFFFFu;
        f |= (uint32_t)(t >= TAG_TOMB) << k;
        e |= t == TAG_EMPTY;
      }
      if (f) __hip_atomic_fetch_or(&L.free[b], (Mask)f << j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (C::DOUBLE && e) L.ends[b] = 1;
    }
  } else {
    for (uint32_t s = tid; s < slots; s += BULK_THREADS) {
      const uint32_t b = s / B, j = s % B;
      const K x = ld(O::key_ptr(tv, slot0 + s));
      L.img[L.img_at(b, j)] = x;
      if (C::CHAIN && j == 7) {
        // a chain of one node: the search ends there
        L.ends[b] = ld((const uint64_t*)O::val_ptr(tv, slot0 + s)) == O::NIL;
        continue;
      }
      if (x == O::EMPTY || x == O::TOMB)
        __hip_atomic_fetch_or(&L.free[b], (Mask)1 << j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (C::DOUBLE && x == O::EMPTY) L.ends[b] = 1;
    }
  }
  if constexpr (!ERASE && C::ICEBERG) {
    // The erase flag counts as read after every bucket (hw_ops.hpp, shortcut
    // safety): each wave reads it after the buckets it read.
    wait_mem();
    if (__lane_id() == 0 && ld(tv.ctrl) != 0) *flag_lds = 1;
  }
  for (uint32_t s = tid; s < slots / 4; s += BULK_THREADS) ((uint64_t*)L.op_of)[s] = ~0ull;
  __syncthreads();
  const bool erased = *flag_lds != 0;

  // ---- find each key in its home bucket.  `op_of` first holds, per slot, the operation
  // that may find its key there: reads and updates then go in slot order too.
  Mask cand[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    cand[r] = 0;
    if (i >= count || lead[r] != i) continue;
    uint8_t s = BULK_SLOW;
    if (key[r] >= Keys<K>::FIRST_INVALID) {
      s = ST_INVALID;
    } else if (!L.held[lb[r]]) {
      s = BULK_PENDING;
    } else {
      if constexpr (C::TAGS) cand[r] = image_equal(L, lb[r], tag_of((uint64_t)key[r]), B);
      else cand[r] = image_equal(L, lb[r], key[r], C::CHAIN ? 7 : B);
      if (cand[r]) L.op_of[lb[r] * B + nth_bit(cand[r], 0)] = (uint16_t)i;
    }
    L.state[i] = s;
  }
  __syncthreads();
  for (uint32_t s = tid; s < slots; s += BULK_THREADS) {
    const uint32_t o = L.op_of[s];
    if (o == BULK_NO_OP) continue;
    bool hit = true;
    if constexpr (C::TAGS) hit = ld(O::key_ptr(tv, slot0 + s)) == L.keys[o];
    if (!hit) {
      L.op_of[s] = (uint16_t)BULK_NO_OP;
    } else if constexpr (ERASE) {
      L.state[o] = ST_DONE;
      st(O::key_ptr(tv, slot0 + s), (K)(C::DOUBLE ? O::TOMB : O::EMPTY));
    } else {
      L.op_of[s] = (uint16_t)BULK_NO_OP;
      L.state[o] = ST_EXISTED;
      O::combine_lane(tv, slot0 + s, L.vals[o], combine);
      count_home_write(tv);
    }
  }
  if constexpr (ERASE && C::TAGS) wait_mem();  // the keys are gone before their tags are
  __syncthreads();
  if constexpr (ERASE && C::TAGS)
    for (uint32_t s = tid; s < slots; s += BULK_THREADS)
      if (L.op_of[s] != BULK_NO_OP) st((uint16_t*)tv.tagw + slot0 + s, (uint16_t)(C::DOUBLE ? TAG_TOMB : TAG_EMPTY));

  // ---- decide the others there, if that bucket can
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= count || lead[r] != i || L.state[i] != BULK_SLOW) continue;
    uint8_t s = BULK_SLOW;
    const uint32_t b = lb[r];
    int32_t j = -1;
    if constexpr (C::TAGS) {
      // other slots of the same tag: rare, one at a time
      if (cand[r]) {
        const uint64_t s0 = slot0 + b * B;
        j = match_key<C, Mask>(tv, s0, cand[r], ld(O::key_ptr(tv, s0 + nth_bit(cand[r], 0))), key[r]);
        if (j >= 0) {
          if constexpr (ERASE) {
            s = ST_DONE;
            st(O::key_ptr(tv, s0 + j), (K)(C::DOUBLE ? O::TOMB : O::EMPTY));
            wait_mem();
            st((uint16_t*)tv.tagw + s0 + j, (uint16_t)(C::DOUBLE ? TAG_TOMB : TAG_EMPTY));
          } else {
            s = ST_EXISTED;
            O::combine_lane(tv, s0 + j, L.vals[i], combine);
            count_home_write(tv);
          }
        }
      }
    }
    if (j < 0) {
      if constexpr (ERASE) {
        if constexpr (C::DOUBLE || C::CHAIN)
          if (L.ends[b]) s = ST_MISS;
      } else {
        // an absent key goes into this bucket while it has room for it
        uint32_t room = (uint32_t)__popcll((unsigned long long)L.free[b]);
        if constexpr (C::ICEBERG) room = erased ? 0 : room;
        else room = L.ends[b] ? room : 0;
        if (room) {
          const uint32_t k = __hip_atomic_fetch_add(&L.taken[b], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (k < room) {
            L.op_of[b * B + nth_bit(L.free[b], k)] = (uint16_t)i;
            s = BULK_NEW;
          }
        }
      }
    }
    if (ALTERNATE && s == BULK_SLOW) {
      const uint32_t at = __hip_atomic_fetch_add(n_slow_lds, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      L.list[at] = (uint16_t)i;
    }
    L.state[i] = s;
  }
  __syncthreads();
  if constexpr (ALTERNATE) {
    const uint32_t n = *n_slow_lds;
    if (n) {
      bulk_alternates<C>(tv, L, n);
      __syncthreads();
      if (tid == 0) *n_slow_lds = 0;
      __syncthreads();
    }
  }

  if constexpr (!ERASE) {
    // ---- claim the new keys' slots: other buckets' writers may claim them too, except
    // in iceberg's front yard and in chains
    if constexpr (C::TAGS && !C::ICEBERG) {
      for (uint32_t w = tid; w < slots / 4; w += BULK_THREADS) {
        const uint64_t ops = ((const uint64_t*)L.op_of)[w];
        if (ops == ~0ull) continue;
        uint64_t cur = *(const uint64_t*)(L.img + L.img_at(w / (B / 4), w % (B / 4) * 4));
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (uint32_t)(ops >> (16 * j)) & 0xFFFFu;
        while (true) {
          uint64_t want = cur;
          bool any = false;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (o[j] == BULK_NO_OP) continue;
            if (((uint32_t)(cur >> (16 * j)) & 0xFFFFu) >= TAG_TOMB) {
              want = (want & ~(0xFFFFull << (16 * j))) | (uint64_t)tag_of((uint64_t)L.keys[o[j]]) << (16 * j);
              any = true;
            } else {  // lost to another bucket's writer
              L.state[o[j]] = BULK_SLOW;
              L.op_of[4 * w + j] = (uint16_t)BULK_NO_OP;
              o[j] = BULK_NO_OP;
            }
          }
          if (!any) break;
          const uint64_t old = cas((uint64_t*)(tv.tagw + slot0 / 2) + w, cur, want);
          if (old == cur) break;
          cur = old;
        }
      }
      __syncthreads();
    } else if constexpr (!C::TAGS && !C::ICEBERG && !C::CHAIN) {
      for (uint32_t s = tid; s < slots; s += BULK_THREADS) {
        const uint32_t o = L.op_of[s];
        if (o == BULK_NO_OP) continue;
        bool won = false;
        if constexpr (sizeof(K) == 8) {
          K* kp = O::key_ptr(tv, slot0 + s);
          K cur = L.img[L.img_at(s / B, s % B)];
          while (cur == O::EMPTY || cur == O::TOMB) {
            const K old = cas(kp, cur, (K)Keys<K>::RESERVED);
            if (old == cur) { won = true; break; }
            cur = old;
          }
        } else {
          // the whole slot at once; a slot never used since the table was cleared reads all-ones
          uint64_t* sp = (uint64_t*)O::key_ptr(tv, slot0 + s);
          uint64_t cur = (uint64_t)L.img[L.img_at(s / B, s % B)] | 0xFFFFFFFF00000000ull;
          const uint64_t want = (uint64_t)L.keys[o] | (uint64_t)L.vals[o] << 32;
          while ((K)cur == O::EMPTY || (K)cur == O::TOMB) {
            const uint64_t old = cas(sp, cur, want);
            if (old == cur) { won = true; break; }
            cur = old;
          }
        }
        if (!won) {
          L.state[o] = BULK_SLOW;
          L.op_of[s] = (uint16_t)BULK_NO_OP;
        }
      }
      __syncthreads();
    }
    // ---- publish in slot order: consecutive lanes write consecutive slots
    for (uint32_t s = tid; s < slots; s += BULK_THREADS) {
      const uint32_t o = L.op_of[s];
      if (o == BULK_NO_OP) continue;
      if constexpr (C::TAGS && C::ICEBERG) st((uint16_t*)tv.tagw + slot0 + s, (uint16_t)tag_of((uint64_t)L.keys[o]));
      if constexpr (C::TAGS || C::ICEBERG || C::CHAIN || sizeof(K) == 8) O::publish(tv, slot0 + s, L.keys[o], L.vals[o]);
      L.state[o] = ST_DONE;
      count_home_write(tv);
    }
    wait_mem();
    __syncthreads();
  }

  // ---- what needs more than the home bucket: tiles, still under its lock.  Keys are
  // distinct here, so tiles may share a bucket and claim free slots with
  // compare-and-swaps, except in chains, whose free slots are taken with plain stores:
  // there one tile takes a bucket's operations one by one.
  // (listed afresh: claims have been lost since, and the alternate buckets decided)
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= count || lead[r] != i || L.state[i] != BULK_SLOW) continue;
    const uint32_t at = __hip_atomic_fetch_add(n_slow_lds, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    L.list[at] = (uint16_t)i;
    if constexpr (Lds::SERIAL)
      L.next[i] = (uint16_t)__hip_atomic_exchange(&L.head[lb[r]], i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  const uint32_t n_slow = *n_slow_lds;
  if (n_slow) {
    const Tile<C::T> tile;
    auto one = [&](uint32_t i) {
      const K k = L.keys[i];
      const typename O::Home h = O::home_of(tv, k);
      const uint32_t tag = C::TAGS ? tag_of((uint64_t)k) : 0u;
      uint8_t s;
      if constexpr (ERASE) s = O::erase_locked(tv, tile, h, k, tag);
      else if (C::ICEBERG && !erased) s = O::upsert_iceberg_backyard(tv, tile, h, k, L.vals[i], tag, combine);
      else s = O::template upsert_locked<true>(tv, tile, h, k, L.vals[i], tag, combine);
      if (tile.leader()) L.state[i] = s;
    };
    const uint32_t at = tid / 64 + tid % 64 / C::T * (BULK_THREADS / 64);  // tiles taken from every wave
    // (in a table that has erased most of them are no backyard choices)
    const uint32_t tiles = erased ? BULK_THREADS / C::T : slow_tiles;
    if (!Lds::SERIAL && at < tiles) {
#pragma unroll 1
      for (uint32_t u = at; u < n_slow; u += tiles) one(L.list[u]);
    }
    if constexpr (Lds::SERIAL) {
#pragma unroll 1
      for (uint32_t b = tid / C::T; b < nb; b += BULK_THREADS / C::T)
        for (uint32_t i = L.head[b]; i; i = L.next[i - 1]) {
          one(i - 1);
          wait_mem();  // the next one sees what this one wrote
        }
    }
  }
  wait_mem();  // every write of the part has completed
  __syncthreads();
  for (uint32_t b = tid; b < nb; b += BULK_THREADS)
    if (L.held[b]) release_try_lock(tv.locks, b0 + b);

  // ---- statuses: a key's first operation has its own, the others follow it
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = r * BULK_THREADS + tid;
    if (i >= count) continue;
    stat[i] = follow<ERASE>(L.state[lead[r]], lead[r] == i);
  }
}

template <class C, bool ERASE>
__global__ void __launch_bounds__(BULK_THREADS)
k_bulk_write(TableDev tv, const typename C::K* __restrict__ rec, const uint32_t* __restrict__ cursor, uint32_t cstride,
             uint32_t cap, uint32_t hash_n, uint32_t shift, uint32_t slow_tiles,
             int combine, uint8_t* __restrict__ stat) {
  extern __shared__ __align__(16) char bulk_lds[];
  BulkLds<C, ERASE> L;
  L.place(bulk_lds, cap, hash_n, 1u << shift);
  const uint32_t p = blockIdx.x, b0 = p << shift, left = Ops<C>::home_buckets(tv) - b0;
  bulk_part<C, ERASE>(tv, L, rec + (uint64_t)p * cap * (ERASE ? 1 : 2), cursor + (uint64_t)p * cstride, cap, hash_n, b0,
                      left < (1u << shift) ? left : 1u << shift, slow_tiles, combine, stat + (uint64_t)p * cap);
}

// Two levels: statuses back to the order of the first level's bins, a wave per 64 places
// of a bin that holds count[] operations (room for `cap`).
template <typename K>
__global__ void __launch_bounds__(256)
k_bulk_back(uint32_t bins, uint32_t cap, const uint32_t* __restrict__ count, const uint32_t* __restrict__ pos,
            const uint8_t* __restrict__ stat, uint8_t* __restrict__ out) {
  const uint32_t per_bin = (cap + 63) / 64, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * 256 + threadIdx.x) / 64);
  for (uint32_t w = wave; w < bins * per_bin; w += gridDim.x * 4) {
    const uint32_t bin = w / per_bin, off = w % per_bin * 64 + lane, have = count[bin * BULK_CSTRIDE];
    if (off >= (have < cap ? have : cap)) continue;
    const uint64_t i = (uint64_t)bin * cap + off;
    const uint32_t p = pos[i];
    out[i] = p == BULK_NONE ? BULK_PENDING : stat[p];
  }
}

// Statuses back to the call's order, and the operations left over (no room in their bin,
// or BULK_PENDING) through the per-tile path, in that order.
//
// bulk_finish: 64 operations from `base` on, by one wave; pos null: none is decided.
//
// What is left over of a skewed call is its hot keys, closer together than in the call
// itself, so equal keys of the 64 merge first: one locked operation each.  Without that, the
// waits for a hot key's lock took longer than in a plain call (27,852 upserts, half of them of one
// key, DOUBLE, 2^15 slots: 30 ms plain, 34 unmerged, 0.79 so).
template <class C, bool ERASE>
__device__ __forceinline__ void bulk_finish(const TableDev& tv, const typename C::K* __restrict__ keys,
                                            const typename C::K* __restrict__ vals, uint64_t base, uint64_t n,
                                            const uint32_t* __restrict__ pos, const uint8_t* __restrict__ stat,
                                            int combine, uint8_t* __restrict__ out) {
  using K = typename C::K;
  struct Rest {
    K key[64], val[64];  // val: of the first of equal keys, all of theirs
    uint8_t order[64], stat[64];
  };
  __shared__ Rest rest_lds[BLOCK / 64];
  const Tile<C::T> tile;
  const uint32_t lane = __lane_id();
  Rest& L = rest_lds[__builtin_amdgcn_readfirstlane(threadIdx.x / 64)];
  bool rest = false;
  if (base + lane < n) {
    const uint32_t p = pos ? pos[base + lane] : BULK_NONE;
    const uint8_t s = p == BULK_NONE ? BULK_PENDING : stat[p];
    rest = s == BULK_PENDING;
    if (!rest && out) out[base + lane] = s;
  }
  const uint64_t m = __ballot(rest);
  if (m == 0) return;
  K key = 0, val = 0;
  if (rest) {
    key = keys[base + lane];
    if constexpr (!ERASE) val = vals[base + lane];
  }
  uint32_t lead = lane;  // the first lane with the same key
  for (uint64_t todo = m; todo;) {
    const uint32_t f = (uint32_t)ffs64(todo);
    const K kf = __shfl(key, (int)f, 64);
    const uint64_t same = __ballot(rest && key == kf);
    if (same >> lane & 1) lead = f;
    todo &= ~same;
  }
  const uint64_t leads = __ballot(rest && lead == lane);
  if (rest && lead == lane) {
    L.order[__popcll(leads & ((1ull << lane) - 1))] = (uint8_t)lane;
    L.key[lane] = key;
    if constexpr (!ERASE) L.val[lane] = val;
  }
  wave_sync();
  if constexpr (!ERASE)
    if (rest && lead != lane) merge_value(&L.val[lead], val, combine);
  wave_sync();
  const uint32_t cnt = (uint32_t)__popcll(leads);
  for (uint32_t u = lane / C::T; u < cnt; u += 64 / C::T) {
    const uint32_t o = L.order[u];
    uint8_t s;
    if constexpr (ERASE) s = Ops<C>::erase(tv, tile, L.key[o]);
    else s = Ops<C>::upsert(tv, tile, L.key[o], L.val[o], combine);
    if (tile.leader()) L.stat[o] = s;
  }
  wave_sync();
  if (rest && out) out[base + lane] = follow<ERASE>(L.stat[lead], lead == lane);
  wave_sync();
}

template <class C, bool ERASE>
__global__ void __launch_bounds__(BLOCK)
k_bulk_finish(TableDev tv, const typename C::K* __restrict__ keys, const typename C::K* __restrict__ vals, uint32_t n,
              const uint32_t* __restrict__ pos, const uint8_t* __restrict__ stat, int combine,
              uint8_t* __restrict__ out) {
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  for (uint64_t base = ((uint64_t)blockIdx.x * (BLOCK / 64) + wid) * 64; base < n; base += (uint64_t)gridDim.x * BLOCK)
    bulk_finish<C, ERASE>(tv, keys, vals, base, n, pos, stat, combine, out);
}

// ---------------------------------------------------------------- groups of tables
//
// One upsert per table of a group of one configuration: the same steps, each one
// launch over all tables.  A step's blocks are numbered through the tables
// (BulkGroup::first); a block looks its table up in that list, a wave at 64 places a
// time, which costs one round trip to the L2 for every 64 tables.

// A table of a group.
struct MultiTable {
  TableDev tv;
  uint32_t cls;          // index in the key width's configuration menu
  uint32_t pad;
  uint64_t fill_words;   // 16-byte words of slots + tags (all-ones when empty)
  uint64_t zero_words;   // 16-byte words of locks + control (zero when empty)
};

// One table's part in the call.
struct BulkJob {
  BulkPlan plan;      // levels 0: its operations are not grouped
  HomeMap home;
  uint32_t table;     // of the group
  uint32_t n;         // operations
  uint64_t begin;     // first operation, in the shared arrays
  uint64_t scratch;   // offset of the plan's memory in the scratch buffer
};

enum : int { GROUP_ZERO, GROUP_SPLIT, GROUP_SPLIT2, GROUP_WRITE, GROUP_BACK, GROUP_FINISH, GROUP_STEPS };
constexpr uint32_t GROUP_ZERO_BYTES = 4096;  // cleared per block of 256
constexpr int GROUP_PER = 8;                 // operations per thread of a split tile

struct BulkGroup {
  const BulkJob* jobs;
  const uint32_t* first;  // [GROUP_STEPS][n]: each job's first block of a step
  uint32_t n;             // jobs
  uint8_t* scratch;
};

// The job of this block, and the block's number within it (`rest`).
template <int STEP>
__device__ __forceinline__ const BulkJob& group_job(const BulkGroup& g, uint32_t* rest) {
  const uint32_t* f = g.first + STEP * g.n;
  const uint32_t lane = __lane_id();
  uint32_t j = 0;  // jobs that start at or before this block
  for (uint32_t i = 0; i < g.n; i += 64)
    j += (uint32_t)__popcll(__ballot(i + lane < g.n && f[i + lane] <= blockIdx.x));
  j = __builtin_amdgcn_readfirstlane(j) - 1;
  *rest = blockIdx.x - __builtin_amdgcn_readfirstlane(f[j]);
  return g.jobs[j];
}

template <typename K>
__global__ void __launch_bounds__(256) k_group_clear(BulkGroup g) {
  uint32_t b;
  const BulkJob& j = group_job<GROUP_ZERO>(g, &b);
  const uint64_t at = (uint64_t)b * GROUP_ZERO_BYTES + threadIdx.x * 16;
  if (at < j.plan.zero_bytes) *(uint4*)(g.scratch + j.scratch + j.plan.off_cursor1 + at) = make_uint4(0, 0, 0, 0);
}

template <typename K, bool REC, int PER>
__global__ void __launch_bounds__(BULK_SPLIT_THREADS)
k_group_split(BulkGroup g, const K* __restrict__ keys, const K* __restrict__ vals) {
  uint32_t b;
  const BulkJob& j = group_job<REC ? GROUP_SPLIT2 : GROUP_SPLIT>(g, &b);
  const BulkPlan& p = j.plan;
  uint8_t* m = g.scratch + j.scratch;
  uint32_t* cursor1 = (uint32_t*)(m + p.off_cursor1);
  if constexpr (REC)
    bulk_split<K, true, true, PER>(b, (const K*)(m + p.off_rec1), nullptr, p.bins * p.cap1, p.cap1, cursor1, j.home,
                                   p.shift, p.sub, 1u << p.sub, p.cap, (uint32_t*)(m + p.off_cursor), 1,
                                   (K*)(m + p.off_rec), (uint32_t*)(m + p.off_pos));
  else
    bulk_split<K, true, false, PER>(b, keys + j.begin, vals + j.begin, j.n, j.n, nullptr, j.home,
                                    p.shift + (p.levels == 2 ? p.sub : 0), 0, p.bins, p.cap1, cursor1, BULK_CSTRIDE,
                                    (K*)(m + p.off_rec1), (uint32_t*)(m + p.off_pos1));
}

template <class C>
__global__ void __launch_bounds__(BULK_THREADS)
k_group_write(BulkGroup g, const MultiTable* __restrict__ tables, int combine) {
  using K = typename C::K;
  extern __shared__ __align__(16) char bulk_lds[];
  uint32_t part;
  const BulkJob& j = group_job<GROUP_WRITE>(g, &part);
  const BulkPlan& p = j.plan;
  const TableDev tv = tables[j.table].tv;
  uint8_t* m = g.scratch + j.scratch;
  const bool two = p.levels == 2;
  BulkLds<C, false> L;
  L.place(bulk_lds, p.cap, p.hash_n, 1u << p.shift);
  const uint32_t b0 = part << p.shift, left = Ops<C>::home_buckets(tv) - b0;
  bulk_part<C, false>(tv, L, (const K*)(m + (two ? p.off_rec : p.off_rec1)) + (uint64_t)part * p.cap * 2,
                      (const uint32_t*)(m + (two ? p.off_cursor : p.off_cursor1)) + (uint64_t)part * (two ? 1 : BULK_CSTRIDE),
                      p.cap, p.hash_n, b0, left < (1u << p.shift) ? left : 1u << p.shift,
                      p.slow_tiles < BULK_THREADS / C::T ? p.slow_tiles : BULK_THREADS / C::T, combine,
                      m + (two ? p.off_stat : p.off_stat1) + (uint64_t)part * p.cap);
}

// (a block per 256 places of a first-level bin)
template <typename K>
__global__ void __launch_bounds__(256) k_group_back(BulkGroup g) {
  uint32_t b;
  const BulkJob& j = group_job<GROUP_BACK>(g, &b);
  const BulkPlan& p = j.plan;
  uint8_t* m = g.scratch + j.scratch;
  const uint32_t per_bin = (p.cap1 + 255) / 256, bin = b / per_bin, off = b % per_bin * 256 + threadIdx.x;
  const uint32_t have = ((const uint32_t*)(m + p.off_cursor1))[bin * BULK_CSTRIDE];
  if (off >= (have < p.cap1 ? have : p.cap1)) return;
  const uint64_t i = (uint64_t)bin * p.cap1 + off;
  const uint32_t at = ((const uint32_t*)(m + p.off_pos))[i];
  (m + p.off_stat1)[i] = at == BULK_NONE ? BULK_PENDING : (m + p.off_stat)[at];
}

// (a block per GROUP_FINISH_OPS operations)
constexpr uint32_t GROUP_FINISH_OPS = 4 * BLOCK;
template <class C>
__global__ void __launch_bounds__(BLOCK)
k_group_finish(BulkGroup g, const MultiTable* __restrict__ tables, const typename C::K* __restrict__ keys,
               const typename C::K* __restrict__ vals, int combine, uint8_t* __restrict__ out) {
  uint32_t b;
  const BulkJob& j = group_job<GROUP_FINISH>(g, &b);
  const TableDev tv = tables[j.table].tv;
  const uint8_t* m = g.scratch + j.scratch;
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const bool grouped = j.plan.levels != 0;
  for (uint32_t k = 0; k < GROUP_FINISH_OPS / BLOCK; ++k) {
    const uint64_t base = (uint64_t)b * GROUP_FINISH_OPS + k * BLOCK + wid * 64;
    if (base < j.n)
      bulk_finish<C, false>(tv, keys + j.begin, vals + j.begin, base, j.n,
                            grouped ? (const uint32_t*)(m + j.plan.off_pos1) : nullptr, m + j.plan.off_stat1, combine,
                            out ? out + j.begin : nullptr);
  }
}

}  // namespace hw

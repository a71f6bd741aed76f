// C-ABI of HashWave (declared in include/hashwave.h): table creation and
// layout, argument checks, dispatch to the kernel instance of the table's
// (key width, design, bucket, tile), and the design-independent kernels
// (initialisation, counting, export, primary-bucket lookup).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "hashwave.h"
#include "hw_launch.hpp"
#include "hw_multi.hpp"

using namespace hw;

static void drop_groups_of(hwave_table* t);

struct hwave_table {
  int device;
  hwave_design design;
  hwave_config cfg;
  uint64_t nb, capacity, bytes;
  uint64_t units;  // (key, value) units in the slot region (chaining: link units too)
  uint64_t n_lock_words;
  void* base;
  bool owns;
  const KernelSet* ks;
  LaunchArgs la;
  bool has_merge;  // HWAVE_F_MERGE_MIXED: workspace for merging mixed calls' upserts
  MergeWs ws;
};

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return HWAVE_EDEVICE;
}

constexpr uint64_t ALIGN = 256;
// A waiter's limit for its bucket lock (hwave_config.lock_timeout_us), converted
// to ticks of the 100 MHz wall clock, which must fit 32 bits.
constexpr uint32_t DEFAULT_LOCK_TIMEOUT_US = 10000000;
constexpr uint32_t MAX_LOCK_TIMEOUT_US = 40000000;
uint64_t round_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

struct Layout {
  uint64_t nb, capacity, units, pool;
  uint64_t off_tags, off_locks, off_lockq, off_ctrl, off_pool_ctr, off_hot, off_merge, total;
  uint64_t n_lock_words;  // 32-bit words of the lock array (one byte per bucket, at a stride)
  uint32_t lock_shift;    // log2 of the lock stride in bytes
  uint64_t n_lockq;       // lock queues (hw_device.hpp): a power of two
};

// Lock bytes at a stride of 1 << lock_shift bytes (hw_device.hpp, LockArray:
// clamp(2^23 / nb, 1, 8) bytes), then the lock queues: the largest power of
// two <= nb, at most LOCK_QUEUES_MAX.  Returns the offset after them.
uint64_t place_locks(uint64_t nb, uint64_t off, Layout* L) {
  L->lock_shift = 0;
  while (L->lock_shift < 3 && (nb << (L->lock_shift + 1)) <= (1ull << 23)) ++L->lock_shift;
  L->off_locks = off;
  L->n_lock_words = ((nb << L->lock_shift) + 3) / 4;
  off += round_up(L->n_lock_words * 4, ALIGN);
  uint64_t nq = 1;
  while (nq * 2 <= nb && nq * 2 <= LOCK_QUEUES_MAX) nq *= 2;
  L->off_lockq = off;
  L->n_lockq = nq;
  return off + round_up(nq * 8, ALIGN);
}

// Hot-key accumulators (hw_ops.hpp, HOT_ROWS): tables that merge duplicates and
// never erase, except cuckoo (it moves keys) and the phased variant.
bool has_hot(hwave_design design, const hwave_config& c) {
  const uint32_t f = c.flags;
  return (f & HWAVE_F_AGGREGATE) && (f & HWAVE_F_NO_ERASE) && !(f & HWAVE_F_BSP) && design != HWAVE_CUCKOO;
}

// Appends the hot-key accumulators (tags, then accumulators) at `off` if the
// table has them; they lie in the zero-filled part of the table.  Then the
// merge workspace of HWAVE_F_MERGE_MIXED tables (hw_merge.hpp: 2 * MERGE_CHUNK
// entries of a key word and 16 bytes, and a word per operation of a chunk), also
// all zero when empty.
constexpr uint64_t MERGE_ENTRIES = 2ull * MERGE_CHUNK;
uint64_t merge_bytes() { return MERGE_ENTRIES * (8 + sizeof(MergeEntry)) + (uint64_t)MERGE_CHUNK * 4; }

uint64_t place_hot(hwave_design design, const hwave_config& c, uint64_t off, Layout* L) {
  L->off_hot = 0;
  L->off_merge = 0;
  if (has_hot(design, c)) {
    L->off_hot = off;
    off += round_up((uint64_t)HOT_N * 16, ALIGN);
  }
  if (c.flags & HWAVE_F_MERGE_MIXED) {
    L->off_merge = off;
    off += round_up(merge_bytes(), ALIGN);
  }
  return off;
}

bool design_tags(int d) { return d == HWAVE_DOUBLE_M || d == HWAVE_P2_M || d == HWAVE_ICEBERG_M; }
bool design_iceberg(int d) { return d == HWAVE_ICEBERG || d == HWAVE_ICEBERG_M; }
bool design_chain(int d) { return d == HWAVE_CHAINING; }

// Iceberg front yard: 83% of the buckets (Section 5), at least one bucket in
// each yard.
uint64_t iceberg_front(uint64_t nb) {
  uint64_t nf = nb * 83 / 100;
  if (nf < 1) nf = 1;
  if (nf > nb - 1) nf = nb - 1;
  return nf;
}

const std::vector<const KernelSet*>& registry() {
  static std::vector<const KernelSet*> all;
  static std::once_flag once;
  std::call_once(once, [] {
    const KernelSet* (*fns[])(size_t*) = {sets_u64_double, sets_u64_p2, sets_u64_iceberg, sets_u64_chain, sets_u64_cuckoo,
                                          sets_u32_double, sets_u32_p2, sets_u32_iceberg, sets_u64_bsp};
    for (auto f : fns) {
      size_t n = 0;
      const KernelSet* s = f(&n);
      for (size_t i = 0; i < n; i++) all.push_back(s + i);
    }
  });
  return all;
}

const KernelSet* find_set(const hwave_config& c, int design) {
  const bool bsp = (c.flags & HWAVE_F_BSP) != 0;
  for (const KernelSet* s : registry())
    if (s->kv_bits == (int)c.kv_bits && s->design == design && s->bucket == (int)c.bucket_slots &&
        s->tile == (int)c.tile && s->bsp == bsp)
      return s;
  return nullptr;
}

// Paper configurations (Section 5) for 64-bit keys; 32-bit keys keep the same
// bucket byte span with 8-byte slots where a design's default bucket is small.
void defaults_for(hwave_design design, uint32_t kv_bits, hwave_config* c) {
  memset(c, 0, sizeof *c);
  c->kv_bits = kv_bits;
  c->bucket_slots = design == HWAVE_DOUBLE ? (kv_bits == 64 ? 8 : 16)
                    : design_chain(design)   ? 7
                    : design == HWAVE_CUCKOO ? 8
                                             : 32;
  c->tile = design_tags(design) || design == HWAVE_CUCKOO ? 4 : 8;
}

int resolve_config(hwave_design design, const hwave_config* in, hwave_config* out) {
  if ((int)design < HWAVE_DOUBLE || (int)design > HWAVE_CUCKOO) return HWAVE_EINVAL;
  const uint32_t kv = in && in->kv_bits ? in->kv_bits : 64;
  if (kv != 64 && kv != 32) return HWAVE_EINVAL;
  hwave_config c;
  defaults_for(design, kv, &c);
  if (in) {
    if (in->bucket_slots) c.bucket_slots = in->bucket_slots;
    if (in->tile) c.tile = in->tile;
    c.probe_cap = in->probe_cap;
    c.flags = in->flags;
    c.lock_timeout_us = in->lock_timeout_us;
  }
  if (c.lock_timeout_us > MAX_LOCK_TIMEOUT_US) return HWAVE_EINVAL;
  *out = c;
  return HWAVE_OK;
}

int layout_of(uint64_t capacity, hwave_design design, const hwave_config& c, Layout* L) {
  if (capacity == 0 || c.bucket_slots == 0) return HWAVE_EINVAL;
  if (design_chain(design)) {
    // Chaining (Section 5): ceil(capacity / 7) buckets, each a 128-byte first
    // node (7 pairs and a link), then an overflow pool of twice as many nodes.
    // A node stays on its chain once linked (lock-free readers may be walking
    // it), so under churn a chain keeps the nodes its longest past content
    // needed; two spare nodes per bucket cover that for long aging runs.  The
    // capacity reported counts every slot of buckets and pool.
    const uint64_t nb = (capacity + 6) / 7;
    if (nb > (1ull << 30)) return HWAVE_EINVAL;
    const uint64_t pool = 2 * nb;
    L->nb = nb;
    L->pool = pool;
    L->units = (nb + pool) * 8;
    L->capacity = (nb + pool) * 7;
    uint64_t off = round_up(L->units * 16, ALIGN);
    L->off_tags = off;
    off = place_locks(nb, off, L);
    L->off_ctrl = off;
    off += ALIGN;
    L->off_pool_ctr = off;  // POOL_PARTS allocation counters, one per 128-byte line
    off += round_up((uint64_t)POOL_PARTS * POOL_CTR_STRIDE * 4, ALIGN);
    L->total = place_hot(design, c, off, L);
    return HWAVE_OK;
  }
  const uint64_t B = c.bucket_slots;
  uint64_t want = (capacity + B - 1) / B;
  uint64_t nb = design_iceberg(design) ? 2 : 1;  // iceberg: a bucket in each yard
  while (nb < want) nb <<= 1;
  if (nb > (1ull << 32)) return HWAVE_EINVAL;
  const uint64_t slot_bytes = c.kv_bits / 4;  // two words
  L->nb = nb;
  L->capacity = nb * B;
  L->units = L->capacity;
  L->pool = 0;
  uint64_t off = round_up(L->capacity * slot_bytes, ALIGN);
  L->off_tags = off;
  if (design_tags(design)) off += round_up(L->capacity * 2, ALIGN);
  off = place_locks(nb, off, L);
  L->off_ctrl = off;
  off += ALIGN;
  L->total = place_hot(design, c, off, L);
  return HWAVE_OK;
}

__global__ void k_fill16(uint4* p, uint64_t n16, uint32_t word) {
  const uint4 v = make_uint4(word, word, word, word);
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

template <typename K>
__global__ void k_count(const K* __restrict__ slots, uint64_t nslots, uint64_t* count) {
  uint64_t c = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nslots;
       i += (uint64_t)gridDim.x * blockDim.x)
    c += slots[2 * i] < Keys<K>::FIRST_INVALID;
  // one atomic per block: one address serves ~80 M of them a second
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  __shared__ uint64_t wave[4];
  if ((threadIdx.x & 63) == 0) wave[threadIdx.x / 64] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    c = wave[0] + wave[1] + wave[2] + wave[3];
    if (c) atomicAdd((unsigned long long*)count, (unsigned long long)c);
  }
}

// Live pairs, in no order.  Bound by memory, once the output cursor is not what
// counts: one address serves ~80 M atomics a second, so a block reserves room for
// EXPORT_PER slots a thread at once (2^21 slots, 1.6 M live: 397 us with an atomic per
// wave and slot, 20 here).
constexpr int EXPORT_PER = 8;
template <typename K>
__global__ void __launch_bounds__(256)
k_export(const K* __restrict__ slots, uint64_t nslots, K* __restrict__ okeys, K* __restrict__ ovals, uint64_t* count) {
  struct alignas(2 * sizeof(K)) Pair {
    K key, val;
  };
  __shared__ uint32_t wave[4];
  __shared__ uint64_t base;
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x / 64;
  for (uint64_t i0 = (uint64_t)blockIdx.x * (256 * EXPORT_PER); i0 < nslots; i0 += (uint64_t)gridDim.x * (256 * EXPORT_PER)) {
    Pair p[EXPORT_PER];
    uint32_t at[EXPORT_PER], n = 0;  // n: the wave's live slots so far
#pragma unroll
    for (int r = 0; r < EXPORT_PER; ++r) {
      const uint64_t i = i0 + r * 256 + threadIdx.x;
      p[r].key = Keys<K>::EMPTY;
      if (i < nslots) p[r] = ((const Pair*)slots)[i];
    }
#pragma unroll
    for (int r = 0; r < EXPORT_PER; ++r) {
      const uint64_t m = __ballot(p[r].key < Keys<K>::FIRST_INVALID);
      at[r] = n + (uint32_t)__popcll(m & ((1ull << lane) - 1));
      n += (uint32_t)__popcll(m);
    }
    if (lane == 0) wave[wid] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint64_t all = (uint64_t)wave[0] + wave[1] + wave[2] + wave[3];
      base = all ? atomicAdd((unsigned long long*)count, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    uint64_t out = base;
    for (uint32_t w = 0; w < wid; ++w) out += wave[w];
#pragma unroll
    for (int r = 0; r < EXPORT_PER; ++r) {
      if (!(p[r].key < Keys<K>::FIRST_INVALID)) continue;
      okeys[out + at[r]] = p[r].key;
      ovals[out + at[r]] = p[r].val;
    }
    __syncthreads();
  }
}

__global__ void k_zero_u64(uint64_t* p) { *p = 0; }

// The bucket whose lock a key's writers take: primary bucket, or the front-yard
// bucket of iceberg tables (nf != 0).
template <typename K>
__global__ void k_primary(const K* __restrict__ keys, uint64_t n, uint32_t mask, uint32_t nf,
                          uint64_t* __restrict__ out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = nf ? front_bucket((uint64_t)keys[i], nf) : hash_key((uint64_t)keys[i], mask).b1;
}

// Every bucket a key may occupy (hwave_candidate_buckets): three per key,
// unused entries all-ones.
template <typename K>
__global__ void k_candidates(const K* __restrict__ keys, uint64_t n, int design, uint32_t mask, uint32_t nf,
                             uint32_t nback, uint64_t* __restrict__ out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t k = (uint64_t)keys[i];
    uint64_t c0 = ~0ull, c1 = ~0ull, c2 = ~0ull;
    if (design == HWAVE_CHAINING) {
      c0 = front_bucket(k, nf);
    } else if (design == HWAVE_ICEBERG || design == HWAVE_ICEBERG_M) {
      const Yard y = yard_of(k, nf, nback);
      c0 = y.front;
      c1 = y.back1;
      c2 = y.back2;
    } else {
      const Hashed h = hash_key(k, mask);
      c0 = h.b1;
      if (design == HWAVE_DOUBLE || design == HWAVE_DOUBLE_M) {
        c1 = (h.h2 & mask) | 1u;  // the probe step
      } else {
        c1 = h.h2 & mask;
        if (design == HWAVE_CUCKOO) c2 = (uint32_t)fmix64(k ^ HASH_SALT_B) & mask;
      }
    }
    out[3 * i] = c0;
    out[3 * i + 1] = c1;
    out[3 * i + 2] = c2;
  }
}

// Grid cap for grid-stride kernels, cached per device (tables may be created
// from several host threads, e.g. beside a serving loop's worker).
unsigned max_blocks_for(int device) {
  static std::atomic<unsigned> cache[64];
  const bool cached = device >= 0 && device < 64;
  if (cached) {
    const unsigned c = cache[device].load(std::memory_order_relaxed);
    if (c) return c;
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0)
    cus = 256;
  const unsigned v = (unsigned)cus * 32;
  if (cached) cache[device].store(v, std::memory_order_relaxed);
  return v;
}

unsigned stream_grid(uint64_t n, int device) {
  uint64_t blocks = (n + 255) / 256;
  uint64_t cap = max_blocks_for(device);
  if (blocks > cap) blocks = cap;
  return (unsigned)(blocks ? blocks : 1);
}

int init_table(hwave_table* t, void* base, uint64_t bytes, const Layout& L, hwave_design design,
               const hwave_config& c, const KernelSet* ks, void* stream) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  t->device = dev;
  t->design = design;
  t->cfg = c;
  t->nb = L.nb;
  t->capacity = L.capacity;
  t->units = L.units;
  t->bytes = bytes;
  t->n_lock_words = L.n_lock_words;
  t->base = base;
  t->ks = ks;
  uint8_t* b = (uint8_t*)base;
  TableDev& tv = t->la.tv;
  tv.slots = b;
  tv.tagw = design_tags(design) ? (uint32_t*)(b + L.off_tags) : nullptr;
  tv.locks.words = (uint32_t*)(b + L.off_locks);
  tv.locks.shift = L.lock_shift;
  tv.lockq = (uint64_t*)(b + L.off_lockq);
  tv.lockq_mask = (uint32_t)(L.n_lockq - 1);
  tv.ctrl = (uint32_t*)(b + L.off_ctrl);
  tv.bucket_mask = (uint32_t)(L.nb - 1);
  tv.nb_front = design_iceberg(design) ? (uint32_t)iceberg_front(L.nb) : (uint32_t)L.nb;
  tv.nb_back = design_iceberg(design) ? (uint32_t)(L.nb - tv.nb_front) : 0u;
  tv.pool_nodes = (uint32_t)L.pool;
  tv.pool_ctr = design_chain(design) ? (uint32_t*)(b + L.off_pool_ctr) : nullptr;
  uint64_t cap = c.probe_cap ? c.probe_cap : L.nb;
  if (cap > L.nb) cap = L.nb;
  tv.probe_cap = (uint32_t)(cap > 0xFFFFFFFFull ? 0xFFFFFFFFull : cap);
  tv.shortcut = (c.flags & HWAVE_F_NO_SHORTCUT) ? 0u : 1u;
  tv.no_erase = (c.flags & HWAVE_F_NO_ERASE) ? 1u : 0u;
  tv.aggregate = (c.flags & HWAVE_F_AGGREGATE) ? 1u : 0u;
  tv.lock_limit = (uint32_t)((c.lock_timeout_us ? c.lock_timeout_us : DEFAULT_LOCK_TIMEOUT_US) * 100ull);
  tv.hot_tag = L.off_hot ? (uint64_t*)(b + L.off_hot) : nullptr;
  tv.hot_acc = L.off_hot ? tv.hot_tag + HOT_N : nullptr;
  t->has_merge = L.off_merge != 0;
  t->ws = MergeWs{};
  if (t->has_merge) {
    uint8_t* m = b + L.off_merge;
    t->ws.key = (uint64_t*)m;
    t->ws.ent = (MergeEntry*)(m + MERGE_ENTRIES * 8);
    t->ws.op_ent = (uint32_t*)(m + MERGE_ENTRIES * (8 + sizeof(MergeEntry)));
    t->ws.ne_mask = (uint32_t)(MERGE_ENTRIES - 1);
    t->ws.chunk = MERGE_CHUNK;
  }
  tv.probe_ctr = nullptr;
#ifdef HW_INSTRUMENT
  {
    const size_t pb = (size_t)PROBE_STRIPES * 16 * sizeof(unsigned long long);
    e = hipMalloc((void**)&tv.probe_ctr, pb);
    if (e != hipSuccess) {
      tv.probe_ctr = nullptr;
      return hip_fail(e);
    }
    hipLaunchKernelGGL(k_fill16, dim3(1), dim3(256), 0, (hipStream_t)stream, (uint4*)tv.probe_ctr, pb / 16, 0u);
  }
#endif
  t->la.max_blocks = max_blocks_for(dev);
  const int rc = hwave_clear(t, stream);
  if (rc && tv.probe_ctr) {
    (void)hipFree(tv.probe_ctr);
    tv.probe_ctr = nullptr;
  }
  return rc;
}

bool bad_ptr(const void* p) { return p == nullptr; }

// Most operations grouped in one go: larger calls run in pieces, one after another in the
// same scratch memory, which so stays bounded (about 50 bytes per operation).  The
// instrumented build has smaller pieces: tests reach their edges there.
#ifndef HW_BULK_CHUNK
#define HW_BULK_CHUNK (1ull << 27)
#endif
constexpr uint64_t BULK_CHUNK = HW_BULK_CHUNK;

// Blocks of k_bulk_write at work at a time: six a CU; and how many fill the chip.
constexpr uint64_t BULK_RESIDENT = 1536;
constexpr uint32_t BULK_FILL = 512;

// Fewest operations of a group's table that are grouped: a block's chain of round trips is
// the same for fewer (400 tables of 2^8 slots, DOUBLE_M, present keys: 33 operations each
// 87 us plain, 106 grouped; 51 104 / 110; 64 123 / 96).
constexpr uint64_t BULK_MIN_MEMBER = 64;

// Fewest operations per configuration for which a group of several is grouped.  Each
// configuration's launches follow the others' (100 to 170 us a configuration however few
// its operations), where one persistent launch runs all together.  Plain against grouped,
// microseconds, 24 tables of 2^20 slots, present keys: nearly all operations on one
// configuration of six, 0.65 M per configuration 773 / 995, 1.3 M 1656 / 1180; on one of four, 0.5 M
// 516 / 667, 1.0 M 799 / 767; evenly on six, 1.26 M 1701 / 841.
constexpr uint64_t GROUP_MIN_CONFIG = 1u << 20;

// Room for a bin that receives `mean` operations on average: seven standard
// deviations of a random spread; keys that are spread worse overflow into the
// per-tile path.
uint32_t bulk_room(double mean) { return (uint32_t)round_up((uint64_t)(mean + 7 * std::sqrt(mean)) + 32, 64); }

// What a plan depends on.
struct BulkShape {
  const KernelSet* ks;
  hwave_design design;
  uint32_t kv_bits, B;  // B: slot units per home bucket
  uint64_t nbh, backs;  // home buckets; iceberg's backyard buckets
  bool stable;          // the table never erases
  bool impatient;       // its writers may not wait for a grouped part's locks
};
// A part's block holds the locks of its buckets while it works on all their operations, where a
// plain writer holds one for one operation.  So tables whose lock_timeout_us is below what a part
// takes keep the plain calls: iceberg's parts place backyard keys with few tiles (ICEBERG, 2^20 slots
// from 0.75 to 0.95 beside small upserts: with 100 us, 744 timed out beside the grouped call, none
// beside the plain one; with 200 none), others' are done in tens of microseconds (plain calls of that
// size time out among themselves with 50).  The lines leave a factor of 20.
constexpr uint32_t BULK_PATIENCE_US = 1000, BULK_PATIENCE_ICEBERG_US = 4000;

BulkShape bulk_shape(const hwave_table* t) {
  const bool iceberg = design_iceberg(t->design);
  const uint64_t patience = (uint64_t)(iceberg ? BULK_PATIENCE_ICEBERG_US : BULK_PATIENCE_US) * 100;  // in ticks
  return BulkShape{t->ks, t->design, t->cfg.kv_bits, design_chain(t->design) ? 8u : t->cfg.bucket_slots,
                   t->la.tv.nb_front, t->la.tv.nb_back, t->la.tv.no_erase != 0,
                   t->la.tv.lock_limit < patience};
}

// What a grouped call does: KEEP upserts are inserts, which mostly bring absent keys.
enum BulkKind { BULK_INSERT, BULK_UPSERT, BULK_ERASE };
BulkKind bulk_kind(int combine) { return combine == HWAVE_KEEP ? BULK_INSERT : BULK_UPSERT; }

// Fewest operations per home slot for which a call is grouped, in percent: where every
// kind of such a call (into an empty table, to loads of 0.85 and 0.95, of present keys;
// erases of present and of absent keys) is within 5% of the plain call or faster, in tables of 2^12
// to 2^25 slots.  Plain against grouped, microseconds, below the line and at it:
//   tags, 32 slots:      inserts and upserts 0.10: 36 / 30 (2^15), 317 / 308 (2^25, present keys)
//   tags, 16 slots:      0.10: DOUBLE_M present 27 / 30 (2^15), P2HT(M) erases of absent keys 21 / 23;
//                        0.13: 32 / 29, 24 / 23
//                        DOUBLE_M with 64-bit keys and tiles of up to 4, from 2^23 buckets on, where the tags are
//                        twice the last-level cache: 32 slots, 2^28, 0.15: present 3758 / 3904, to
//                        0.95 4855 / 5441; 0.20: 4950 / 4445, 6204 / 5653; 16 slots, 2^27, 0.15: to 0.95 2866 /
//                        3152, 0.20: 3592 / 3204 (2^27 of 32 slots 0.15: 1983 / 1905, 2799 / 2666)
//   32-bit keys:         8 slots 0.16: present 25 / 30 (2^15); 0.21: 30 / 29.  16 and more 0.16: 31 / 29
//   64-bit, no tags:     8 slots 0.25: inserts to 0.95 69 / 84 (2^16), present 25 / 30 (2^14), but 2^13
//                        fresh 32 / 27; 0.29: 73 / 73, 28 / 29.  Erases 0.25: absent 30 / 41, 0.29
//                        present 30 / 34 (2^13); 0.33 35 / 35.  16 and more 0.25: P2HT erases 96 / 89 (2^21).
//                        ICEBERG 0.21: upserts of present keys 115 / 43 (2^19)
//   chaining:            erases of absent keys 0.29: 20 / 26 (2^14), 0.37: 24 / 25; upserts walk whole
//                        chains under the lock with one tile: 0.69: 83 / 74 (2^19), inserts to 0.95 86 / 83
uint64_t bulk_min_percent(const BulkShape& t, BulkKind kind) {
  if (design_chain(t.design)) return kind == BULK_ERASE ? 33 : 60;
  if (design_iceberg(t.design)) return design_tags(t.design) ? 10 : 12;
  if (design_tags(t.design)) {
    if (kind != BULK_ERASE && t.kv_bits == 64 && t.ks->tile <= 4 && t.nbh >= 1u << 23) return 20;
    return t.B < 32 ? 13 : 10;
  }
  if (t.kv_bits == 32) return t.B < 16 ? 21 : 16;
  if (t.B >= 16) return 25;
  if (kind == BULK_ERASE) return 32;
  return kind == BULK_INSERT && t.nbh * t.B <= 1u << 13 ? 25 : 29;
}

// Whether an upsert of a table that never erases is grouped.  Its plain upserts of present
// keys take no lock: one look and one atomic, which grouping beats only where several
// operations meet in a key, and where memory or a launch's many tables bound the plain call.
// Plain against grouped, microseconds, present keys unless noted: DOUBLE_M 0.2 operations per
// slot 11 / 30 (2^15), 421 / 576 (2^25); 1.7 per slot 31 / 43 (2^18), 339 / 367 (2^22), 1478 / 1507
// (2^24; fresh 2863 / 1619); CHAINING 1451 / 1720 (2^24).  Groups with 1.7 per slot: 400
// tables of 2^12 slots 294 / 195 (fresh 851 / 203), 40 of 2^10 48 / 50; ICEBERG_M 56 / 77.
bool bulk_stable(const BulkShape& t, uint64_t n, uint64_t call) {
  if (n < t.nbh * t.B || design_iceberg(t.design)) return false;
  return call ? call >= 1u << 17 : !design_chain(t.design) && t.nbh * t.B >= 1u << 24;
}

// How a call of n operations (at most BULK_CHUNK) is grouped (hw_bulk.hpp), or
// false where one tile per operation is better.  `call`: the operations of all tables of a
// group's call, which fill the chip together; 0 for a table's own call.
bool bulk_plan(const BulkShape& t, uint64_t n, BulkKind kind, uint64_t call, BulkPlan* p) {
  const bool member = call != 0;
  const bool erase = kind == BULK_ERASE;
  if (!(erase ? t.ks->bulk_erase : t.ks->bulk_upsert) || t.impatient) return false;
  if (n < (member ? BULK_MIN_MEMBER : BULK_MIN_OPS) || n > BULK_CHUNK) return false;
  const uint32_t B = t.B;
  const uint64_t nbh = t.nbh;
  if (!erase && t.stable && !bulk_stable(t, n, call)) return false;
  if (nbh == 0 || n * 100 < nbh * B * bulk_min_percent(t, kind)) return false;
  const double per_bucket = (double)n / (double)nbh;
  uint32_t shift = 0;
  while ((2u << shift) * B <= (uint32_t)t.ks->bulk_slots) ++shift;
  auto fits = [&](uint32_t sh) { return bulk_room(per_bucket * (double)(1u << sh)) <= (uint32_t)BULK_CAP; };
  // as many buckets as a block takes, but enough blocks to fill the chip
  while (shift > 0 && (!fits(shift) || (!member && ((nbh - 1) >> shift) + 1 < BULK_FILL && per_bucket * (double)(1u << shift) > 256)))
    --shift;
  if (!fits(shift)) return false;
  p->shift = shift;
  p->parts = (uint32_t)(((nbh - 1) >> shift) + 1);
  const double mean = per_bucket * (double)(1u << shift);
  p->cap = bulk_room(mean);
  p->hash_n = 256;
  while (p->hash_n * 2 < p->cap * 3) p->hash_n *= 2;
  // Iceberg inserts: no more tiles choose between two backyard buckets at a time than
  // there are backyard buckets, as in a plain call, where such choices are spread
  // over the call's time.  All at once they meet equal fills and take the first choice
  // (ICEBERG, 2^20 slots filled to 0.9 in one call: 2.91 lines per query with all tiles,
  // 2.95 with the limit, 2.96 plain; 202, 308 and 582 us).  Calls of few blocks, or of few
  // operations for the table, take twice as many tiles (per 32 slots of a bucket): with the limit they were
  // slower than plain calls in nearly full tables (2^15 slots from 0.75 to 0.95: 149 us plain,
  // 188 with the limit, 156 so), and a few choices at a time leave the backyard as even
  // (the standard deviation of its fills is 0.95 in all three).
  p->slow_tiles = BULK_THREADS;
  if (!erase && design_iceberg(t.design)) {
    const uint64_t blocks = std::min<uint64_t>(p->parts, BULK_RESIDENT);
    const bool few = (member ? call < BULK_FILL * 256 : p->parts < BULK_FILL) || n * 4 < nbh * B;
    p->slow_tiles = (uint32_t)std::min<uint64_t>(BULK_THREADS, t.backs * (few ? B / 16 : 1) / blocks + 1);
  }
  p->sub = 0;
  p->levels = p->parts <= (uint32_t)BULK_BINS ? 1 : 2;
  if (p->levels == 2) {
    while ((1u << (2 * p->sub)) < p->parts) ++p->sub;  // both levels about the square root
    p->bins = ((p->parts - 1) >> p->sub) + 1;
    p->cap1 = bulk_room(mean * (double)(1u << p->sub));
  } else {
    p->bins = p->parts;
    p->cap1 = p->cap;
  }
  if ((1u << p->sub) > (uint32_t)BULK_BINS) return false;
  const uint64_t pair = t.kv_bits / 8 * (erase ? 1 : 2);
  const uint64_t room1 = (uint64_t)p->bins * p->cap1, room = p->levels == 2 ? (uint64_t)p->parts * p->cap : 0;
  uint64_t off = 0;
  auto place = [&](uint64_t bytes) {
    const uint64_t at = off;
    off += round_up(bytes, ALIGN);
    return at;
  };
  p->off_cursor1 = place((uint64_t)p->bins * BULK_CSTRIDE * 4);
  p->off_cursor = place(p->levels == 2 ? (uint64_t)p->parts * 4 : 0);
  p->zero_bytes = off;
  p->off_pos1 = place(n * 4);
  p->off_pos = place(p->levels == 2 ? room1 * 4 : 0);
  p->off_rec1 = place(room1 * pair);
  p->off_rec = place(room * pair);
  p->off_stat1 = place(room1);
  p->off_stat = place(room);
  p->bytes = off;
  return room1 < 0xFFFFFFFFull && room < 0xFFFFFFFFull;
}

// Operations per piece of a grouped call, all pieces but the last of the same size.
uint64_t bulk_piece(uint64_t n) {
  const uint64_t pieces = (n + BULK_CHUNK - 1) / BULK_CHUNK;
  return (n + pieces - 1) / pieces;
}

bool upsert_groups(const hwave_table* t, int combine) {
  // tables that merge duplicates keep their own path for what it merges
  return !(t->la.tv.aggregate && combine != HWAVE_REPLACE);
}

// A grouped call, piece by piece; false (nothing enqueued) where the call is not
// grouped or the scratch memory does not hold it.
bool bulk_run(hwave_table* t, bool erase, const void* keys, const void* vals, uint64_t n, int combine, uint8_t* status,
              void* scratch, uint64_t scratch_bytes, hipStream_t s, hipError_t* err) {
  BulkPlan p;
  const uint64_t piece = bulk_piece(n), w = t->cfg.kv_bits / 8;
  if (!scratch || ((uintptr_t)scratch % ALIGN) ||
      !bulk_plan(bulk_shape(t), piece, erase ? BULK_ERASE : bulk_kind(combine), 0, &p) || p.bytes > scratch_bytes)
    return false;
  *err = hipSuccess;
  for (uint64_t at = 0; at < n && *err == hipSuccess; at += piece) {
    const uint64_t m = n - at < piece ? n - at : piece;
    *err = (erase ? t->ks->bulk_erase : t->ks->bulk_upsert)(
        t->la, p, (uint8_t*)scratch, (const uint8_t*)keys + at * w, vals ? (const uint8_t*)vals + at * w : nullptr,
        (uint32_t)m, combine, status ? status + at : nullptr, s);
  }
  return true;
}

}  // namespace

extern "C" {

int hwave_config_default(hwave_design design, hwave_config* out) {
  if (!out || (int)design < HWAVE_DOUBLE || (int)design > HWAVE_CUCKOO) return HWAVE_EINVAL;
  defaults_for(design, 64, out);
  return HWAVE_OK;
}

int hwave_table_bytes(uint64_t capacity, hwave_design design, const hwave_config* cfg, uint64_t* bytes) {
  if (!bytes) return HWAVE_EINVAL;
  hwave_config c;
  int rc = resolve_config(design, cfg, &c);
  if (rc) return rc;
  if (!find_set(c, design)) return HWAVE_EUNSUPPORTED;
  Layout L;
  rc = layout_of(capacity, design, c, &L);
  if (rc) return rc;
  *bytes = L.total;
  return HWAVE_OK;
}

int hwave_create(hwave_table** out, uint64_t capacity, hwave_design design, const hwave_config* cfg,
                 void* stream) {
  if (!out) return HWAVE_EINVAL;
  *out = nullptr;
  hwave_config c;
  int rc = resolve_config(design, cfg, &c);
  if (rc) return rc;
  const KernelSet* ks = find_set(c, design);
  if (!ks) return HWAVE_EUNSUPPORTED;
  Layout L;
  rc = layout_of(capacity, design, c, &L);
  if (rc) return rc;
  void* base = nullptr;
  hipError_t e = hipMalloc(&base, L.total);
  if (e != hipSuccess) {
    g_last_hip_error = (int)e;
    (void)hipGetLastError();
    return HWAVE_ENOMEM;
  }
  hwave_table* t = new hwave_table;
  t->owns = true;
  rc = init_table(t, base, L.total, L, design, c, ks, stream);
  if (rc) {
    (void)hipFree(base);
    delete t;
    return rc;
  }
  *out = t;
  return HWAVE_OK;
}

int hwave_create_in(hwave_table** out, void* d_buffer, uint64_t buffer_bytes, uint64_t capacity,
                    hwave_design design, const hwave_config* cfg, void* stream) {
  if (!out || !d_buffer || ((uintptr_t)d_buffer % ALIGN)) return HWAVE_EINVAL;
  *out = nullptr;
  hwave_config c;
  int rc = resolve_config(design, cfg, &c);
  if (rc) return rc;
  const KernelSet* ks = find_set(c, design);
  if (!ks) return HWAVE_EUNSUPPORTED;
  Layout L;
  rc = layout_of(capacity, design, c, &L);
  if (rc) return rc;
  if (buffer_bytes < L.total) return HWAVE_ENOMEM;
  hwave_table* t = new hwave_table;
  t->owns = false;
  rc = init_table(t, d_buffer, L.total, L, design, c, ks, stream);
  if (rc) {
    delete t;
    return rc;
  }
  *out = t;
  return HWAVE_OK;
}

int hwave_destroy(hwave_table* t) {
  if (!t) return HWAVE_EINVAL;
  drop_groups_of(t);
  hipError_t e = hipDeviceSynchronize();
  int rc = e == hipSuccess ? HWAVE_OK : hip_fail(e);
  if (t->la.tv.probe_ctr) (void)hipFree(t->la.tv.probe_ctr);
  if (t->owns) {
    e = hipFree(t->base);
    if (e != hipSuccess && rc == HWAVE_OK) rc = hip_fail(e);
  }
  delete t;
  return rc;
}

int hwave_clear(hwave_table* t, void* stream) {
  if (!t) return HWAVE_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  // Every region size is a multiple of 256 bytes.  Slots and tags: all-ones
  // (empty); locks and control word: zero.
  const uint64_t fill_end = (uint64_t)((uint8_t*)t->la.tv.locks.words - (uint8_t*)t->base);
  hipLaunchKernelGGL(k_fill16, dim3(stream_grid(fill_end / 16, t->device)), dim3(256), 0, s,
                     (uint4*)t->base, fill_end / 16, 0xFFFFFFFFu);
  const uint64_t zero_bytes = t->bytes - fill_end;
  hipLaunchKernelGGL(k_fill16, dim3(stream_grid(zero_bytes / 16, t->device)), dim3(256), 0, s,
                     (uint4*)t->la.tv.locks.words, zero_bytes / 16, 0u);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_insert(hwave_table* t, const void* d_keys, const void* d_vals, uint64_t n, uint8_t* d_status,
                 void* stream) {
  return hwave_upsert(t, d_keys, d_vals, n, HWAVE_KEEP, d_status, stream);
}

int hwave_upsert(hwave_table* t, const void* d_keys, const void* d_vals, uint64_t n, hwave_combine combine,
                 uint8_t* d_status, void* stream) {
  if (!t || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_keys) || bad_ptr(d_vals)) return HWAVE_EINVAL;
  hipError_t e = t->ks->upsert(t->la, d_keys, d_vals, n, (int)combine, d_status, (hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_write_scratch(const hwave_table* t, hwave_op op, uint64_t n, hwave_combine combine, uint64_t* bytes) {
  if (!t || !bytes || (int)op < HWAVE_OP_INSERT || (int)op > HWAVE_OP_ERASE) return HWAVE_EINVAL;
  BulkPlan p;
  const int comb = op == HWAVE_OP_INSERT ? (int)HWAVE_KEEP : (int)combine;
  const bool grouped = n != 0 && (op == HWAVE_OP_ERASE || upsert_groups(t, comb)) &&
                       bulk_plan(bulk_shape(t), bulk_piece(n), op == HWAVE_OP_ERASE ? BULK_ERASE : bulk_kind(comb), 0, &p);
  *bytes = grouped ? p.bytes : 0;
  return HWAVE_OK;
}

int hwave_upsert_scratch(hwave_table* t, const void* d_keys, const void* d_vals, uint64_t n, hwave_combine combine,
                         uint8_t* d_status, void* d_scratch, uint64_t scratch_bytes, void* stream) {
  if (!t || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_keys) || bad_ptr(d_vals)) return HWAVE_EINVAL;
  hipError_t e;
  if (upsert_groups(t, (int)combine) && bulk_run(t, false, d_keys, d_vals, n, (int)combine, d_status, d_scratch,
                                                 scratch_bytes, (hipStream_t)stream, &e))
    return e == hipSuccess ? HWAVE_OK : hip_fail(e);
  return hwave_upsert(t, d_keys, d_vals, n, combine, d_status, stream);
}

int hwave_erase_scratch(hwave_table* t, const void* d_keys, uint64_t n, uint8_t* d_found, void* d_scratch,
                        uint64_t scratch_bytes, void* stream) {
  if (!t || t->la.tv.no_erase) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_keys)) return HWAVE_EINVAL;
  hipError_t e;
  if (bulk_run(t, true, d_keys, nullptr, n, HWAVE_KEEP, d_found, d_scratch, scratch_bytes, (hipStream_t)stream, &e))
    return e == hipSuccess ? HWAVE_OK : hip_fail(e);
  return hwave_erase(t, d_keys, n, d_found, stream);
}

int hwave_query(hwave_table* t, const void* d_keys, uint64_t n, void* d_vals_out, uint8_t* d_found,
                void* stream) {
  if (!t) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_keys)) return HWAVE_EINVAL;
  hipError_t e = t->ks->query(t->la, d_keys, n, d_vals_out, d_found, (hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_erase(hwave_table* t, const void* d_keys, uint64_t n, uint8_t* d_found, void* stream) {
  if (!t || t->la.tv.no_erase) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_keys)) return HWAVE_EINVAL;
  hipError_t e = t->ks->erase(t->la, d_keys, n, d_found, (hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_mixed(hwave_table* t, const uint8_t* d_ops, const void* d_keys, const void* d_vals, uint64_t n,
                hwave_combine combine, void* d_vals_out, uint8_t* d_status, void* stream) {
  if (!t || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_ops) || bad_ptr(d_keys)) return HWAVE_EINVAL;
  // Values are read only for inserts/upserts; a batch without them may pass NULL,
  // in which case the keys array stands in (never dereferenced for other ops).
  const void* vals = d_vals ? d_vals : d_keys;
  hipError_t e = t->ks->mixed(t->la, d_ops, d_keys, vals, n, (int)combine, d_vals_out, d_status,
                              t->has_merge ? &t->ws : nullptr, (hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

}  // extern "C"

namespace {

// The workspace of hwave_mixed_noalloc: one merge workspace (hw_merge.hpp) for
// chunks of NOALLOC_OPS operations, in a fixed device array that each device
// holds for the life of the process.  In host code `scratch` names a host-side
// stand-in, never the device memory: its device address comes from
// hipGetSymbolAddress, once per device (noalloc_ws), and only that address is
// ever given to kernels.
constexpr uint32_t NOALLOC_OPS = 1u << 18;
constexpr uint64_t NOALLOC_ENTRIES = 2ull * NOALLOC_OPS;
constexpr uint64_t NOALLOC_ZERO_BYTES = NOALLOC_ENTRIES * (8 + sizeof(MergeEntry));  // key words + entries
constexpr uint64_t NOALLOC_BYTES = NOALLOC_ZERO_BYTES + (uint64_t)NOALLOC_OPS * 4;  // + per-op words
static __device__ __align__(256) uint8_t scratch[NOALLOC_BYTES];

std::mutex g_noalloc_mu;
void* g_noalloc_ptr[64];

// Device address of this device's `scratch`, looked up on the first call per
// device (with that device current).  NULL on failure (*err set).
uint8_t* noalloc_base(int device, hipError_t* err) {
  if (device < 0 || device >= 64) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> g(g_noalloc_mu);
  if (!g_noalloc_ptr[device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      *err = e != hipSuccess ? e : hipErrorInvalidSymbol;
      return nullptr;
    }
    g_noalloc_ptr[device] = ptr;
  }
  return (uint8_t*)g_noalloc_ptr[device];
}

}  // namespace

extern "C" {

int hwave_mixed_noalloc(hwave_table* t, const uint8_t* d_ops, const void* d_keys, const void* d_vals, uint64_t n,
                        hwave_combine combine, void* d_vals_out, uint8_t* d_status, void* stream) {
  if (!t || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  if (n > NOALLOC_OPS) return HWAVE_ETOOBIG;
  if (n == 0) return HWAVE_OK;
  if (bad_ptr(d_ops) || bad_ptr(d_keys)) return HWAVE_EINVAL;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return hip_fail(e);
  if (cur != t->device) return HWAVE_EINVAL;  // the table's device must be current
  uint8_t* base = noalloc_base(cur, &e);
  if (!base) return hip_fail(e);
  MergeWs ws;
  ws.key = (uint64_t*)base;
  // entries for this call: twice its operations, as the whole array has for the largest call
  // (20,000 operations: 1.5 MB to clear, not 12.6, 2.4 us, not 4.4)
  uint64_t entries = 1ull << 10;
  while (entries < 2 * n) entries <<= 1;
  ws.ent = (MergeEntry*)(base + entries * 8);
  ws.op_ent = (uint32_t*)(base + NOALLOC_ZERO_BYTES);
  ws.ne_mask = (uint32_t)(entries - 1);
  ws.chunk = NOALLOC_OPS;
  hipStream_t s = (hipStream_t)stream;
  // the array keeps the last call's contents: the entries must start empty (all
  // zero); a fill kernel, not a memset, so the call can be captured in a graph
  const uint64_t zero16 = entries * (8 + sizeof(MergeEntry)) / 16;
  hipLaunchKernelGGL(k_fill16, dim3(stream_grid(zero16, cur)), dim3(256), 0, s, (uint4*)base, zero16, 0u);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  const void* vals = d_vals ? d_vals : d_keys;
  e = t->ks->mixed(t->la, d_ops, d_keys, vals, n, (int)combine, d_vals_out, d_status, &ws, s);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_size(hwave_table* t, uint64_t* d_count, void* stream) {
  if (!t || !d_count) return HWAVE_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(1), 0, s, d_count);
  const unsigned g = stream_grid(t->units, t->device);
  if (t->cfg.kv_bits == 64)
    hipLaunchKernelGGL(k_count<uint64_t>, dim3(g), dim3(256), 0, s, (const uint64_t*)t->base, t->units, d_count);
  else
    hipLaunchKernelGGL(k_count<uint32_t>, dim3(g), dim3(256), 0, s, (const uint32_t*)t->base, t->units, d_count);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_export(hwave_table* t, void* d_keys, void* d_vals, uint64_t* d_count, void* stream) {
  if (!t || !d_keys || !d_vals || !d_count) return HWAVE_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(1), 0, s, d_count);
  const unsigned g = stream_grid((t->units + EXPORT_PER - 1) / EXPORT_PER, t->device);
  if (t->cfg.kv_bits == 64)
    hipLaunchKernelGGL(k_export<uint64_t>, dim3(g), dim3(256), 0, s, (const uint64_t*)t->base, t->units,
                       (uint64_t*)d_keys, (uint64_t*)d_vals, d_count);
  else
    hipLaunchKernelGGL(k_export<uint32_t>, dim3(g), dim3(256), 0, s, (const uint32_t*)t->base, t->units,
                       (uint32_t*)d_keys, (uint32_t*)d_vals, d_count);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

uint64_t hwave_num_buckets(const hwave_table* t) { return t ? t->nb : 0; }
uint64_t hwave_capacity(const hwave_table* t) { return t ? t->capacity : 0; }

int hwave_primary_bucket(hwave_table* t, const void* d_keys, uint64_t n, uint64_t* d_out, void* stream) {
  if (!t || (n && (!d_keys || !d_out))) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  hipStream_t s = (hipStream_t)stream;
  const unsigned g = stream_grid(n, t->device);
  const uint32_t nf = design_iceberg(t->design) || design_chain(t->design) ? t->la.tv.nb_front : 0u;
  if (t->cfg.kv_bits == 64)
    hipLaunchKernelGGL(k_primary<uint64_t>, dim3(g), dim3(256), 0, s, (const uint64_t*)d_keys, n,
                       t->la.tv.bucket_mask, nf, d_out);
  else
    hipLaunchKernelGGL(k_primary<uint32_t>, dim3(g), dim3(256), 0, s, (const uint32_t*)d_keys, n,
                       t->la.tv.bucket_mask, nf, d_out);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_candidate_buckets(hwave_table* t, const void* d_keys, uint64_t n, uint64_t* d_out, void* stream) {
  if (!t || (n && (!d_keys || !d_out))) return HWAVE_EINVAL;
  if (n == 0) return HWAVE_OK;
  hipStream_t s = (hipStream_t)stream;
  const unsigned g = stream_grid(n, t->device);
  const TableDev& tv = t->la.tv;
  if (t->cfg.kv_bits == 64)
    hipLaunchKernelGGL(k_candidates<uint64_t>, dim3(g), dim3(256), 0, s, (const uint64_t*)d_keys, n,
                       (int)t->design, tv.bucket_mask, tv.nb_front, tv.nb_back, d_out);
  else
    hipLaunchKernelGGL(k_candidates<uint32_t>, dim3(g), dim3(256), 0, s, (const uint32_t*)d_keys, n,
                       (int)t->design, tv.bucket_mask, tv.nb_front, tv.nb_back, d_out);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_probe_counters(hwave_table* t, hwave_probe_stats* out, int reset, void* stream) {
  if (!t || !out) return HWAVE_EINVAL;
  memset(out, 0, sizeof *out);
  unsigned long long* d = t->la.tv.probe_ctr;
  if (!d) return HWAVE_EUNSUPPORTED;  // not an instrumented build
  hipStream_t s = (hipStream_t)stream;
  std::vector<unsigned long long> h((size_t)PROBE_STRIPES * 16);
  hipError_t e = hipMemcpyAsync(h.data(), d, h.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e);
  for (uint32_t i = 0; i < PROBE_STRIPES; i++) {
    out->bucket_lines += h[i * 16 + PC_BUCKET];
    out->slot_lines += h[i * 16 + PC_SLOT];
    out->queries += h[i * 16 + PC_QUERY];
    out->writes += h[i * 16 + PC_WRITE];
    out->write_visits += h[i * 16 + PC_VISIT];
  }
  if (reset) {
    hipLaunchKernelGGL(k_fill16, dim3(1), dim3(256), 0, s, (uint4*)d, h.size() * sizeof(unsigned long long) / 16, 0u);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
  }
  return HWAVE_OK;
}

int hwave_raw(const hwave_table* t, hwave_raw_view* out) {
  if (!t || !out) return HWAVE_EINVAL;
  out->slots = t->la.tv.slots;
  out->tags = (uint16_t*)t->la.tv.tagw;
  out->locks = t->la.tv.locks.words;
  out->n_lock_words = t->n_lock_words;
  out->lock_stride = 1u << t->la.tv.locks.shift;
  out->lock_queues = t->la.tv.lockq;
  out->n_lock_queues = (uint64_t)t->la.tv.lockq_mask + 1;
  out->num_buckets = t->nb;
  out->bucket_slots = t->cfg.bucket_slots;
  out->tile = t->cfg.tile;
  out->kv_bits = t->cfg.kv_bits;
  out->design = (uint32_t)t->design;
  out->slot_bytes = t->units * (t->cfg.kv_bits / 4);
  return HWAVE_OK;
}

const char* hwave_strerror(int code) {
  switch (code) {
    case HWAVE_OK: return "ok";
    case HWAVE_EINVAL: return "invalid argument";
    case HWAVE_ENOMEM: return "out of device memory or buffer too small";
    case HWAVE_EDEVICE: return "HIP error (see hwave_last_hip_error)";
    case HWAVE_EUNSUPPORTED: return "no kernel instance for this configuration";
    case HWAVE_EIO: return "file could not be read or written, or is malformed";
    case HWAVE_ETOOBIG: return "batch larger than the allocation-free call's fixed workspace";
  }
  return "unknown error";
}

int hwave_last_hip_error(void) { return g_last_hip_error; }

// ---------------------------------------------------------------- multi-table

}  // extern "C"

struct hwave_multi {
  int device;
  int kv_bits;
  int menu;  // MENU_BASE, MENU_EXT or MENU_SOLO
  int solo;  // menu entry shared by every table (MENU_SOLO), else -1
  bool agg;  // some table merges duplicate keys (64-bit solo kernels: the merging path)
  uint32_t n_tables;
  std::vector<uint64_t> table_bytes;  // footprint per table (queue placement)
  std::vector<BulkShape> shapes;      // per table, for grouped upserts
  std::vector<HomeMap> homes;
  std::vector<uint32_t> order;        // the tables, those of one configuration together
  MultiTable* d_tables = nullptr;
  uint32_t* d_heads = nullptr;
  uint32_t* d_hot = nullptr;  // indices of the tables with hot-key accumulators the kernel fills
  uint32_t n_hot = 0;
  MultiItem* d_items = nullptr;
  size_t items_cap = 0;
  MultiItem* h_stage = nullptr;  // pinned staging of the item list
  size_t stage_cap = 0;
  hipEvent_t staged = nullptr;   // recorded after the last item upload
  bool staged_pending = false;
  unsigned grid = 0;
  std::vector<MultiItem> build;  // host scratch
  std::vector<uint32_t> qcount;
};

namespace {

// Items are split into chunks of at most this many ops so the queues balance big
// tables; the chunk shrinks (down to MULTI_CHUNK_MIN) when a launch has too little
// work to give every wave of the persistent grid several chunks.
constexpr uint64_t MULTI_CHUNK = 16384;
constexpr uint64_t MULTI_CHUNK_MIN = 256;
// A wave works through a chunk one tile-full after the other, so calls of few operations
// get smaller ones (16 tables of 2^20 slots, 8000 queries each: 151 us with 256, 82 with
// 64; 60,000 each 179 with 256, 197 with 117).  Writes only while the chunks put no more tiles
// to work than the table has home buckets: more of them queue longer for its locks
// (40 tables of 2^12 slots, 1.7 operations per slot: 630 us with 256, 761 with 64).
constexpr uint64_t MULTI_CHUNK_LEAST = 64;
// Tables whose footprint fits comfortably in one XCD's L2 keep all their items on
// one queue.
constexpr uint64_t L2_RESIDENT_BYTES = 2ull << 20;

int multi_reserve(hwave_multi* m, size_t n) {
  if (n <= m->items_cap && n <= m->stage_cap) return HWAVE_OK;
  size_t cap = 1024;
  while (cap < n) cap <<= 1;
  hipError_t e = hipDeviceSynchronize();  // the old buffers may still be read by a launch
  if (e != hipSuccess) return hip_fail(e);
  if (m->d_items) (void)hipFree(m->d_items);
  if (m->h_stage) (void)hipHostFree(m->h_stage);
  m->d_items = nullptr;
  m->h_stage = nullptr;
  m->items_cap = m->stage_cap = 0;
  e = hipMalloc(&m->d_items, cap * sizeof(MultiItem));
  if (e != hipSuccess) { g_last_hip_error = (int)e; return HWAVE_ENOMEM; }
  e = hipHostMalloc((void**)&m->h_stage, cap * sizeof(MultiItem), hipHostMallocDefault);
  if (e != hipSuccess) { g_last_hip_error = (int)e; return HWAVE_ENOMEM; }
  m->items_cap = m->stage_cap = cap;
  m->staged_pending = false;
  return HWAVE_OK;
}

}  // namespace

extern "C" {

int hwave_multi_supported(uint32_t kv_bits, hwave_design design, uint32_t bucket_slots, uint32_t tile) {
  for (int menu : {MENU_BASE, MENU_EXT})
    if (multi_menu_index((int)kv_bits, menu, (int)design, (int)bucket_slots, (int)tile) >= 0) return 1;
  return 0;
}

int hwave_multi_create(hwave_multi** out, hwave_table* const* tables, uint32_t n_tables, void* stream) {
  if (!out || !tables || n_tables == 0) return HWAVE_EINVAL;
  *out = nullptr;
  const int kv = (int)tables[0]->cfg.kv_bits;
  const int dev = tables[0]->device;
  // the base menu when it holds every table's configuration, else the extended one
  int menu = MENU_BASE;
  for (uint32_t i = 0; i < n_tables; i++) {
    const hwave_table* t = tables[i];
    if (!t || (int)t->cfg.kv_bits != kv || t->device != dev) return HWAVE_EINVAL;
    if (t->cfg.flags & HWAVE_F_BSP) return HWAVE_EUNSUPPORTED;
    if (multi_menu_index(kv, MENU_BASE, (int)t->design, (int)t->cfg.bucket_slots, (int)t->cfg.tile) < 0)
      menu = MENU_EXT;
  }
  std::vector<MultiTable> h(n_tables);
  for (uint32_t i = 0; i < n_tables; i++) {
    const hwave_table* t = tables[i];
    int cls = multi_menu_index(kv, menu, (int)t->design, (int)t->cfg.bucket_slots, (int)t->cfg.tile);
    if (cls < 0) return HWAVE_EUNSUPPORTED;
    h[i].tv = t->la.tv;
    h[i].cls = (uint32_t)cls;
    h[i].pad = 0;
    const uint64_t locks_off = (uint64_t)((uint8_t*)t->la.tv.locks.words - (uint8_t*)t->base);
    h[i].fill_words = locks_off / 16;
    h[i].zero_words = (t->bytes - locks_off) / 16;
  }
  std::vector<uint32_t> order(n_tables);
  for (uint32_t i = 0; i < n_tables; i++) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return h[a].cls < h[b].cls; });
  // every table on one configuration: that configuration's own kernel (its
  // entry in the 32-bit menu or in the 64-bit extended menu)
  int solo = (int)h[0].cls;
  for (uint32_t i = 1; i < n_tables && solo >= 0; i++)
    if ((int)h[i].cls != solo) solo = -1;
  if (solo >= 0) {
    const hwave_table* t = tables[0];
    solo = multi_menu_index(kv, MENU_SOLO, (int)t->design, (int)t->cfg.bucket_slots, (int)t->cfg.tile);
    if (solo < 0) return HWAVE_EUNSUPPORTED;
    menu = MENU_SOLO;
    for (uint32_t i = 0; i < n_tables; i++) h[i].cls = 0;
  }
  hwave_multi* m = new hwave_multi;
  m->device = dev;
  m->kv_bits = kv;
  m->menu = menu;
  m->solo = solo;
  m->agg = false;
  m->order = std::move(order);
  for (uint32_t i = 0; i < n_tables; i++) m->agg = m->agg || tables[i]->la.tv.aggregate;
  m->n_tables = n_tables;
  for (uint32_t i = 0; i < n_tables; i++) {
    const TableDev& tv = tables[i]->la.tv;
    m->table_bytes.push_back(tables[i]->bytes);
    m->shapes.push_back(bulk_shape(tables[i]));
    m->homes.push_back(HomeMap{tv.bucket_mask, design_iceberg(tables[i]->design) || design_chain(tables[i]->design) ? tv.nb_front : 0u});
  }
  // only the 64-bit menu carries the merging path that fills the accumulators
  std::vector<uint32_t> hot;
  for (uint32_t i = 0; i < n_tables; i++)
    if (kv == 64 && tables[i]->la.tv.hot_tag) hot.push_back(i);
  m->n_hot = (uint32_t)hot.size();
  hipError_t e = hipMalloc(&m->d_tables, n_tables * sizeof(MultiTable));
  if (e == hipSuccess && m->n_hot) e = hipMalloc(&m->d_hot, m->n_hot * sizeof(uint32_t));
  if (e == hipSuccess && m->n_hot)
    e = hipMemcpyAsync(m->d_hot, hot.data(), m->n_hot * sizeof(uint32_t), hipMemcpyHostToDevice,
                       (hipStream_t)stream);
  if (e == hipSuccess) e = hipMalloc(&m->d_heads, NQ * HEAD_STRIDE * sizeof(uint32_t));
  if (e == hipSuccess) e = hipMemcpyAsync(m->d_tables, h.data(), n_tables * sizeof(MultiTable),
                                          hipMemcpyHostToDevice, (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&m->staged, hipEventDisableTiming);
  if (e != hipSuccess) {
    hwave_multi_destroy(m);
    return hip_fail(e);
  }
  // Persistent grid: full occupancy of the multi-table kernel.
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
  m->grid = (unsigned)cus * (4 * multi_waves(kv, menu, solo, m->agg) * 64 / BLOCK);
  *out = m;
  return HWAVE_OK;
}

int hwave_multi_kernel(const hwave_multi* m, uint32_t* kernel, uint32_t* waves) {
  if (!m) return HWAVE_EINVAL;
  static_assert(HWAVE_MULTI_MENU == MENU_BASE && HWAVE_MULTI_EXTENDED == MENU_EXT && HWAVE_MULTI_SOLO == MENU_SOLO,
                "kernel codes");
  if (kernel) *kernel = (uint32_t)m->menu;
  if (waves) *waves = (uint32_t)multi_waves(m->kv_bits, m->menu, m->solo, m->agg);
  return HWAVE_OK;
}

int hwave_multi_destroy(hwave_multi* m) {
  if (!m) return HWAVE_EINVAL;
  (void)hipDeviceSynchronize();
  if (m->d_tables) (void)hipFree(m->d_tables);
  if (m->d_heads) (void)hipFree(m->d_heads);
  if (m->d_hot) (void)hipFree(m->d_hot);
  if (m->d_items) (void)hipFree(m->d_items);
  if (m->h_stage) (void)hipHostFree(m->h_stage);
  if (m->staged) (void)hipEventDestroy(m->staged);
  delete m;
  return HWAVE_OK;
}

int hwave_multi_run(hwave_multi* m, const hwave_item* h_items, uint32_t n_items, const void* d_keys,
                    const void* d_vals, void* d_vals_out, uint8_t* d_status, void* stream) {
  if (!m || (n_items && (!h_items || !d_keys))) return HWAVE_EINVAL;
  if (n_items == 0) return HWAVE_OK;
  // Split items into chunks and deal them to queues: small tables to queue
  // table % NQ, big tables' chunks round-robin over all queues.
  m->build.clear();
  std::vector<std::vector<MultiItem>> per_q(NQ);
  uint32_t rr = 0;
  uint64_t total_ops = 0;
  bool merging = false;  // an upsert whose combine merges (it may fill hot-key accumulators)
  for (uint32_t i = 0; i < n_items; i++)
    if (h_items[i].end > h_items[i].begin) total_ops += h_items[i].end - h_items[i].begin;
  const uint64_t waves = (uint64_t)m->grid * (BLOCK / 64);
  uint64_t chunk = total_ops / (4 * waves);
  if (chunk > MULTI_CHUNK) chunk = MULTI_CHUNK;
  const uint64_t least = std::max(chunk, std::min(MULTI_CHUNK_MIN, std::max(MULTI_CHUNK_LEAST, 4 * total_ops / waves)));
  if (chunk < MULTI_CHUNK_MIN) chunk = MULTI_CHUNK_MIN;
  for (uint32_t i = 0; i < n_items; i++) {
    const hwave_item& it = h_items[i];
    if (it.table >= m->n_tables || it.end < it.begin) return HWAVE_EINVAL;
    const int op = (int)(it.op & 0xFF);
    if (op > HWAVE_OP_ERASE || ((it.op >> 8) & 0xFF) > HWAVE_MAX) return HWAVE_EINVAL;
    if ((op == HWAVE_OP_INSERT || op == HWAVE_OP_UPSERT) && !d_vals) return HWAVE_EINVAL;
    const int comb = (int)((it.op >> 8) & 0xFF);
    if (op == HWAVE_OP_UPSERT && (comb == HWAVE_SUM || comb == HWAVE_MIN || comb == HWAVE_MAX)) merging = true;
    const bool small = m->table_bytes[it.table] <= L2_RESIDENT_BYTES;
    uint64_t step = least;
    if (op != HWAVE_OP_QUERY)
      step = std::min(std::max(least, 16 * (it.end - it.begin) / std::max<uint64_t>(1, m->shapes[it.table].nbh)), std::max(least, chunk));
    for (uint64_t b = it.begin; b < it.end; b += step) {
      MultiItem c;
      c.table = it.table;
      c.op = it.op;
      c.begin = b;
      c.end = b + step < it.end ? b + step : it.end;
      const uint32_t q = small ? it.table % NQ : (rr++ % NQ);
      per_q[q].push_back(c);
    }
  }
  size_t total = 0;
  for (auto& v : per_q) total += v.size();
  if (total == 0) return HWAVE_OK;
  if (total > 0xFFFFFFFFull) return HWAVE_EINVAL;
  int rc = multi_reserve(m, total);
  if (rc) return rc;
  // the staging buffer may still be in flight from the previous call
  if (m->staged_pending) {
    hipError_t e = hipEventSynchronize(m->staged);
    if (e != hipSuccess) return hip_fail(e);
  }
  MultiQueues qs;
  size_t at = 0;
  for (int q = 0; q < NQ; q++) {
    qs.start[q] = (uint32_t)at;
    memcpy(m->h_stage + at, per_q[q].data(), per_q[q].size() * sizeof(MultiItem));
    at += per_q[q].size();
    qs.end[q] = (uint32_t)at;
  }
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(m->d_items, m->h_stage, total * sizeof(MultiItem), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipEventRecord(m->staged, s);
  if (e != hipSuccess) return hip_fail(e);
  m->staged_pending = true;
  // Two waves per item where that is fewer than the chip holds: every wave looks at every
  // queue's head before it ends, and one address serves ~80 M atomics a second (2560
  // queries on 10 tables: 143 us with the whole grid, 29 so).
  const unsigned grid = (unsigned)std::min<uint64_t>(m->grid, (2 * total + BLOCK / 64 - 1) / (BLOCK / 64));
  e = launch_multi(m->kv_bits, m->menu, m->solo, m->agg, grid, m->d_tables, m->d_items, qs, m->d_heads, d_keys,
                   d_vals ? d_vals : d_keys, d_vals_out, d_status, s);
  if (e == hipSuccess && merging) e = launch_multi_hot_flush(m->kv_bits, m->d_tables, m->d_hot, m->n_hot, s);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_multi_clear(hwave_multi* m, void* stream) {
  if (!m) return HWAVE_EINVAL;
  const unsigned grid = m->n_tables < 4096 ? m->n_tables : 4096;
  hipError_t e = launch_multi_clear(grid, m->d_tables, m->n_tables, (hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

int hwave_multi_upsert(hwave_multi* m, const uint64_t* h_offsets, const void* d_keys, const void* d_vals,
                       hwave_combine combine, uint8_t* d_status, void* stream) {
  if (!m || !h_offsets || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  std::vector<hwave_item> items;
  items.reserve(m->n_tables);
  for (uint32_t i = 0; i < m->n_tables; i++) {
    if (h_offsets[i + 1] < h_offsets[i]) return HWAVE_EINVAL;
    if (h_offsets[i + 1] == h_offsets[i]) continue;
    items.push_back(hwave_item{i, (uint32_t)HWAVE_OP_UPSERT | ((uint32_t)combine << 8), h_offsets[i],
                               h_offsets[i + 1]});
  }
  return hwave_multi_run(m, items.data(), (uint32_t)items.size(), d_keys, d_vals, nullptr, d_status, stream);
}

}  // extern "C"

namespace {

// A group's upsert, grouped by bucket (hw_bulk.hpp), as runs of tables of one
// configuration and at most BULK_CHUNK operations (a larger table in pieces): one after
// another on the stream, all in the same scratch memory.
struct GroupRun {
  const KernelSet* ks;
  size_t job;                 // first of its jobs
  uint32_t n;                 // jobs
  size_t list;                // offset of its list in the staging buffer: jobs, then `first`
  std::vector<uint32_t> first;  // per step, the blocks before each job's
  GroupArgs args;
  size_t first_at() const { return round_up(n * sizeof(BulkJob), ALIGN); }
  size_t list_bytes() const { return first_at() + round_up(first.size() * 4, ALIGN); }
};
struct GroupPlan {
  std::vector<BulkJob> jobs;
  std::vector<GroupRun> runs;
  uint64_t bytes = 0;  // scratch memory: the largest run's
  size_t staged = 0;   // bytes of all runs' lists
};

// Lays out a run's lists, blocks and scratch memory; false for more blocks than a launch takes.
bool group_run_layout(GroupPlan* g, GroupRun* r) {
  const uint32_t n = r->n;
  r->first.assign((size_t)GROUP_STEPS * n, 0);
  uint64_t at = r->list_bytes(), blocks[GROUP_STEPS] = {};
  constexpr uint64_t TILE = (uint64_t)BULK_SPLIT_THREADS * GROUP_PER;
  for (uint32_t i = 0; i < n; i++) {
    BulkJob& j = g->jobs[r->job + i];
    const BulkPlan& p = j.plan;
    const bool on = p.levels != 0, two = p.levels == 2;
    const uint64_t step[GROUP_STEPS] = {on ? (p.zero_bytes + GROUP_ZERO_BYTES - 1) / GROUP_ZERO_BYTES : 0,
                                        on ? (j.n + TILE - 1) / TILE : 0,
                                        two ? p.bins * ((p.cap1 + TILE - 1) / TILE) : 0,
                                        on ? p.parts : 0,
                                        two ? (uint64_t)p.bins * ((p.cap1 + 255) / 256) : 0,
                                        ((uint64_t)j.n + GROUP_FINISH_OPS - 1) / GROUP_FINISH_OPS};
    for (int k = 0; k < GROUP_STEPS; k++) {
      r->first[(size_t)k * n + i] = (uint32_t)blocks[k];
      blocks[k] += step[k];
    }
    j.scratch = at;
    at += p.bytes;
  }
  for (int k = 0; k < GROUP_STEPS; k++) {
    // a launch takes fewer than 2^32 threads
    if (blocks[k] >= (1ull << 32) / BULK_SPLIT_THREADS) return false;
    r->args.blocks[k] = (uint32_t)blocks[k];
  }
  r->list = g->staged;
  g->staged += r->list_bytes();
  g->bytes = std::max(g->bytes, at);
  return true;
}

// The runs of a call; false where one tile per operation is better: few operations, or
// most of them in tables that get too few.
//
// One tile per operation against grouped, microseconds, 32-bit DOUBLE tables filled to
// 0.85: 40 of 2^12 slots 360 / 65, 400 of 2^10 370 / 129, 4 of 2^20 658 / 216, 20 of 2^20 with 1.7
// operations per slot 5125 / 1714; ICEBERG_M, 64-bit, 10 of 2^13 564 / 125, 20 of 2^20 5265 / 2041.
bool group_plan(const hwave_multi* m, const uint64_t* offsets, int combine, GroupPlan* g) try {
  if (m->agg && combine != HWAVE_REPLACE) return false;
  uint64_t total = 0, grouped = 0;
  for (uint32_t i = 0; i < m->n_tables; i++) {
    if (offsets[i + 1] < offsets[i]) return false;
    total += offsets[i + 1] - offsets[i];
  }
  if (total < BULK_MIN_OPS) return false;
  auto ops = [&](uint32_t at) { return offsets[m->order[at] + 1] - offsets[m->order[at]]; };
  uint64_t configs = 0;
  for (uint32_t at = 0, end; at < m->n_tables; at = end) {  // tables of one configuration
    const KernelSet* ks = m->shapes[m->order[at]].ks;
    uint64_t call = 0, in_run = 0;
    for (end = at; end < m->n_tables && m->shapes[m->order[end]].ks == ks; end++) call += ops(end);
    if (call == 0) continue;
    if (!ks->group_upsert) return false;
    ++configs;
    for (uint32_t k = at; k < end; k++) {
      const uint32_t i = m->order[k];
      const uint64_t n = ops(k);
      if (n == 0) continue;
      const uint64_t piece = bulk_piece(n);
      BulkPlan plan{};
      if (bulk_plan(m->shapes[i], piece, bulk_kind(combine), call, &plan)) grouped += n;
      else plan = BulkPlan{};
      for (uint64_t from = 0; from < n; from += piece) {
        BulkJob j{};
        j.plan = plan;
        j.home = m->homes[i];
        j.table = i;
        j.n = (uint32_t)std::min(piece, n - from);
        j.begin = offsets[i] + from;
        if (in_run == 0 || in_run + j.n > BULK_CHUNK) {
          g->runs.push_back(GroupRun{ks, g->jobs.size(), 0, 0, {}, {}});
          in_run = 0;
        }
        in_run += j.n;
        g->runs.back().n++;
        g->jobs.push_back(j);
      }
    }
  }
  if (configs > 1 && total < configs * GROUP_MIN_CONFIG) return false;
  if (2 * grouped < total) return false;
  for (GroupRun& r : g->runs)
    if (!group_run_layout(g, &r)) return false;
  return true;
} catch (const std::bad_alloc&) {
  return false;
}

}  // namespace

extern "C" {

int hwave_multi_scratch(const hwave_multi* m, const uint64_t* h_offsets, hwave_combine combine, uint64_t* bytes) {
  if (!m || !h_offsets || !bytes || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  GroupPlan g;
  *bytes = group_plan(m, h_offsets, (int)combine, &g) ? g.bytes : 0;
  return HWAVE_OK;
}

int hwave_multi_upsert_scratch(hwave_multi* m, const uint64_t* h_offsets, const void* d_keys, const void* d_vals,
                               hwave_combine combine, uint8_t* d_status, void* d_scratch, uint64_t scratch_bytes,
                               void* stream) {
  if (!m || !h_offsets || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX) return HWAVE_EINVAL;
  GroupPlan g;
  if (!d_scratch || (uintptr_t)d_scratch % ALIGN || bad_ptr(d_keys) || bad_ptr(d_vals) ||
      !group_plan(m, h_offsets, (int)combine, &g) || g.bytes > scratch_bytes)
    return hwave_multi_upsert(m, h_offsets, d_keys, d_vals, combine, d_status, stream);
  // The lists go to the scratch buffer through the staging buffer, which may still be
  // in flight from the previous call.
  const int rc = multi_reserve(m, g.staged / sizeof(MultiItem) + 1);
  if (rc) return rc;
  hipError_t e = m->staged_pending ? hipEventSynchronize(m->staged) : hipSuccess;
  hipStream_t s = (hipStream_t)stream;
  uint8_t* scratch = (uint8_t*)d_scratch;
  for (size_t i = 0; i < g.runs.size() && e == hipSuccess; i++) {
    GroupRun& r = g.runs[i];
    uint8_t* stage = (uint8_t*)m->h_stage + r.list;
    memcpy(stage, &g.jobs[r.job], r.n * sizeof(BulkJob));
    memcpy(stage + r.first_at(), r.first.data(), r.first.size() * 4);
    e = hipMemcpyAsync(scratch, stage, r.list_bytes(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipEventRecord(m->staged, s);
    m->staged_pending = true;
    r.args.g = BulkGroup{(const BulkJob*)scratch, (const uint32_t*)(scratch + r.first_at()), r.n, scratch};
    r.args.tables = m->d_tables;
    if (e == hipSuccess)
      e = r.ks->group_upsert(r.args, &g.jobs[r.job], d_keys, d_vals, (int)combine, d_status, s);
  }
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

}  // extern "C"

namespace {

// Groups made by hwave_multi_upsert_tables, one per distinct table list, kept
// until one of their tables is destroyed.
std::mutex g_groups_mu;
std::vector<std::pair<std::vector<hwave_table*>, hwave_multi*>> g_groups;

}  // namespace

// Called by hwave_destroy: groups that hold `t` go with it.
static void drop_groups_of(hwave_table* t) {
  std::lock_guard<std::mutex> g(g_groups_mu);
  for (size_t i = 0; i < g_groups.size();) {
    const auto& v = g_groups[i].first;
    if (std::find(v.begin(), v.end(), t) != v.end()) {
      hwave_multi_destroy(g_groups[i].second);
      g_groups.erase(g_groups.begin() + (long)i);
    } else {
      ++i;
    }
  }
}

extern "C" {

int hwave_multi_upsert_tables(hwave_table* const* tables, uint32_t n_tables, const uint64_t* d_offsets,
                              const void* d_keys, const void* d_vals, hwave_combine combine, uint8_t* d_status,
                              void* stream) {
  if (!tables || n_tables == 0 || !d_offsets || (int)combine < HWAVE_SUM || (int)combine > HWAVE_MAX)
    return HWAVE_EINVAL;
  std::vector<hwave_table*> key(tables, tables + n_tables);
  hwave_multi* m = nullptr;
  {
    std::lock_guard<std::mutex> g(g_groups_mu);
    for (auto& e : g_groups)
      if (e.first == key) m = e.second;
    if (!m) {
      const int rc = hwave_multi_create(&m, tables, n_tables, stream);
      if (rc) return rc;
      g_groups.emplace_back(key, m);
    }
  }
  std::vector<uint64_t> h(n_tables + 1);
  hipError_t e = hipMemcpyAsync(h.data(), d_offsets, h.size() * sizeof(uint64_t), hipMemcpyDeviceToHost,
                                (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e);
  if (h[0] != 0) return HWAVE_EINVAL;
  return hwave_multi_upsert(m, h.data(), d_keys, d_vals, combine, d_status, stream);
}

int hwave_stream_sync(void* stream) {
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  return e == hipSuccess ? HWAVE_OK : hip_fail(e);
}

}  // extern "C"

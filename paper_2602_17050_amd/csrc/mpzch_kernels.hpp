// Device code of the MPZCH batched remap for gfx950 (wave64).
//
// Kernel sequence of one training remap (paper Sec. 3.2 / Algorithm 1, Sec. 3.4, Sec. 3.6):
//   k_discover   Pass 1 for every position.  An 8-lane group reads the aligned block of 8 slots
//                that holds the id's home slot with one coalesced access; ids and results travel
//                between the id's lane and the lanes that load for it through LDS (probe_first);
//                the few ids whose window continues are parked in LDS and scanned 8 slots at
//                a time.  Hits store metadata = step and the output slot.  (k_lookup is the
//                same body without writes, k_discover_tables / k_lookup_tables the bodies for
//                several tables, k_discover_records the one for a table of 16-byte records,
//                k_discover_tables_chunk a shorter one for groups of small batches.)  Each
//                wavefront owns a contiguous range of positions (a segment) and appends the
//                positions that missed to its segment's list; at the end it enters them into a
//                scratch hash set that elects, per distinct missed id, the position of its first
//                occurrence (input de-duplication of the ids that must allocate).
//   k_allocate   the elected positions claim slots.  A claim is a 64-bit atomic min of a tag
//                (round, first position) into the identities word, so a slot always ends up
//                with the claimant of the lowest (round, position); a claimant that is
//                displaced is carried on by the displacing lane from its next round.  The
//                fixed point is the unique stable assignment, the same one a sequential
//                round-major / position-minor sweep produces.  The outcomes are counted here.
//   k_finalize   every listed position finds the slot that carries its id's claim; the elected one
//                replaces the tag by the id, sets the metadata and reports evicted slots; ids
//                without a claim fall back to home.  The scratch set entries that were used are
//                emptied again; a workgroup of its own publishes the call's counters meanwhile.
// k_allocate / k_finalize work with one lane per claimant.  Tables under the LRU policy allocate in
// k_allocate_lru (a group of lanes per claimant) or k_allocate_lru_long (probe ranges beyond 64 slots).
//
// No kernel funnels work through one hot address: an atomic on a single address costs about
// 12 ns on this GPU however many lanes it serves, so miss lists are per wavefront (no shared
// cursor), counters are accumulated per workgroup and added to one of several copies, and evicted
// slots are staged in LDS and appended with one reservation per workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace mpzch {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxTables = 64;
constexpr int kDies = 8;               // the dies of the GPU, each with an L2 of its own, take the workgroups of a launch in turn
constexpr int kStatCount = 9;
constexpr int kEvBuf = 256;            // evicted slots staged per wavefront before a flush

enum Stat { kHitPos = 0, kMissPos, kDistinctMiss, kInserts, kEvictions, kCollisions, kInvalidPos, kHitProbeSum, kMissProbeSum };

struct TableDesc {
    int64_t *I;            // identities
    int32_t *M;            // metadata (last-seen step)
    int64_t N;             // slots
    uint64_t seed;
    int32_t P;             // min(max_probe, N)
    int32_t ttl;
    int32_t evict;         // 0 = off, 1 = TTL (metadata = last-seen step), 2 = LRU, 3 = TTL with metadata = expiry step
    int32_t sh;            // 0: identities and metadata are two dense tensors; 1: one tensor of 16-byte records
                           // {int64 id; int32 metadata; int32 unused}, I = &record[0].id, M = &record[0].metadata
    int64_t ev_begin;      // where this table's evicted list starts in out_evicted
    int64_t ev_cap;
};

// Counters of one call.  Every workgroup adds its partial counts once, into one of kBins copies of the
// counters chosen by its index: an atomic on ONE address costs about 12 ns whatever it adds, so a
// few thousand workgroups on one address would take longer than the kernel, spread over kBins addresses
// they vanish in it.  Pass 1 and the allocation count; a workgroup of k_finalize sums the copies, publishes the
// totals and clears them (publish_counters), while the others work: the counters are zero between calls (so a captured
// launch sequence can be replayed).
constexpr int kBins = 16;
// One table: k_allocate's wavefronts, workgroups of one, have this many times as many copies, the other tables' counters.
constexpr int kSpread = 8;
struct Control {
    unsigned long long num_evicted[kMaxTables];       // k_finalize: how much of the evicted lists is taken (cleared by the allocation)
    unsigned long long stats[kBins][kMaxTables][kStatCount];
    unsigned long long done;       // counting lookups: workgroups that have finished
};
// Workgroups of 16 wavefronts: at 12 ns each the reservations of 2 048 workgroups of four took 25 us, however little
// there was to do (batch of 700 K positions 35 -> 19 us).
constexpr int kFinalizeBlock = 1024;
constexpr int kFinalizeWaves = kFinalizeBlock / kWave;
constexpr int kFinalizeExtra = 1;      // workgroups of k_finalize beside those that walk the lists

struct Params {
    const int64_t *ids;
    const int32_t *ttls;           // evict == 3: retention of every position's feature, or null (= the table's ttl)
    int64_t n;
    int32_t step;
    int32_t num_tables;            // 1 => t0 is used and offsets/descs are ignored
    int64_t *out_slots;
    uint8_t *out_found;            // lookup only, may be null
    // scratch.  Segment s (one wavefront of k_discover) covers the 64-position chunks
    // [s * seg_chunks, (s + 1) * seg_chunks); its missed positions are list[s * seg_chunks * 64 + k]
    // for k < seg_cnt[s]; ent, list_id and first_of run parallel to list.
    uint32_t *list;
    uint32_t *ent;                 // entry of the position's id in the scratch set
    int64_t *list_id;              // the position's id (read back in one piece: in the batch it is one of a line of sixteen)
    uint32_t *first_of;            // position of the first occurrence of the position's id
    uint8_t *hint;                 // by batch position: round at which k_allocate placed the claim of the id
                                   // elected there (written for elected positions only)
    uint32_t *seg_cnt;
    // one chunk per wavefront (mpzch_chunk_kernels.hpp): by batch position, where the claim of the id elected there
    // ended up; by workgroup, the slots evicted by its claimants; and three words of counters per workgroup
    uint32_t *place;
    uint8_t *note;                 // ... by batch position, 0 between calls: 1 = somebody else has met the id that was entered
                                   // in the scratch set for it (also where lists are kept, of one table; of groups: that the
                                   // claim made there was displaced)
    int64_t *evicted;
    uint64_t *wg_words;
    int32_t seg_chunks;
    int32_t num_segs;
    int32_t short_shift;           // k_lookup_short: a wavefront takes 64 >> short_shift ids
    int32_t front_shift;           // the first try of the scratch set is made in the front 1 / 2^front_shift of it (set_insert)
    uint32_t *set_slot;            // scratch hash set of batch positions, empty = 0xFFFFFFFF
    Control *ctl;
    // several tables
    const TableDesc *descs;        // device array [num_tables]
    const int64_t *offsets;        // device array [num_tables + 1]
    TableDesc t0;
    // lookup fused with the embedding gather: out[pos, :] <- rows[slot mod num_rows, :]
    const char *g_rows;
    char *g_out;
    int64_t g_num_rows;
    int64_t g_stride;              // bytes between rows
    int32_t g_chunks;              // 16-byte (g_wide) or 4-byte pieces per row
    int32_t g_wide;
    int32_t all_records;           // several tables: every one of them is kept as records
    int32_t g_shift;               // log2(g_chunks) when that is a power of two, else -1
    // training remap that also resets the rows of the slots it evicts (one table; geometry in g_num_rows,
    // g_stride, g_chunks, g_wide, g_shift): rows[slot mod num_rows, :] <- init row, or zero bits
    char *r_rows;
    const void *r_init;
    // outputs
    int64_t *out_evicted;
    int64_t *out_num_evicted;
    int64_t *out_stats;
};

// What the kernel of a lookup gets.  The runtime writes the arguments of a launch into device memory, and beyond 112 bytes
// that takes the host 0.7 to 1 us longer (3.0 to 3.5 instead of 2.3 to 2.8): a small lookup is bound by it.
struct LookupBatch {
    const int64_t *ids;
    int64_t *out_slots;
    uint8_t *out_found;
    int32_t n;                     // (at most 2^30)
    int32_t spread;                // Params::short_shift, or Params::seg_chunks
};
struct LookupTable {
    int64_t *I;
    int64_t N;
    uint64_t seed;
    int32_t P;
    int32_t sh;
};
struct LookupTables {
    const TableDesc *descs;
    const int64_t *offsets;
    int32_t num_tables;
};
struct LookupRows {
    const char *rows;
    char *out;
    int64_t num_rows;
    int64_t stride;
    int32_t chunks;
    int16_t wide;
    int16_t shift;
};
struct Nothing {};
template <bool MULTI, bool GATHER>
struct LookupArgs {
    LookupBatch batch;
    std::conditional_t<MULTI, LookupTables, LookupTable> tables;
    std::conditional_t<GATHER, LookupRows, Nothing> rows;
};
static_assert(sizeof(LookupArgs<false, true>) <= 112 && sizeof(LookupArgs<true, true>) <= 112, "see above");

template <bool MULTI, bool GATHER>
inline LookupArgs<MULTI, GATHER> lookup_args(const Params &p, int32_t spread)
{
    LookupArgs<MULTI, GATHER> a{};
    a.batch = {p.ids, p.out_slots, p.out_found, (int32_t)p.n, spread};
    if constexpr (MULTI) a.tables = {p.descs, p.offsets, p.num_tables};
    else a.tables = {p.t0.I, p.t0.N, p.t0.seed, p.t0.P, p.t0.sh};
    if constexpr (GATHER) a.rows = {p.g_rows, p.g_out, p.g_num_rows, p.g_stride, p.g_chunks, (int16_t)p.g_wide, (int16_t)p.g_shift};
    return a;
}
template <bool MULTI, bool GATHER>
__device__ __forceinline__ Params lookup_params(const LookupArgs<MULTI, GATHER> &a)
{
    Params p{};
    p.ids = a.batch.ids;
    p.out_slots = a.batch.out_slots;
    p.out_found = a.batch.out_found;
    p.n = a.batch.n;
    p.short_shift = p.seg_chunks = a.batch.spread;
    p.num_tables = 1;
    if constexpr (MULTI) {
        p.descs = a.tables.descs;
        p.offsets = a.tables.offsets;
        p.num_tables = a.tables.num_tables;
    } else {
        p.t0.I = a.tables.I;
        p.t0.N = a.tables.N;
        p.t0.seed = a.tables.seed;
        p.t0.P = a.tables.P;
        p.t0.sh = a.tables.sh;
    }
    if constexpr (GATHER) {
        p.g_rows = a.rows.rows;
        p.g_out = a.rows.out;
        p.g_num_rows = a.rows.num_rows;
        p.g_stride = a.rows.stride;
        p.g_chunks = a.rows.chunks;
        p.g_wide = a.rows.wide;
        p.g_shift = a.rows.shift;
    }
    return p;
}

// ------------------------------------------------------------------ arithmetic
__device__ __forceinline__ uint64_t mix64(uint64_t x)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t hash_of(int64_t id, uint64_t seed) { return mix64((uint64_t)id ^ seed); }
__device__ __forceinline__ int64_t home_of(uint64_t hash, int64_t n_slots) { return (int64_t)__umul64hi(hash, (uint64_t)n_slots); }
__device__ __forceinline__ int64_t home_slot(int64_t id, uint64_t seed, int64_t n_slots) { return home_of(hash_of(id, seed), n_slots); }

// Claim tags live in the identities word while a call is in flight.  They are below every
// valid id and below the empty marker, and a smaller tag is a better claim.
constexpr uint64_t kTagBase = 0x8000000000000000ull;
constexpr int kTagRoundShift = 33;

__device__ __forceinline__ int64_t make_tag(uint32_t round, uint32_t pos, uint32_t was_occupied)
{
    return (int64_t)(kTagBase | ((uint64_t)round << kTagRoundShift) | ((uint64_t)pos << 1) | was_occupied);
}
__device__ __forceinline__ bool is_tag(int64_t v) { return v < -1; }
__device__ __forceinline__ uint32_t tag_pos(int64_t v) { return (uint32_t)(((uint64_t)v >> 1) & 0xFFFFFFFFull); }
__device__ __forceinline__ uint32_t tag_round(int64_t v) { return (uint32_t)(((uint64_t)v & ~kTagBase) >> kTagRoundShift); }
__device__ __forceinline__ uint32_t tag_occ(int64_t v) { return (uint32_t)((uint64_t)v & 1u); }

// Under the LRU policy claims rank by the number of the choice.  The round, which tells a displaced claimant's home slot, is kept
// below the position.
constexpr int kLruRoundBits = 11, kLruPosShift = 1 + kLruRoundBits, kLruChoiceShift = kLruPosShift + 32;
static_assert(MPZCH_MAX_PROBE_LRU <= 1 << kLruRoundBits, "rounds (and choices, of which a window has no more) fit an LRU claim tag");
static_assert(MPZCH_MAX_BATCH <= (int64_t)1 << 32, "positions fit an LRU claim tag");
__device__ __forceinline__ int64_t make_lru_tag(uint32_t choice, uint32_t pos, uint32_t round, uint32_t was_occupied)
{
    return (int64_t)(kTagBase | ((uint64_t)choice << kLruChoiceShift) | ((uint64_t)pos << kLruPosShift) | (round << 1 | was_occupied));
}
__device__ __forceinline__ uint32_t lru_tag_pos(int64_t v) { return (uint32_t)((uint64_t)v >> kLruPosShift); }
__device__ __forceinline__ uint32_t lru_tag_choice(int64_t v) { return (uint32_t)(((uint64_t)v & ~kTagBase) >> kLruChoiceShift); }
__device__ __forceinline__ uint32_t lru_tag_round(int64_t v) { return (uint32_t)v >> 1 & ((1u << kLruRoundBits) - 1u); }

__device__ __forceinline__ int64_t shfl64(int64_t v, int src)
{
    int lo = __shfl((int)(uint32_t)(uint64_t)v, src);
    int hi = __shfl((int)(uint32_t)((uint64_t)v >> 32), src);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
// This wavefront's number in the workgroup, in a scalar register: what follows from it (segments, chunks, loop ends) then
// costs scalar instructions, and the loops are branches instead of masks.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)); }
// how many of the lanes below this one are in the mask
__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// table owning position pos (largest f with offsets[f] <= pos)
__device__ __forceinline__ int find_table(const int64_t *offsets, int num_tables, int64_t pos)
{
    int lo = 0, hi = num_tables - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (offsets[mid] <= pos) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The same for a position that is the same in every lane: lane f holds offsets[f] (table_offsets, read once per
// wavefront), so one comparison over the lanes replaces a chain of dependent loads.
__device__ __forceinline__ int64_t table_offsets(const int64_t *offsets, int num_tables)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    return lane < num_tables ? offsets[lane] : 0x7FFFFFFFFFFFFFFFll;
}
__device__ __forceinline__ int find_table_wave(int64_t lane_offset, int64_t pos)
{
    const int below = __popcll(__ballot(lane_offset <= pos));
    return below > 0 ? below - 1 : 0;
}
static_assert(kMaxTables <= kWave, "one lane per table");

__device__ __forceinline__ int64_t wrap(int64_t s, int64_t n) { return s >= n ? s - n : s; }

// Device-side view of a TableDesc.  A pointer read from a descriptor in memory has lost the
// "global" address space that kernel arguments carry, and accesses through it become flat_
// instructions, which also count against the LDS wait counter.  All table state is device memory,
// and the view's pointer types say so.
template <typename T>
using global_ptr = T __attribute__((address_space(1))) *;

struct Tab {
    global_ptr<int64_t> I;
    global_ptr<int32_t> M;
    int64_t N;
    uint64_t seed;
    int32_t P;
    int32_t ttl;
    int32_t evict;
    int32_t sh;
};

// The arguments that the kernel is about to use are requested together, here.  (Else each where its first use is, and a row of
// loads becomes a chain of as many scalar loads, each waited for.)
template <typename T>
__device__ __forceinline__ void wait_for_scalar(T x) { asm volatile("" ::"s"(x)); }
template <typename... T>
__device__ __forceinline__ void args_now(T... args) { (wait_for_scalar(args), ...); }

// Where slot s lives.  Two dense tensors (sh = 0): I[s], M[s].  One tensor of 16-byte records (sh = 1): the id of
// slot s is the int64 at I + 2 s, its metadata the int32 at M + 4 s -- the line that a probe fetches then also
// holds the metadata word that a hit refreshes.
__device__ __forceinline__ global_ptr<int64_t> id_at(const Tab &d, int64_t s) { return d.I + (s << d.sh); }
__device__ __forceinline__ global_ptr<int32_t> meta_at(const Tab &d, int64_t s) { return d.M + (s << (2 * d.sh)); }
// identities of slot s's aligned block of 8 (64 bytes, or 128 bytes of records): how far s lies into it
__device__ __forceinline__ int block_offset(const Tab &d, int64_t s, int slots)
{
    return (int)((s + (int64_t)(((uintptr_t)d.I >> (3 + d.sh)) & (uintptr_t)(slots - 1))) & (slots - 1));
}

__device__ __forceinline__ Tab view(const TableDesc &d)
{
    Tab t;
    t.I = (global_ptr<int64_t>)d.I;
    t.M = (global_ptr<int32_t>)d.M;
    t.N = d.N;
    t.seed = d.seed;
    t.P = d.P;
    t.ttl = d.ttl;
    t.evict = d.evict;
    t.sh = d.sh;
    return t;
}

// A value that is the same in every lane, read from lane 0 so that the compiler keeps it in scalar
// registers (a descriptor loaded from memory arrives in vector registers: the kernels also store to
// global memory, so the load cannot be a scalar one).
__device__ __forceinline__ int32_t uniform32(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t readlane64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ Tab uniform(const Tab &d)
{
    Tab t;
    t.I = (global_ptr<int64_t>)(uintptr_t)uniform64((int64_t)(uintptr_t)(int64_t *)d.I);
    t.M = (global_ptr<int32_t>)(uintptr_t)uniform64((int64_t)(uintptr_t)(int32_t *)d.M);
    t.N = uniform64(d.N);
    t.seed = (uint64_t)uniform64((int64_t)d.seed);
    t.P = uniform32(d.P);
    t.ttl = uniform32(d.ttl);
    t.evict = uniform32(d.evict);
    t.sh = uniform32(d.sh);
    return t;
}

// find_table for a position of a segment that begins in table f, without a look at the memory: one comparison for every table that begins
// before the segment's `end`.  (In k_allocate_lru the lanes' offsets cost more registers than the search costs time: 8 x 100 000 values in LRU
// tables of records 664 -> 691 us for six steps.)
__device__ __forceinline__ int find_table_from(int64_t lane_offset, int num_tables, int f, int64_t end, int64_t pos)
{
    for (int k = f + 1; k < num_tables; ++k) {
        const int64_t begin = readlane64(lane_offset, k);
        if (begin >= end) break;
        if (begin <= pos) f = k;
    }
    return f;
}

// The descriptors of a group, in LDS: to be reached by all `threads` of the workgroup.  (Segments of short features belong to several tables, one after
// the other, and each change waited for a descriptor, each position for a search through the offsets in memory, each list of
// evicted slots for its place.  With the lanes' offsets and a copy of the descriptors, whole steps, us: 26 tables with 10 400 values 36.5 -> 35.4, with
// 320 K 50.2 -> 49.0, 4 with 20 K 32.7 -> 32.4, 26 with 1.1 M 74.5 -> 73.4, 41.6 M values the same.)
__device__ __forceinline__ void copy_descs(const Params &p, TableDesc *s_desc, int threads)
{
    const uint64_t *src = reinterpret_cast<const uint64_t *>(p.descs);
    uint64_t *dst = reinterpret_cast<uint64_t *>(s_desc);
    for (int i = threadIdx.x; i < p.num_tables * (int)(sizeof(TableDesc) / 8); i += threads) dst[i] = src[i];
    __syncthreads();
}

// Metadata written for the id at batch position pos: the step (last seen), or with per-feature TTL
// (Sec. 3.4) the step after which the id is expired: now + duration of its feature.
__device__ __forceinline__ int32_t meta_value(const Params &p, const Tab &d, int64_t pos)
{
    if (d.evict != 3) return p.step;
    return p.step + (p.ttls ? p.ttls[pos] : d.ttl);
}
// The same in two parts, for kernels that request the duration ahead.
__device__ __forceinline__ int32_t duration_of(const Params &p, const Tab &d, int64_t pos)
{
    int32_t t = d.ttl;
    if (d.evict == 3 && p.ttls) t = p.ttls[pos];
    return t;
}
__device__ __forceinline__ int32_t metadata_for(const Params &p, const Tab &d, int32_t duration)
{
    return d.evict == 3 ? p.step + duration : p.step;
}

// Metadata write on behalf of one batch position.  With last-seen metadata every writer of a call
// stores the same step.  With per-feature expiry times (Sec. 3.4, second paragraph) the writers of one
// slot -- the copies of the id that lives there, which may come from features of different retention,
// and the ids that fall back to it as their home -- carry different values; the slot keeps the latest
// expiry step any of them asks for: a refresh never moves it backward, so a short-lived feature
// cannot cut short the retention a long-lived one gave the slot, and the result does not depend on
// the order of the writers.  (A slot that is claimed held -1 or an expired value, which is below
// every value written at this step.)
// Of a record the id that moves in is stored after the atomic: one on a line that a store has just made dirty waits for the
// line to be written back (500 000 new ids in a table of 1 M records with expiry steps: k_finalize_chunk 64.5 us the other way
// round, 28 so; 1 M in 4 M, k_finalize 150 -> 58).  Not so in k_remap_block, whose few atomics wait for nobody and whose last
// store would come later: 1 024 positions per step 1 to 3 % slower.
__device__ __forceinline__ void store_meta(const Tab &d, int64_t s, int32_t value)
{
    if (d.evict == 3) __hip_atomic_fetch_max(meta_at(d, s), value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *meta_at(d, s) = value;
}

// ------------------------------------------------------------------ scratch set
constexpr uint64_t kSetSeed = 0x2545F4914F6CDD1Dull;
constexpr uint32_t kSetEmpty = 0xFFFFFFFFu;

// The scratch set elects, per distinct missed id, the smallest batch position holding it.  An
// entry is one 32-bit word: a batch position (the id it stands for is ids[position]) or empty.
// Inserting (id, pos) into the region [base, base + size): claim the first empty entry of the
// probe sequence with one compare-and-swap, or, on meeting an entry of the same id, lower it to
// min(entry, pos).  An entry never changes the id it stands for, so concurrent inserts agree.
// size >= 2 * (number of inserts into the region), so the unbounded probe always ends.
// Returns the entry index, with kEntered if pos was the first to stand there.  NOTE: whoever meets an entry of its id leaves a
// note under the position that stands there, so that who comes first need not be read back where there is no note, and with
// k_allocate's notes of displaced claims k_finalize need not look at the table (a random read less in each, for each missed
// id: 2.5 M positions, 10 % of them new, on 400 M slots 208 -> 203 us, on 50 M 194 -> 188; 5 %, on 300 M, 165 -> 161).  New
// ids that are popular: nobody loses by notes and merging together.  2.5 M positions on 50 M slots, a call and the add
// that moves its ids, us, neither / notes alone / both: new ids 10 % of the positions, each once 194 / 191 / 191; each ten
// times 155.5 / 157 / 157; drawn by a power law 173 / 173 / 162; the most popular a tenth of the new positions 208 / 206 /
// 177, of all 895 / 890 / 203; all positions new, by a power law (a table's first batch), 1 472 / 1 469 / 620.  600 000
// positions: within 1 % but for the last, 253 / 252 / 110.
constexpr uint32_t kEntered = 0x80000000u;       // (entries are below 2^31)
// one entry: what was there (kSetEmpty: `mine` is there now)
__device__ __forceinline__ uint32_t try_entry(const Params &p, uint64_t e, uint32_t mine)
{
    uint32_t seen = kSetEmpty;
    __hip_atomic_compare_exchange_strong(&p.set_slot[e], &seen, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return seen;
}
// entry e is taken: by the id at hand?  Then `pos` is noted there.
__device__ __forceinline__ bool meets_own(const Params &p, int64_t id, uint32_t pos, uint64_t e, uint32_t seen, bool notes)
{
    if ((int64_t)seen >= p.n || p.ids[seen] != id) return false;      // (an entry is always a position of this batch)
    if (notes) p.note[seen] = 1;
    if (pos < seen) __hip_atomic_fetch_min(&p.set_slot[e], pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}
// the rest of it, entry e having been tried
template <bool NOTE>
__device__ __forceinline__ uint32_t set_insert_from(const Params &p, int64_t id, uint32_t pos, uint64_t e, uint32_t seen, uint64_t base,
                                                    uint64_t end, bool notes = NOTE)
{
    while (seen != kSetEmpty) {
        if (meets_own(p, id, pos, e, seen, NOTE && notes)) return (uint32_t)e;
        if (++e == end) e = base;
        seen = try_entry(p, e, pos);
    }
    return NOTE ? (uint32_t)e | kEntered : (uint32_t)e;           // first of its id so far
}
// Long calls (front_shift) make the first try in the front quarter of the region, the others in the rest of it.  The region must be large
// enough for a batch of new ids, but of nearly every batch a tenth or less is new, and spread over all of it each id is a line of its
// own, fetched and written back three times (entered, read, emptied): 333 MB of them for 41.6 M values, more than the memory-side cache
// holds.  (Three quarters have 1.5 entries for each position of the region, so the rest never fills up.)
// The question whether there is a front costs the calls without one up to 0.3 %, groups up to 1 %: without / with it, us, one table, 0.54 M
// positions 60.9 / 61.0, 1.2 M 95.2 / 95.3, 1.9 M 183.6 / 183.8; 26 tables, 0.33 M values 51.1 / 50.9, 0.64 M 63.4 / 63.8, 1.1 M 82.5 / 83.3, 2.5 M
// 131.7 / 132.5, 5.6 M 238.5 / 239.4.  (Entries in 32 bits, which take back half of the scalar registers that it needs, are no faster.)
template <bool NOTE>
__device__ __forceinline__ uint32_t set_insert(const Params &p, int64_t id, uint64_t hash, uint32_t pos, uint64_t base, uint64_t size,
                                               bool notes = NOTE)
{
    const uint64_t front = size >> p.front_shift, end = base + size;
    uint64_t e = base + __umul64hi(hash, front);
    const uint32_t seen = try_entry(p, e, pos);
    if (seen == kSetEmpty) return NOTE ? (uint32_t)e | kEntered : (uint32_t)e;
    if (meets_own(p, id, pos, e, seen, NOTE && notes)) return (uint32_t)e;
    uint64_t rest = base;
    if (p.front_shift) {
        rest += front;
        e = rest + __umul64hi(hash << 32 | hash >> 32, size - front);
    } else if (++e == end) {
        e = base;
    }
    return set_insert_from<NOTE>(p, id, pos, e, try_entry(p, e, pos), rest, end, notes);
}

// Is it certain that nobody else has the id that was entered at `ent`?
__device__ __forceinline__ bool entered_alone(uint32_t ent, uint8_t note) { return (ent & kEntered) && !note; }

// ------------------------------------------------------------------ small wavefront helpers
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long x)
{
    // rotation sum: afterwards every lane holds the wavefront total
    const int lane = lane_id();
    for (int o = 32; o > 0; o >>= 1) x += (unsigned long long)shfl64((int64_t)x, (lane + o) & 63);
    return x;
}

// Hands the next (64 / G) set bits of amask to the G-lane groups of the wavefront: returns this
// group's bit index or -1, and removes the bits that were handed out.
template <int G>
__device__ __forceinline__ int next_bits(uint64_t &amask, int g)
{
    constexpr int GPW = kWave / G;
    int b = -1;
    uint64_t m = amask;
#pragma unroll
    for (int gg = 0; gg < GPW; ++gg) {
        const int bb = m ? __ffsll((unsigned long long)m) - 1 : -1;
        if (gg == g) b = bb;
        m &= m - 1;
    }
    amask = m;
    return b;
}

// Sum over the wavefront of 32-bit values whose total fits 32 bits, in every lane.
__device__ __forceinline__ uint32_t wave_sum32(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);      // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);      // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);      // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);      // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);      // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);      // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}

__device__ __forceinline__ unsigned long long *stat_word(const Params &p, int table, int k)
{
    return &p.ctl->stats[blockIdx.x % kBins][table][k];
}

// Sums counters (each the wavefront's total) over the workgroup and adds them to this workgroup's copy of the call's
// counters: one atomic per counter when all its wavefronts ended on the same table (the rule), one
// per wavefront and counter otherwise.  Must be reached by all threads of the workgroup.
template <int WAVES>
__device__ __forceinline__ void block_stat_add(const Params &p, const int *idx, const unsigned long long *vals,
                                               int count, int table, unsigned long long (&s_red)[WAVES][kStatCount],
                                               int (&s_tab)[WAVES])
{
    const int lane = lane_id(), w = threadIdx.x / kWave;
    if (lane == 0) {
        for (int k = 0; k < count; ++k) s_red[w][idx[k]] = vals[k];
        s_tab[w] = table;
    }
    __syncthreads();
    if ((int)threadIdx.x < count) {
        const int k = idx[threadIdx.x];
        bool same = true;
        for (int i = 1; i < WAVES; ++i) same = same && s_tab[i] == s_tab[0];
        if (same) {
            unsigned long long v = 0;
            for (int i = 0; i < WAVES; ++i) v += s_red[i][k];
            if (v) atomicAdd(stat_word(p, s_tab[0], k), v);
        } else {
            for (int i = 0; i < WAVES; ++i)
                if (s_red[i][k]) atomicAdd(stat_word(p, s_tab[i], k), s_red[i][k]);
        }
    }
}

// Sums the copies of the call's counters, writes out_num_evicted / out_stats and clears them.  Run by a workgroup of
// k_finalize of its own; of a counting lookup by the one that finishes last.
template <int THREADS>
__device__ __forceinline__ void publish_counters(const Params &p, unsigned long long (*s_sum)[kStatCount])
{
    const bool multi = p.num_tables > 1;
    const int tables = multi ? p.num_tables : 1, words = (multi ? p.num_tables : kSpread) * kStatCount;
    unsigned long long *const sum = &s_sum[0][0];
    for (int i = threadIdx.x; i < tables * kStatCount; i += THREADS) sum[i] = 0;
    __syncthreads();
    for (int k = threadIdx.x; k < words; k += THREADS) {
        // (all copies requested at once)
        unsigned long long *const at = &p.ctl->stats[0][0][0] + k;
        constexpr int kNext = kMaxTables * kStatCount;
        unsigned long long v[kBins], total = 0;
#pragma unroll
        for (int b = 0; b < kBins; ++b) v[b] = __hip_atomic_load(at + b * kNext, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int b = 0; b < kBins; ++b) {
            total += v[b];
            if (v[b]) at[b * kNext] = 0;
        }
        if (total) atomicAdd(&sum[multi ? k : k % kStatCount], total);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tables * kStatCount; i += THREADS) {
        const unsigned long long *const t = s_sum[i / kStatCount];
        const int k = i % kStatCount;
        if (p.out_stats) p.out_stats[i] = (int64_t)(k == kCollisions ? t[kDistinctMiss] - t[kInserts] - t[kEvictions] : t[k]);
        if (p.out_num_evicted && k == kEvictions) p.out_num_evicted[i / kStatCount] = (int64_t)t[k];
    }
}

// The outcomes of the claimants that a wavefront of the allocation has served.  A claim that meets a slot nobody has claimed yet is
// an insert or an eviction whatever displacements follow, and it ends the chain of the lane or group that carries it: so the
// lane that holds a claimant's list entry knows one outcome when its chain has ended, keeps it with the claimant's hint, which it holds
// anyway, and the wavefront counts a chunk's by ballot.  (Counted where a claim stands, in words of the lanes in LDS, they cost the
// claims registers, a wavefront per SIMD in LRU groups.  Before any were counted here / so counted / now, both builds in turn on the same
// tables, us, windows of 16 unless said: the allocation of 26 x 400 000 values, LRU, 250 / 263 / 251, of 64 541 / 556 / 543; whole steps 924 /
// 937 / 922, 1 762 / 1 778 / 1 764; 8 x 100 000, LRU, of 100, 490 / 511 / 485, of 8 90 / 91 / 87; TTL 26 x 20 000 74 / 68 / 68.)
// A word counts positions of the call, MPZCH_MAX_BATCH of them at most, however many a wavefront gets.
struct Outcomes {
    uint32_t word[3][kMaxTables];                    // ids, inserts, evictions
};
static_assert(MPZCH_MAX_BATCH <= UINT32_MAX, "outcomes are counted in 32 bits");
static_assert(kMaxTables == kWave, "a lane per table");
static_assert(kInserts == kDistinctMiss + 1 && kEvictions == kDistinctMiss + 2, "three counters side by side");
constexpr uint32_t kOutcomeInsert = 0x200u, kOutcomeEvict = 0x400u;      // (above what first_of takes of a hint)
__device__ __forceinline__ uint32_t outcome_of(int64_t old) { return is_tag(old) ? 0u : old == -1 ? kOutcomeInsert : kOutcomeEvict; }

// (the kernels of the allocation also clear what k_finalize counts in: it is all zero for it, whatever it left behind)
__device__ __forceinline__ void clear_outcomes(const Params &p, Outcomes &o)
{
    const int lane = lane_id();
    if (blockIdx.x == 0) p.ctl->num_evicted[lane] = 0;
    for (int k = 0; k < 3; ++k) o.word[k][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// Claimants of table t (the same in all lanes), hint: theirs and its outcome.
__device__ __forceinline__ void count_outcomes(Outcomes &o, bool agent, uint32_t hint, int t)
{
    int lane = lane_id();
    asm volatile("" : "+v"(lane));                   // (compared here: the masks would else be kept, or spilled, through the loops of claims)
    const uint64_t agents = __ballot(agent);
    const uint32_t ids = (uint32_t)__popcll(agents), inserts = (uint32_t)__popcll(__ballot((hint & kOutcomeInsert) != 0) & agents),
                   evictions = (uint32_t)__popcll(__ballot((hint & kOutcomeEvict) != 0) & agents);
    if (lane < 3)
        __hip_atomic_fetch_add(&o.word[lane][t], lane == 0 ? ids : lane == 1 ? inserts : evictions, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
// Claimants of several tables, f being each one's own.
template <bool MULTI>
__device__ __forceinline__ void count_outcomes_of(Outcomes &o, bool agent, uint32_t hint, int f)
{
    if constexpr (MULTI) {
        for (uint64_t m = __ballot(agent); m;) {
            const int t = __builtin_amdgcn_readlane(f, __ffsll((unsigned long long)m) - 1);
            const bool of_table = agent && f == t;
            count_outcomes(o, of_table, hint, t);
            m &= ~__ballot(of_table);
        }
    } else {
        count_outcomes(o, agent, hint, 0);
    }
}
template <bool MULTI>
__device__ __forceinline__ void add_outcomes(const Params &p, Outcomes &o)
{
    const int lane = lane_id();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if constexpr (MULTI) {
        if (o.word[0][lane] == 0) return;
        for (int k = 0; k < 3; ++k) {
            const uint32_t v = o.word[k][lane];
            if (v) atomicAdd(stat_word(p, lane, kDistinctMiss + k), (unsigned long long)v);
        }
    } else if (lane < 3) {
        const uint32_t v = o.word[lane][0];
        if (v) atomicAdd(stat_word(p, (int)(blockIdx.x / kBins) % kSpread, kDistinctMiss + lane), (unsigned long long)v);
    }
}

// ------------------------------------------------------------------ Pass 1 (discovery)
// A probe pass compares the ids held one per lane with 8 consecutive slots each (or several times 8: probe_more).  Eight
// lanes read the slots of one id with one access, eight ids per load instruction, and all loads of a pass are in flight
// together.  What the lanes that load need to know goes through LDS (ProbeReq), what each saw (1 = the id, 2 = an empty
// slot, 0 = neither; 4 added to 1 over records: the metadata is what the hit would store) goes back through LDS as one
// byte per slot, and the id's own lane reads its bytes at once and drops those of rounds that do not exist: no
// cross-lane operation depends on a load, and nothing branches.  A pass returns the round of the match; kProbeGoOn when
// the id is not among these slots; or, when in addition one of them is empty, a value <= kProbeAbsent that names the round
// of the first empty slot (probe_absent / absent_len): a slot never becomes empty again once it was
// occupied, so no resident id lies beyond an empty slot of its window and the search can end there.
constexpr int kFirstG = 8;             // slots looked at by the first pass: the aligned 64 bytes that hold the home slot
constexpr int kProbeGoOn = -1;
constexpr int kProbeAbsent = -2;

__device__ __forceinline__ int probe_absent(int empty_round) { return kProbeAbsent - empty_round; }
// slots of the window read until the search ended: up to and including the first empty one
__device__ __forceinline__ int absent_len(int code) { return -code - 1; }

// What the lane that holds an id leaves in LDS for the lanes that load for it: the id, and the address of the identity of
// the first slot to read.
struct alignas(16) ProbeReq {
    int64_t id;
    uint64_t where;
};

// The reads of one pass: 64 blocks of 8 slots, 1 << m of them side by side for each request; 8 lanes read one block, and
// lane_bytes is how far this lane's slot lies from its request's first one.  rows: how many of the blocks anybody asks for.
// What was seen goes to s_code, a byte per slot in the order of requests and slots.
// NT: the loads are marked non-temporal (see k_discover_streaming).  REC: a table of records, read with the
// metadata (12 bytes per lane, the same line): what comes back besides the id is the slot's metadata.
//
// The blocks are read as they lie and nothing is asked per slot: whoever made the request chose a first slot from which
// all of them are in the table, and its own lane knows which bytes are rounds of its window.  (A lookup spends more than
// half of its time issuing instructions.  1 M ids, windows of 32 slots, 80 % load: 903 -> 554 vector instructions per
// wavefront of two chunks, 21.4 -> 19.5 us; 10 K values over 26 tables 5.6 -> 5.1.)
//
// The forms for 8, 4 and 2 rows are copies of one loop of loads behind a wave-uniform branch.  An earlier lookup built that way,
// with nothing to hold the copies apart, gave wrong and varying results on tables of 100 M slots, for a reason that was not
// found, and right ones with a scheduling barrier behind the branch.  The two barriers below therefore stay, whatever their
// effect on the speed: with them every form, in the assembly of each kernel, issues its own loads behind the branch and
// waits for the last of them before the last byte is stored.
template <int T, bool NT, bool REC>
__device__ __forceinline__ void probe_rows(const ProbeReq *req, int next, uint8_t *s_code, uint32_t lane_bytes, int32_t fresh_meta)
{
    int64_t v[T];
    int32_t meta[T];
    // (without: the compiler starts what the forms have in common before it branches to one of them, and waits there)
    asm volatile("" ::"i"(T) : "memory");
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint64_t a = req[t * next].where + lane_bytes;
        if constexpr (REC) {
            const u32x3 rec = *(global_ptr<u32x3>)(uintptr_t)a;
            v[t] = (int64_t)(((uint64_t)rec.y << 32) | rec.x);
            meta[t] = (int32_t)rec.z;
        } else if constexpr (NT) {
            v[t] = __builtin_nontemporal_load((global_ptr<int64_t>)(uintptr_t)a);
        } else {
            v[t] = *(global_ptr<int64_t>)(uintptr_t)a;
        }
    }
    __builtin_amdgcn_sched_barrier(0);          // (the ids are read now, not kept meanwhile)
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const bool same = v[t] == req[t * next].id;
        // (only an empty slot has a high word of all ones: ids are not negative, and the rounds of tags stay below 2^21)
        const uint32_t empty = __builtin_elementwise_sub_sat((uint32_t)((uint64_t)v[t] >> 32), 0xFFFFFFFDu);       // 2 or 0
        uint32_t hit = 1;
        if constexpr (REC) hit = meta[t] == fresh_meta ? 5u : 1u;
        s_code[t * kWave] = (uint8_t)(same ? hit : empty);
    }
}

// (Which of the 64 blocks anybody asks for: the last few searches of a wavefront ask for a quarter of them.)
template <bool NT, bool REC>
__device__ __forceinline__ void probe_blocks(const ProbeReq *s_req, uint8_t *s_code, int m, int rows, uint32_t lane_bytes,
                                             int32_t fresh_meta)
{
    const int lane = lane_id();
    const ProbeReq *const req = s_req + ((lane / 8) >> m);
    const int next = 8 >> m;
    if (rows > 32) probe_rows<8, NT, REC>(req, next, s_code + lane, lane_bytes, fresh_meta);
    else if (rows > 16) probe_rows<4, NT, REC>(req, next, s_code + lane, lane_bytes, fresh_meta);
    else probe_rows<2, NT, REC>(req, next, s_code + lane, lane_bytes, fresh_meta);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// probe_first's lane_bytes (tables of fewer than 8 slots have no block to read: the lanes past the last slot read that one)
__device__ __forceinline__ uint32_t first_lane_bytes(const Tab &d)
{
    const int r = lane_id() % kFirstG;
    return (uint32_t)((int64_t)r < d.N ? r : (int)d.N - 1) << (3 + d.sh);
}

// The first pass: the aligned block of 8 slots that holds the home slot or, ALIGNED not set, the 8 slots from the home slot
// on.  d is wave-uniform; s_req, s_code: this wavefront's own areas of LDS; next: the round to go on with; fresh: whether
// the record of a hit holds fresh_meta already.  A block that reaches out of the table is moved to its edge.  (With the
// tables of a group looked at one at a time, see discover_body: 41 M values over 26 tables 961 -> 882 us; lookup of 1 M ids
// 19.8 -> 18.4 us.)
template <bool NT, bool REC, bool ALIGNED = true>
__device__ __forceinline__ int probe_first(const Tab &d, int64_t id, int64_t home, uint32_t lane_bytes, ProbeReq *s_req,
                                           uint8_t *s_code, int32_t fresh_meta, bool *fresh, int *next)
{
    constexpr int G = kFirstG;
    const int lane = lane_id();
    const int64_t last = d.N > G ? d.N - G : 0;
    int64_t first = home;
    if constexpr (ALIGNED) {
        first -= block_offset(d, home, G);
        first = first > 0 ? first : 0;
    }
    first = first < last ? first : last;
    const int o = (int)(home - first);
    s_req[lane] = ProbeReq{id, (uint64_t)(uintptr_t)(int64_t *)id_at(d, first)};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    probe_blocks<NT, REC>(s_req, s_code, 0, kWave, lane_bytes, fresh_meta);
    const uint64_t x = *reinterpret_cast<const uint64_t *>(s_code + lane * G) >> (8 * o);
    const int bit = __ffsll((unsigned long long)x) - 1;
    const int round = bit >> 3;
    const int there = (d.N < G ? (int)d.N : G) - o;
    const int count = d.P < there ? d.P : there;
    if constexpr (REC) *fresh = x != 0 && ((x >> (bit & 63)) & 4ull) != 0;
    *next = count;
    int found = (bit & 1) ? probe_absent(round) : round;
    if (x == 0 || round >= count) found = count == d.P ? probe_absent(d.P - 1) : kProbeGoOn;   // (or: the whole window was read)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // the areas are written again by the next pass
    return found;
}

// How many blocks of 8 slots each of `count` lanes gets in one pass over 64 blocks, as a shift; no more than `left` rounds
// have use for.
__device__ __forceinline__ int blocks_shift(int count, int left)
{
    const int m = count <= 8 ? 3 : count <= 16 ? 2 : count <= 32 ? 1 : 0;
    const int most = left <= 8 ? 0 : left <= 16 ? 1 : left <= 32 ? 2 : 3;
    return m < most ? m : most;
}

// A later pass: rounds q, q + 1, ... of the lanes with `need` set (the others' arguments are ignored).  The 64 blocks of
// 8 slots that one pass reads are shared out among those lanes: the fewer are left, the more of its window each one
// sees per round trip (8 slots, up to 64 when 8 lanes or fewer are left; a window at 95 % load is often longer than
// 8 slots).  q is moved on past the slots that were looked at; left: how many rounds any of the lanes has left, as far as
// is known (blocks past the end of every window are lines read for nothing).  The slots of one request lie side by side: a window that
// goes on at the table's start does so in the next pass.  The lanes may be of several tables, d being each one's own, if
// these have kWidest slots or more; sh: the layout, the same for all of them; slots: the table's slots, or kWidest if it
// has more.
constexpr int kWidest = 64;
__device__ __forceinline__ int slots_up_to_widest(const Tab &d) { return d.N < kWidest ? (int)d.N : kWidest; }
template <bool NT = false, bool REC = false>
__device__ __forceinline__ int probe_more(const Tab &d, int sh, int slots, int64_t id, int64_t home, int &q, int &left,
                                          bool need, ProbeReq *s_req, uint8_t *s_code, int32_t fresh_meta = 0,
                                          bool *fresh = nullptr)
{
    constexpr int G = 8;
    const int lane = lane_id();
    const uint64_t nm = __ballot(need);
    const int requests = uniform32(__popcll(nm));
    int m = blocks_shift(requests, left);
    if (slots < kWidest) m = slots < 2 * G ? 0 : slots < 4 * G ? (m < 1 ? m : 1) : (m < 2 ? m : 2);
    const int width = slots < G ? slots : G << m;                           // slots of a request
    const int at = lanes_below(nm);
    const int64_t slot = wrap(home + q, d.N);
    const int64_t last = d.N - width;
    const int64_t first = slot < last ? slot : last;
    const int o = (int)(slot - first);
    const int count = d.P - q < width - o ? d.P - q : width - o;           // rounds among them
    // What nobody asks for is read where the first of them reads.  (Not in this lane's own table: it may be one of those
    // with fewer slots than a request is wide.)
    const uint64_t where = (uint64_t)(uintptr_t)(int64_t *)(d.I + (first << sh));
    const uint64_t there = (uint64_t)readlane64((int64_t)where, __ffsll((unsigned long long)nm) - 1);
    s_req[need ? at : requests + lane - at] = ProbeReq{id, need ? where : there};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int r = lane & ((G << m) - 1);                                    // this lane's slot of its request
    probe_blocks<NT, REC>(s_req, s_code, m, requests << m, (uint32_t)(r < width ? r : width - 1) << (3 + sh), fresh_meta);
    const bool moved = __any(need && o != 0);
    int found = kProbeGoOn;
    if (need) {
        // the first byte that is not 0, from the o-th on
        const uint8_t *const mine = s_code + (at << (m + 3));
        uint64_t x = 0;
        int from = 0;
        auto see = [&](int j, int skip) {
            uint64_t y = reinterpret_cast<const uint64_t *>(mine)[j];
            if (skip > 0) y = skip < G ? y & (~0ull << (8 * skip)) : 0;
            if (y) {
                x = y;
                from = G * j;
            }
        };
        if (moved) {
#pragma unroll 1
            for (int j = (1 << m) - 1; j >= 0; --j) see(j, o - G * j);
        } else {
            if (m == 3) {
                see(7, 0);
                see(6, 0);
                see(5, 0);
                see(4, 0);
            }
            if (m >= 2) {
                see(3, 0);
                see(2, 0);
            }
            if (m >= 1) see(1, 0);
            see(0, 0);
        }
        const int bit = __ffsll((unsigned long long)x) - 1;
        const int k = from + (bit >> 3) - o;
        if (x && k < count) {
            if constexpr (REC) *fresh = ((x >> bit) & 4ull) != 0;
            found = (bit & 1) ? probe_absent(q + k) : q + k;
        }
        q += count;
    }
    left -= width;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // the areas are written again by the next pass
    return found;
}

// store_meta for the lanes with `active` set, of which many may hold the same slot (the copies of a popular id).  With
// expiry steps every store is an atomic maximum, and those on one address follow each other at some 12 ns: 20 011
// positions of which the most popular id holds a tenth spent 20 of 24 us on it.  So lanes of one slot first agree on
// their maximum in LDS: of the lanes that write their number into one of 64 (or, over a workgroup, 512) words the
// winner collects the values of those that share its slot; a lane that lost to another slot stores for itself.
struct MetaMerge {
    int64_t slot;
    int32_t value;
    uint32_t winner;
};
static_assert(sizeof(MetaMerge) == sizeof(ProbeReq), "a wavefront's requests lie idle meanwhile");

__device__ __forceinline__ void store_meta_wave(const Tab &d, bool active, int64_t slot, int32_t value, MetaMerge *s_m)
{
    if (d.evict != 3) {
        if (active) *meta_at(d, slot) = value;
        return;
    }
    const int lane = lane_id();
    const int cell = (int)((uint32_t)slot * 0x9E3779B1u >> 26);
    s_m[lane].slot = active ? slot : -1;
    s_m[lane].value = value;
    if (active) s_m[cell].winner = (uint32_t)lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    bool store = active;
    if (active) {
        const uint32_t o = s_m[cell].winner;
        if (o != (uint32_t)lane && s_m[o].slot == slot) {
            __hip_atomic_fetch_max(&s_m[o].value, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            store = false;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (store) __hip_atomic_fetch_max(meta_at(d, slot), s_m[lane].value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Copies of one id within the wavefront (those that find each other in LDS) enter the scratch set once, with the smallest
// of their positions: an id that is new and popular at once -- the first batch of a table, of a feature -- otherwise has
// thousands of atomics on one word, 12 ns each (65 536 positions, the most popular id a fourteenth of them: 67 -> 27 us; over
// the workgroup instead, 14 us, but the barriers cost every other call 0.7).
// miss: the lanes with an id to enter; cell: bits of its hash.  Returns the lane that enters it, and the position in `pos`.
// TABLES: the lanes may be of several tables, f being each one's own; s_f: the wavefront's area for them.
template <bool TABLES = false>
__device__ __forceinline__ int merge_copies(bool miss, int64_t id, int cell, uint32_t &pos, MetaMerge *s_m, uint8_t *s_f = nullptr, int f = 0)
{
    const int lane = lane_id();
    s_m[lane].slot = miss ? id : -1;
    s_m[lane].value = (int32_t)pos;
    if (miss) s_m[cell].winner = (uint32_t)lane;
    if constexpr (TABLES) s_f[lane] = (uint8_t)f;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int from = lane;
    if (miss) {
        const int o = (int)s_m[cell].winner;
        if (o != lane && s_m[o].slot == id && (!TABLES || s_f[o] == f)) {
            __hip_atomic_fetch_min(&s_m[o].value, (int32_t)pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            from = o;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    pos = (uint32_t)s_m[from].value;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return from;
}

// out[pos, :] <- rows[slot mod num_rows, :] for the positions of the active lanes (Sec. 3.7: the lookup
// fused with the embedding gather).  The 64 rows are copied by the whole wavefront, consecutive lanes
// moving consecutive 16-byte (or 4-byte) pieces of a row, several loads in flight per lane.
template <typename VEC>
__device__ __forceinline__ void gather_rows_wave(const Params &p, uint64_t am, int64_t pos, int64_t row)
{
    constexpr int U = 4;
    const int lane = lane_id();
    const int C = p.g_chunks;
    const int total = (kWave - __clzll((long long)am)) * C;          // up to the last active lane (am is not 0)
    for (int i0 = 0; i0 < total; i0 += kWave * U) {
        VEC v[U];
        int64_t dst[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = i0 + u * kWave + lane;
            const bool in = idx < total;
            const int src = in ? (p.g_shift >= 0 ? idx >> p.g_shift : idx / C) : 0;
            const int c = in ? idx - src * C : 0;
            const int64_t srow = shfl64(row, src);
            const int64_t spos = shfl64(pos, src);
            ok[u] = in && ((am >> src) & 1ull);
            dst[u] = spos * C + c;
            // (no branch between the loads: lanes without a piece read the first piece of a row, which is row 0 for
            // positions that are not active)
            v[u] = reinterpret_cast<const VEC *>(p.g_rows + srow * p.g_stride)[c];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<VEC *>(p.g_out) + dst[u]);
    }
}

__device__ __forceinline__ void gather_wave(const Params &p, bool active, int64_t pos, int64_t slot)
{
    const uint64_t am = __ballot(active);
    if (!am) return;
    int64_t row = active ? slot : 0;
    if (row >= p.g_num_rows) row %= p.g_num_rows;
    if (p.g_wide) gather_rows_wave<u32x4>(p, am, pos, row);
    else gather_rows_wave<uint32_t>(p, am, pos, row);
}

// Every wavefront owns one segment of positions.  Per 64-position chunk it probes the line that
// holds each id's home slot.  Ids that were not found there but whose window goes on are parked
// in LDS (position, next round) and resolved later, 64 at a time, so that the second
// memory round trip is paid once per 64 parked ids instead of once per chunk.  What remains
// unfound is the segment's miss list.
//
// REC (training, every table of the call kept as records): a hit whose record already holds the metadata it would
// get is not written again.  A batch draws its popular ids many times, and only the first of them has to dirty the
// line: a read costs the memory system half of what a read and a narrow write of one line cost (48 against 20 G
// lines/s on tables of 8 to 24 GB).  The value read may be older than the table (another die's refresh not yet seen), which
// costs a second store of the same value and nothing else.
template <bool TRAIN, bool MULTI, bool GATHER, bool COUNT = TRAIN, bool NT = false, bool REC = false>
__device__ __forceinline__ void discover_body(const Params &p)
{
    // undecided positions parked per wavefront before they are resolved.  (A lookup's wavefront has two chunks as a rule; with
    // room for 256 in 22 KB of LDS, and one register more than 64, seven of its workgroups were resident on a compute unit and
    // the last twelfth of 1 M ids waited for another's end: 15.8 -> 15.0 us, 19.2 -> 18.4 on batches that the caches do not
    // hold.  With the gather, which has the waiting to do elsewhere, the larger area is the better one: 1.5 M rows of
    // 128 bytes 85.4 against 87.0.)
    constexpr int kStage = TRAIN || GATHER ? 256 : 128;
    __shared__ uint32_t s_pos[kWavesPerBlock][kStage];
    __shared__ int32_t s_q[kWavesPerBlock][kStage];      // >= 0: next round to look at; < 0: absent, -(slots read)
    __shared__ int64_t s_id[kWavesPerBlock][kStage];
    __shared__ unsigned long long s_red[kWavesPerBlock][kStatCount];
    __shared__ int s_tab[kWavesPerBlock];
    __shared__ ProbeReq s_req[kWavesPerBlock][kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_code[kWavesPerBlock][kWave * kFirstG];
    __shared__ TableDesc s_desc[MULTI ? kMaxTables : 1];

    const int lane = lane_id();
    const int w = wave_id();
    int block = blockIdx.x;
    if constexpr (MULTI && TRAIN) {
        // Which workgroup takes which part of the batch.  The dies take workgroups in turn; here each gets whole
        // sixteenths of the batch, so that the popular ids of a feature are in the L2 of one or two dies instead of all
        // eight (41 M values over 26 tables: lines read 23.1 M -> 16.3 M, 877 -> 848 us; eighths 855, for some dies then
        // have the large tables, 32nds 852, 128ths 906).  Whole calls, dealt in turn against sixteenths, us: records 8.1 M
        // values 268 / 252, 16.2 M 490 / 463, 28.6 M 772 / 727, 41.6 M 1 077 / 1 030; two tensors 332 / 323, 576 / 554,
        // 992 / 937, 1 603 / 1 513.  The line at 16 chunks per wavefront is a cautious one: 4.1 M values 171 / 164 and
        // 186 / 183.  Not for lookups, which do not write the lines they share: 12.2 M values 152 / 159, 16.2 M 201 / 210,
        // 41.6 M 495 / 494.
        constexpr int kParts = 16;
        if (p.seg_chunks >= 16 && gridDim.x % kParts == 0) {
            const int per = (int)gridDim.x / kParts, j = block / kDies;
            block = (j / per * kDies + block % kDies) * per + j % per;
        }
    }
    // (positions are below 2^30: 32 bits, of which the scalar unit compares any two)
    const int n = (int)p.n;
    const int seg = block * kWavesPerBlock + w;                         // this wavefront's segment
    const int num_chunks = (n + kWave - 1) / kWave;
    const int c_begin = seg * p.seg_chunks;
    const int c_end = c_begin + p.seg_chunks < num_chunks ? c_begin + p.seg_chunks : num_chunks;
    const int64_t seg_base = (int64_t)c_begin * kWave;
    constexpr bool multi = MULTI;
    const bool want_stats = COUNT && p.out_stats != nullptr;

    // counters of the table currently being processed: positions per wavefront, probe lengths per lane
    unsigned long long st_hit = 0, st_miss = 0, st_inv = 0, st_probe = 0, st_mlen = 0;
    int staged = 0, flushed = 0;                 // wave-uniform: parked ids in LDS / misses already listed

    // Several tables: the table that owns the positions this wavefront is working through, with the
    // range of positions it owns (all wave-uniform).  Positions arrive in ascending order, so the
    // search through the offsets and the load of the descriptor -- a chain of dependent loads in
    // front of every hash -- are paid when the range is left, not once per chunk.
    // (The descriptors are copied to LDS and the offsets to one lane each at the start, together with the first
    // ids: from then on a change of table waits for no memory.  A request of 10 K values over 26 tables, one chunk
    // per wavefront, took 11 us, five of them for the search and the descriptor.)
    int t_f = 0;
    int t_lo = 0, t_hi = 0;
    Tab t_d = view(p.t0);
    // the ids of the next chunk are requested while the current one is probed
    auto ids_of = [&](int chunk) {
        int64_t id = -1;
        if (chunk < c_end && lane < n - chunk * kWave) id = (p.ids + (int64_t)chunk * kWave)[lane];
        return id;
    };
    int64_t id_next = ids_of(c_begin);
    int64_t lane_offset = 0;
    if constexpr (multi) {
        lane_offset = table_offsets(p.offsets, p.num_tables);
        copy_descs(p, s_desc, kBlock);
    }
    // hands the counters of the present table over (when the table changes inside this wavefront's range)
    auto hand_over = [&]() {
        if (!want_stats) return;
        const unsigned long long y = wave_sum(st_probe), z = wave_sum(st_mlen);
        if (lane == 0) {
            if (st_hit) atomicAdd(stat_word(p, t_f, kHitPos), st_hit);
            if (st_miss) atomicAdd(stat_word(p, t_f, kMissPos), st_miss);
            if (st_inv) atomicAdd(stat_word(p, t_f, kInvalidPos), st_inv);
            if (y) atomicAdd(stat_word(p, t_f, kHitProbeSum), y);
            if (z) atomicAdd(stat_word(p, t_f, kMissProbeSum), z);
        }
        st_hit = st_miss = st_inv = st_probe = st_mlen = 0;
    };
    auto enter_table = [&](int64_t upos) {
        t_f = find_table_wave(lane_offset, upos);
        // the search skips empty features that share this offset; the clamps keep every loop
        // finite and every range inside the batch even if the offsets break their contract
        int64_t lo = shfl64(lane_offset, t_f), hi = shfl64(lane_offset, (t_f + 1) & (kWave - 1));
        if (t_f == p.num_tables - 1 || hi > p.n) hi = p.n;
        if (hi <= upos) hi = upos + 1;
        if (lo > upos) lo = upos;
        if (lo < 0) lo = 0;
        t_lo = uniform32((int)lo);
        t_hi = uniform32((int)hi);
        t_d = uniform(view(s_desc[t_f]));
    };
    // a position whose id is resident at `dist` probes from home
    // (the first pass stores the outputs of its whole chunk itself: emit = false)
    // (called by all lanes; `active`: the lane's position is a hit)
    auto finish_hit = [&](const Tab &d, bool active, int64_t pos, int64_t home, int dist, bool emit, bool fresh) {
        const int64_t slot = wrap(home + dist, d.N);
        if (TRAIN)            // "Update": refresh the resident's metadata
            store_meta_wave(d, active && !(REC && fresh && d.evict != 3), slot, active ? meta_value(p, d, pos) : 0,
                            reinterpret_cast<MetaMerge *>(s_req[w]));
        if (!active) return;
        if (COUNT) st_probe += (unsigned long long)(dist + 1);
        if (emit) {
            // (Non-temporal, as are the few that k_finalize rewrites: kept in the L2, such a word is a line of it that the call does not read
            // again.  Both so, us: 41.6 M values over 26 tables 1 266 -> 1 243, 22 M 720 -> 706, 5.6 M 240 -> 237, 1.2 M over 22 79.1 -> 78.3;
            // one table, 3 M positions under LRU 304 -> 295, 4 M 290 -> 289, 0.54 M 61.2 -> 60.7; lookups of 1 M 13.4 -> 13.1, of 0.44 M 8.53 ->
            // 8.41.  What the next kernel of the caller pays for it, the same with a copy of out_slots behind each call: groups 1 412 -> 1 387,
            // 805 -> 793, 262.3 -> 261.9, 84.7 -> 83.9; one table 318 -> 312, 308.5 -> 310, 64.8 -> 64.4, but 2 M on 500 M slots 178.8 -> 181.1 and
            // 2 M on 30 M 150.8 -> 152.2; lookups 18.2 -> 18.0, 11.24 -> 11.18, 4 M 64.5 -> 64.4.  With the rows gathered by them all are
            // within 0.3 %, LRU 944 -> 937.  Not in calls of one chunk: 51 of 65 536 positions 906 -> 923.)
            if (!GATHER || p.out_slots) __builtin_nontemporal_store(slot, &p.out_slots[pos]);
            if (!TRAIN && p.out_found) p.out_found[pos] = 1;
        }
    };

    // probes the parked ids (all of the present table) until found or their window ends; enters the rest into the
    // scratch set
    auto resolve_stage = [&]() {
        // what the first pass stored comes before what any lane of this wavefront stores below
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const Tab d = t_d;
        int nmiss = 0;
        for (int e0 = 0; e0 < staged; e0 += kWave) {
            const bool have = e0 + lane < staged;
            const uint32_t pos = have ? s_pos[w][e0 + lane] : 0;
            const int q0 = have ? s_q[w][e0 + lane] : -1;
            const int64_t id = have ? s_id[w][e0 + lane] : -1;
            const int64_t home = have ? home_slot(id, d.seed, d.N) : 0;
            int dist = -1;
            bool fresh = false;
            int mlen = q0 < 0 ? -q0 : 0;                // > 0: the search has ended at an empty slot
            int q = q0, left = d.P - 1;
            for (;;) {
                const bool need = have && dist < 0 && mlen == 0 && q < d.P;
                if (!__any(need)) break;
                bool got_fresh = false;
                const int got = probe_more<NT, REC>(d, d.sh, slots_up_to_widest(d), id, home, q, left, need, s_req[w], s_code[w], p.step, &got_fresh);
                if (need) {
                    if (got >= 0) { dist = got; fresh = got_fresh; }
                    else if (got <= kProbeAbsent) mlen = absent_len(got);   // an empty slot ends the search
                }
            }
            finish_hit(d, have && dist >= 0, (int64_t)pos, home, dist, true, fresh);
            const bool miss = have && dist < 0;
            const uint64_t mb = __ballot(miss);
            if (miss && TRAIN) {
                const int at = nmiss + lanes_below(mb);      // slots already consumed
                s_pos[w][at] = pos;
                s_id[w][at] = id;
            }
            if (COUNT) {
                st_hit += __popcll(__ballot(have && dist >= 0));
                st_miss += __popcll(mb);
                if (miss) st_mlen += (unsigned long long)(mlen ? mlen : d.P);
            }
            // lookup: the first pass has already stored home and "not found"
            if (GATHER) gather_wave(p, have, (int64_t)pos, dist >= 0 ? wrap(home + dist, d.N) : home);
            nmiss += __popcll(mb);
        }
        if (TRAIN) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            // the region of the scratch set that serves this table: twice as many entries as the table has positions, so
            // that it can never fill up
            const uint64_t sb = multi ? 2ull * (uint64_t)t_lo : 0, ss = 2ull * (uint64_t)(multi ? t_hi - t_lo : p.n);
            // (The copies of an id are merged, but leave notes with one table only: in groups, with batches of 320 K values of
            // which the new ones are popular, Pass 1 took 21 instead of 17 us with both.  No notes for an LRU table either: its
            // claims read the set and its finalize looks, whatever they say; read and cleared they cost finalize 3 of 40 us for
            // 360 000 new ids.  Merged or not, groups, whole steps, new ids popular: 26 x 12 000 values 64.1 / 52.6 us, 8 x
            // 100 000 254 / 88, 4 x 1 M 2 066 / 512, the less so the faster Pass 1 reaches the atomics; new ids rare, 26 x 12 000
            // to 41 M values, the same to 0.6 %.)
            constexpr bool NOTE = !MULTI;
            const bool notes = d.evict != 2;
            for (int j0 = 0; j0 < nmiss; j0 += kWave) {
                const int j = j0 + lane;
                const bool miss = j < nmiss;
                const uint32_t pos = miss ? s_pos[w][j] : 0;
                const int64_t id = miss ? s_id[w][j] : -1;
                const uint64_t hash = mix64((uint64_t)id ^ kSetSeed);
                uint32_t e = 0, first = pos;
                const int from = merge_copies(miss, id, (int)hash & (kWave - 1), first, reinterpret_cast<MetaMerge *>(s_req[w]));
                if (miss && from == lane) e = set_insert<NOTE>(p, id, hash, first, sb, ss, notes);
                e = (uint32_t)__shfl((int)e, from);
                if constexpr (NOTE) {
                    if (miss && from != lane && notes) p.note[first] = 1;
                    if (first != pos) e &= ~kEntered;
                }
                if (miss) {
                    p.list[seg_base + flushed + j] = pos;
                    p.ent[seg_base + flushed + j] = e;
                    p.list_id[seg_base + flushed + j] = id;
                }
            }
            flushed += nmiss;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        staged = 0;
    };

    // One step looks at the lanes of the present chunk that belong to one table (all of them unless the chunk straddles a
    // feature boundary); parked ids are resolved when the stage is full, when the next lanes belong to another table and
    // at the end.  (One place each for the two, or the code is there several times over and needs more registers.)
    int c = c_begin;
    int64_t id = -1;
    bool todo = false;                           // lanes of chunk c that have not been looked at
    bool fetch = true, done = c_begin >= c_end;
    // The first ids are waited for here: a wait inside the loop would be one for everything under way, among it the stores
    // of the chunk before.
    asm volatile("" : "+v"(id_next));
    for (;;) {
        bool resolve = done;
        if (!done) {
            const int pos = c * kWave + lane;
            if (fetch) {
                id = id_next;
                todo = pos < n;
            }
            if (multi) {
                const int upos = c * kWave + __ffsll((unsigned long long)__ballot(todo)) - 1;
                if (upos < t_lo || upos >= t_hi) {
                    resolve = staged > 0;        // what is parked belongs to the table that is left
                    if (!resolve) {
                        hand_over();
                        enter_table(upos);
                    }
                }
            }
            if (!resolve) {
                const Tab d = t_d;
                const bool mine = todo && (!multi || pos < t_hi);
                const bool valid = mine && id >= 0;
                const int64_t home = mine ? home_slot(id, d.seed, d.N) : 0;
                // (behind the hash, or the hash waits for this load too)
                if (fetch) id_next = ids_of(c + 1);
                fetch = false;
                const uint32_t lane_bytes = first_lane_bytes(d);
                bool fresh = false;
                int next = 0;
                const int res = probe_first<NT, REC>(d, id, home, lane_bytes, s_req[w], s_code[w], p.step, &fresh, &next);
                const bool hit = valid && res >= 0;
                finish_hit(d, hit, pos, home, res, false, fresh);
                if (COUNT) {
                    st_hit += __popcll(__ballot(hit));
                    st_inv += __popcll(__ballot(mine && !valid));
                }
                if (COUNT && !TRAIN) {                                       // a lookup miss decided here is final
                    const bool final_miss = valid && res <= kProbeAbsent;
                    st_miss += __popcll(__ballot(final_miss));
                    if (final_miss) st_mlen += (unsigned long long)absent_len(res);
                }
                // One store for the whole chunk keeps the 64-byte sectors of the outputs complete (a
                // sector written with holes leaves the cache as narrow writes).  A position that is
                // not decided yet gets its home slot: final for a negative id (home of its bit
                // pattern) and for a lookup miss, rewritten later otherwise.
                const int64_t slot = hit ? wrap(home + res, d.N) : home;
                if (mine) {
                    // (non-temporal: the outputs are not read by this call; nine in ten are final here)
                    const int64_t base = (int64_t)c * kWave;
                    if (!GATHER || p.out_slots) __builtin_nontemporal_store(slot, &(p.out_slots + base)[lane]);
                    if (!TRAIN && p.out_found) (p.out_found + base)[lane] = hit ? 1 : 0;
                }
                // not found so far: parked when its window goes on, or (training) to be listed as a miss
                const bool park = valid && (res == kProbeGoOn || (TRAIN && res <= kProbeAbsent));
                const uint64_t pb = __ballot(park);
                if (park) {
                    const int at = staged + lanes_below(pb);
                    s_pos[w][at] = (uint32_t)pos;
                    s_id[w][at] = id;
                    s_q[w][at] = res <= kProbeAbsent ? -absent_len(res) : next;
                }
                staged += __popcll(pb);
                if (GATHER) gather_wave(p, mine && !park, pos, slot);
                todo = todo && !mine;
                if (!__any(todo)) {
                    ++c;
                    fetch = true;
                    done = c >= c_end;
                }
                resolve = done || staged > kStage - kWave;
            }
        }
        if (resolve) {
            resolve_stage();
            if (done) break;
        }
    }
    if (TRAIN && lane == 0 && seg < p.num_segs) p.seg_cnt[seg] = (uint32_t)flushed;
    if (want_stats) {
        const int idx[5] = {kHitPos, kMissPos, kInvalidPos, kHitProbeSum, kMissProbeSum};
        const unsigned long long vals[5] = {st_hit, st_miss, st_inv, wave_sum(st_probe), wave_sum(st_mlen)};
        block_stat_add(p, idx, vals, 5, t_f, s_red, s_tab);
    }
    if constexpr (COUNT && !TRAIN) {
        // a counting lookup publishes its own counters (see k_finalize for the training remap)
        __shared__ unsigned long long s_bins[kMaxTables][kStatCount];
        __shared__ bool s_last;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        if (threadIdx.x == 0) s_last = atomicAdd(&p.ctl->done, 1ull) == (unsigned long long)(gridDim.x - 1);
        __syncthreads();
        if (s_last) {
            publish_counters<kBlock>(p, s_bins);
            if (threadIdx.x == 0) p.ctl->done = 0;
        }
    }
}

// The kernels around the one body.  At least four wavefronts per SIMD are asked for (128 registers); with the 70 to 78
// registers that training on one table needs six are resident, with the 80 and 96 of a group six and five (41 M values over
// 26 tables as records, the whole step: held to four 1 221 us, five 1 173, six, with spills, 1 375), of the lookup with gather
// seven, of the plain ones, held to 64 registers, eight.  Training is bound by memory, and measured within 2 % of its best from three
// to six wavefronts for both table layouts.
__global__ __launch_bounds__(kBlock, 4) void k_discover(Params p)
{
    discover_body<true, false, false>(p);
}

// The same pass with the identities read by non-temporal loads, for a two-tensor table far larger than the
// caches: a line of identities is not used again before it is evicted anyway, and not keeping it leaves the L2
// to the lines of metadata that the hits write into (1 B slots, 4 M ids: 0.295 -> 0.253 ms).  Not for
// records -- there the refresh goes into the very line the probe has fetched (0.218 -> 0.277 ms with such
// loads) -- and not for lookups, whose repeated ids do hit in the L2 (100 M slots, 1 M ids: 0.029 -> 0.034 ms).
__global__ __launch_bounds__(kBlock, 4) void k_discover_streaming(Params p)
{
    discover_body<true, false, false, true, true>(p);
}

// the same pass over a table kept as 16-byte records: the metadata store lands in the line just read, and is left
// out when the record shows that an earlier copy of the id has refreshed it (16 % of 4 M positions, 1 B slots:
// 205 -> 202 us)
__global__ __launch_bounds__(kBlock, 4) void k_discover_records(Params p)
{
    discover_body<true, false, false, true, false, true>(p);
}

__global__ __launch_bounds__(kBlock, 8) void k_lookup(LookupArgs<false, false> a)
{
    discover_body<false, false, false>(lookup_params(a));
}

__global__ __launch_bounds__(kBlock, 5) void k_lookup_gather(LookupArgs<false, true> a)
{
    discover_body<false, false, true>(lookup_params(a));
}

__global__ __launch_bounds__(kBlock, 3) void k_lookup_counting(Params p)
{
    discover_body<false, false, false, true>(p);
}

__global__ __launch_bounds__(kBlock, 4) void k_discover_tables(Params p)
{
    discover_body<true, true, false>(p);
}

// A group whose tables are all kept as records: popular ids are refreshed once (41 M values over 26 tables: 1 494 ->
// 1 045 us, at 40 G ids/s near the rate of random line reads).
// (Two dense tensors keep the plain store: a
// look at the metadata first is a random read of its own there, and Pass 1 over 500 M slots went from 111 to 133 us.)
__global__ __launch_bounds__(kBlock, 4) void k_discover_tables_records(Params p)
{
    discover_body<true, true, false, true, false, true>(p);
}

__global__ __launch_bounds__(kBlock, 4) void k_lookup_tables(LookupArgs<true, false> a)
{
    discover_body<false, true, false>(lookup_params(a));
}

// Lookups of few ids.  The chip is idle and round trips are what counts, so a wavefront takes only as many ids as lets the
// 64 blocks of one pass hold the whole window of each (32 ids with windows of 16 slots, 8 with 64; longer ones take
// more passes): a lookup is ids, one look at the table, outputs.  Used while the blocks of a call are no more than
// kShortBlocks (lookup of 5 000 ids, windows of 32 slots, 5.8 -> 3.9 us; 10 K values over 26 tables 7.9 -> 5.6 us; at the
// limit, 128 000 ids with windows of 16 slots 5.2 -> 4.6, 32 000 with 64 7.0 -> 5.9; at twice as many blocks, 64 000 with
// 64, 7.3 against 8.2).
constexpr int64_t kShortBlocks = (int64_t)1 << 18;
constexpr int window_shift(int P) { return P <= 8 ? 0 : P <= 16 ? 1 : P <= 32 ? 2 : 3; }

// Several tables: a wavefront's ids are looked up together whatever their tables, each lane with its own (tables of one
// layout at a time, and those of fewer slots than a request is wide one by one).  One table after the other was a chain
// of its own for each, 1.1 us: 26 ids over 26 tables 32 -> 4 us, 10 K values over them 5.1 -> 3.8.
template <bool MULTI, bool GATHER>
__global__ __launch_bounds__(kBlock, 4) void k_lookup_short(LookupArgs<MULTI, GATHER> a)
{
    const Params p = lookup_params(a);
    __shared__ ProbeReq s_req[kWavesPerBlock][kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_code[kWavesPerBlock][kWave * kFirstG];
    __shared__ TableDesc s_desc[MULTI ? kMaxTables : 1];
    const int lane = lane_id(), w = wave_id();
    const int per = kWave >> p.short_shift;                      // ids of a wavefront
    const int64_t pos0 = ((int64_t)blockIdx.x * kWavesPerBlock + w) * per, pos = pos0 + lane;
    bool todo = lane < per && pos < p.n;
    const int64_t id = todo ? p.ids[pos] : -1;
    Tab d = view(p.t0);
    int f = 0;
    if constexpr (MULTI) {
        const int64_t lane_offset = table_offsets(p.offsets, p.num_tables);
        copy_descs(p, s_desc, kBlock);
        f = find_table_from(lane_offset, p.num_tables, find_table_wave(lane_offset, pos0), pos0 + per, pos);
        d = view(s_desc[f]);
    }
    const int64_t home = home_slot(id, d.seed, d.N);
    while (__any(todo)) {
        bool mine = todo;
        int sh = d.sh, slots = slots_up_to_widest(d);
        if constexpr (MULTI) {
            const int head = __ffsll((unsigned long long)__ballot(todo)) - 1;
            sh = __builtin_amdgcn_readlane(d.sh, head);
            const int of_head = __builtin_amdgcn_readlane(slots, head);
            mine = todo && (of_head < kWidest ? f == __builtin_amdgcn_readlane(f, head) : slots == kWidest && d.sh == sh);
            slots = of_head;
        }
        const bool valid = mine && id >= 0;
        int res = kProbeGoOn, q = 0;
        int left = p.short_shift == 3 ? 1 << 30 : kFirstG << p.short_shift;
        for (;;) {
            const bool need = valid && res == kProbeGoOn && q < d.P;
            if (!__any(need)) break;
            const int got = probe_more<false, false>(d, sh, slots, id, home, q, left, need, s_req[w], s_code[w]);
            if (need) res = got;
        }
        const bool hit = valid && res >= 0;
        const int64_t slot = hit ? wrap(home + res, d.N) : home;
        if (mine) {
            if (!GATHER || p.out_slots) p.out_slots[pos] = slot;
            if (p.out_found) p.out_found[pos] = hit ? 1 : 0;
        }
        if constexpr (GATHER) gather_wave(p, mine, pos, slot);
        todo = todo && !mine;
    }
}

// store_meta_wave where the lanes may be of several tables, d being each one's own: what is shared is told by its address.
__device__ __forceinline__ void store_meta_tables(const Tab &d, bool active, int64_t slot, int32_t value, MetaMerge *s_m)
{
    if (active && d.evict != 3) *meta_at(d, slot) = value;
    const bool latest = active && d.evict == 3;
    if (!__any(latest)) return;
    const int lane = lane_id();
    const int64_t key = latest ? (int64_t)(uintptr_t)meta_at(d, slot) : -1;
    const int cell = (int)((uint32_t)(key >> 2) * 0x9E3779B1u >> 26);
    s_m[lane].slot = key;
    s_m[lane].value = value;
    if (latest) s_m[cell].winner = (uint32_t)lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    bool store = latest;
    if (latest) {
        const uint32_t o = s_m[cell].winner;
        if (o != (uint32_t)lane && s_m[o].slot == key) {
            __hip_atomic_fetch_max(&s_m[o].value, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            store = false;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (store) __hip_atomic_fetch_max(meta_at(d, slot), s_m[lane].value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Pass 1 of a group where every wavefront has one chunk: its positions are looked at together whatever their tables, as in
// k_lookup_short, and nothing is parked, so a chunk in which features end is no longer a chain than another.  Bound by that
// chain: descriptors and ids, looks, set, stores.  Whole steps, k_discover_tables* / this, us: 4 tables with 20 K values 38.3 /
// 33.8, 26 with 320 K 56.3 / 51.4, 26 x 400 values 40.1 / 34.7, 8 x 60 000 on two tensors each 60.0 / 55.2, of four policies
// 101.4 / 85.9 (8 slots), 116.2 / 97.0 (64).
// OVERLAP: what else there is to store goes out beside the scratch set's compare-and-swap, as in k_discover_chunk: 2 x 300 values
// 22.9 -> 22.4 us, 4 x 5 000 25.1 -> 24.7, 26 x 6 000 32.8 -> 32.5 (records), 31.5 -> 31.0; 26 x 12 000 the same, 26 x 19 000 59.6 -> 60.0,
// 55.6 -> 56.1, which is beyond the line that launch_discover draws.
template <bool REC, bool OVERLAP>
__global__ __launch_bounds__(kBlock, 4) void k_discover_tables_chunk(Params p)
{
    __shared__ ProbeReq s_req[kWavesPerBlock][kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_code[kWavesPerBlock][kWave * kFirstG];
    __shared__ uint8_t s_table[kWavesPerBlock][kWave];
    __shared__ TableDesc s_desc[kMaxTables];
    const int lane = lane_id(), w = wave_id();
    const int seg = (int)blockIdx.x * kWavesPerBlock + w;
    const int pos0 = seg * kWave, pos = pos0 + lane, n = (int)p.n;
    const bool in = pos < n;
    const int64_t id = in ? p.ids[pos] : -1;
    const int64_t lane_offset = table_offsets(p.offsets, p.num_tables);
    copy_descs(p, s_desc, kBlock);
    const int f = find_table_from(lane_offset, p.num_tables, find_table_wave(lane_offset, pos0), pos0 + kWave, pos);
    const Tab d = view(s_desc[f]);
    const int64_t home = home_slot(id, d.seed, d.N);
    const bool valid = in && id >= 0;
    int res = kProbeGoOn;
    bool fresh = false, todo = valid;
    while (__any(todo)) {
        // the lanes whose tables are of one layout, or of one table of fewer slots than a request is wide
        const int head = __ffsll((unsigned long long)__ballot(todo)) - 1;
        const int widest = slots_up_to_widest(d), slots = __builtin_amdgcn_readlane(widest, head);
        const int sh = __builtin_amdgcn_readlane(d.sh, head), f_head = __builtin_amdgcn_readlane(f, head);
        const bool mine = todo && (slots < kWidest ? f == f_head : widest == kWidest && d.sh == sh);
        int q = 0, left = __any(mine && f != f_head) ? 1 << 30 : __builtin_amdgcn_readlane(d.P, head);
        for (;;) {
            const bool need = mine && res == kProbeGoOn && q < d.P;
            if (!__any(need)) break;
            bool got_fresh = false;
            const int got = probe_more<false, REC>(d, sh, slots, id, home, q, left, need, s_req[w], s_code[w], p.step, &got_fresh);
            if (need) { res = got; fresh = got_fresh; }
        }
        todo = todo && !mine;
    }
    const bool hit = valid && res >= 0, miss = valid && res < 0;
    MetaMerge *const s_m = reinterpret_cast<MetaMerge *>(s_req[w]);
    const int64_t slot = hit ? wrap(home + res, d.N) : home;
    if (in) __builtin_nontemporal_store(slot, &p.out_slots[pos]);      // (of a missed id: rewritten by k_finalize)
    const uint64_t mb = __ballot(miss);
    uint64_t base = 0, end = 0, entry = 0;
    uint32_t first = (uint32_t)pos, seen = kSetEmpty;
    int from = lane;
    if (mb) {
        // the region of the scratch set that serves the table, and the clamps: see discover_body
        int64_t lo = shfl64(lane_offset, f), hi = shfl64(lane_offset, (f + 1) & (kWave - 1));
        if (f == p.num_tables - 1 || hi > n) hi = n;
        if (hi <= pos) hi = pos + 1;
        if (lo > pos) lo = pos;
        if (lo < 0) lo = 0;
        const uint64_t hash = mix64((uint64_t)id ^ kSetSeed);
        base = 2ull * (uint64_t)lo;
        end = 2ull * (uint64_t)hi;
        entry = base + __umul64hi(hash, end - base);
        from = merge_copies<true>(miss, id, ((int)hash + f) & (kWave - 1), first, s_m, s_table[w], f);
        if (miss && from == lane) seen = try_entry(p, entry, first);
        if (miss) {
            const int at = pos0 + lanes_below(mb);
            p.list[at] = (uint32_t)pos;
            p.list_id[at] = id;
        }
    }
    auto finish = [&]() {
        if (!mb) return;
        uint32_t e = 0;
        if (miss && from == lane) e = set_insert_from<false>(p, id, first, entry, seen, base, end);
        e = (uint32_t)__shfl((int)e, from);
        if (miss) p.ent[pos0 + lanes_below(mb)] = e;
    };
    if constexpr (!OVERLAP) finish();
    if (lane == 0 && seg < p.num_segs) p.seg_cnt[seg] = (uint32_t)__popcll(mb);
    store_meta_tables(d, hit && !(REC && fresh && d.evict != 3), slot, hit ? meta_value(p, d, pos) : 0, s_m);
    for (uint64_t m = p.out_stats ? __ballot(in) : 0; m;) {
        const int t = __builtin_amdgcn_readlane(f, __ffsll((unsigned long long)m) - 1);
        const uint64_t of_table = __ballot(in && f == t);
        const uint32_t hits = (uint32_t)__popcll(__ballot(hit) & of_table), misses = (uint32_t)__popcll(mb & of_table);
        const uint32_t hit_len = wave_sum32(hit && f == t ? (uint32_t)res + 1u : 0u);
        const uint32_t miss_len = wave_sum32(miss && f == t ? (uint32_t)(res <= kProbeAbsent ? absent_len(res) : d.P) : 0u);
        const uint32_t invalid = (uint32_t)__popcll(of_table) - hits - misses;
        const uint32_t v = lane == kHitPos ? hits : lane == kMissPos ? misses : lane == kInvalidPos ? invalid
                         : lane == kHitProbeSum ? hit_len : lane == kMissProbeSum ? miss_len : 0u;
        if (v) atomicAdd(stat_word(p, t, lane), (unsigned long long)v);
        m &= ~of_table;
    }
    if constexpr (OVERLAP) finish();
}

// Several tables: the table of a whole segment of positions [seg_base, seg_base + seg_len), when one
// table owns them all (the rule: a segment is a few thousand positions, a feature's share of the
// batch many times that).  Its number and descriptor are then wave-uniform and read once per segment
// instead of once per lane and list entry.  Returns false when the segment straddles a boundary.
__device__ __forceinline__ bool segment_table(const Params &p, int64_t lane_offset, int64_t seg_base, int64_t seg_len,
                                              int &f, Tab &d, const TableDesc *descs)
{
    f = find_table_wave(lane_offset, seg_base);
    d = uniform(view(descs[f]));
    return f == p.num_tables - 1 || uniform64(seg_base) + seg_len <= uniform64(shfl64(lane_offset, (f + 1) & (kWave - 1)));
}

// ------------------------------------------------------------------ allocation
// One workgroup = one wavefront, every lane carries one claimant.  In one stage the next block of 8 slots of every
// claimant's window (identities and metadata) is read cooperatively -- 8 lanes read the slots of one block with one
// coalesced access, all accesses in flight together -- and what may be claimed goes through LDS to the claimant's own
// lane, one byte per slot.  A lane whose claim displaces another claimant carries that one on.  When few claimants
// are left they get several blocks each, up to 64 slots: a stage costs one round trip, however many it serves.
// (The last claimants used to be served one after the other by the whole wavefront; long windows then took a
// round trip per claimant: 262 K ids into a table of 3 M slots near its capacity, max_probe 64, 69 -> 47 us, the
// last call 104 -> 37 us.)
// The round at which a lane's own claimant was placed is left as a hint for k_finalize.
constexpr uint32_t kHintNone = 0xFF;       // not an elected position
constexpr uint32_t kHintUnplaced = 0xFE;   // ran out of slots: falls back to home (final)
constexpr uint32_t kHintUnknown = 0xFD;    // placed, but not at a round that fits the hint: search the window

// What k_allocate leaves in first_of for k_finalize: the position of the first occurrence of the entry's id, or, for
// that position itself, kAgentEntry | hint, with kAgentOcc if the slot there held an id (and the outcome, which is counted already).  Of tables that are not LRU that stands
// unless a note says that the claim was displaced.
constexpr uint32_t kAgentEntry = 0x80000000u;
constexpr uint32_t kAgentOcc = 0x100u;

// What a claimant's lane leaves in LDS for the lanes that load for it: the address of the identity of the first slot to
// read, that slot's number, and the claim: the claimant's position and the round that the first slot would be for it.
struct alignas(16) ClaimReq {
    uint64_t where;
    int64_t slot;
    int32_t round;
    uint32_t pos;
};

// The TTL test of Sec. 3.4 on a slot that holds an id: expired <=> metadata < bound
__device__ __forceinline__ int32_t expiry_bound(const Tab &d, int32_t step)
{
    if (d.evict == 1) return step - d.ttl;
    if (d.evict == 3) return step;
    return (int32_t)0x80000000;
}

// Blocks.  The first one is aligned: a claimant placed in the block of its home slot -- nearly every one, in a table with room
// or with expired ids -- costs the memory system one line (8 slots counted from the home slot straddle two in seven
// of eight cases; 1 B slots of records, 345 K claimants: 51.5 -> 37 us).  In a table that the memory-side cache holds,
// lines are cheap and round trips are what counts: there a block is simply the next 8 slots.
constexpr int64_t kCachedTableBytes = (int64_t)256 << 20;
constexpr int kAllocG = 8;                           // slots of a block = lanes that read one block together

// A claimant on its way: its position, home slot and next round.
struct Claimant {
    bool active;
    uint32_t pos;
    int32_t q;
    int64_t home;
};

// The claim as an atomic minimum of the tag into the identities word.
__device__ __forceinline__ int64_t claim_in_table(uint64_t address, int64_t tag, uint32_t)
{
    return __hip_atomic_fetch_min((global_ptr<int64_t>)(uintptr_t)address, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The loads of one stage, T for each lane.  As in probe_rows every lane adds a constant to its request's address and nothing
// is asked per slot (51 calls of 65 536 positions 1 026 -> 1 006 us, 12 of 262 144 792 -> 775, 8 of 1 024 90 -> 85).  What the
// claimant's lane needs to know of a slot goes to s_code, one byte: 1 = it may be claimed (empty, holds an expired id, or a
// worse claim), 2 = it held an id when the call began, 4 = it is claimed already.
template <int T, bool REC>
__device__ __forceinline__ void claim_rows(const Tab &d, const ClaimReq *req, int next, uint8_t *s_code, int slot_of_request, bool in,
                                           int32_t bound)
{
    int64_t v[T];
    int32_t meta[T];
    const uint32_t id_bytes = (uint32_t)slot_of_request << (3 + d.sh);
    asm volatile("" ::"i"(T) : "memory");          // (see probe_rows)
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint64_t a = req[t * next].where + id_bytes;
        if constexpr (REC) {
            const u32x3 rec = *(global_ptr<u32x3>)(uintptr_t)a;
            v[t] = (int64_t)(((uint64_t)rec.y << 32) | rec.x);
            meta[t] = (int32_t)rec.z;
        } else {
            v[t] = *(global_ptr<int64_t>)(uintptr_t)a;
        }
    }
    if constexpr (!REC) {
#pragma unroll
        for (int t = 0; t < T; ++t) meta[t] = 0;
        if (d.evict != 0) {
#pragma unroll
            for (int t = 0; t < T; ++t) meta[t] = *meta_at(d, req[t * next].slot + slot_of_request);
        }
    }
    uint32_t code[T];
    uint64_t tags = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        code[t] = v[t] < 0 ? 1u : meta[t] < bound ? 3u : 2u;
        tags |= __ballot(is_tag(v[t]));
    }
    if (tags) {                                    // (hardly ever in the first stage)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t occ = tag_occ(v[t]);
            const bool worse = v[t] > make_tag((uint32_t)(req[t * next].round + slot_of_request), req[t * next].pos, occ);
            if (is_tag(v[t])) code[t] = 4u | (occ << 1) | (worse ? 1u : 0u);
        }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) s_code[t * kWave] = in ? (uint8_t)code[t] : (uint8_t)0;
}

// One stage: reads the next slots of every active claimant's window (am: who is active), 8 << m of them side by side, the
// first ones from the claimant's next round on or, with `aligned`, in the aligned block that holds it.  d is wave-uniform.
// What may be claimed goes to s_code, a byte per slot, 8 << m for each claimant in the order of the lanes.
struct ClaimStage {
    int m;                                           // 8 << m slots per claimant
    int width;                                       // of these, how many there are (all but in tables of fewer than 8 slots)
    int at;                                          // number of this lane's claimant
    int skip;                                        // its first slot is the skip-th that was read
};
template <bool REC>
__device__ __forceinline__ ClaimStage claim_blocks(const Tab &d, const Claimant &c, uint64_t am, int m, int32_t bound, bool aligned,
                                                   uint8_t *s_code, ClaimReq *s_req)
{
    constexpr int G = kAllocG;
    const int lane = lane_id();
    const int slots = slots_up_to_widest(d);
    if (slots < kWidest) m = slots < 2 * G ? 0 : slots < 4 * G ? (m < 1 ? m : 1) : (m < 2 ? m : 2);
    ClaimStage st;
    st.m = m;
    st.width = slots < G ? slots : G << m;
    st.at = lanes_below(am);
    const int claimants = uniform32(__popcll(am));
    const int64_t slot = c.active ? wrap(c.home + c.q, d.N) : 0;
    const int64_t last = d.N - st.width;
    int64_t first = slot;
    if (aligned) {
        first -= block_offset(d, slot, G);
        first = first > 0 ? first : 0;
    }
    first = first < last ? first : last;
    st.skip = (int)(slot - first);
    const ClaimReq rq{(uint64_t)(uintptr_t)(int64_t *)id_at(d, first), first, c.q - st.skip, c.pos};
    s_req[c.active ? st.at : claimants + lane - st.at] = rq;        // (what nobody asks for: slots that are there)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int r = lane & ((G << m) - 1), rows = claimants << m;
    const bool in = r < st.width;
    const ClaimReq *const req = s_req + ((lane / G) >> m);
    const int next = kWave / G >> m, k = in ? r : st.width - 1;
    if (rows > 32) claim_rows<8, REC>(d, req, next, s_code + lane, k, in, bound);
    else if (rows > 16) claim_rows<4, REC>(d, req, next, s_code + lane, k, in, bound);
    else claim_rows<2, REC>(d, req, next, s_code + lane, k, in, bound);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return st;
}

// The claimant's lane walks the slots of the stage and claims.  A claimant that it displaces is carried on at once, from
// the next slot of the same stage (its next round is that slot: displaced at round r of slot s its home is s - r, and
// what was read of empty and expired slots holds for it too; claimed ones it tries) -- a displacement costs the
// round trip of its atomic and no other.  placed(pos, round, slot, old) is called for every claim that stands, old being
// what the slot held before; lost(pos) for a claimant that has run out of slots.  On return c is the claimant to go on
// with, if c.active.
// claim(address of the identity, tag, whether the slot held an id when the call began) makes the claim and returns what the
// slot held before.
//
// Reached by all lanes, who walk in step: one claim each, whichever word of the stage they are at, and what becomes of a lane is a
// number that it carries.  A claim is a round trip and what lies between two of them, which was a third of it: a loop per
// word and lane that ended in five places kept its lanes and their outcomes in masks, some 60 scalar instructions each time around, and
// those that had come to the next word waited for the others.  And where windows are longer than LEAVE slots (0: never) the walk ends
// when, after its first claims, more than WAITS times as many lanes wait for the next stage as walk: those go on there too, with what others have
// claimed meanwhile.  Before / in step / and left early, us: 12 calls of 262 144 new ids 722 / 704 / 686, two of 126 000 and 83 000 into a table of
// 238 000 slots, windows of 256, 163 / 149 / 137, four of 30 000 into 120 000, of 512, 262 / 251 / 202; 51 steps of 65 536 positions 907 /
// 881, 12 of 20 011 309 / 298, 12 of 50 000 on 100 000 slots of records, windows of 32, 411 / 394 / 378; one workgroup, 12 steps of 1 024
// 147 / 141.  (The lists of long calls gain nothing by either, crowded ones lose by the second: 600 000 positions on 3 M slots 167.0 /
// 165.3 / 169.7.)
// WAITS: one in calls of one workgroup, two in those of one chunk for each wavefront.  With more ids than slots most lanes walk to the end of their
// windows, and what is read again for the others is lost.  Walks not in step / never left / left with one / two / four, us, 20 000 positions on 9 000 slots,
// windows of 64, 207 / 204 / 212 / 209 / 207, 66 000 on 30 000 258 / 254 / 262 / 260 / 257; otherwise 5 000 on 20 000 217 / 194 / 194 / 192 / 194, 30 000 new
// ids into 120 000, of 256, 210 / 192 / 172 / 169 / 172, 262 144 into 3 M, of 512, 1 111 / 1 007 / 954 / 954 / 964; one workgroup, 300 on 400, of 200, 845 / - /
// 766 / 790 / 813.
template <int LEAVE, int WAITS, typename Claim, typename Placed, typename Lost>
__device__ __forceinline__ void claim_walk(const Tab &d, Claimant &c, const ClaimStage &st, const uint8_t *s_code,
                                           const ClaimReq *s_req, Claim claim, Placed placed, Lost lost)
{
    constexpr int G = kAllocG;
    constexpr uint64_t kOnes = 0x0101010101010101ull;
    enum : uint32_t { kDone, kWalks, kWaits, kLost };                // kWaits: for the next stage
    uint32_t state = c.active ? kWalks : kDone;
    const int at = c.active ? st.at : 0;
    const uint8_t *const mine = s_code + (at << (st.m + 3));
    const uint64_t where = s_req[at].where;
    uint32_t carried = 0;                                            // all ones: of a displaced claimant, claimed slots are tried
    int32_t round0 = c.q - st.skip;                                  // the round that the first slot read is for the claimant
    int j = 0, skip = st.skip;
    bool claims = false;                                             // (nobody leaves before the stage's first claims)
    uint64_t word = reinterpret_cast<const uint64_t *>(mine)[0], x = word & kOnes;
    if (skip > 0) x = skip < G ? x & (~0ull << (8 * skip)) : 0;
    for (;;) {
        if (__any(state == kWalks && x == 0)) {
            while (state == kWalks && x == 0) {
                ++j;
                if (j == (1 << st.m) || round0 + G * j >= d.P) {
                    c.q = round0 + st.width;                         // (beyond the window's end if the second is why)
                    state = c.q >= d.P ? kLost : kWaits;
                } else {
                    skip -= G;
                    word = reinterpret_cast<const uint64_t *>(mine)[j];
                    x = (word | (word >> 2 & ((uint64_t)carried << 32 | carried))) & kOnes;
                    if (skip > 0) x = skip < G ? x & (~0ull << (8 * skip)) : 0;
                }
            }
        }
        const uint64_t walking = __ballot(state == kWalks);
        if (!walking) break;
        if (LEAVE != 0 && d.P > LEAVE && claims) {
            if (__popcll(__ballot(state == kWaits)) > WAITS * __popcll(walking)) break;
        }
        claims = true;
        const int bit = __ffsll((unsigned long long)x) - 1;
        const int k = G * j + (bit >> 3);
        const int32_t round = round0 + k;
        const uint32_t occ = (uint32_t)(word >> ((bit + 1) & 63)) & 1u;
        const int64_t tag = make_tag((uint32_t)round, c.pos, occ);
        const bool tries = state == kWalks && round < d.P;
        int64_t old = 0;
        if (tries) old = claim(where + ((uint32_t)k << (3 + d.sh)), tag, occ);
        const bool stands = tries && old >= tag;                     // (else a better claim got there first)
        const bool displaces = stands && is_tag(old);
        const int64_t slot = wrap(c.home + round, d.N);
        if (stands) placed(c.pos, round, slot, old);
        x &= x - 1;
        if (state == kWalks && !tries) state = kLost;
        if (stands && !displaces) state = kDone;
        if (displaces) {
            c.pos = tag_pos(old);
            c.home = slot - (int64_t)tag_round(old);
            if (c.home < 0) c.home += d.N;
            round0 = (int32_t)tag_round(old) - k;
            carried = ~0u;
            x = ((word | (word >> 2)) & kOnes) & ~((1ull << bit) | ((1ull << bit) - 1ull));
        }
    }
    if (state == kWalks) {
        c.q = round0 + G * j + ((__ffsll((unsigned long long)x) - 1) >> 3);
        if (c.q >= d.P) state = kLost;
    }
    if (state == kLost) lost(c.pos);
    c.active = state == kWalks || state == kWaits;
}

// One wavefront serves the segments vblock, vblock + vgrid, ...; s_code and s_req are its own areas of LDS.  REC: every
// table of the call is kept as records (identity and metadata come with one load).  Several tables: the claimants of one
// table at a time (nearly always all of them: a segment is a few thousand positions, a feature's share many times that).
template <bool MULTI, bool REC>
__device__ __forceinline__ void allocate_body(const Params &p, int64_t vblock, int64_t vgrid,
                                              uint8_t *s_code, ClaimReq *s_req, Outcomes &outcomes, TableDesc *s_desc)
{
    const int lane = lane_id();
    const Tab d0 = view(p.t0);
    const int64_t lane_offset = MULTI ? table_offsets(p.offsets, p.num_tables) : 0;
    if constexpr (MULTI) copy_descs(p, s_desc, kWave);
    clear_outcomes(p, outcomes);
    for (int64_t seg = vblock; seg < p.num_segs; seg += vgrid) {
        const uint32_t cnt = p.seg_cnt[seg];
        const int64_t seg_base = seg * p.seg_chunks * kWave;
        if ((int32_t)seg_base >= (int32_t)p.n) break;         // segments past the batch hold nothing
        int seg_f = 0;
        Tab seg_d = d0;
        bool seg_one = true;
        if constexpr (MULTI) seg_one = segment_table(p, lane_offset, seg_base, p.seg_chunks * kWave, seg_f, seg_d, s_desc);
        for (uint32_t j0 = 0; j0 == 0 || j0 < cnt; j0 += kWave) {
            // the first entries are requested before the count is known: the count is at most the
            // number of positions of the segment and the arrays have room for n + 128 entries, so
            // the addresses are valid whatever the count turns out to be
            const int64_t idx = seg_base + j0 + lane;
            const uint32_t pos = p.list[idx];
            const uint32_t e = p.ent[idx];
            const int64_t id = p.list_id[idx];
            if (j0 >= cnt) break;
            const bool have = j0 + lane < cnt;
            uint32_t first = 0;
            bool alone = false;
            int f = seg_f;
            if (MULTI && !seg_one) f = find_table_from(lane_offset, p.num_tables, seg_f, seg_base + p.seg_chunks * kWave, (int64_t)pos);
            if (have) {
                if constexpr (MULTI) {
                    first = p.set_slot[e];
                } else {
                    const uint8_t note = p.note[pos];
                    first = pos;
                    if (!(e & kEntered)) first = p.set_slot[e];       // (under way together with the note)
                    alone = entered_alone(e, note);
                    if ((e & kEntered) && note) first = p.set_slot[e & ~kEntered];
                }
            }
            const bool elected = have && first == pos;        // else: a later copy of the id
            if (have && !elected) p.first_of[idx] = first;
            bool todo = elected;
            while (__any(todo)) {
                Tab d = seg_d;
                bool agent = todo;
                int of_table = seg_f;
                if constexpr (MULTI) {
                    if (!seg_one) {
                        of_table = __builtin_amdgcn_readlane(f, __ffsll((unsigned long long)__ballot(todo)) - 1);
                        agent = todo && f == of_table;
                        d = uniform(view(s_desc[of_table]));
                    }
                    todo = todo && !agent;
                    // claimants of LRU tables are served by k_allocate_lru
                    if (d.evict == 2) {
                        if (agent) p.first_of[idx] = first;
                        continue;
                    }
                } else {
                    todo = false;
                }
                const int32_t bound = expiry_bound(d, p.step);
                const bool aligned = (d.N << (3 + d.sh)) > kCachedTableBytes;
                uint32_t hint = kHintUnplaced;        // (and kAgentOcc, and the outcome)
                // the claimant this lane carries
                Claimant c;
                c.active = agent;
                c.pos = pos;
                c.q = 0;
                c.home = home_slot(id, d.seed, d.N);
                for (bool later = false;; later = true) {
                    const uint64_t am = __ballot(c.active);
                    if (!am) break;
                    // the 64 blocks of a stage are shared out among the claimants that are left (but one block each is
                    // what nearly every claimant needs at first)
                    const ClaimStage st = claim_blocks<REC>(d, c, am, later ? blocks_shift(uniform32(__popcll(am)), d.P) : 0, bound,
                                                            aligned && !later, s_code, s_req);
                    claim_walk<0, 0>(d, c, st, s_code, s_req, claim_in_table,
                               [&](uint32_t who, int32_t round, int64_t, int64_t old) {
                                   const uint32_t at = round < (int32_t)kHintUnknown ? (uint32_t)round : kHintUnknown;
                                   if (who == pos) {
                                       hint = at | ((is_tag(old) ? tag_occ(old) != 0 : old >= 0) ? kAgentOcc : 0u);
                                   } else {
                                       p.hint[who] = (uint8_t)at;
                                   }
                                   hint |= outcome_of(old);
                                   if (is_tag(old)) p.note[tag_pos(old)] = 1;
                               },
                               [](uint32_t) {});
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // s_code and s_req are written again
                }
                count_outcomes(outcomes, agent, hint, MULTI ? of_table : 0);
                if (agent) {
                    if (!alone) p.hint[pos] = (uint8_t)hint;  // for the copies of the id
                    p.first_of[idx] = kAgentEntry | hint;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    add_outcomes<MULTI>(p, outcomes);
}

// Two tensors, one table: six wavefronts per SIMD, for the walk in step takes 73 registers.  At seven two go to memory; whole steps, seven / six, us:
// 540 K positions on 20 M slots 59.6 / 59.0, 2 M on 500 M 170.2 / 169.0, 2.5 M on 30 M 247.2 / 245.3, 600 K on 5 M, half of them new, 207.9 / 206.5, 840 K and
// 1.2 M, of which a tenth or a fifth is new, the same to 0.4 %.
template <bool MULTI, bool REC>
__global__ __launch_bounds__(kWave, MULTI ? 5 : REC ? 7 : 6) void k_allocate(Params p)
{
    __shared__ __attribute__((aligned(16))) uint8_t s_code[kWave * kAllocG];
    __shared__ ClaimReq s_req[kWave];
    __shared__ Outcomes s_outcomes;
    __shared__ TableDesc s_desc[MULTI ? kMaxTables : 1];
    allocate_body<MULTI, REC>(p, blockIdx.x, gridDim.x, s_code, s_req, s_outcomes, s_desc);
}

// ------------------------------------------------------------------ allocation, LRU policy
// LRU (Sec. 3.4, last paragraph): a missed id takes the first empty slot of its range, else it
// evicts the entry with the oldest time stamp (ties: the earlier probe round), never one seen at
// the current step.  Its preference list -- empty slots in probe order, then evictable slots
// oldest first -- follows from the state at the start of allocation, which stays readable while
// claims are in flight: a tag keeps the was-occupied bit and metadata is not written before
// k_finalize.  The tag ranks by the CHOICE number (make_lru_tag), so a slot ends with the claimant
// of the lowest (choice, position).  A group of 8 lanes serves one claimant, lane r holding the slots of rounds r, 8 + r, ...
// of its window (T of them, max_probe <= 8 T <= 64; longer ranges: claim_wave_lru_long), so a wavefront works on
// 8 claimants at a time; a displaced claimant is carried on by the group that displaced it, from its next choice.
//
// A claimant is a chain of two round trips, window and atomic, some 2 us, and what counts is how many of them are under way
// (with one lane per slot of the window, two claimants to a wavefront for windows of 32 slots, calls of 300 007
// positions took 53.5 instead of 50.2 us, with windows of 64 of 400 000 78 instead of 72) and the
// number of instructions in between: the list is not ranked, its next choice is drawn when it is needed, which for nearly
// every claimant is once (2 M positions, windows of 32, 220 K claimants: ranked by two shuffles per slot of the window
// more than twice as long, ranked through LDS 78, drawn 56 us).
constexpr int kLruG = 8;
constexpr int kLruGroups = kWave / kLruG;

// What a lane of a claimant's group has read of its slots of the window.
template <int T>
struct LruSlots {
    int64_t v[T];
    int32_t m[T];
};
template <int T, bool REC>
__device__ __forceinline__ LruSlots<T> load_lru_slots(const Tab &d, bool active, int64_t home)
{
    const int r = lane_id() % kLruG;
    LruSlots<T> x;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        // (a lane without a slot reads one that is there)
        const int round = kLruG * t + r;
        const int64_t s = active && round < d.P ? wrap(home + round, d.N) : 0;
        if constexpr (REC) {
            const u32x3 rec = *(global_ptr<u32x3>)id_at(d, s);
            x.v[t] = (int64_t)(((uint64_t)rec.y << 32) | rec.x);
            x.m[t] = (int32_t)rec.z;
        } else {
            x.v[t] = *id_at(d, s);
            x.m[t] = *meta_at(d, s);
        }
    }
    return x;
}

// Minimum over the 8 lanes of a group, in every lane of it.
template <int CTRL>
__device__ __forceinline__ int32_t min_with(int32_t x)
{
    const int32_t y = __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
    return y < x ? y : x;
}
__device__ __forceinline__ int32_t group_min(int32_t x)
{
    x = min_with<0xB1>(x);                           // quad_perm 1 0 3 2
    x = min_with<0x4E>(x);                           // quad_perm 2 3 0 1
    return min_with<0x141>(x);                       // row_half_mirror: 8 lanes
}

// The slots of a window as a mask, bit 8 t + r for lane r's slot t; its union over the 8 lanes of a group, in every lane.
template <int T>
using LruMask = std::conditional_t<(T <= 4), uint32_t, uint64_t>;
template <int CTRL>
__device__ __forceinline__ uint32_t or_with(uint32_t x)
{
    return x | (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t group_or(uint32_t x) { return or_with<0x141>(or_with<0x4E>(or_with<0xB1>(x))); }
__device__ __forceinline__ uint64_t group_or(uint64_t x)
{
    return (uint64_t)group_or((uint32_t)(x >> 32)) << 32 | group_or((uint32_t)x);
}

// active, cpos and home are uniform within a group, x: what its lanes have read of the window.  placed(pos, choice, round,
// slot, old) is called for every claim that stands, old being what the slot held before; lost(pos) for a claimant that
// has run out of slots; both by all lanes of the group.
//
// The list is drawn class by class: the empty slots, then those of the oldest time stamp, of the next one and so on.  A class is
// a mask that all lanes of the group hold, so its choices, and the first `choice` ones that a displaced claimant has behind
// it, cost no exchange between lanes.  (Each choice drawn by three minima over the group, from the first one again for every
// displaced claimant: 12 547 positions on 6 964 slots, windows of 32, 140 -> 99 us; calls of 300 007 on 60 M slots 11.15 -> 10.95.)
//
// A displaced claimant's home slot comes with its tag: by its id it was a round trip of the three that carry a claimant on.  SEEN: a slot that
// was read with a better claim than the claimant's first choice would make is passed over, since claims only get better; the atomic
// that it would lose is another round trip.  Before / home from the tag / and passed over, us: 12 steps under LRU of 684 positions 251.6 /
// 247.0 / 245.7, of 5 000 on 20 000 slots, windows of 32, 373 / 361 / 358, of 20 011 on 12 000 609 / 588 / 558, of 12 000 on 8 000, of 64,
// 1 049 / 1 024 / 889.  (Where few are displaced it costs 1 to 2 %: crowded_lru.  Not in the lists of long calls, where few claims meet and
// windows of 64 have no registers left for it.)
// The wavefront goes through the loops as one: a branch for each group cost windows of 8, which hardly need the classes, what
// they gave (360 000 claimants 56.3 -> 53.9).
template <int T, bool REC, bool SEEN, typename Placed, typename Lost>
__device__ __forceinline__ void claim_group_lru(const Params &p, const Tab &d, bool active, uint32_t cpos, int64_t home,
                                                LruSlots<T> x, Placed placed, Lost lost)
{
    using Mask = LruMask<T>;
    const int lane = lane_id();
    const int r = lane % kLruG, gbase = lane - r;
    int32_t choice = 0;
    while (__any(active)) {
        Mask empties = 0;
        Mask evictable = 0;                          // bit 8 t: the slot of round 8 t + r may be evicted and has not been drawn
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const bool in = active && kLruG * t + r < d.P;
            const bool occ = is_tag(x.v[t]) ? tag_occ(x.v[t]) != 0 : x.v[t] >= 0;     // it held an id when the call began
            if (in && !occ) empties |= (Mask)1 << (kLruG * t + r);
            if (in && occ && x.m[t] != p.step) evictable |= (Mask)1 << (kLruG * t);
        }
        Mask left = group_or(empties);               // of the present class: the slots that have not been drawn
        Mask beaten = 0;                             // SEEN: the slots that were read with a better claim
        if constexpr (SEEN) {
            const int64_t best = make_lru_tag((uint32_t)choice, cpos, 0, 0);
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (is_tag(x.v[t]) && x.v[t] < best) beaten |= (Mask)1 << (kLruG * t + r);
            if (__any(beaten != 0)) beaten = group_or(beaten);
        }
        uint32_t class_occ = 0;                      // ... whether they held ids
        int32_t skip = choice;
        int64_t displaced = 0;
        bool trying = active;
        while (__any(trying)) {
            // on to the class of the present choice
            for (;;) {
                int32_t count = sizeof(Mask) == 4 ? __popc((uint32_t)left) : __popcll(left);
                bool used_up = trying && skip >= count;
                if (SEEN && trying && !used_up) {
                    for (; skip > 0; --skip) left &= left - 1;
                    if (!(left & ~beaten)) {
                        choice += sizeof(Mask) == 4 ? __popc((uint32_t)left) : __popcll(left);
                        count = 0;
                        used_up = true;
                    }
                }
                if (!__any(used_up)) break;
                // (metadata is the caller's: any value may be a time stamp, so a class is told by its members)
                int32_t next = 0x7FFFFFFF;
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if ((evictable >> (kLruG * t) & 1u) && x.m[t] < next) next = x.m[t];
                next = group_min(next);
                Mask members = 0;
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if (x.m[t] == next) members |= (Mask)1 << (kLruG * t);
                members = group_or((members & evictable) << r);
                if (used_up) {
                    skip -= count;
                    class_occ = 1;
                    evictable &= ~(members >> r);
                    left = members;
                    if (!members) {
                        lost(cpos);
                        trying = false;
                    }
                }
            }
            if (!trying) continue;
            if (!SEEN)
                for (; skip > 0; --skip) left &= left - 1;
            const Mask open = left & ~beaten, below = (open & (0 - open)) - 1;
            const int32_t round = __ffsll((unsigned long long)open) - 1;
            if (SEEN) choice += sizeof(Mask) == 4 ? __popc((uint32_t)(left & below)) : __popcll(left & below);
            left &= ~(below << 1 | 1);
            const int64_t mine = make_lru_tag((uint32_t)choice, cpos, (uint32_t)round, class_occ);
            const int64_t s = wrap(home + round, d.N);
            int64_t old = 0;
            if (r == 0) old = __hip_atomic_fetch_min(id_at(d, s), mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            old = shfl64(old, gbase);
            if (is_tag(old) && old < mine) {
                ++choice;                                               // a better claim holds this slot
            } else {
                placed(cpos, choice, round, s, old);
                displaced = is_tag(old) ? old : 0;
                home = s;
                trying = false;
            }
        }
        active = active && displaced != 0;
        if (active) {
            cpos = lru_tag_pos(displaced);                               // same table: same slot
            choice = (int32_t)lru_tag_choice(displaced) + 1;
            home -= (int64_t)lru_tag_round(displaced);
            if (home < 0) home += d.N;
        }
        if (__any(active)) x = load_lru_slots<T, REC>(d, active, home);
    }
}

// One workgroup = one wavefront.  With several tables this kernel runs after k_allocate, which has
// written the hints of every list entry and skipped the claimants of LRU tables; here only those
// claimants are served and only their hints are written.  The windows of the next claimants are requested before the
// present ones are served.
//
// The 8 192 wavefronts of a long call are to run in one go where the registers allow it, with windows of up to 8 slots: 64
// vector registers, and no more than 80 scalar ones, for each wavefront gets 16 more than it uses (with 92 seven of
// eight were resident: 3 M positions, 360 000 claimants, 53.9 -> 48.4 us).
template <int T, bool MULTI, bool REC>
__global__ __launch_bounds__(kWave, MULTI ? (T == 8 ? 3 : 4) : T == 8 ? 4 : T == 1 ? 8 : 5) void k_allocate_lru(Params p)
{
    constexpr int G = kLruG, NG = kLruGroups;
    const int lane = threadIdx.x;
    const int g = lane / G;
    const Tab d0 = view(MULTI ? p.descs[0] : p.t0);
    __shared__ Outcomes outcomes;
    clear_outcomes(p, outcomes);
    for (int64_t seg = blockIdx.x; seg < p.num_segs; seg += gridDim.x) {
        const uint32_t cnt = (uint32_t)uniform32((int)p.seg_cnt[seg]);
        const int64_t seg_base = seg * p.seg_chunks * kWave;
        if ((int32_t)seg_base >= (int32_t)p.n) break;
        for (uint32_t j0 = 0; j0 < cnt; j0 += kWave) {
            const uint32_t idx = (uint32_t)seg_base + j0 + (uint32_t)lane;
            const bool have = j0 + lane < cnt;
            uint32_t pos = 0, e = 0, first = 0;
            int64_t home = 0;
            bool agent = false;
            int f = 0;
            if (have) {
                pos = p.list[idx];
                e = p.ent[idx] & ~kEntered;
                const int64_t id = p.list_id[idx];
                first = p.set_slot[e];
                agent = first == pos;
                if (MULTI && agent) {
                    f = find_table(p.offsets, p.num_tables, (int64_t)pos);
                    const TableDesc &t = p.descs[f];
                    agent = t.evict == 2;
                    home = home_slot(id, t.seed, t.N);
                } else {
                    home = home_slot(id, d0.seed, d0.N);
                }
            }
            uint32_t hint = kHintNone;
            uint64_t am = __ballot(agent);
            // the next NG claimants, one per group of lanes: the lane that holds this group's one, or -1
            int src = next_bits<G>(am, g);
            uint32_t cpos = __shfl(pos, src >= 0 ? src : lane);
            int64_t chome = shfl64(home, src >= 0 ? src : lane);
            const int f1 = __shfl(f, src >= 0 ? src : lane);
            Tab d = d0;
            if (MULTI && src >= 0) d = view(p.descs[f1]);
            LruSlots<T> x = load_lru_slots<T, REC>(d, src >= 0, chome);
            while (__any(src >= 0)) {
                const int src2 = next_bits<G>(am, g);
                const uint32_t cpos2 = __shfl(pos, src2 >= 0 ? src2 : lane);
                const int64_t chome2 = shfl64(home, src2 >= 0 ? src2 : lane);
                const int f2 = __shfl(f, src2 >= 0 ? src2 : lane);
                Tab d2 = d0;
                if (MULTI && src2 >= 0) d2 = view(p.descs[f2]);
                const LruSlots<T> x2 = load_lru_slots<T, REC>(d2, src2 >= 0, chome2);
                uint32_t fr = kHintUnplaced;         // (and the outcome)
                claim_group_lru<T, REC, false>(p, d, src >= 0, cpos, chome, x,
                                        [&](uint32_t who, int32_t, int32_t round, int64_t, int64_t old) {
                                            if (who == cpos) fr = (uint32_t)round;
                                            fr |= outcome_of(old);
                                        },
                                        [](uint32_t) {});
                // the outcome goes to the lane that holds the claimant's list entry
#pragma unroll
                for (int k = 0; k < NG; ++k) {
                    const int sk = __shfl(src, k * G);
                    const uint32_t frk = __shfl(fr, k * G);
                    if (lane == sk) hint = frk;
                }
                src = src2;
                cpos = cpos2;
                chome = chome2;
                d = d2;
                x = x2;
            }
            count_outcomes_of<MULTI>(outcomes, agent, hint, f);
            if (agent) p.hint[pos] = (uint8_t)hint;
            if (agent) p.first_of[idx] = kAgentEntry | hint;
            else if (!MULTI && have) p.first_of[idx] = first;     // (several tables: k_allocate has written it)
        }
    }
    add_outcomes<MULTI>(p, outcomes);
}

// LRU for probe ranges of 65 .. 1 024 slots: the whole wavefront serves one claimant, a lane holds
// the slots of rounds lane, lane + 64, ...  The preference list is not materialised: choice k is
// the k-th empty slot in probe order while k < number of empty slots, else the (k - empties)-th
// evictable slot in (time stamp, round) order, drawn by repeated wavefront-wide minimum of the
// keys above the previous draw.  Same outcome rule as claim_group_lru.
constexpr int kLruLongSlots = 16;          // slots per lane
constexpr int kLruLongProbe = kLruLongSlots * kWave;

__device__ __forceinline__ uint64_t wave_min64(uint64_t x)
{
    const int lane = lane_id();
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t y = (uint64_t)shfl64((int64_t)x, (lane + o) & 63);
        x = y < x ? y : x;
    }
    return x;
}

__device__ __forceinline__ int32_t claim_wave_lru_long(const Params &p, const Tab &d, uint32_t cpos, int32_t choice, uint32_t &outcome)
{
    const int lane = lane_id();
    const int C = (d.P + kWave - 1) / kWave;             // <= kLruLongSlots (checked when the table is created)
    int32_t first_round = -1;
    bool is_first = true;
    for (;;) {
        // (Of a displaced claimant too, by its id: the home slot from its tag, as in claim_group_lru, has to be kept through the loop of
        // choices, and the claim itself took longer.  One table, windows of 100, by the id / from the tag, us: 300 000 positions of records
        // 168 / 180, 700 000 325 / 350, of two tensors 289 / 312; of 1 024, 40 000 positions 280 / 294.  Groups the same either way.)
        const int64_t home = home_slot(p.ids[cpos], d.seed, d.N);
        uint32_t emp = 0, evi = 0;                        // bit c: the slot of round c * 64 + lane is empty / evictable
        int32_t m[kLruLongSlots];
#pragma unroll
        for (int c = 0; c < kLruLongSlots; ++c) {
            const int round = c * kWave + lane;
            const bool in = c < C && round < d.P;
            const int64_t s = in ? wrap(home + round, d.N) : home;      // a valid address either way
            const int64_t v = __hip_atomic_load(id_at(d, s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            m[c] = *meta_at(d, s);
            const bool be = v == -1 || (is_tag(v) && !tag_occ(v));
            const bool oc = v >= 0 || (is_tag(v) && tag_occ(v));
            if (in && be) emp |= 1u << c;
            if (in && oc && m[c] != p.step) evi |= 1u << c;
        }
        int n_empty = 0, n_evict = 0;
        for (int c = 0; c < C; ++c) {
            n_empty += __popcll(__ballot((emp >> c) & 1u));
            n_evict += __popcll(__ballot((evi >> c) & 1u));
        }
        const int n_choices = n_empty + n_evict;
        bool placed = false;
        int64_t displaced = 0;
        uint64_t prev_key = 0;                            // key of the last evictable slot drawn (keys are >= 1)
        int drawn = 0;                                    // evictable slots drawn so far
        for (; choice < n_choices && !placed; ++choice) {
            int round = -1;
            uint32_t occ = 0;
            if (choice < n_empty) {
                int k = choice;
                for (int c = 0; c < C && round < 0; ++c) {
                    uint64_t mask = __ballot((emp >> c) & 1u);
                    const int pc = __popcll(mask);
                    if (k < pc) {
                        for (int i = 0; i < k; ++i) mask &= mask - 1;
                        round = c * kWave + __ffsll((unsigned long long)mask) - 1;
                    } else {
                        k -= pc;
                    }
                }
            } else {
                const int j = choice - n_empty;
                while (drawn <= j) {
                    uint64_t best = ~0ull;
#pragma unroll
                    for (int c = 0; c < kLruLongSlots; ++c) {
                        const uint64_t key =
                            (((uint64_t)((uint32_t)m[c] ^ 0x80000000u) << 32) | (uint32_t)(c * kWave + lane)) + 1ull;
                        if (((evi >> c) & 1u) && key > prev_key && key < best) best = key;
                    }
                    prev_key = wave_min64(best);
                    ++drawn;
                }
                round = (int)(uint32_t)((prev_key - 1ull) & 0xFFFFFFFFull);
                occ = 1;
            }
            if (round < 0) break;                                        // (cannot happen: choice < n_choices)
            const int who = round % kWave;
            int64_t old = 0, mine = 0;
            if (lane == who) {
                mine = make_lru_tag((uint32_t)choice, cpos, (uint32_t)round, occ);
                old = __hip_atomic_fetch_min(id_at(d, wrap(home + round, d.N)), mine, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
            }
            old = shfl64(old, who);
            mine = shfl64(mine, who);
            if (is_tag(old) && old < mine) continue;                    // a better claim holds this slot
            placed = true;
            displaced = is_tag(old) ? old : 0;
            outcome = outcome_of(old);
            if (is_first) first_round = round;
        }
        is_first = false;
        if (!placed || !displaced) break;
        cpos = lru_tag_pos(displaced);                                   // same table: same slot
        choice = (int32_t)lru_tag_choice(displaced) + 1;
    }
    return first_round;
}

template <bool MULTI>
__global__ __launch_bounds__(kWave) void k_allocate_lru_long(Params p)
{
    const int lane = threadIdx.x;
    const Tab d0 = view(MULTI ? p.descs[0] : p.t0);
    __shared__ Outcomes outcomes;
    clear_outcomes(p, outcomes);
    for (int64_t seg = blockIdx.x; seg < p.num_segs; seg += gridDim.x) {
        const uint32_t cnt = p.seg_cnt[seg];
        const int64_t seg_base = seg * p.seg_chunks * kWave;
        if ((int32_t)seg_base >= (int32_t)p.n) break;
        for (uint32_t j0 = 0; j0 < cnt; j0 += kWave) {
            const int64_t idx = seg_base + j0 + lane;
            const bool have = j0 + lane < cnt;
            uint32_t pos = 0, e = 0, first = 0;
            bool agent = false;
            int f = 0;
            if (have) {
                pos = p.list[idx];
                e = p.ent[idx] & ~kEntered;
                first = p.set_slot[e];
                agent = first == pos;
                if (MULTI && agent) {
                    f = find_table(p.offsets, p.num_tables, (int64_t)pos);
                    agent = p.descs[f].evict == 2;
                }
            }
            uint32_t hint = kHintNone;
            uint64_t am = __ballot(agent);
            while (am) {
                const int src = __ffsll((unsigned long long)am) - 1;
                am &= am - 1;
                const uint32_t cpos = __shfl(pos, src);
                const int fs = __shfl(f, src);
                const Tab d = MULTI ? view(p.descs[fs]) : d0;
                uint32_t outcome = 0;
                const int32_t fr = claim_wave_lru_long(p, d, cpos, 0, outcome);
                if (lane == src)
                    hint = (fr < 0 ? kHintUnplaced : (fr < (int32_t)kHintUnknown ? (uint32_t)fr : kHintUnknown)) | outcome;
            }
            count_outcomes_of<MULTI>(outcomes, agent, hint, f);
            if (agent) p.hint[pos] = (uint8_t)hint;
            if (agent) p.first_of[idx] = kAgentEntry | hint;
            else if (!MULTI && have) p.first_of[idx] = first;     // (several tables: k_allocate has written it)
        }
    }
    add_outcomes<MULTI>(p, outcomes);
}

// ------------------------------------------------------------------ finalize
// Sec. 3.4, fused with the remap: the rows of the evicted slots that this wavefront has staged (row numbers in
// rows_buf) get their initial value.  A row is written by consecutive lanes, 16 (or 4) bytes each.
template <typename VEC>
__device__ __forceinline__ void reset_rows_wave(const Params &p, const int64_t *rows_buf, int count)
{
    const int lane = lane_id();
    const int C = p.g_chunks;
    const int64_t total = (int64_t)count * C;
    for (int64_t i = lane; i < total; i += kWave) {
        const int k = p.g_shift >= 0 ? (int)(i >> p.g_shift) : (int)(i / C);
        const int c = (int)(i - (int64_t)k * C);
        VEC v = VEC(0);
        if (p.r_init) v = reinterpret_cast<const VEC *>(p.r_init)[c];
        __builtin_nontemporal_store(v, reinterpret_cast<VEC *>(p.r_rows + rows_buf[k] * p.g_stride) + c);
    }
}

__device__ __forceinline__ void reset_staged_rows(const Params &p, const int64_t *rows_buf, int count)
{
    if (!p.r_rows || count == 0) return;
    if (p.g_wide) reset_rows_wave<u32x4>(p, rows_buf, count);
    else reset_rows_wave<uint32_t>(p, rows_buf, count);
}

// Appends the staged evicted slots of one wavefront to table `table`'s list (and resets their rows).
__device__ __forceinline__ void flush_evicted(const Params &p, const int64_t *buf, const int64_t *rows_buf, int &count,
                                              int table, const TableDesc *s_desc)
{
    if (count == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    reset_staged_rows(p, rows_buf, count);
    const int lane = lane_id();
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&p.ctl->num_evicted[table], (unsigned long long)count);
    base = (unsigned long long)shfl64((int64_t)base, 0);
    // (separate statements: a choice between the descriptor in the kernel arguments and one in global memory,
    // written as one expression, is compiled into loads through a generic pointer)
    int64_t ev_begin = p.t0.ev_begin, ev_cap = p.t0.ev_cap;
    if (p.num_tables > 1) {
        ev_begin = s_desc[table].ev_begin;
        ev_cap = s_desc[table].ev_cap;
    }
    for (int i = lane; i < count; i += kWave) {
        const int64_t at = (int64_t)base + i;
        if (at < ev_cap) p.out_evicted[ev_begin + at] = buf[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    count = 0;
}

// Evicted slots staged per wavefront in LDS (all members are the same in every lane).
struct Staged {
    int count = 0, table = 0;
};

// Called by all lanes of the wavefront.  `evicted` lanes hold an evicted slot s of table f.
__device__ __forceinline__ void stage_evicted(const Params &p, Staged &st, int64_t *s_ev_w, int64_t *s_row_w, bool evicted, int64_t s, int f, const TableDesc *s_desc)
{
    const int lane = lane_id();
    // all entries of the buffer belong to one table
    uint64_t evm = __ballot(evicted);
    while (evm) {
        const int tf = __shfl(f, __ffsll((unsigned long long)evm) - 1);
        const bool sel = evicted && f == tf;
        const uint64_t selm = __ballot(sel);
        const int add = __popcll(selm);
        if ((st.count > 0 && tf != st.table) || st.count + add > kEvBuf) flush_evicted(p, s_ev_w, s_row_w, st.count, st.table, s_desc);
        st.table = tf;
        if (sel) {
            const int at = st.count + __popcll(selm & ((1ull << lane) - 1ull));
            s_ev_w[at] = s;
            if (p.r_rows) s_row_w[at] = s >= p.g_num_rows ? s % p.g_num_rows : s;
        }
        st.count += add;
        evm &= ~selm;
    }
}

// End of k_finalize, reached by all threads: the workgroup reserves its part of the evicted list (one reservation when all its
// wavefronts staged for the same table) and writes it.
__device__ __forceinline__ void list_evicted(const Params &p, Staged &st, int64_t (*s_ev)[kEvBuf], int64_t (*s_row)[kEvBuf],
                                             int *s_cnt, int (&s_tab)[kFinalizeWaves], unsigned long long *s_base, const TableDesc *s_desc)
{
    const int lane = lane_id(), w = threadIdx.x / kWave;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (lane == 0) { s_cnt[w] = st.count; s_tab[w] = st.table; }
    __syncthreads();
    int total = 0, before = 0, tab = -1;
    bool same = true;
    for (int i = 0; i < kFinalizeWaves; ++i) {
        if (s_cnt[i] == 0) continue;
        if (tab < 0) tab = s_tab[i];
        else if (s_tab[i] != tab) same = false;
        if (i < w) before += s_cnt[i];
        total += s_cnt[i];
    }
    if (total == 0) return;
    if (!same) {
        flush_evicted(p, s_ev[w], s_row[0], st.count, st.table, s_desc);
        return;
    }
    if (threadIdx.x == 0) *s_base = atomicAdd(&p.ctl->num_evicted[tab], (unsigned long long)total);
    __syncthreads();
    const int64_t base = (int64_t)*s_base + before;
    int64_t ev_begin = p.t0.ev_begin, ev_cap = p.t0.ev_cap;
    if (p.num_tables > 1) {
        ev_begin = s_desc[tab].ev_begin;
        ev_cap = s_desc[tab].ev_cap;
    }
    for (int i = lane; i < st.count; i += kWave)
        if (base + i < ev_cap) p.out_evicted[ev_begin + base + i] = s_ev[w][i];
}

// Every entry of the miss lists -- the elected position of an id (its agent) and the other copies of
// the id alike -- finds the slot that carries the agent's claim.  The agent of a table that is not LRU knows where it is unless a
// note says that it was displaced (or, with one table, has copies); else it and its copies look where k_allocate left the claim (the hint, kept
// under the agent's batch position, which every copy knows), and the whole wavefront searches the window of a claimant
// displaced after its hint was written.  A copy may find the claim tag or, when the agent has been quicker, already the id.  The agent turns the tag into the id,
// writes the metadata and lists the slot that it evicted; every entry stores its output slot.  Entries
// without a claim fall back to the home slot (Case 3).
// NOTES: one table, not LRU (see set_insert).  Groups have notes of displaced claims alone: the claim is looked at by few, and a
// random line less is read for each (same tables, both builds in turn, whole steps: 26 x 400 000 values, 10 % of them new, records 670 ->
// 660 us, two tensors 822 -> 813; 8 x 500 000 239 -> 237, 271 -> 269; 26 x 12 000 the same).
template <bool MULTI, bool NOTES>
__device__ __forceinline__ void finalize_body(const Params &p)
{
    __shared__ int64_t s_ev[kFinalizeWaves][kEvBuf];
    __shared__ int64_t s_row[MULTI ? 1 : kFinalizeWaves][kEvBuf];  // fused row reset (one table): the rows of the staged slots
    __shared__ unsigned long long s_sum[MULTI ? kMaxTables : 1][kStatCount];
    __shared__ int s_cnt[kFinalizeWaves];
    __shared__ int s_tab[kFinalizeWaves];
    __shared__ unsigned long long s_base;

    // The call's counters, complete since the allocation, are the work of a workgroup of its own, the last one, which starts when
    // another has ended where all compute units are full.  (Outcomes counted here, by workgroups that reported in and of which the
    // last summed the counters and cleared 74 KB, ended the kernel 7 us after its last list entry, now 2.4; the allocation takes
    // 0.5 longer for it.  600 K positions on two tensors, k_finalize 19.7 -> 15.8 us, the step 80.4 -> 76.8; 4 tables with 20 K
    // values 42.0 -> 38.3; 500 M slots, 2 M positions, k_finalize 23.4 -> 20.0.)
    if (blockIdx.x == gridDim.x - kFinalizeExtra) {
        publish_counters<kFinalizeBlock>(p, s_sum);
        return;
    }
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    const int64_t wave_global = ((int64_t)blockIdx.x * kFinalizeBlock + threadIdx.x) / kWave;
    const int64_t num_waves = (int64_t)(gridDim.x - kFinalizeExtra) * kFinalizeWaves;
    constexpr bool multi = MULTI;
    Staged staged;
    const int64_t lane_offset = multi ? table_offsets(p.offsets, p.num_tables) : 0;
    __shared__ TableDesc s_desc[MULTI ? kMaxTables : 1];
    if constexpr (MULTI) copy_descs(p, s_desc, kFinalizeBlock);

    for (int64_t seg = wave_global; seg < p.num_segs; seg += num_waves) {
        const uint32_t cnt = p.seg_cnt[seg];
        const int64_t seg_base = seg * p.seg_chunks * kWave;
        int seg_f = 0;
        Tab seg_d{};
        if (!multi) seg_d = view(p.t0);
        bool seg_one = true;
        if (multi) seg_one = segment_table(p, lane_offset, seg_base, p.seg_chunks * kWave, seg_f, seg_d, s_desc);
        if ((int32_t)seg_base >= (int32_t)p.n) break;         // segments past the batch hold nothing
        for (uint32_t j0 = 0; j0 == 0 || j0 < cnt; j0 += kWave) {
            // (as in k_allocate, the first entries are requested before the count is known)
            const int64_t idx = seg_base + j0 + lane;
            const uint32_t pos = p.list[idx];
            const uint32_t word = p.first_of[idx];
            const uint32_t e = p.ent[idx];
            const int64_t id = p.list_id[idx];
            if (j0 >= cnt) break;
            const bool have = j0 + lane < cnt;
            bool agent = false;
            uint32_t first = 0, h = kHintUnplaced;
            int outcome = 2, f = 0;
            int64_t s_final = 0, home = 0;
            Tab d = seg_d;
            int at = -1;
            uint32_t occ = 0;
            // does slot value v carry the claim of the id whose first occurrence is `fst`?
            auto is_claim_of = [](int64_t v, uint32_t fst, int64_t cid, bool lru) {
                return is_tag(v) ? (lru ? lru_tag_pos(v) : tag_pos(v)) == fst : v == cid;
            };
            bool search = false, sure = false;
            if (multi && !seg_one) f = find_table_from(lane_offset, p.num_tables, seg_f, seg_base + p.seg_chunks * kWave, (int64_t)pos);
            if (have) {
                agent = (word & kAgentEntry) != 0;
                first = agent ? pos : word;
                h = agent ? word & 0xFFu : (uint32_t)p.hint[first];
                p.set_slot[e & ~kEntered] = kSetEmpty;         // the scratch set is left empty again
                if (multi) {
                    if (seg_one) {
                        f = seg_f;
                    } else {
                        d = view(s_desc[f]);
                    }
                }
                if (MULTI ? d.evict != 2 : NOTES) {
                    const uint8_t note = p.note[pos];
                    if (note) p.note[pos] = 0;                 // no note is left behind
                    sure = agent && !note;
                }
                home = home_slot(id, d.seed, d.N);
                if (sure && h < kHintUnknown) {
                    at = (int)h;
                    occ = (word & kAgentOcc) ? 1u : 0u;
                } else if (h < kHintUnknown) {
                    const int64_t v = *id_at(d, wrap(home + (int)h, d.N));
                    if (is_claim_of(v, first, id, d.evict == 2)) { at = (int)h; occ = tag_occ(v); }
                }
                search = at < 0 && h != kHintUnplaced;
            }
            // the hint did not lead to the claim (the claimant was displaced afterwards): the window is
            // searched; searches are served one after the other by the whole wavefront, 64 slots per access
            uint64_t sm = __ballot(search);
            while (sm) {
                const int src = __ffsll((unsigned long long)sm) - 1;
                sm &= sm - 1;
                const uint32_t cfirst = __shfl(first, src);
                const int64_t cid = shfl64(id, src);
                const int64_t chome = shfl64(home, src);
                Tab dw = seg_d;
                if (multi) dw = uniform(view(p.descs[__shfl(f, src)]));
                int found_round = -1;
                uint32_t found_occ = 0;
                for (int32_t c0 = 0; c0 < dw.P && found_round < 0; c0 += kWave) {
                    const int32_t round = c0 + lane;
                    bool mine = false;
                    uint32_t o = 0;
                    if (round < dw.P) {
                        const int64_t v = *id_at(dw, wrap(chome + round, dw.N));
                        mine = is_claim_of(v, cfirst, cid, dw.evict == 2);
                        o = tag_occ(v);
                    }
                    const uint64_t mb = __ballot(mine);
                    if (mb) {
                        const int ml = __ffsll((unsigned long long)mb) - 1;
                        found_round = c0 + ml;
                        found_occ = __shfl(o, ml);
                    }
                }
                if (lane == src) { at = found_round; occ = found_occ; }
            }
            if (have) {
                s_final = at >= 0 ? wrap(home + at, d.N) : home;
                if (agent) {
                    // the claim becomes the id, metadata gets its value (Algorithm 1, Pass 2); without a
                    // claim: Case 3, the home slot's metadata is refreshed.  (The agent always meets its
                    // own tag: nobody else replaces it.)
                    if (at >= 0) outcome = (int)occ;
                    const int32_t m = meta_value(p, d, pos);
                    if (at >= 0 && d.sh == 1 && d.evict != 3) {
                        // (one store for both)
                        *(global_ptr<u32x3>)id_at(d, s_final) = u32x3{(uint32_t)(uint64_t)id, (uint32_t)((uint64_t)id >> 32), (uint32_t)m};
                    } else {
                        store_meta(d, s_final, m);
                        if (at >= 0) *id_at(d, s_final) = id;
                    }
                } else if (p.ttls && d.evict == 3) {
                    // per-feature retention: a later copy may ask for a later expiry step than the first
                    store_meta(d, s_final, meta_value(p, d, pos));
                }
                __builtin_nontemporal_store(s_final, &p.out_slots[pos]);             // (see finish_hit in discover_body)
            }
            stage_evicted(p, staged, s_ev[w], s_row[MULTI ? 0 : w], agent && outcome == 1, s_final, f, s_desc);
        }
    }
    if constexpr (!MULTI) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        reset_staged_rows(p, s_row[w], staged.count);
    }
    list_evicted(p, staged, s_ev, s_row, s_cnt, s_tab, &s_base, s_desc);
}

// WAVES = 8 wavefronts per SIMD (one table: 47 vector registers and 66 KB of LDS for 16 wavefronts, several: 61 and 44 KB, 4 of them the
// descriptors; no vector register goes to memory, 67 to 76 scalar ones are kept in lanes of vector registers), so that
// the 8 192 wavefronts, each a chain of three round trips, run in one go.  (Several tables with 66 registers and the rows'
// buffer that only one table has use for: one workgroup per compute unit and two turns, 41 M values over 26 tables 152 -> 145
// us.)  A batch of 4 M positions, 10 % of them new, with
// the row reset: 56 -> 46 us by the ids in the miss lists (a line read for each of them before), one store for id and
// metadata of a record, and rows reset before the workgroup's barrier instead of behind it, 45.5 -> 41 us by the claims that
// need no look; 41 M values over 26 tables
// 242 -> 178 us.
// WAVES = 4, several tables: more scalar registers, 38 kept in vector lanes, which is time that the chain of a small call
// sees: steps of 600 values over 2 tables 35.6 -> 34.8 us, 10 400 over 26 41.4 -> 40.6.
template <bool MULTI, bool NOTES, int WAVES = 8>
__global__ __launch_bounds__(kFinalizeBlock, WAVES) void k_finalize(Params p)
{
    finalize_body<MULTI, NOTES>(p);
}

// ------------------------------------------------------------------ fills and row reset
__global__ __launch_bounds__(kBlock) void k_fill64(long long *dst, int64_t count, long long value)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (int64_t)gridDim.x * kBlock)
        dst[i] = value;
}

// initial state of a table kept as 16-byte records: id = -1, metadata = -1, the unused word 0
__global__ __launch_bounds__(kBlock) void k_init_records(u32x4 *dst, int64_t count)
{
    const u32x4 v = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (int64_t)gridDim.x * kBlock)
        dst[i] = v;
}

// initial state of a table kept as two tensors (one launch: a second one takes longer than a small table)
__global__ __launch_bounds__(kBlock) void k_init_tensors(long long *ids, int32_t *metadata, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (int64_t)gridDim.x * kBlock) {
        ids[i] = -1;
        metadata[i] = -1;
    }
}

__global__ __launch_bounds__(kBlock) void k_fill32(int32_t *dst, int64_t count, int32_t value)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (int64_t)gridDim.x * kBlock)
        dst[i] = value;
}

}  // namespace mpzch

// The training remap of batches that give every wavefront at most one chunk of 64 positions (one table; up to
// about half a million positions on 256 compute units).
//
// Such a call is bound by latency: every kernel is a chain of dependent round trips to memory (0.6 to 1 us each),
// and the kernels wait for each other.  The kernels of mpzch_kernels.hpp compact the missed positions into lists, add
// their counters to shared words and reserve their parts of the evicted list by atomics; none of that pays here.
// In these kernels lane L of wavefront W works on position 64 W + L in all three phases, what one phase leaves for the
// next is stored by position, and counters are stored per workgroup and summed by the last kernel: no shared
// counter, no reservation, no list.
//   k_discover_chunk   Pass 1; the whole window of every id is looked at in registers (nothing is parked); missed
//                      ids enter the scratch set.
//   k_allocate_chunk   claims.  The first block of every window is requested together with the election of the
//                      first occurrence.  A slot that is claimed for the first time is an insert or an eviction
//                      whatever displacements follow, so the outcome is counted here, and the evicted slots are left for
//                      the last kernel, per workgroup.  Where its own lane has placed a claimant is stored once; lanes
//                      that carry on displaced ones note it in place[position], and since rounds only grow while a
//                      claimant is displaced an atomic maximum makes the larger of the two words final when the
//                      kernel ends.  So the last kernel need not look at the table at all.
//   k_finalize_chunk   ids and metadata of the placed claimants, outputs, evicted list (its place in the list
//                      comes from the counts of the workgroups before), row reset, counters.
#pragma once
#include "mpzch_kernels.hpp"

namespace mpzch {

constexpr uint32_t kNoEntry = 0xFFFFFFFFu;       // ent[pos]: the position did not miss
                                                 // (with the entry: kEntered)
// Where a claimant ends up: round + 1 (under the LRU policy choice << 16 | round + 1), 0: nowhere so far, kPlaceNone:
// displaced and out of slots.
constexpr uint32_t kPlaceNone = 0x7FFFFFFEu;      // (with kOwnPlace it is not kNoEntry)
constexpr uint32_t kOwnPlace = 0x80000000u;      // list[pos] of the first occurrence of a missed id: this bit and its place
                                                 // as far as its own lane knows.  Of a later copy: the position of the
                                                 // first; kNoEntry: the position did not miss

// Scratch set of these calls: an entry is the batch position with 12 bits of the id's hash above it, so that two ids that
// meet in one entry tell each other apart without a look at the batch (a round trip per collision; with every
// id missed and half of the set full, that was 8 of 40 us for 262 144 ids).  Otherwise as set_insert.  The hash is the one
// that gave the home slot: that takes its highest bits, an entry its low word and the 12 bits above.  (Three hashes per
// position before: 51 calls of 65 536 positions 1 006 -> 996 us, 8 of 1 024 85 -> 83.)
//
// Four entries per position: the GPU performs 27 G atomics/s on memory that its 256 MB cache holds, as it does this set of
// 8 MB at most (17 to 18 G/s on gigabytes), so where every id is missed the lanes of all wavefronts queue 10 us for their
// first one, and every collision queues again (262 144 ids,
// Pass 1: 36 -> 24 us; two entries per position and 1.5 atomics per id took 27 of 36).
// (With the notes of set_insert: 12 calls of 262 144 new ids 772 -> 749 us, 51 of 65 536 positions 998 -> 986.)
constexpr int kChunkSetEntries = 4;              // per position
constexpr int64_t kChunkMaxBatch = (int64_t)1 << 19;
constexpr int kChunkPosBits = 20;
constexpr uint32_t kChunkPosMask = (1u << kChunkPosBits) - 1u;

// A missed id enters it in two halves: begin_insert requests the first compare-and-swap, and what the kernel has to store besides goes
// out while that is under way (OVERLAP of k_discover_chunk).
struct SetInsert {
    uint32_t mine, e;                // what is entered, and where next
    uint32_t seen;                   // what was there
    uint32_t first;                  // the lowest position among the copies of the id in this wavefront
    int from;                        // the lane that enters the id
};
// for the lanes with `miss` set
__device__ __forceinline__ SetInsert begin_insert(const Params &p, bool miss, int64_t id, uint64_t hash, uint32_t pos, MetaMerge *s_m)
{
    SetInsert x;
    x.first = pos;
    x.from = merge_copies(miss, id, (int)(hash >> 44) & (kWave - 1), x.first, s_m);
    x.mine = ((uint32_t)(hash >> 32) << kChunkPosBits) | x.first;
    x.e = __umulhi((uint32_t)hash, (uint32_t)kChunkSetEntries * (uint32_t)p.n);
    x.seen = kSetEmpty;
    if (miss && x.from == lane_id()) x.seen = try_entry(p, x.e, x.mine);
    return x;
}
// The entry to try after e, which another id holds: the next one that was empty, or had the hash bits of `mine`, when looked at.  (What
// was seen of an entry that an id holds stays true: none is given up or handed on during the call.)
__device__ __forceinline__ uint32_t next_entry(const Params &p, uint32_t e, uint32_t size, uint32_t mine)
{
    for (;;) {
        if (++e == size) e = 0;
        const uint32_t g = e & ~3u, h = g + 4 == size ? 0 : g + 4;       // (size is a multiple of four)
        const u32x4 a = *reinterpret_cast<const u32x4 *>(p.set_slot + g), b = *reinterpret_cast<const u32x4 *>(p.set_slot + h);
        uint32_t stop = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (a[k] == kSetEmpty || ((a[k] ^ mine) & ~kChunkPosMask) == 0) stop |= 1u << k;
            if (b[k] == kSetEmpty || ((b[k] ^ mine) & ~kChunkPosMask) == 0) stop |= 16u << k;
        }
        stop &= ~0u << (e & 3);
        if (stop) {
            const uint32_t k = (uint32_t)__ffs((int)stop) - 1u;
            return k < 4 ? g + k : h + k - 4;
        }
        e = h + 3;
    }
}
// LOOKS: after a collision a wavefront most of which has missed looks at the entries that follow and goes on at the first that may serve.
// Where all ids are new the last entries of a call are a quarter full, and the last wavefronts had chains of eleven compare-and-swaps, a
// round trip each; so they are three trips long.  Where few are new the one after the next is nearly always free, and the look is one
// more, so calls of less than a workgroup per compute unit do without.  Loads of new ids, us: 12 calls of 262 144 677 / 662, 15 of 100 000 429 /
// 422, 6 of 262 144 into records 304 / 298, of 233 000 133 / 130.  (In all calls and wavefronts: sessions 1 to 3 % longer.)
template <bool LOOKS>
__device__ __forceinline__ uint32_t finish_insert(const Params &p, bool miss, int64_t id, uint32_t pos, const SetInsert &x)
{
    uint32_t ent = kNoEntry;
    const bool many = LOOKS && __popcll(__ballot(miss)) > kWave / 2;
    if (miss && x.from == lane_id()) {
        const uint32_t size = (uint32_t)kChunkSetEntries * (uint32_t)p.n;
        uint32_t e = x.e, seen = x.seen;
        ent = kEntered;                                       // first of its id so far
        while (seen != kSetEmpty) {
            if (((seen ^ x.mine) & ~kChunkPosMask) == 0) {
                const uint32_t other = seen & kChunkPosMask;
                if ((int64_t)other < p.n && p.ids[other] == id) {
                    p.note[other] = 1;
                    if (x.mine < seen) __hip_atomic_fetch_min(&p.set_slot[e], x.mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ent = 0;
                    break;
                }
            }
            if (LOOKS && many) e = next_entry(p, e, size, x.mine);
            else if (++e == size) e = 0;
            seen = try_entry(p, e, x.mine);
        }
        ent |= e;
    }
    ent = (uint32_t)__shfl((int)ent, x.from);
    return miss && x.first != pos ? ent & ~kEntered : ent;
}

// hint[pos] of a missed position: the first round at which its id may find a slot to claim, as far as Pass 1 can tell
// (without eviction: the first empty slot), at most kStartMax; kStartNever: there is none in its window.  (Of the others 0: a
// line that is written as a whole need not be fetched.)
constexpr uint32_t kStartMax = 0xFE, kStartNever = 0xFF;

// counters of one workgroup, three words: positions (hit, miss, invalid), probe lengths (hits, misses), outcomes
// (distinct ids, inserts, evictions); the first ones of all workgroups, then the second ones, then the third ones
__device__ __forceinline__ uint64_t pack3(uint32_t a, uint32_t b, uint32_t c)
{
    return (uint64_t)a | ((uint64_t)b << 16) | ((uint64_t)c << 32);
}
__device__ __forceinline__ uint32_t unpack3(uint64_t w, int k) { return (uint32_t)(w >> (16 * k)) & 0xFFFFu; }

// store_meta_wave over the workgroup (all threads reach it; barriers only where metadata is expiry steps).
template <int THREADS, int CELLS>
struct MergeArea {
    int64_t slot[THREADS];
    int32_t value[THREADS];
    uint16_t winner[CELLS];
};
template <int THREADS, int CELLS>
__device__ __forceinline__ void store_meta_block(const Tab &d, bool active, int64_t slot, int32_t value,
                                                 MergeArea<THREADS, CELLS> &s_m)
{
    static_assert((CELLS & (CELLS - 1)) == 0 && CELLS >= 2, "cells by the high bits of a product");
    if (d.evict != 3) {
        if (active) *meta_at(d, slot) = value;
        return;
    }
    const int t = threadIdx.x;
    const int cell = (int)((uint32_t)slot * 0x9E3779B1u >> (32 - __builtin_ctz(CELLS)));
    __syncthreads();                                 // the area may still be read from the call before
    s_m.slot[t] = active ? slot : -1;
    s_m.value[t] = value;
    if (active) s_m.winner[cell] = (uint16_t)t;
    __syncthreads();
    bool store = active;
    if (active) {
        const int o = s_m.winner[cell];
        if (o != t && s_m.slot[o] == slot) {
            __hip_atomic_fetch_max(&s_m.value[o], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            store = false;
        }
    }
    __syncthreads();
    if (store) __hip_atomic_fetch_max(meta_at(d, slot), s_m.value[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The first position of the id that was entered at ent[pos].
__device__ __forceinline__ uint32_t first_occurrence(const Params &p, uint32_t pos, uint32_t ent, uint8_t note)
{
    if (entered_alone(ent, note)) return pos;
    return p.set_slot[ent & ~kEntered] & kChunkPosMask;
}

// ALIGNED: the first look is at an aligned block (aligned_first says when).  A parameter of the kernel: with both looks in it, and a
// branch, 51 calls of 65 536 positions took 885 us instead of 862, sessions of ten steps of 4 000 positions of records 196 to 201 instead of 190
// to 196, of 60 000 255 to 260 instead of 251 to 257.
//
// SHIFT 1: a wavefront takes 32 positions, so that one pass holds the whole windows of up to 16 slots (see k_lookup_short),
// and the workgroup's 256 positions have 512 threads (whole_windows says when).  Longer windows gain nothing by it: what a look
// less saves, the barriers of 1 024 threads and the copies of an id that no longer meet in one wavefront cost.
//
// EVEN: where there are several workgroups per compute unit its memory pipe has more requests than it takes at a time, and the
// older wavefronts go first, with all their looks, so that the youngest come to their first one when the others are
// through (300 007 positions, windows of 32 slots at 95 % load: the first look is there after 2 to 15 us) and their
// chain of looks ends the call, alone.  With a priority that falls from look to look they end together.  even_looks says when.
//
// OVERLAP: metadata, outputs and counters are stored between the request of the scratch set's compare-and-swap and its answer, a round
// trip that nothing else then waits for; overlap_insert says when.  (With the durations of expiry steps requested together with
// the ids, here and in k_finalize_chunk: calls of 2 000 to 20 000 positions 15.0 to 16.0 -> 14.5 to 15.4 us, 51 of 65 536 in a row
// 924 -> 894, 12 of 262 144 new ids 726 -> 718.)
template <bool REC, int SHIFT, bool EVEN, bool OVERLAP, bool ALIGNED, bool LOOKS>
__global__ __launch_bounds__(kBlock << SHIFT, 4) void k_discover_chunk(Params p)
{
    constexpr int THREADS = kBlock << SHIFT, WAVES = THREADS / kWave, PER = kWave >> SHIFT;
    __shared__ ProbeReq s_req[WAVES][kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_code[WAVES][kWave * kFirstG];
    __shared__ uint32_t s_red[WAVES][5];
    __shared__ MergeArea<THREADS, 2 * kBlock> s_merge;

    const int lane = lane_id(), w = wave_id();
    const int64_t pos = (int64_t)blockIdx.x * kBlock + w * PER + lane;
    const bool in = lane < PER && pos < p.n;
    const Tab d = view(p.t0);
    const int64_t id = in ? p.ids[pos] : -1;
    int32_t duration = duration_of(p, d, in ? pos : 0);
    const bool valid = in && id >= 0;
    const uint64_t hash = hash_of(id, d.seed);
    const int64_t home = home_of(hash, d.N);
    bool fresh = false;
    int res = kProbeGoOn, q = 0;
    if constexpr (EVEN) __builtin_amdgcn_s_setprio(3);
    if constexpr (SHIFT == 0) {
        // the first block: the aligned one that holds the home slot, or the 8 slots from there on
        res = probe_first<false, REC, ALIGNED>(d, id, home, first_lane_bytes(d), s_req[w], s_code[w], p.step, &fresh, &q);
    }
    if constexpr (EVEN) __builtin_amdgcn_s_setprio(2);
    int left = SHIFT == 0 ? d.P - 1 : d.P;
    for (bool second = true;; second = false) {
        const bool need = valid && res == kProbeGoOn && q < d.P;
        if (!__any(need)) break;
        bool f = false;
        const int got = probe_more<false, REC>(d, d.sh, slots_up_to_widest(d), id, home, q, left, need, s_req[w], s_code[w], p.step, &f);
        if (need) { res = got; fresh = f; }
        if constexpr (EVEN) {
            if (second) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
    }
    if constexpr (EVEN) __builtin_amdgcn_s_setprio(3);
    const bool hit = valid && res >= 0, miss = valid && res < 0;
    asm volatile("" : "+v"(duration));               // (not added to before: made right behind the load, the sum waits for it)
    const SetInsert insert = begin_insert(p, miss, id, hash, (uint32_t)pos, reinterpret_cast<MetaMerge *>(s_req[w]));
    uint32_t e = kNoEntry;
    if constexpr (!OVERLAP) e = finish_insert<LOOKS>(p, miss, id, (uint32_t)pos, insert);
    const int64_t slot = hit ? wrap(home + res, d.N) : home;
    store_meta_block(d, hit && !(REC && fresh && d.evict != 3), slot, metadata_for(p, d, duration), s_merge);
    if (in) {
        p.out_slots[pos] = slot;
        if constexpr (!OVERLAP) p.ent[pos] = e;
        p.place[pos] = 0;
        uint32_t start = 0;
        if (d.evict == 0 && miss) {
            const uint32_t r = (uint32_t)(absent_len(res) - 1);
            start = res > kProbeAbsent ? kStartNever : r < kStartMax ? r : kStartMax;
        }
        p.hint[pos] = (uint8_t)start;
    }
    if (p.out_stats) {
        const uint32_t hits = (uint32_t)__popcll(__ballot(hit)), misses = (uint32_t)__popcll(__ballot(miss));
        const uint32_t invalid = (uint32_t)__popcll(__ballot(in && !valid));
        const uint32_t hit_len = wave_sum32(hit ? (uint32_t)res + 1u : 0u);
        const uint32_t miss_len = wave_sum32(miss ? (uint32_t)(res <= kProbeAbsent ? absent_len(res) : d.P) : 0u);
        if (lane == 0) {
            s_red[w][0] = hits;
            s_red[w][1] = misses;
            s_red[w][2] = invalid;
            s_red[w][3] = hit_len;
            s_red[w][4] = miss_len;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t[5] = {0, 0, 0, 0, 0};
            for (int i = 0; i < WAVES; ++i)
                for (int k = 0; k < 5; ++k) t[k] += s_red[i][k];
            p.wg_words[blockIdx.x] = pack3(t[0], t[1], t[2]);
            p.wg_words[gridDim.x + blockIdx.x] = (uint64_t)t[3] | ((uint64_t)t[4] << 32);
        }
    }
    if constexpr (OVERLAP) {
        e = finish_insert<LOOKS>(p, miss, id, (uint32_t)pos, insert);
        if (in) p.ent[pos] = e;
    }
}

// What the lanes of a workgroup leave for k_finalize_chunk: which evicted which slot (evicted: lanes with a slot in
// `slot`), and the workgroup's outcome counts.  Reached by all threads.
template <int WAVES>
__device__ __forceinline__ void leave_outcomes(const Params &p, bool agent, bool inserted, bool evicted, int64_t slot,
                                               uint32_t (&s_red)[WAVES][3])
{
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const uint64_t em = __ballot(evicted);
    const uint32_t agents = (uint32_t)__popcll(__ballot(agent)), ins = (uint32_t)__popcll(__ballot(inserted));
    if (lane == 0) {
        s_red[w][0] = agents;
        s_red[w][1] = ins;
        s_red[w][2] = (uint32_t)__popcll(em);
    }
    __syncthreads();
    uint32_t before = 0;
    for (int i = 0; i < w; ++i) before += s_red[i][2];
    if (evicted) p.evicted[(int64_t)blockIdx.x * kBlock + before + __popcll(em & ((1ull << lane) - 1ull))] = slot;
    if (threadIdx.x == 0) {
        uint32_t t[3] = {0, 0, 0};
        for (int i = 0; i < WAVES; ++i)
            for (int k = 0; k < 3; ++k) t[k] += s_red[i][k];
        p.wg_words[2 * gridDim.x + blockIdx.x] = pack3(t[0], t[1], t[2]);
    }
}

__device__ __forceinline__ void note_place(const Params &p, uint32_t pos, uint32_t place)
{
    __hip_atomic_fetch_max(&p.place[pos], place, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// READ_BACK: a wavefront of which most have missed reads the set back for all of them, notes or not: calls of about one to two
// workgroups per compute unit (read_back_groups).  There the claims of all wavefronts, if they read their
// windows at once, go out within a microsecond or two, and the atomics then run at 9 instead of 27 G/s: 131 000 new ids in a
// table of five times as many slots, the same 151 K atomics either way (0.3 % apart), of which each wavefront waits 15 us for
// its first and k_allocate_chunk takes 22.7 us (14 to 28); with the set read in front 17.7.  From 145 000 ids on the wait is 5.5
// us without it.  Why a burst of that length is slow, and longer ones are not, is not known.
template <bool REC, bool READ_BACK>
__global__ __launch_bounds__(kBlock, 4) void k_allocate_chunk(Params p)
{
    __shared__ __attribute__((aligned(16))) uint8_t s_code[kWavesPerBlock][kWave * kAllocG];
    __shared__ ClaimReq s_req[kWavesPerBlock][kWave];
    __shared__ uint32_t s_red[kWavesPerBlock][3];

    const int w = wave_id();
    const int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool in = pos < p.n;
    const Tab d = view(p.t0);
    const int64_t from = in ? pos : 0;               // (no branch between the loads)
    args_now(p.ent, p.ids, p.hint, p.note, p.set_slot, p.list, p.step, d.I, d.M, d.N, d.seed, d.P, d.ttl, d.evict, d.sh);
    uint32_t e = p.ent[from];
    const int64_t id = p.ids[from];
    uint32_t start = (uint32_t)p.hint[from];         // (anything where the position did not miss)
    const uint8_t note = p.note[from];
    if (!in) e = kNoEntry;
    const bool have = e != kNoEntry;
    uint32_t first = 0;
    const bool read_back = READ_BACK && __popcll(__ballot(have)) > kWave / 2;
    // (looked at here: compared in the branch that reads it, calls of 262 144 and 400 000 new ids 23.5 -> 24.1 and 31.4 -> 32.2)
    uint32_t met = read_back ? 1u : note;
    asm volatile("" : "+v"(met));
    if (have) first = first_occurrence(p, (uint32_t)pos, e, (uint8_t)met);
    else start = kStartNever;

    Claimant c;
    c.active = start != kStartNever;                 // the first blocks are requested before the election is known
    c.pos = (uint32_t)pos;
    c.home = home_slot(id, d.seed, d.N);
    c.q = (int32_t)start;
    const int32_t bound = expiry_bound(d, p.step);
    const bool aligned = (d.N << (3 + d.sh)) > kCachedTableBytes;
    int64_t was = (int64_t)kTagBase;                // what the slot of the lane's last claim held
    int64_t slot = 0;
    uint32_t own = 0;
    for (bool later = false;; later = true) {
        const uint64_t am = __ballot(c.active);
        if (!am) break;
        const ClaimStage st = claim_blocks<REC>(d, c, am, later || !aligned ? blocks_shift(uniform32(__popcll(am)), d.P) : 0, bound,
                                                aligned && !later, s_code[w], s_req[w]);
        if (!later) c.active = c.active && first == (uint32_t)pos;      // else: a later copy of the id
        claim_walk<16, 2>(d, c, st, s_code[w], s_req[w], claim_in_table,
                   [&](uint32_t who, int32_t round, int64_t at, int64_t old) {
                       if (who == (uint32_t)pos) own = (uint32_t)round + 1u;
                       else note_place(p, who, (uint32_t)round + 1u);
                       was = old;
                       slot = at;
                   },
                   // (also for the lane's own: its chain may come back to it, in a table hardly longer than a window)
                   [&](uint32_t who) {
                       if (who == (uint32_t)pos) own = kPlaceNone;
                       else note_place(p, who, kPlaceNone);
                   });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // s_code and s_req are written again
    }
    if (in) p.list[pos] = !have ? kNoEntry : first == (uint32_t)pos ? kOwnPlace | own : first;
    leave_outcomes<kWavesPerBlock>(p, have && first == (uint32_t)pos, was == -1, was >= 0, slot, s_red);
}

// The claims under the LRU policy (max_probe <= 8 T <= 64).  The workgroup first lists its claimants, so that its groups of
// 8 lanes get them evenly: a wavefront of 64 positions has a handful, which it would serve one or two at a time
// (300 007 positions, 10 % of them claimants with windows of 32 slots: 43 -> 16 us).  Claimants beyond the groups wait for
// the first ones' chains, so the workgroup is as large as the compute unit has room for (lru_chunk_threads).  SEEN: crowded_lru.
template <int T, bool REC, bool SEEN, int THREADS>
__global__ __launch_bounds__(THREADS, T == 8 || THREADS > kBlock ? 4 : 6) void k_allocate_lru_chunk(Params p)
{
    constexpr int G = kLruG, WAVES = THREADS / kWave, GROUPS = THREADS / G;
    __shared__ int64_t s_home[kBlock];
    __shared__ int64_t s_slot[kBlock];               // of the claimant's chain of claims: the slot not claimed before
    __shared__ uint32_t s_pos[kBlock];
    __shared__ uint32_t s_own[kBlock];               // its place
    __shared__ uint8_t s_outcome[kBlock];            // 0: none, 1: it was empty, 2: it held an id
    __shared__ uint32_t s_red[WAVES][3];
    const int lane = lane_id(), w = wave_id();
    const Tab d = view(p.t0);
    const int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool in = (int)threadIdx.x < kBlock && pos < p.n;
    const int64_t from = in ? pos : 0;               // (no branch between the loads, see k_finalize_chunk: 20 011 positions 24.7 -> 24.3 us)
    args_now(p.ent, p.ids, p.note, p.set_slot, p.list, p.place, p.evicted, p.wg_words, p.step, d.I, d.M, d.N, d.seed, d.P, d.sh);
    uint32_t e = p.ent[from];
    const int64_t id = p.ids[from];
    const uint8_t note = p.note[from];
    if (!in) e = kNoEntry;
    const bool have = e != kNoEntry;
    uint32_t first = 0;
    if (have) first = first_occurrence(p, (uint32_t)pos, e, note);
    const bool agent = have && first == (uint32_t)pos;
    if (in && !agent) p.list[pos] = have ? first : kNoEntry;
    const uint64_t am = __ballot(agent);
    if (lane == 0) s_red[w][0] = (uint32_t)__popcll(am);
    __syncthreads();
    int at = __popcll(am & ((1ull << lane) - 1ull)), count = 0;
    for (int i = 0; i < WAVES; ++i) {
        if (i < w) at += (int)s_red[i][0];
        count += (int)s_red[i][0];
    }
    if (agent) {
        s_pos[at] = (uint32_t)pos;
        s_home[at] = home_slot(id, d.seed, d.N);
        s_own[at] = 0;
        s_outcome[at] = 0;
    }
    __syncthreads();
    const int g = (int)threadIdx.x / G;
    int i = g;
    int64_t home = i < count ? s_home[i] : 0;
    LruSlots<T> x = load_lru_slots<T, REC>(d, i < count, home);
    for (; __any(i < count); i += GROUPS) {
        // the window of the next claimant is requested before this one is served
        const bool more = i + GROUPS < count;
        const int64_t home2 = more ? s_home[i + GROUPS] : 0;
        const LruSlots<T> x2 = load_lru_slots<T, REC>(d, more, home2);
        claim_group_lru<T, REC, SEEN>(p, d, i < count, i < count ? s_pos[i] : 0u, home, x,
                                [&](uint32_t who, int32_t choice, int32_t round, int64_t slot, int64_t old) {
                                    if (lane % G != 0) return;
                                    const uint32_t place = (uint32_t)choice << 16 | (uint32_t)(round + 1);
                                    if (who == s_pos[i]) s_own[i] = place;
                                    else note_place(p, who, place);
                                    if (is_tag(old)) return;
                                    s_slot[i] = slot;
                                    s_outcome[i] = old == -1 ? 1 : 2;
                                },
                                [&](uint32_t who) {
                                    if (lane % G != 0) return;
                                    if (who == s_pos[i]) s_own[i] = kPlaceNone;
                                    else note_place(p, who, kPlaceNone);
                                });
        home = home2;
        x = x2;
    }
    __syncthreads();
    const bool mine = (int)threadIdx.x < count;
    if (mine) p.list[s_pos[threadIdx.x]] = kOwnPlace | s_own[threadIdx.x];
    const int outcome = mine ? s_outcome[threadIdx.x] : 0;
    leave_outcomes<WAVES>(p, mine, outcome == 1, outcome == 2, outcome == 2 ? s_slot[threadIdx.x] : 0, s_red);
}

// Sum over the workgroup, in every thread.  s_sum: one word per wavefront; to be reached by all threads.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long x, unsigned long long *s_sum)
{
    const unsigned long long t = wave_sum(x);
    __syncthreads();                                 // s_sum may still be read from an earlier sum
    if (lane_id() == 0) s_sum[threadIdx.x / kWave] = t;
    __syncthreads();
    unsigned long long v = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) v += s_sum[i];
    return v;
}

// The call's counters, from the words of all `groups` workgroups: three tasks, each the work of a workgroup of its own in
// front of the others: at the end of the first three it was the last 1.7 us of the kernel.  Together with the counts of
// the workgroups before being requested at the start: 51 calls of 65 536 positions 1 057 -> 1 027 us, 12 of 262 144
// 806 -> 796.
constexpr int kPublishTasks = 3;
// Workgroups in front of the others: one for each die, of which those beyond the tasks have nothing to do.  The dies take the
// workgroups of a launch in turn, so a workgroup then runs on the die that has discovered and allocated for its positions and finds
// what it reads and overwrites (words, places, notes, its part of the set, outputs) in that die's L2.  (Three in front: 51 calls
// of 65 536 positions 1 028 us, 12 of 20 011 with expiry steps 328; eight 1 014 and 324.  A launch that reads and writes 16 MB
// which the launch before has written takes 4.7 us on the same die, 12.8 on another.)
constexpr int kPublishGroups = kDies;
static_assert(kPublishTasks <= kPublishGroups, "one workgroup per task");
__device__ __forceinline__ void publish_words(const Params &p, int task, int groups, unsigned long long *s_sum)
{
    if (task < 2 && !p.out_stats) return;
    unsigned long long a = 0, b = 0, c = 0;
    for (int i = threadIdx.x; i < groups; i += kBlock) {
        const uint64_t v = p.wg_words[task * groups + i];
        if (task == 1) {
            a += (uint32_t)v;
            b += v >> 32;
        } else {
            a += unpack3(v, 0);
            b += unpack3(v, 1);
            c += unpack3(v, 2);
        }
    }
    a = block_sum(a, s_sum);
    b = block_sum(b, s_sum);
    c = block_sum(c, s_sum);
    if (threadIdx.x != 0) return;
    if (task == 0) {
        p.out_stats[kHitPos] = (int64_t)a;
        p.out_stats[kMissPos] = (int64_t)b;
        p.out_stats[kInvalidPos] = (int64_t)c;
    } else if (task == 1) {
        p.out_stats[kHitProbeSum] = (int64_t)a;
        p.out_stats[kMissProbeSum] = (int64_t)b;
    } else {
        p.out_num_evicted[0] = (int64_t)c;
        if (p.out_stats) {
            p.out_stats[kDistinctMiss] = (int64_t)a;
            p.out_stats[kInserts] = (int64_t)b;
            p.out_stats[kEvictions] = (int64_t)c;
            p.out_stats[kCollisions] = (int64_t)(a - b - c);
        }
    }
}

__global__ __launch_bounds__(kBlock, 8) void k_finalize_chunk(Params p)
{
    __shared__ int64_t s_row[kBlock];
    __shared__ unsigned long long s_sum[kWavesPerBlock];
    __shared__ uint32_t s_base[kWavesPerBlock];
    __shared__ MergeArea<kBlock, 2 * kBlock> s_merge;

    const int groups = (int)gridDim.x - kPublishGroups, group = (int)blockIdx.x - kPublishGroups;
    if (group < 0) {
        if ((int)blockIdx.x < kPublishTasks) publish_words(p, (int)blockIdx.x, groups, s_sum);
        return;
    }
    const int64_t pos = (int64_t)group * kBlock + threadIdx.x;
    const bool in = pos < p.n;
    const Tab d = view(p.t0);
    // Nothing is asked between the loads and nothing is done with one before the last of them has been requested: two round
    // trips, this workgroup's words and then, for copies, those of their first occurrences.  (A choice or a scalar made right
    // behind a load waits for it, and for all stores before it: the counts of the workgroups before were a chain of their own,
    // one to eight round trips long.  With k_allocate_chunk's loads likewise: 51 calls of 65 536 positions 972 -> 926 us, 12 of
    // 20 011 with expiry steps 321 -> 309, 12 of 262 144 new ids 753 -> 731.)
    const int64_t at = in ? pos : 0;
    args_now(p.list, p.ids, p.place, p.set_slot, p.note, p.wg_words, p.evicted, p.out_slots, p.r_rows, p.ttls, p.step, p.g_num_rows, d.I, d.M, d.N,
             d.seed, d.evict, d.sh);
    uint32_t word = p.list[at];
    const int64_t id = p.ids[at];
    uint32_t moved = p.place[at];
    int32_t duration = duration_of(p, d, at);
    // what the evicted slots of this workgroup need, requested now: the slots, and the counts of the workgroups before (the
    // upper halves of their words)
    const uint64_t *const outcomes = p.wg_words + 2 * groups;
    uint32_t evicted_word = reinterpret_cast<const uint32_t *>(outcomes)[2 * group + 1];
    constexpr int kMostBefore = (int)(kChunkMaxBatch / kBlock / kBlock);
    uint32_t before[kMostBefore];
#pragma unroll
    for (int k = 0; k < kMostBefore; ++k) {
        before[k] = 0;
        const int i = k * kBlock + (int)threadIdx.x;
        if (d.evict != 0 && k * kBlock < group) before[k] = reinterpret_cast<const uint32_t *>(outcomes)[2 * (i < group ? i : group) + 1];
    }
    const int64_t evicted_slot = d.evict != 0 ? p.evicted[at] : 0;     // (of the threads below `evicted`)
    if (!in) word = kNoEntry;
    const bool have = word != kNoEntry, agent = have && (word & kOwnPlace) != 0;
    uint32_t place = word & ~kOwnPlace;
    if (have && !agent) {
        moved = p.place[word];
        place = p.list[word] & ~kOwnPlace;
    }
    // (meanwhile: where this workgroup's part of the evicted list begins, and the rows to reset)
    asm volatile("" : "+v"(evicted_word));           // (a scalar from here on: made one right behind the load it waits for it)
    const int evicted = uniform32((int)(evicted_word & 0xFFFFu));
    if (evicted > 0) {
        uint32_t base = 0;
#pragma unroll
        for (int k = 0; k < kMostBefore; ++k) {
            asm volatile("" : "+v"(before[k]));      // (selected here: a choice right behind a load waits for it)
            if (k * kBlock + (int)threadIdx.x < group) base += before[k] & 0xFFFFu;
        }
        base = wave_sum32(base);
        if (lane_id() == 0) s_base[wave_id()] = base;
        if (p.r_rows && (int)threadIdx.x < evicted)
            s_row[threadIdx.x] = evicted_slot >= p.g_num_rows ? evicted_slot % p.g_num_rows : evicted_slot;
    }
    const bool refresh = agent || (have && p.ttls && d.evict == 3);
    bool moves_in = false;
    int64_t slot = 0;
    if (have) {
        place = moved > place ? moved : place;
        const bool placed = place != 0 && place != kPlaceNone;
        const int64_t home = home_slot(id, d.seed, d.N);
        if (d.evict == 2) place &= 0xFFFFu;
        slot = placed ? wrap(home + (int64_t)(place - 1u), d.N) : home;
        // the claim becomes the id, metadata gets its value (Algorithm 1, Pass 2); without a claim: Case 3, the home
        // slot's metadata is refreshed; with per-feature retention a later copy may ask for a later expiry step
        if (agent && placed) {
            if (d.evict != 3) *id_at(d, slot) = id;
            else moves_in = true;
        }
        p.out_slots[pos] = slot;
    }
    // the scratch set is left empty again (all of it, in one coalesced store, instead of the entries that were used, one at
    // a time; behind all loads, none of which then waits for it)
    static_assert(kChunkSetEntries == 4, "cleared as one vector of four");
    if (in) {
        reinterpret_cast<u32x4 *>(p.set_slot)[pos] = u32x4(kSetEmpty);
        p.note[pos] = 0;
    }
    asm volatile("" : "+v"(duration));               // (see k_discover_chunk)
    store_meta_block(d, refresh, slot, metadata_for(p, d, duration), s_merge);
    if (moves_in) *id_at(d, slot) = id;              // (expiry steps: see store_meta)
    if (evicted > 0) {
        __syncthreads();
        uint32_t base = 0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock; ++i) base += s_base[i];
        const int64_t at = (int64_t)base + threadIdx.x;
        if ((int)threadIdx.x < evicted && at < p.t0.ev_cap) p.out_evicted[at] = evicted_slot;
        if (p.r_rows) {
            // every wavefront resets a quarter of the rows
            const int per = (evicted + kWavesPerBlock - 1) / kWavesPerBlock, w = wave_id();
            const int lo = w * per < evicted ? w * per : evicted;
            const int hi = lo + per < evicted ? lo + per : evicted;
            reset_staged_rows(p, s_row + lo, hi - lo);
        }
    }
}

}  // namespace mpzch

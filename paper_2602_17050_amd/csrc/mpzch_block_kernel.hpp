// The training remap of the smallest batches: one workgroup, one launch.
//
// Three launches cost the host some 12 us and the GPU two waits of 1.6 us between kernels, which is most of a step of
// a thousand ids.  One workgroup of up to 1 024 threads has barriers instead of launches, and what the phases hand to
// each other (scratch set, claims, places, counters, evicted rows) stays in LDS, so the call needs no scratch memory.  The
// phases are those of mpzch_chunk_kernels.hpp.  Remap with row reset, us per call, against three launches: 64 to 512
// positions 14 to 17.5 -> 7 to 9, 1 024 positions 13.8 to 17.7 -> 7.0 to 12.4; with two positions per thread (2 048) the
// one compute unit took as long as three launches do (10.8 to 21.8 against 13.8 to 19.2), so the line is drawn at 1 024.
// (Claimants listed, so that they take up as few wavefronts as they can, 83.9 against 82.6 us for the 8-step pass: a list
// costs a barrier, and a stage of few claimants loads only the rows they ask for.)
#pragma once
#include "mpzch_chunk_kernels.hpp"

namespace mpzch {

constexpr int kOneBlock = 1024;
constexpr int kOneBlockWaves = kOneBlock / kWave;
// Entries of the scratch set for each thread.  Every collision is a chain of two LDS operations, which the wavefront waits for.
// Sessions of 12 steps, us, two entries / four / eight: 256 positions 98.5 / 97.2 / 97.6 and, of records, 109.4 / 108.1 / 108.3; 700 with
// expiry steps 175.7 / 173.6 / 174.1; 1 024 121.6 / 121.1 / 122.2.  (Four of the claims' map as well: 0.2 % less time, 32 KB more LDS.)
constexpr int kOneBlockSet = 4;

struct OneBlockArea {
    ClaimReq req[kOneBlockWaves][kWave];                     // (Pass 1: the requests of its probes)
    alignas(16) uint8_t code[kOneBlockWaves][kWave * kAllocG];
    int64_t id[kOneBlock];
    int64_t row[kOneBlock];                                  // rows to reset
    uint32_t set[kOneBlockSet * kOneBlock];
    uint64_t claim_slot[2 * kOneBlock];                      // claims: address of the slot's identity (0: free entry)
    int64_t claim_tag[2 * kOneBlock];                        // and the best claim of it so far (0: none)
    uint32_t place[kOneBlock];
    uint32_t count[kStatCount];                              // (probe lengths of 1 024 positions fit 32 bits)
    MergeArea<kOneBlock, 2 * kOneBlock> merge;
};

template <bool REC>
__global__ __launch_bounds__(kOneBlock) void k_remap_block(Params p)
{
    __shared__ OneBlockArea s;
    const int lane = lane_id(), w = wave_id(), t = threadIdx.x, threads = blockDim.x;
    const int n = (int)p.n;
    const Tab d = view(p.t0);
    ProbeReq *const s_probe = reinterpret_cast<ProbeReq *>(s.req[w]);

    const bool in = t < n;
    const uint32_t pos = (uint32_t)t;
    const int64_t id = in ? p.ids[t] : -1;
    const bool valid = in && id >= 0;
    const uint64_t hash = hash_of(id, d.seed);
    const int64_t home = home_of(hash, d.N);
    for (int i = 2 * threads + t; i < kOneBlockSet * threads; i += threads) s.set[i] = kSetEmpty;
    for (int i = t; i < 2 * threads; i += threads) {
        s.set[i] = kSetEmpty;
        s.claim_slot[i] = 0;
        s.claim_tag[i] = 0;
    }
    if (t < kStatCount) s.count[t] = 0;
    s.id[t] = id;
    s.place[t] = 0;
    __syncthreads();

    // Pass 1.  (Blocks of the next 8 slots: round trips count here, not lines.)
    bool fresh = false;
    int q = 0;
    int res = probe_first<false, REC, false>(d, id, home, first_lane_bytes(d), s_probe, s.code[w], p.step, &fresh, &q);
    int left = d.P - 1;
    for (;;) {
        const bool need = valid && res == kProbeGoOn && q < d.P;
        if (!__any(need)) break;
        bool f = false;
        const int got = probe_more<false, REC>(d, d.sh, slots_up_to_widest(d), id, home, q, left, need, s_probe, s.code[w], p.step, &f);
        if (need) { res = got; fresh = f; }
    }
    const bool hit = valid && res >= 0, miss = valid && res < 0;
    int64_t slot = hit ? wrap(home + res, d.N) : home;
    uint32_t e = kNoEntry;
    if (miss) {
        const uint32_t size = (uint32_t)(kOneBlockSet * threads);
        uint32_t at = __umulhi((uint32_t)hash, size);
        for (;;) {
            uint32_t expected = kSetEmpty;
            if (__hip_atomic_compare_exchange_strong(&s.set[at], &expected, pos, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP))
                break;
            if (s.id[expected] == id) {
                if (pos < expected)
                    __hip_atomic_fetch_min(&s.set[at], pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                break;
            }
            if (++at == size) at = 0;
        }
        e = at;
    }
    store_meta_block(d, hit && !(REC && fresh && d.evict != 3), slot, hit ? meta_value(p, d, pos) : 0, s.merge);
    if (p.out_stats) {
        const uint32_t hits = (uint32_t)__popcll(__ballot(hit)), misses = (uint32_t)__popcll(__ballot(miss));
        const uint32_t invalid = (uint32_t)__popcll(__ballot(in && !valid));
        const uint32_t hit_len = wave_sum32(hit ? (uint32_t)res + 1u : 0u);
        const uint32_t miss_len = wave_sum32(miss ? (uint32_t)(res <= kProbeAbsent ? absent_len(res) : d.P) : 0u);
        if (lane == 0) {
            atomicAdd(&s.count[kHitPos], hits);
            atomicAdd(&s.count[kMissPos], misses);
            atomicAdd(&s.count[kInvalidPos], invalid);
            atomicAdd(&s.count[kHitProbeSum], hit_len);
            atomicAdd(&s.count[kMissProbeSum], miss_len);
        }
    }
    // every id that was resident has been refreshed, every first occurrence is elected
    __syncthreads();

    // A claim is an atomic minimum of the claimant's tag, as in the table, but on an entry of a map in LDS: all claimants of
    // the call are in this workgroup, and the table keeps what it held until every claim stands.  (Claims are made one after
    // the other, each waiting for the one before.  8 steps of 1 024 positions on 4 096 slots, the whole pass: 94.9 us with
    // the claims in memory, 90.3 so.)  An entry comes with a claim that
    // stands, if only until a better one, so there are no more entries than claimants: at most half of the map.
    auto claim_in_map = [&](uint64_t address, int64_t tag, uint32_t occ) -> int64_t {
        const uint32_t size = 2u * (uint32_t)threads;
        uint32_t at = __umulhi((uint32_t)(address >> 3) * 0x9E3779B1u, size);
        for (;;) {
            uint64_t holds = 0;
            if (__hip_atomic_compare_exchange_strong(&s.claim_slot[at], &holds, address, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP) ||
                holds == address)
                break;
            if (++at == size) at = 0;
        }
        const int64_t old = __hip_atomic_fetch_min(&s.claim_tag[at], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return old != 0 ? old : occ ? 0 : -1;
    };

    // claims
    const int32_t bound = expiry_bound(d, p.step);
    const uint32_t first = e != kNoEntry ? s.set[e] : kNoEntry;
    uint32_t outcome = 0;                                    // 1 = this lane's last claim was an insert, 2 = an eviction
    int64_t claimed = 0;
    Claimant cl;
    cl.active = first == pos;
    cl.pos = pos;
    cl.q = 0;
    cl.home = home;
    const uint32_t distinct = (uint32_t)__popcll(__ballot(cl.active));
    for (;;) {
        const uint64_t am = __ballot(cl.active);
        if (!am) break;
        const ClaimStage st = claim_blocks<REC>(d, cl, am, blocks_shift(uniform32(__popcll(am)), d.P), bound, false, s.code[w], s.req[w]);
        claim_walk<32, 1>(d, cl, st, s.code[w], s.req[w], claim_in_map,
                   [&](uint32_t who, int32_t round, int64_t at, int64_t old) {
                       atomicMax(&s.place[who], (uint32_t)round + 1u);
                       outcome = old == -1 ? 1u : old >= 0 ? 2u : 0u;
                       claimed = at;
                   },
                   [&](uint32_t who) { atomicMax(&s.place[who], kPlaceNone); });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    const uint64_t em = __ballot(outcome == 2u);
    const uint32_t ins = (uint32_t)__popcll(__ballot(outcome == 1u));
    uint32_t base = 0;
    if (lane == 0 && distinct) atomicAdd(&s.count[kDistinctMiss], distinct);
    if (lane == 0 && ins) atomicAdd(&s.count[kInserts], ins);
    if (lane == 0 && em) base = atomicAdd(&s.count[kEvictions], (uint32_t)__popcll(em));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (outcome == 2u) {
        const uint32_t at = base + (uint32_t)__popcll(em & ((1ull << lane) - 1ull));
        if ((int64_t)at < p.t0.ev_cap) p.out_evicted[at] = claimed;
        if (p.r_rows) s.row[at] = claimed >= p.g_num_rows ? claimed % p.g_num_rows : claimed;
    }
    // every claim stands
    __syncthreads();

    bool refresh = false;
    if (first != kNoEntry) {
        const uint32_t place = s.place[first];
        const bool placed = place != 0 && place != kPlaceNone, agent = first == pos;
        if (placed) slot = wrap(home + (int64_t)(place - 1u), d.N);
        if (agent && placed) *id_at(d, slot) = id;
        refresh = agent || (p.ttls && d.evict == 3);
    }
    if (in) p.out_slots[pos] = slot;
    store_meta_block(d, refresh, slot, refresh ? meta_value(p, d, pos) : 0, s.merge);
    const int evicted = (int)s.count[kEvictions];
    if (p.r_rows && evicted > 0) {
        const int waves = (threads + kWave - 1) / kWave, per = (evicted + waves - 1) / waves;
        const int lo = w * per < evicted ? w * per : evicted;
        const int hi = lo + per < evicted ? lo + per : evicted;
        reset_staged_rows(p, s.row + lo, hi - lo);
    }
    if (t == 0) p.out_num_evicted[0] = evicted;
    if (p.out_stats && t < kStatCount)
        p.out_stats[t] = t == kCollisions ? (int64_t)(s.count[kDistinctMiss] - s.count[kInserts] - s.count[kEvictions])
                                          : (int64_t)s.count[t];
}

}  // namespace mpzch

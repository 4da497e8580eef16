// Host side of the C ABI declared in include/mpzch.h: argument checks, scratch management and
// kernel launches on the caller's stream.  No call here synchronises with the host except
// where the header says so (scratch growth, descriptor upload, timing read-out, destroy).
#include "../../include/mpzch.h"
#include "mpzch_block_kernel.hpp"
#include "mpzch_row_kernels.hpp"

#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

using namespace mpzch;

namespace {

struct TableCfg {
    int64_t num_slots;
    int32_t max_probe;
    int32_t kind;
    int32_t ttl;
    uint64_t seed;
    int32_t layout;                // MPZCH_LAYOUT_*
};

// ---- per-kernel timing --------------------------------------------------------------------
enum KernelId { KDiscover = 0, KAllocate, KFinalize, KLookup, KernelCount };
const char *const kKernelNames[KernelCount] = {"k_discover", "k_allocate", "k_finalize", "k_lookup"};

struct Timing {
    bool enabled = false;
    bool pass1_only = false;       // bracket k_discover / k_lookup only (two events per call instead of eight)
    int every = 1;                 // ... and of those launches only every `every`-th
    int64_t pass1_seen = 0;
    bool skipped = false;          // the launch between the last begin and end is not bracketed
    void set_mode(int32_t enable)
    {
        enabled = enable != 0;
        pass1_only = enable == 2 || enable == 3;
        every = enable == 3 ? 4 : 1;
        pass1_seen = 0;
    }
    struct Rec { int kernel; hipEvent_t a, b; };
    std::vector<Rec> used;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;

    bool begin(int kernel, hipStream_t s)
    {
        skipped = !enabled || (pass1_only && kernel != KDiscover && kernel != KLookup);
        if (!skipped && pass1_only) skipped = (pass1_seen++ % every) != every - 1;
        if (skipped) return true;
        std::pair<hipEvent_t, hipEvent_t> ev;
        if (!pool.empty()) {
            ev = pool.back();
            pool.pop_back();
        } else {
            if (hipEventCreate(&ev.first) != hipSuccess) return false;
            if (hipEventCreate(&ev.second) != hipSuccess) { (void)hipEventDestroy(ev.first); return false; }
        }
        used.push_back({kernel, ev.first, ev.second});
        return hipEventRecord(ev.first, s) == hipSuccess;
    }
    bool end(hipStream_t s)
    {
        if (skipped) return true;
        return hipEventRecord(used.back().b, s) == hipSuccess;
    }
    mpzch_status_t collect(const char **names, double *ms, int64_t *launches, int32_t cap, int32_t *count)
    {
        double acc[KernelCount] = {0};
        int64_t cnt[KernelCount] = {0};
        for (auto &r : used) {
            if (hipEventSynchronize(r.b) != hipSuccess) return MPZCH_ERR_HIP;
            float t = 0.f;
            if (hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) return MPZCH_ERR_HIP;
            acc[r.kernel] += t;
            cnt[r.kernel]++;
            pool.push_back({r.a, r.b});
        }
        used.clear();
        int32_t k = 0;
        for (int i = 0; i < KernelCount && k < cap; ++i) {
            if (!cnt[i]) continue;
            names[k] = kKernelNames[i];
            ms[k] = acc[i];
            launches[k] = cnt[i];
            ++k;
        }
        *count = k;
        return MPZCH_OK;
    }
    void destroy()
    {
        for (auto &r : used) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
        for (auto &e : pool) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
        used.clear();
        pool.clear();
    }
};

// ---- device scratch -----------------------------------------------------------------------
// Grid caps in workgroups per compute unit.  8 is the measured best for Pass 1 (4 M positions: 197 us; 4 and 16 per unit
// 222 and 210) and for the kernels that walk the miss lists.  From 16 M positions on, where a wavefront has 32 chunks
// and more, twice as many even the ends out: whole calls over 26 tables, 8 / 16 per unit, us: records 20.8 M values
// 614 / 618, 28.6 M 727 / 727, 41.6 M 1 030 / 1 007; two tensors 763 / 751, 937 / 924, 1 513 / 1 466; below the line it
// costs (12.2 M values 354 / 373 and 430 / 440).  One table, 8 to 40 M positions, either layout: no difference beyond
// the runs' own.  Scratch is sized for up to kDiscoverBlocksPerCuMax.
constexpr int kDiscoverBlocksPerCuMax = 16;
constexpr int discover_blocks_per_cu() { return 8; }
constexpr int64_t kLongBatch = (int64_t)1 << 24;
constexpr int train_blocks_per_cu(int64_t n) { return n < kLongBatch ? discover_blocks_per_cu() : kDiscoverBlocksPerCuMax; }
static_assert(3 * sizeof(uint64_t) * discover_blocks_per_cu() <= sizeof(uint32_t) * kDiscoverBlocksPerCuMax * kWavesPerBlock, "the counter words of the workgroups of a one-chunk call fit seg_cnt");
constexpr int group_blocks_per_cu() { return 8; }

// Compute units of the current device, asked once per device and process (no handle state: read-only
// entry points take const handles).
mpzch_status_t device_cus(int *out)
{
    static std::mutex mu;
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MPZCH_ERR_HIP;
    if (dev < 0 || dev >= 64) return MPZCH_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!cus[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) return MPZCH_ERR_HIP;
        cus[dev] = n;
    }
    *out = cus[dev];
    return MPZCH_OK;
}

struct Scratch {
    char *base = nullptr;
    int64_t cap_n = 0;
    uint32_t *list = nullptr;
    uint32_t *ent = nullptr;
    uint32_t *first_of = nullptr;
    int64_t *list_id = nullptr;
    uint8_t *hint = nullptr;
    uint32_t *seg_cnt = nullptr;
    uint32_t *set_slot = nullptr;
    Control *ctl = nullptr;
    uint8_t *note = nullptr;
    Control *lookup_ctl = nullptr; // counter block of counting lookups while there is no scratch area
    bool dirty = false;            // a launch sequence was cut short: set and counters must be cleared before use
    bool owned = true;             // base came from hipMalloc (false: it points into the file-scope scratch array)
    int num_cus = 0;

    static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

    mpzch_status_t query_device()
    {
        if (num_cus) return MPZCH_OK;
        return device_cus(&num_cus);
    }

    // Where each array sits inside an area that serves batches of up to n positions: 30 bytes per
    // position (38 for the first kChunkMaxBatch) and a few small fixed areas.  What a call leaves empty: the set from o_set
    // to o_ctl (ones), counters and notes from there on (zeros).
    struct Layout {
        size_t o_list, o_ent, o_first, o_list_id, o_hint, o_seg, o_set, o_ctl, o_note, total;
    };
    static int64_t set_entries(int64_t n)
    {
        const int64_t chunk = kChunkSetEntries * (n < kChunkMaxBatch ? n : kChunkMaxBatch);
        return 2 * n > chunk ? 2 * n : chunk;
    }
    static Layout layout_for(int64_t n, int num_cus)
    {
        Layout L;
        const size_t max_blocks = (size_t)num_cus * kDiscoverBlocksPerCuMax;
        const size_t per_pos = 4 * ((size_t)n + 2 * kWave);   // list-shaped arrays: n + 128 entries
        L.o_list = 0;
        L.o_ent = L.o_list + align_up(per_pos);
        L.o_first = L.o_ent + align_up(per_pos);
        L.o_list_id = L.o_first + align_up(per_pos);
        L.o_hint = L.o_list_id + align_up(2 * per_pos);
        L.o_seg = L.o_hint + align_up((size_t)n + kWave);
        L.o_set = L.o_seg + align_up(4 * max_blocks * kWavesPerBlock);
        L.o_ctl = L.o_set + align_up(4 * (size_t)set_entries(n));
        L.o_note = L.o_ctl + align_up(sizeof(Control));
        L.total = L.o_note + align_up((size_t)n);
        return L;
    }
    void bind(char *area, const Layout &L, int64_t n)
    {
        base = area;
        list = (uint32_t *)(base + L.o_list);
        ent = (uint32_t *)(base + L.o_ent);
        first_of = (uint32_t *)(base + L.o_first);
        list_id = (int64_t *)(base + L.o_list_id);
        hint = (uint8_t *)(base + L.o_hint);
        seg_cnt = (uint32_t *)(base + L.o_seg);
        set_slot = (uint32_t *)(base + L.o_set);
        ctl = (Control *)(base + L.o_ctl);
        note = (uint8_t *)(base + L.o_note);
        cap_n = n;
    }

    mpzch_status_t ensure(int64_t n)
    {
        mpzch_status_t st = query_device();
        if (st != MPZCH_OK) return st;
        if (n <= cap_n && base) return MPZCH_OK;
        if (n < 1024) n = 1024;
        if (base) {
            if (hipDeviceSynchronize() != hipSuccess) return MPZCH_ERR_HIP;
            (void)hipFree(base);
            base = nullptr;
            cap_n = 0;
        }
        const Layout L = layout_for(n, num_cus);
        char *area = nullptr;
        if (hipMalloc((void **)&area, L.total) != hipSuccess) return MPZCH_ERR_ALLOC;
        bind(area, L, 0);
        // empty set (0xFFFFFFFF) and zero counters; set entries are re-emptied by every call, so
        // this is the only full clear
        if (hipMemset(base + L.o_set, 0xFF, (L.o_ctl - L.o_set)) != hipSuccess) return MPZCH_ERR_HIP;
        if (hipMemset(base + L.o_ctl, 0, L.total - L.o_ctl) != hipSuccess) return MPZCH_ERR_HIP;
        if (hipDeviceSynchronize() != hipSuccess) return MPZCH_ERR_HIP;
        cap_n = n;
        return MPZCH_OK;
    }
    // the counter block alone (a counting lookup needs nothing else): the scratch area's when there is one
    mpzch_status_t ensure_ctl(Control **out)
    {
        if (base) { *out = ctl; return MPZCH_OK; }
        if (!lookup_ctl) {
            if (hipMalloc((void **)&lookup_ctl, sizeof(Control)) != hipSuccess) { lookup_ctl = nullptr; return MPZCH_ERR_ALLOC; }
            if (hipMemset(lookup_ctl, 0, sizeof(Control)) != hipSuccess) return MPZCH_ERR_HIP;
            if (hipDeviceSynchronize() != hipSuccess) return MPZCH_ERR_HIP;
        }
        *out = lookup_ctl;
        return MPZCH_OK;
    }
    void release()
    {
        if (base && owned) { (void)hipDeviceSynchronize(); (void)hipFree(base); }
        if (lookup_ctl) { (void)hipDeviceSynchronize(); (void)hipFree(lookup_ctl); lookup_ctl = nullptr; }
        base = nullptr;
        cap_n = 0;
    }
};

int grid_for(int64_t items, int64_t items_per_block, int num_cus, int blocks_per_cu)
{
    int64_t b = (items + items_per_block - 1) / items_per_block;
    const int64_t cap = (int64_t)num_cus * blocks_per_cu;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

static_assert(kLruLongProbe == MPZCH_MAX_PROBE_LRU, "the LRU kernels hold max_probe / 64 slots per lane");

int32_t p_eff(const TableCfg &c) { return (int64_t)c.max_probe < c.num_slots ? c.max_probe : (int32_t)c.num_slots; }

TableDesc make_desc(const TableCfg &c, int64_t *I, int32_t *M, int64_t ev_begin, int64_t ev_cap)
{
    TableDesc d;
    d.I = I;
    d.M = M;
    d.N = c.num_slots;
    d.seed = c.seed;
    d.P = p_eff(c);
    d.ttl = c.ttl;
    d.evict = c.kind == MPZCH_EVICT_TTL ? 1 : c.kind == MPZCH_EVICT_LRU ? 2 : c.kind == MPZCH_EVICT_TTL_EXPIRY ? 3 : 0;
    d.sh = c.layout == MPZCH_LAYOUT_RECORDS ? 1 : 0;
    d.ev_begin = ev_begin;
    d.ev_cap = ev_cap;
    return d;
}

#define TRY(...)                                    \
    do {                                            \
        mpzch_status_t st__ = (__VA_ARGS__);        \
        if (st__ != MPZCH_OK) return st__;          \
    } while (0)

// A launch without the runtime's push and pop of its configuration and a look at the last error: 2.6 instead of 2.9 us on
// the host.  (Arguments in braces: one that does not fit its parameter, another pointer or a number that would be narrowed,
// does not compile.)
template <typename... P, typename... A>
mpzch_status_t launch(void (*kernel)(P...), int grid, int block, hipStream_t s, const A &...args)
{
    auto go = [&](P... values) {
        void *pointers[] = {&values...};
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), pointers, 0, s);
    };
    if (go(P{args}...) == hipSuccess) return MPZCH_OK;
    (void)hipGetLastError();
    return MPZCH_ERR_HIP;
}

// two-tensor tables from this size on (1 GiB of identities, four times the memory-side cache) are probed with
// non-temporal loads in training
constexpr int64_t kStreamingSlots = (int64_t)1 << 27;

// Workgroups of a lookup: two chunks per wavefront where there are enough to go round -- the second chunk's ids are under
// way while the first is looked up, and what both leave open is resolved at once -- and one below (500 K ids, windows of
// 32 slots, 13.9 -> 12.6 us; 4 M, four to eight chunks each before, 66 -> 59; 300 K would lose 3 %).
int lookup_grid(int64_t n, int num_cus)
{
    const bool two = n > (int64_t)6 * num_cus * kBlock;
    return grid_for(n, two ? 2 * kBlock : kBlock, num_cus, 16);
}

// Calls whose stores go out while the compare-and-swap of the scratch set is under way (k_discover_chunk): up to four workgroups per
// compute unit, of records two, of expiry steps three.  Beyond, the stores of the others are in the way of it.  Whole calls, behind / beside it, us, of 66 K 100 K 131 K
// 150 K 200 K 240 K 262 144 300 007 positions; steps in steady state with a tenth of the ids new, sessions of 12 steps on 1 M slots, loads of new ids:
//   records, 10 M slots, TTL, of 64   20.6/20.5 22.8/22.6 24.1/23.9 26.8/26.9 30.7/30.7 33.7/33.8 35.0/35.2 39.3/39.6
//   records, 80 M slots, TTL, of 24   20.4/20.1 22.6/22.4 23.6/23.5 25.9/26.2 30.0/30.3 33.6/34.1 35.4/35.9 39.8/39.2
//   records, sessions, TTL, of 64     250/249 288/285 319/317 348/346 397/397 438/436 471/467 518/520   loads 187/185 226/224 276/273 291/289 354/351 398/394 434/430
//   tensors, 20 M slots, TTL, of 64   20.7/20.3 23.1/22.9 24.6/24.4 26.8/26.8 30.3/30.3 33.8/33.9 36.5/36.2 40.8/40.5
//   tensors, 80 M slots, TTL, of 24   20.9/20.6 23.0/22.8 24.2/24.2 26.4/26.8 30.8/30.9 34.8/35.0 36.3/36.6 40.6/40.8
//   tensors, sessions, TTL, of 64     247/244 291/288 322/318 351/349 402/400 443/442 470/470 515/516   loads 188/186 225/222 276/272 282/281 349/346 393/391 428/425
// (Expiry steps, whose stores have barriers between them, lose where tables have room, sessions of 12 on 4 M slots, windows of 40, 66 K 567 / 573, 131 K
// 678 / 684, records 568 / 577, 675 / 693, and gain where they are crowded, on 1 M, of 16, 131 K 596 / 580, 180 K 729 / 688, records 609 / 584;
// 262 144, windows of 40, on 1 M 762 / 766, on 4 M 911 / 927, of 64, on 1 M, 638 / 646.)
constexpr bool overlap_insert(int64_t groups, int num_cus, bool records, bool expiry)
{
    return groups <= (records ? 2 : expiry ? 3 : 4) * (int64_t)num_cus;
}

// The longest windows, min(max_probe, num_slots), of the tables involved: of those under the LRU policy and of the others; 0 where
// there is none.
struct Windows {
    int32_t lru, other;
};
Windows windows_of(const TableDesc &d) { return d.evict == 2 ? Windows{d.P, 0} : Windows{0, d.P}; }
Windows longest(Windows a, Windows b) { return {a.lru > b.lru ? a.lru : b.lru, a.other > b.other ? a.other : b.other}; }

// Groups with one chunk per wavefront (up to 524 288 values on 256 compute units) run k_discover_tables_chunk where searches end
// early.  It looks from the home slot on, so every look of 8 slots of records is two lines, where k_discover_tables_records, whose
// first look is an aligned block, goes on with one each: long searches cost it more than the round trip that it saves, and the more
// so the more wavefronts share the memory.  How long they are the windows tell: an absent id's search ends at an empty slot, and LRU tables
// have none once they are full.  26 tables, Pass 1 of this over that of the other kernels, by workgroups per compute unit
// (1, 2, 3, 4, 6, 8); TTL at 95 % load, LRU full, 4 slots a value, in brackets 8:
//   records      LRU, of 32     0.69 0.82 0.87 0.93 0.92 1.00       of 64   0.79 0.82 0.93 1.03 1.03 1.12
//                of 110       (0.83 0.84 1.03 1.12 1.15 1.18)       of 520 (0.93 0.98 1.10 1.20 1.18 1.26)
//                TTL, of 128    0.81 0.88 0.86 0.91 0.95 0.99       of 256  0.81 0.85 0.86 0.92 0.95 1.03
//                of 520       (0.77 0.81 0.96 1.00 1.02 1.05)       of 1 000, whole steps (0.86 0.95 0.90 0.99 1.00 1.03)
//   two tensors  LRU, of 100    0.79 0.79 0.82 0.83 0.90 0.99       of 200 (0.83 0.86 0.86 1.02 1.02 1.15)
//   (8 slots are of 520       (0.88 0.94 0.94 1.07 1.05 1.17)
//   half a line) TTL, of 520  (0.74 0.81 0.96 0.97 0.94 0.94)       of 1 000, whole steps (0.86 0.96 0.88 0.95 0.90 0.95)
// (Eviction off counts as the others: its tables are full only when they are too small for their ids, and then windows of 520 take whole
// steps 0.85 0.93 1.11 1.15 1.15 1.17 over records, 0.86 0.86 0.95 1.12 1.05 1.12 over two tensors; half full they gain like the others.)
constexpr bool tables_by_chunk(int64_t groups, int num_cus, bool records, Windows w)
{
    int per_cu = 8;
    if (records) per_cu = w.lru > 64 ? 2 : w.lru > 32 ? 3 : w.other > 128 ? 6 : 8;
    else if (w.lru > 100) per_cu = w.lru > 256 ? 3 : 6;
    return groups <= (int64_t)per_cu * num_cus;
}

mpzch_status_t launch_discover(const Params &p, int grid, int num_cus, Windows windows, hipStream_t s)
{
    if (p.num_tables > 1 && p.seg_chunks == 1 && tables_by_chunk(grid, num_cus, p.all_records, windows)) {
        const bool overlap = overlap_insert(grid, num_cus, false, false);
        if (p.all_records && overlap) TRY(launch(k_discover_tables_chunk<true, true>, grid, kBlock, s, p));
        else if (p.all_records) TRY(launch(k_discover_tables_chunk<true, false>, grid, kBlock, s, p));
        else if (overlap) TRY(launch(k_discover_tables_chunk<false, true>, grid, kBlock, s, p));
        else TRY(launch(k_discover_tables_chunk<false, false>, grid, kBlock, s, p));
    }
    else if (p.num_tables > 1 && p.all_records) TRY(launch(k_discover_tables_records, grid, kBlock, s, p));
    else if (p.num_tables > 1) TRY(launch(k_discover_tables, grid, kBlock, s, p));
    else if (p.t0.sh) TRY(launch(k_discover_records, grid, kBlock, s, p));
    else if (p.t0.N >= kStreamingSlots) TRY(launch(k_discover_streaming, grid, kBlock, s, p));
    else TRY(launch(k_discover, grid, kBlock, s, p));
    return MPZCH_OK;
}

mpzch_status_t launch_lookup(const Params &p, int grid, hipStream_t s)
{
    if (p.num_tables > 1) TRY(launch(k_lookup_tables, grid, kBlock, s, lookup_args<true, false>(p, p.seg_chunks)));
    else TRY(launch(k_lookup, grid, kBlock, s, lookup_args<false, false>(p, p.seg_chunks)));
    return MPZCH_OK;
}

// A lookup of few ids (k_lookup_short).  max_p: the longest window of the tables involved.
bool short_lookup(Params &p, int32_t max_p)
{
    p.short_shift = window_shift(max_p);
    return p.n << p.short_shift <= kShortBlocks;
}
template <bool GATHER>
mpzch_status_t launch_lookup_short(const Params &p, hipStream_t s)
{
    const int per_block = kBlock >> p.short_shift;
    const int grid = (int)((p.n + per_block - 1) / per_block);
    if constexpr (!GATHER) {
        if (p.num_tables > 1) {
            TRY(launch(k_lookup_short<true, false>, grid, kBlock, s, lookup_args<true, false>(p, p.short_shift)));
            return MPZCH_OK;
        }
    }
    TRY(launch(k_lookup_short<false, GATHER>, grid, kBlock, s, lookup_args<false, GATHER>(p, p.short_shift)));
    return MPZCH_OK;
}

// max_p_lru: Windows::lru
template <bool MULTI, bool REC>
mpzch_status_t launch_allocate_lru(int32_t max_p_lru, const Params &p, int grid, hipStream_t s)
{
    // 8 lanes per claimant, with 1, 2, 4 or 8 slots each, whichever holds its window; the whole wavefront
    // with several slots per lane for longer probe ranges
    if (max_p_lru > kWave) TRY(launch(k_allocate_lru_long<MULTI>, grid, kWave, s, p));
    else if (max_p_lru <= 8) TRY(launch(k_allocate_lru<1, MULTI, REC>, grid, kWave, s, p));
    else if (max_p_lru <= 16) TRY(launch(k_allocate_lru<2, MULTI, REC>, grid, kWave, s, p));
    else if (max_p_lru <= 32) TRY(launch(k_allocate_lru<4, MULTI, REC>, grid, kWave, s, p));
    else TRY(launch(k_allocate_lru<8, MULTI, REC>, grid, kWave, s, p));
    return MPZCH_OK;
}

// The same where every wavefront has one chunk (max_p_lru <= 64).  Threads that serve the up to 256 claimants of a workgroup:
// 1 024 while there is one workgroup per compute unit, 512 up to two, with windows of up to 16 slots (48 and 57 registers)
// up to five, and 256 beyond, where more of them only keep other workgroups out.  Full tables, ten steps of mostly claimants that
// contend, us, 256 / 512 / 1 024 threads: 15 194 positions, windows of 8, 485 / 366 / 345, of 16 720 / 524 / 470, of 32
// 1 205 / 830 / 730, of 64 2 220 / - / 1 320; 100 000 positions, of 8 543 / 424 / -, of 64 2 260 / 1 590 / -; 200 000, of 8
// 517 / 456 / -, 300 000 604 / 582 / -, 400 000 660 / 647 / -.  Steps of which a tenth are claimants, on 30 M slots: 65 000
// positions 21.5 / 21.4 / 21.6 (8), 25.0 / 25.7 / 25.1 (32); 200 000, 30.7 / 29.8 / 33.1 (8), 38.1 / 41.8 / - (32); 300 000,
// 39.7 / 40.5 / - (8); 500 000, 56.1 / 57.9 / - (8).
template <int T>
constexpr int lru_chunk_threads(int grid, int num_cus)
{
    return grid <= num_cus ? 4 * kBlock : grid <= (T <= 2 ? 5 : 2) * num_cus ? 2 * kBlock : kBlock;
}
// Calls whose LRU claims pass over slots that were read with a better claim (SEEN of claim_group_lru): up to four slots of the table for a
// position.  With more of them claims hardly meet, and the look for better ones costs each claimant some twenty instructions more.
// Steps at 95 % load, a tenth of the ids new, with / without, us: 70 000 positions, one slot for a position 97.6 / 123.1, two 57.4 / 60.1, a little over
// four 34.4 / 33.7, eight 26.5 / 26.2, 64 26.9 / 26.5; 200 000 149 / 186, 78.8 / 82.4, 48.1 / 47.2, 33.7 / 33.3, 39.3 / 38.1; 400 000 210 / 252, 112 / 116,
// 68.4 / 67.9, 49.4 / 49.2, 65.4 / 64.5.  (Twelve steps of 5 000 on 20 000 slots, the table filling up, 358 / 361.)
constexpr bool crowded_lru(const Params &p) { return p.t0.N <= 4 * p.n; }

template <int T, bool REC, bool SEEN>
mpzch_status_t launch_allocate_lru_chunk(const Params &p, int grid, int num_cus, hipStream_t s)
{
    const int threads = lru_chunk_threads<T>(grid, num_cus);
    if (threads == 4 * kBlock) TRY(launch(k_allocate_lru_chunk<T, REC, SEEN, 4 * kBlock>, grid, threads, s, p));
    else if (threads == 2 * kBlock) TRY(launch(k_allocate_lru_chunk<T, REC, SEEN, 2 * kBlock>, grid, threads, s, p));
    else TRY(launch(k_allocate_lru_chunk<T, REC, SEEN, kBlock>, grid, threads, s, p));
    return MPZCH_OK;
}
template <bool REC, bool SEEN>
mpzch_status_t launch_allocate_lru_chunk(int32_t max_p_lru, const Params &p, int grid, int num_cus, hipStream_t s)
{
    if (max_p_lru <= 8) TRY((launch_allocate_lru_chunk<1, REC, SEEN>(p, grid, num_cus, s)));
    else if (max_p_lru <= 16) TRY((launch_allocate_lru_chunk<2, REC, SEEN>(p, grid, num_cus, s)));
    else if (max_p_lru <= 32) TRY((launch_allocate_lru_chunk<4, REC, SEEN>(p, grid, num_cus, s)));
    else TRY((launch_allocate_lru_chunk<8, REC, SEEN>(p, grid, num_cus, s)));
    return MPZCH_OK;
}
template <bool REC>
mpzch_status_t launch_allocate_lru_chunk(int32_t max_p_lru, const Params &p, int grid, int num_cus, hipStream_t s)
{
    if (crowded_lru(p)) return launch_allocate_lru_chunk<REC, true>(max_p_lru, p, grid, num_cus, s);
    return launch_allocate_lru_chunk<REC, false>(max_p_lru, p, grid, num_cus, s);
}

mpzch_status_t launch_allocate(int32_t max_p_lru, const Params &p, int num_cus, hipStream_t s)
{
    // one wavefront per workgroup, one segment per workgroup pass
    const int grid = grid_for((int64_t)p.num_segs, 1, num_cus, 4 * group_blocks_per_cu());
    if (p.num_tables > 1) {
        // several tables: TTL / no-eviction claimants first (this also writes every hint), then
        // the claimants of LRU tables
        if (p.all_records) TRY(launch(k_allocate<true, true>, grid, kWave, s, p));
        else TRY(launch(k_allocate<true, false>, grid, kWave, s, p));
        if (max_p_lru > 0 && p.all_records) TRY(launch_allocate_lru<true, true>(max_p_lru, p, grid, s));
        else if (max_p_lru > 0) TRY(launch_allocate_lru<true, false>(max_p_lru, p, grid, s));
    } else if (max_p_lru > 0) {
        if (p.t0.sh) TRY(launch_allocate_lru<false, true>(max_p_lru, p, grid, s));
        else TRY(launch_allocate_lru<false, false>(max_p_lru, p, grid, s));
    } else {
        if (p.t0.sh) TRY(launch(k_allocate<false, true>, grid, kWave, s, p));
        else TRY(launch(k_allocate<false, false>, grid, kWave, s, p));
    }
    return MPZCH_OK;
}

// Groups of at most one workgroup of k_finalize per compute unit have no use for a second one beside it (k_finalize: WAVES).
mpzch_status_t launch_finalize(const Params &p, int grid, int num_cus, hipStream_t s)
{
    if (p.num_tables > 1 && grid <= num_cus) TRY(launch(k_finalize<true, false, 4>, kFinalizeExtra + grid, kFinalizeBlock, s, p));
    else if (p.num_tables > 1) TRY(launch(k_finalize<true, false>, kFinalizeExtra + grid, kFinalizeBlock, s, p));
    else if (p.t0.evict == 2) TRY(launch(k_finalize<false, false>, kFinalizeExtra + grid, kFinalizeBlock, s, p));
    else TRY(launch(k_finalize<false, true>, kFinalizeExtra + grid, kFinalizeBlock, s, p));
    return MPZCH_OK;
}

#define TIMED(tm, id, s, launch)                    \
    do {                                            \
        if (!(tm).begin((id), (s))) return MPZCH_ERR_HIP; \
        TRY(launch);                                \
        if (!(tm).end((s))) return MPZCH_ERR_HIP;   \
    } while (0)

mpzch_status_t fill64(int64_t *dst, int64_t count, long long value, hipStream_t s);
mpzch_status_t fill32(int32_t *dst, int64_t count, int32_t value, hipStream_t s);

// One workgroup (mpzch_block_kernel.hpp).  Timed as Pass 1.
bool one_block(const Params &p) { return p.num_tables == 1 && p.t0.evict != 2 && p.n <= kOneBlock; }
mpzch_status_t launch_remap_block(Timing &tm, const Params &p, hipStream_t s)
{
    const int threads = (int)((p.n + kWave - 1) / kWave) * kWave;
    if (!tm.begin(KDiscover, s)) return MPZCH_ERR_HIP;
    if (p.t0.sh) TRY(launch(k_remap_block<true>, 1, threads, s, p));
    else TRY(launch(k_remap_block<false>, 1, threads, s, p));
    if (!tm.end(s)) return MPZCH_ERR_HIP;
    return MPZCH_OK;
}

// The launch sequence of one training remap (single table or group).
mpzch_status_t launch_remap(Scratch &sc, Timing &tm, Params p, Windows windows, hipStream_t s);

// Every call leaves the scratch set and the notes empty and, of the counter block, `stats` and `done` zero -- unless its launch
// sequence was cut short by a HIP error; the next call then clears all of it before it starts.  num_evicted is left as it is: it is
// k_finalize's alone, and the kernels of the allocation, which run before every k_finalize, clear it (clear_outcomes).
mpzch_status_t run_remap(Scratch &sc, Timing &tm, const Params &p, Windows windows, hipStream_t s)
{
    if (one_block(p)) return launch_remap_block(tm, p, s);        // uses no scratch
    if (sc.dirty) {
        TRY(fill32((int32_t *)sc.set_slot, Scratch::set_entries(sc.cap_n), -1, s));
        const Scratch::Layout L = Scratch::layout_for(sc.cap_n, sc.num_cus);
        TRY(fill64((int64_t *)sc.ctl, (int64_t)((L.total - L.o_ctl) / sizeof(int64_t)), 0, s));
    }
    sc.dirty = true;
    const mpzch_status_t st = launch_remap(sc, tm, p, windows, s);
    if (st == MPZCH_OK) sc.dirty = false;
    return st;
}

template <int SHIFT, bool EVEN, bool OVERLAP, bool ALIGNED, bool LOOKS>
mpzch_status_t launch_discover_chunk(const Params &p, int grid, hipStream_t s)
{
    if (p.t0.sh) TRY(launch(k_discover_chunk<true, SHIFT, EVEN, OVERLAP, ALIGNED, LOOKS>, grid, kBlock << SHIFT, s, p));
    else TRY(launch(k_discover_chunk<false, SHIFT, EVEN, OVERLAP, ALIGNED, LOOKS>, grid, kBlock << SHIFT, s, p));
    return MPZCH_OK;
}
template <bool OVERLAP, bool LOOKS>
mpzch_status_t launch_discover_chunk(const Params &p, int grid, bool aligned, hipStream_t s)
{
    if (aligned) return launch_discover_chunk<0, false, OVERLAP, true, LOOKS>(p, grid, s);
    return launch_discover_chunk<0, false, OVERLAP, false, LOOKS>(p, grid, s);
}

// Calls of so many workgroups of 256 positions read the scratch set back (k_allocate_chunk says why).  Measured on 256 compute
// units, loads of new ids by the notes alone / with the set read back, us, two calls into a table that ends 0.4 full, windows of
// 16 slots, records: 50 K ids 60.3 / 60.0, 57 K 69.2 / 63.5, 66 K 75.4 / 64.7, 100 K 93.2 / 77.3, 131 K 105.7 / 88.5, 145 K 87.4 /
// 91.1, 200 K 105.9 / 110.9; one call, 0.2 full, 30.5 / 31.0, 34.8 / 33.5, 40.1 / 35.0, 48.1 / 40.2, 53.0 / 46.1, 45.7 / 47.5, 53.9 /
// 56.0; eight calls, 0.95 full, 222 / 225, 243 / 235, 283 / 252, 324 / 286, 373 / 341, 344 / 350, 406 / 425; windows of 64 and
// two tensors have the same lines.  (Below 50 K the read costs what it is, 1 to 2 %.)
constexpr bool read_back_groups(int64_t groups, int num_cus) { return 8 * groups > 7 * (int64_t)num_cus && groups <= 2 * (int64_t)num_cus; }

template <bool REC>
mpzch_status_t launch_allocate_chunk(const Params &p, int grid, int num_cus, hipStream_t s)
{
    if (read_back_groups(grid, num_cus)) TRY(launch(k_allocate_chunk<REC, true>, grid, kBlock, s, p));
    else TRY(launch(k_allocate_chunk<REC, false>, grid, kBlock, s, p));
    return MPZCH_OK;
}

// Calls whose first looks go before the later ones (k_discover_chunk): windows of up to 32 slots, more than three workgroups per
// compute unit, and no more than leave the even end something to give.  In a table that the memory-side cache holds looks are
// short: up to four.  Beyond the cache five, of records, which need more registers, four; under the LRU policy, whose full windows make
// long chains of looks, one more, but over two tensors with windows of more than 16 slots.  Whole steps with a tenth of the ids new, without /
// with, us, of 230 K 262 144 300 007 330 K 393 216 480 K positions, each table as two tensors and as records:
//   60 M slots, TTL, 90 % load, of 16  42.8/41.7 45.2/43.2 48.0/46.5 50.5/47.4 58.2/53.7 65.8/62.5  41.5/40.5 44.2/42.1 47.0/45.6 49.8/46.8 57.3/53.0 65.1/63.5
//   60 M slots, TTL, 90 %, of 32       43.2/41.6 45.6/43.1 48.4/46.4 50.7/47.5 58.5/54.2 66.4/64.1  41.9/40.6 44.4/41.5 47.2/45.3 49.6/47.6 57.3/54.9 65.0/66.0
//   300 M slots, TTL, 95 %, of 24      43.1/41.8 46.1/43.8 48.4/46.4 50.7/47.5 58.1/54.3 65.8/63.2  41.8/41.7 44.7/43.4 47.3/45.3 49.6/48.4 57.2/57.5 64.9/67.3
//   60 M slots, LRU, full, of 16       35.8/35.2 38.4/37.5 41.8/41.3 44.0/43.5 50.5/50.6 58.2/60.1  38.6/38.8 42.0/41.7 45.7/45.0 48.0/47.4 54.2/54.8 62.5/66.4
//   300 M slots, LRU, full, of 24      38.2/37.1 41.1/39.5 44.9/45.0 47.3/48.0 54.0/57.0 63.0/67.8  41.4/41.0 45.0/44.2 49.0/49.9 51.9/54.4 59.3/63.0 68.7/73.5
// (TTL tables would gain beyond their lines as well, but calls of new ids lose there: half of the ids new, 300 M slots as two tensors, 400 K
// 68.6/70.6, 500 K 81.9/85.5, nearly all 97.2/102.4, 115.5/122.9, as records, 300 K, 73.2/76.1.)
// In the cache (20 M slots as two tensors, 10 M as records), 262 144 positions: TTL, of 24, 43.3/42.2, records 39.1/39.3, LRU, of 32, 43.5/43.3,
// records 48.9/48.5; sessions of eight steps of 200 000 on 2 M slots 450/438, records 421/421, loads of new ids 341/347, records 344/346.  Windows of up to
// 8 slots have no later looks there, all having been looked at from the home slot on: TTL, 200 000, 262 144, 27.4/27.5 32.4/32.6, records 28.6/28.9 32.6/32.8.
constexpr bool even_looks(int64_t groups, int num_cus, const TableDesc &t)
{
    const bool cached = (t.N << (3 + t.sh)) <= kCachedTableBytes;
    const int most = cached ? 4 : 5 - (t.sh ? 1 : 0) + (t.evict == 2 && (t.sh || t.P <= 16) ? 1 : 0);
    return t.P <= 32 && !(cached && t.P <= 8) && groups > 3 * (int64_t)num_cus && groups <= (int64_t)most * num_cus;
}

// Calls whose windows of 9 to 16 slots are read whole (SHIFT 1 of k_discover_chunk): up to one workgroup for two compute units.  Of records
// that is three lines an id, where a first look reads one or two, and beyond it is their number that counts: 65 536 ids were 196 K lines,
// 3.4 us of the kernel's 6.8.  Sessions of ten steps on six slots a position, whole windows / two looks, us: 2 000 positions of two tensors 177
// / 183, of records 175 / 183, 9 000 188 / 191, 187 / 192, 20 000 203 / 205, 203 / 207, 40 000 227 / 226, 225 / 224, 65 000 285 / 276, 284 /
// 273; six steps of 100 000 on 1 M slots 452 / 403, 444 / 395.
// Up to one workgroup per compute unit where the lines are fewer or nearly every absent id needs its whole window: tables of two tensors
// that the memory-side cache holds and the L2 does not, unless eviction is off, and, beyond that cache, LRU tables, which are full.  Steps
// in steady state, windows of 16, whole / two looks, 36 000, 45 000, 55 000 and 65 536 positions, us: LRU, 80 M slots as two tensors 19.4 / 20.6,
// 20.1 / 21.3, 20.9 / 21.9, 21.6 / 22.6, as records 19.8 / 20.9, 20.7 / 21.6, 21.7 / 22.2, 22.5 / 23.1; two tensors, 20 M slots, TTL 17.9 / 18.5,
// 18.4 / 19.1, 19.3 / 19.6, 19.5 / 19.8; sessions on 2.1 M slots 628 / 631, 637 / 643, 650 / 655, 662 / 667.  On the other sides: TTL, 80 M slots as
// records 18.8 / 18.6, 19.8 / 19.2, 20.7 / 19.7, 21.6 / 20.3, as two tensors, of 65 536, 20.8 / 20.7; sessions on 1 M slots, 50 000 positions, 330 / 324, on
// 300 000 448 / 371; loads of new ids into 3 M 231 / 229, 242 / 241, 264 / 259, 287 / 279; LRU, windows of 9, 80 M slots as records, of 50 000, 20.6 /
// 20.2; 72 000 positions, LRU, 80 M slots as two tensors 22.7 / 22.9, as records 24.2 / 23.2.
constexpr int64_t kL2Slots = (int64_t)1 << 21;
constexpr bool whole_windows(int64_t groups, int num_cus, const TableDesc &t)
{
    if (window_shift(t.P) != 1 || groups > num_cus) return false;
    const bool cached = (t.N << (3 + t.sh)) <= kCachedTableBytes;
    return 2 * groups <= num_cus || (cached ? !t.sh && t.evict != 0 && t.N >= kL2Slots : t.evict == 2 && t.P > 9);
}

// One-chunk calls whose first look is at the aligned block that holds the home slot: one line an id, and a second look where the id is
// not in its part of the window.  In tables beyond the memory-side cache all of them (see k_allocate).  Otherwise the 8 slots from the home slot
// on, which are two lines of records and one and a half of two tensors, decide more of the ids, and only calls with enough
// workgroups for the lines to count do better without: from one per compute unit on over records, from two and a half over two tensors.
// From the home slot on / aligned, us, 49 K 57 K 65 536 72 K 80 K 100 K 131 K 160 K 200 K positions; steps in steady state, sessions of 12 steps on
// 1 M slots, which the L2 holds, loads of new ids into 3 M:
//   records, 10 M slots, TTL, of 24   20.8/18.6 20.6/19.0 20.2/19.4 21.6/19.9 21.5/20.2 22.8/21.2 24.7/23.0 27.2/25.0 30.1/27.2
//   records, 10 M slots, LRU, of 16   22.1/20.9 22.1/21.6 22.8/22.7 23.0/22.9 23.6/23.3 25.0/24.6 27.8/27.0 30.8/29.8 34.4/32.0
//   records, sessions, TTL, of 16     224/238 232/239 241/245 250/253 260/260 283/280 309/307 341/344 384/374
//   ... of 24                         225/241 233/242 243/249 253/257 261/265 286/284 312/313 348/353 399/387
//   records, loads, of 16             171/172 181/181 189/186 200/197 205/203 226/222 281/271 304/295 357/345
//   tensors, from 100 K: 20 M slots, TTL, of 24, 22.4/21.4 24.0/23.3 26.1/25.1 29.2/27.9; LRU, of 16, 23.5/23.3 25.8/25.9 28.3/27.9 31.3/30.5; sessions, TTL, of 24, 289/287
//   317/322 356/358 400/399; loads, of 16, 221/221 272/271 288/287 350/348
// (Fuller sessions, filled to 0.3 before, gain from 65 536 records on: 51 steps of that many 883 / 860.)  Windows of up to 8 slots, which a look from the
// home slot on decides, have it in all of them: sessions, records, 57 K 228 / 242, 72 K 248 / 249, 160 K 330 / 333.
constexpr bool aligned_first(int64_t groups, int num_cus, const TableDesc &t)
{
    if ((t.N << (3 + t.sh)) > kCachedTableBytes) return true;
    return t.P > 8 && 2 * groups >= (t.sh ? 2 : 5) * (int64_t)num_cus;
}

// One chunk per wavefront (mpzch_chunk_kernels.hpp): grid = workgroups of 256 positions.
mpzch_status_t launch_remap_chunks(Timing &tm, const Params &p, int32_t max_p_lru, int grid, int num_cus, hipStream_t s)
{
    const bool rec = p.t0.sh != 0;
    const bool aligned = aligned_first(grid, num_cus, p.t0);
    if (!tm.begin(KDiscover, s)) return MPZCH_ERR_HIP;
    if (whole_windows(grid, num_cus, p.t0)) TRY((launch_discover_chunk<1, false, true, false, false>(p, grid, s)));
    else if (even_looks(grid, num_cus, p.t0)) TRY((launch_discover_chunk<0, true, false, true, true>(p, grid, s)));     // (all of them are `aligned`)
    else if (grid < num_cus) TRY((launch_discover_chunk<true, false>(p, grid, aligned, s)));
    else if (overlap_insert(grid, num_cus, rec, p.t0.evict == 3)) TRY((launch_discover_chunk<true, true>(p, grid, aligned, s)));
    else TRY((launch_discover_chunk<false, true>(p, grid, aligned, s)));
    if (!tm.end(s) || !tm.begin(KAllocate, s)) return MPZCH_ERR_HIP;
    if (max_p_lru > 0 && rec) TRY(launch_allocate_lru_chunk<true>(max_p_lru, p, grid, num_cus, s));
    else if (max_p_lru > 0) TRY(launch_allocate_lru_chunk<false>(max_p_lru, p, grid, num_cus, s));
    else if (rec) TRY(launch_allocate_chunk<true>(p, grid, num_cus, s));
    else TRY(launch_allocate_chunk<false>(p, grid, num_cus, s));
    if (!tm.end(s) || !tm.begin(KFinalize, s)) return MPZCH_ERR_HIP;
    TRY(launch(k_finalize_chunk, kPublishGroups + grid, kBlock, s, p));
    if (!tm.end(s)) return MPZCH_ERR_HIP;
    return MPZCH_OK;
}

// Where the first try of the scratch set is made (set_insert), as a shift.  Calls, everywhere / front half / quarter / eighth, us: 41.6 M
// values over 26 tables 1 282 / 1 272 / 1 259 / 1 250, 22 M 645 / 639 / 639, 11 M 364.5 / 364.1 / 363.7, 5.6 M 230.0 / 230.3 / 230.3, 2.8 M
// 142.8 / 143.2 / 143.9, 1.4 M 92.0 / 92.8 / 93.5 (a set that the caches hold: there the second try is what it costs).  One table, a
// tenth of the ids new: 4 M positions on 1 B slots 295 / 291 / 288 / 287, 2.4 M under LRU 281 / 278 / 277 / 277, 2 M on 500 M 173.0 / 171.8 /
// 171.6 / 171.6, 1.4 M 121.7 / 122.0 / 121.7 / 121.9.  All positions new: 1 M 218 / 207 / 219 / 235, 4 M 938 / 893 / 932 / 981, 16 M
// 3 792 / 3 599 / 3 711 / 3 935, nine tenths of 26 x 1.6 M 12 552 / 12 430 / 12 498 / 12 734: first tries meet, and of the parts that gain
// otherwise the quarter is the smallest that costs these nothing.
constexpr int front_shift(int64_t n, bool group) { return n >= (group ? (int64_t)1 << 23 : (int64_t)1 << 21) ? 2 : 0; }

mpzch_status_t launch_remap(Scratch &sc, Timing &tm, Params p, Windows windows, hipStream_t s)
{
    p.list = sc.list;
    p.ent = sc.ent;
    p.first_of = sc.first_of;
    p.hint = sc.hint;
    p.list_id = sc.list_id;
    p.evicted = sc.list_id;
    p.seg_cnt = sc.seg_cnt;
    p.set_slot = sc.set_slot;
    p.ctl = sc.ctl;

    p.place = sc.first_of;
    p.note = sc.note;
    p.wg_words = (uint64_t *)sc.seg_cnt;

    // one table, and no wavefront of Pass 1 has more than one chunk
    const int64_t groups = (p.n + kBlock - 1) / kBlock;
    // (the LRU policy with windows of more than 64 slots gives a claimant the whole wavefront)
    if (p.num_tables == 1 && windows.lru <= kWave && groups <= (int64_t)sc.num_cus * discover_blocks_per_cu() &&
        p.n <= kChunkMaxBatch)
        return launch_remap_chunks(tm, p, windows.lru, (int)groups, sc.num_cus, s);

    const int64_t num_chunks = (p.n + kWave - 1) / kWave;
    // k_discover: every wavefront owns one segment of seg_chunks 64-position chunks
    const int g_disc = grid_for(p.n, kBlock, sc.num_cus, train_blocks_per_cu(p.n));
    p.num_segs = g_disc * kWavesPerBlock;
    p.seg_chunks = (int32_t)((num_chunks + p.num_segs - 1) / p.num_segs);
    p.front_shift = front_shift(p.n, p.num_tables > 1);
    // the other kernels walk the segments' miss lists, one segment per wavefront pass.  (Two workgroups of 16 wavefronts
    // per compute unit.)
    const int g_grp = grid_for((int64_t)p.num_segs, kFinalizeWaves, sc.num_cus, 2);

    TIMED(tm, KDiscover, s, launch_discover(p, g_disc, sc.num_cus, windows, s));
    TIMED(tm, KAllocate, s, launch_allocate(windows.lru, p, sc.num_cus, s));
    TIMED(tm, KFinalize, s, launch_finalize(p, g_grp, sc.num_cus, s));
    return MPZCH_OK;
}

int fill_grid(int64_t count) { return (int)((count + kBlock - 1) / kBlock < 4096 ? (count + kBlock - 1) / kBlock : 4096); }

mpzch_status_t fill64(int64_t *dst, int64_t count, long long value, hipStream_t s)
{
    if (count <= 0) return MPZCH_OK;
    TRY(launch(k_fill64, fill_grid(count), kBlock, s, (long long *)dst, count, value));
    return MPZCH_OK;
}

mpzch_status_t fill32(int32_t *dst, int64_t count, int32_t value, hipStream_t s)
{
    if (count <= 0) return MPZCH_OK;
    TRY(launch(k_fill32, fill_grid(count), kBlock, s, dst, count, value));
    return MPZCH_OK;
}

// one tensor of 16-byte records: identities points at record 0 (16-byte aligned), metadata at its third word
bool records_ok(const int64_t *identities, const int32_t *metadata)
{
    return !((uintptr_t)identities & 15) && (const void *)metadata == (const void *)((const int32_t *)identities + 2);
}
// no device address of this GPU has more than 48 bits: a pointer that cannot be one is refused here instead of faulting in a
// kernel
bool addresses_ok(const TableCfg &c, const int64_t *identities)
{
    const uint64_t bytes = (uint64_t)c.num_slots << (c.layout == MPZCH_LAYOUT_RECORDS ? 4 : 3);
    const uint64_t begin = (uint64_t)(uintptr_t)identities;
    return identities && !(begin >> 48) && !((begin + bytes) >> 48);
}
bool layout_ok(const TableCfg &c, const int64_t *identities, const int32_t *metadata)
{
    return addresses_ok(c, identities) && (c.layout != MPZCH_LAYOUT_RECORDS || records_ok(identities, metadata));
}
// the read-only entry points see the identities only: records start at a multiple of 16 bytes
bool identities_ok(const TableCfg &c, const int64_t *identities)
{
    return addresses_ok(c, identities) && (c.layout != MPZCH_LAYOUT_RECORDS || !((uintptr_t)identities & 15));
}

bool valid_cfg(int64_t num_slots, int32_t max_probe, mpzch_eviction_policy_t policy)
{
    if (num_slots < 1 || num_slots > MPZCH_MAX_SLOTS || max_probe < 1 || max_probe > MPZCH_MAX_PROBE) return false;
    if (policy.kind != MPZCH_EVICT_NONE && policy.kind != MPZCH_EVICT_TTL && policy.kind != MPZCH_EVICT_LRU &&
        policy.kind != MPZCH_EVICT_TTL_EXPIRY)
        return false;
    if (policy.ttl < 0) return false;
    return true;
}

}  // namespace

// ---- the entry point that allocates nothing ------------------------------------------------------
// Its scratch is this file-scope array in device memory (every GPU the library runs on holds its own
// copy until the process ends).  In host code the array's name is only a handle for
// hipGetSymbolAddress: the address that kernels and fills receive is the one that call returns,
// queried once per device and kept in g_static.
constexpr size_t kStaticScratchBytes = (size_t)MPZCH_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
struct StaticState {
    bool ready = false;
    Scratch sc;
};
StaticState g_static[kMaxDevices];
std::mutex g_static_mutex;

// Set-up on the current device (first call on it): the array's address on this device, the layout of
// the scratch arrays inside it, and the one full clear (empty set, zero counters).
mpzch_status_t static_scratch(hipStream_t s, Scratch **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MPZCH_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MPZCH_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticState &st = g_static[dev];
    if (!st.ready) {
        TRY(st.sc.query_device());
        const Scratch::Layout L = Scratch::layout_for(MPZCH_NOALLOC_MAX_BATCH, st.sc.num_cus);
        if (L.total > kStaticScratchBytes) return MPZCH_ERR_UNSUPPORTED;     // a GPU with far more compute units
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MPZCH_ERR_HIP;
        st.sc.owned = false;
        st.sc.bind((char *)ptr, L, MPZCH_NOALLOC_MAX_BATCH);
        // fill kernels, not memsets: the first call may sit in a stream whose work a caller replays
        TRY(fill32((int32_t *)st.sc.set_slot, (int64_t)((L.o_ctl - L.o_set) / 4), -1, s));
        TRY(fill64((int64_t *)(st.sc.base + L.o_ctl), (int64_t)((L.total - L.o_ctl) / 8), 0, s));
        st.ready = true;
    }
    *out = &st.sc;
    return MPZCH_OK;
}
}  // namespace

struct mpzch_table {
    TableCfg cfg;
    Scratch sc;
    mutable Timing tm;             // benchmark instrumentation: also records the launches of read-only calls
};

// A device copy of per-table descriptors of a group, re-uploaded only when one of them changes.
template <typename D>
struct DevCache {
    D *dev = nullptr;
    std::vector<D> host;                 // what dev holds
    bool uploaded = false;

    mpzch_status_t put(const std::vector<D> &descs, hipStream_t s)
    {
        if (!dev && hipMalloc((void **)&dev, sizeof(D) * MPZCH_MAX_GROUP_TABLES) != hipSuccess) {
            dev = nullptr;
            return MPZCH_ERR_ALLOC;
        }
        const size_t bytes = sizeof(D) * descs.size();
        if (!uploaded || host.size() != descs.size() || std::memcmp(host.data(), descs.data(), bytes) != 0) {
            // earlier calls on this stream may still read the old descriptors
            if (hipStreamSynchronize(s) != hipSuccess) return MPZCH_ERR_HIP;
            if (hipMemcpy(dev, descs.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) return MPZCH_ERR_HIP;
            host = descs;
            uploaded = true;
        }
        return MPZCH_OK;
    }
    void release()
    {
        if (dev) (void)hipFree(dev);
        dev = nullptr;
        uploaded = false;
    }
};

struct mpzch_group {
    std::vector<TableCfg> cfgs;
    Scratch sc;
    Timing tm;
    DevCache<TableDesc> train;           // descriptors of mpzch_remap_jagged (identities + metadata)
    DevCache<TableDesc> infer;           // descriptors of mpzch_lookup_jagged (identities only)
    DevCache<JagRows> rows;              // descriptors of mpzch_reset_rows_jagged
};

extern "C" {

mpzch_status_t mpzch_create(int64_t num_slots, int32_t max_probe, mpzch_eviction_policy_t policy,
                            uint64_t hash_seed, mpzch_table_t **out)
{
    return mpzch_create_with_layout(num_slots, max_probe, policy, hash_seed, MPZCH_LAYOUT_SEPARATE, out);
}

mpzch_status_t mpzch_create_with_layout(int64_t num_slots, int32_t max_probe, mpzch_eviction_policy_t policy,
                                        uint64_t hash_seed, int32_t layout, mpzch_table_t **out)
{
    if (!out) return MPZCH_ERR_INVALID_ARG;
    *out = nullptr;
    if (layout != MPZCH_LAYOUT_SEPARATE && layout != MPZCH_LAYOUT_RECORDS) return MPZCH_ERR_INVALID_ARG;
    if (!valid_cfg(num_slots, max_probe, policy)) return MPZCH_ERR_INVALID_ARG;
    if (policy.kind == MPZCH_EVICT_LRU && max_probe > MPZCH_MAX_PROBE_LRU) return MPZCH_ERR_UNSUPPORTED;
    mpzch_table *t = new (std::nothrow) mpzch_table();
    if (!t) return MPZCH_ERR_ALLOC;
    t->cfg = {num_slots, max_probe, policy.kind, policy.ttl, hash_seed, layout};
    *out = t;
    return MPZCH_OK;
}

mpzch_status_t mpzch_destroy(mpzch_table_t *t)
{
    if (!t) return MPZCH_OK;
    t->sc.release();
    t->tm.destroy();
    delete t;
    return MPZCH_OK;
}

mpzch_status_t mpzch_reserve(mpzch_table_t *t, int64_t max_n)
{
    if (!t || max_n < 0 || max_n > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    return t->sc.ensure(max_n);
}

mpzch_status_t mpzch_init_tensors(const mpzch_table_t *t, int64_t *identities, int32_t *metadata, void *stream)
{
    if (!t || !identities) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (t->cfg.layout == MPZCH_LAYOUT_RECORDS) {
        if (!records_ok(identities, metadata)) return MPZCH_ERR_INVALID_ARG;
        const int64_t count = t->cfg.num_slots;
        TRY(launch(k_init_records, fill_grid(count), kBlock, s, (u32x4 *)identities, count));
        return MPZCH_OK;
    }
    if (!metadata) return fill64(identities, t->cfg.num_slots, -1, s);
    TRY(launch(k_init_tensors, fill_grid(t->cfg.num_slots), kBlock, s, (long long *)identities, metadata, t->cfg.num_slots));
    return MPZCH_OK;
}

namespace {
// geometry shared by the row movers: 16-byte chunks when everything is 16-byte aligned, else 4-byte
struct RowGeom { bool ok; bool wide; int64_t chunks; };
RowGeom row_geom(const void *rows, int64_t row_bytes, int64_t row_stride_bytes, const void *other)
{
    RowGeom g{false, false, 0};
    if (row_bytes < 4 || row_stride_bytes < row_bytes || (row_bytes & 3) || (row_stride_bytes & 3)) return g;
    if (((uintptr_t)rows & 3) || ((uintptr_t)other & 3)) return g;
    g.wide = !(row_bytes & 15) && !(row_stride_bytes & 15) && !((uintptr_t)rows & 15) && !((uintptr_t)other & 15);
    g.chunks = g.wide ? row_bytes / 16 : row_bytes / 4;
    g.ok = g.chunks <= 0x7FFFFFFF;
    return g;
}
// (the number of rows lives on the device: the grid is sized for the capacity of the list and bounded, the kernels stride.
// `most`: 2 048 workgroups, eight on each of 256 compute units, are all that run at a time.  The reset of one tensor is
// as fast with them as with more (0.6 M rows of 256 bytes 34 / 33 us with 8 192), and those without work cost a short list
// time.  Where the last ones would end late the kernel's bound is a multiple of it.)
int row_grid(int64_t items, int64_t per_block = kBlock, int64_t most = 2048)
{
    int64_t want = (items + per_block - 1) / per_block;
    if (want > most) want = most;
    if (want < 1) want = 1;
    return (int)want;
}
}  // namespace

namespace {
// rows that a remap resets itself (mpzch_remap_reset), or none
struct ResetRows {
    void *rows = nullptr;
    int64_t num_rows = 0, row_bytes = 0, row_stride_bytes = 0;
    const void *init_row = nullptr;
};

mpzch_status_t remap_one(mpzch_table_t *t, int64_t *identities, int32_t *metadata, const int64_t *ids,
                         const int32_t *ttls, int64_t n, int32_t step, int64_t *out_slots,
                         int64_t *out_evicted_slots, int64_t evicted_cap, int64_t *out_num_evicted,
                         int64_t *out_stats, const ResetRows &rr, void *stream)
{
    if (!t || !identities || !metadata || !out_num_evicted) return MPZCH_ERR_INVALID_ARG;
    if (n < 0 || n > MPZCH_MAX_BATCH || step < 0 || evicted_cap < 0) return MPZCH_ERR_INVALID_ARG;
    if (ttls && t->cfg.kind != MPZCH_EVICT_TTL_EXPIRY) return MPZCH_ERR_INVALID_ARG;
    if (!layout_ok(t->cfg, identities, metadata)) return MPZCH_ERR_INVALID_ARG;
    if (n > 0 && (!ids || !out_slots)) return MPZCH_ERR_INVALID_ARG;
    if (evicted_cap > 0 && !out_evicted_slots) return MPZCH_ERR_INVALID_ARG;
    RowGeom g{true, false, 0};
    if (rr.rows) {
        if (rr.num_rows < 1) return MPZCH_ERR_INVALID_ARG;
        g = row_geom(rr.rows, rr.row_bytes, rr.row_stride_bytes, rr.init_row);
        if (!g.ok) return MPZCH_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        TRY(fill64(out_num_evicted, 1, 0, s));
        if (out_stats) TRY(fill64(out_stats, MPZCH_STAT_COUNT, 0, s));
        return MPZCH_OK;
    }
    TRY(t->sc.ensure(n));
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = ids;
    p.ttls = ttls;
    p.n = n;
    p.step = step;
    p.num_tables = 1;
    p.out_slots = out_slots;
    p.t0 = make_desc(t->cfg, identities, metadata, 0, evicted_cap);
    p.out_evicted = out_evicted_slots;
    p.out_num_evicted = out_num_evicted;
    p.out_stats = out_stats;
    if (rr.rows) {
        p.r_rows = (char *)rr.rows;
        p.r_init = rr.init_row;
        p.g_num_rows = rr.num_rows;
        p.g_stride = rr.row_stride_bytes;
        p.g_chunks = (int32_t)g.chunks;
        p.g_wide = g.wide ? 1 : 0;
        p.g_shift = -1;
        for (int b = 0; b < 31; ++b)
            if (g.chunks == ((int64_t)1 << b)) p.g_shift = b;
    }
    return run_remap(t->sc, t->tm, p, windows_of(p.t0), s);
}
}  // namespace

mpzch_status_t mpzch_remap_feature_ttl(mpzch_table_t *t, int64_t *identities, int32_t *metadata,
                                       const int64_t *ids, const int32_t *ttls, int64_t n, int32_t step,
                                       int64_t *out_slots,
                                       int64_t *out_evicted_slots, int64_t evicted_cap, int64_t *out_num_evicted,
                                       int64_t *out_stats, void *stream)
{
    return remap_one(t, identities, metadata, ids, ttls, n, step, out_slots, out_evicted_slots, evicted_cap,
                     out_num_evicted, out_stats, ResetRows{}, stream);
}

mpzch_status_t mpzch_remap(mpzch_table_t *t, int64_t *identities, int32_t *metadata,
                           const int64_t *ids, int64_t n, int32_t step,
                           int64_t *out_slots,
                           int64_t *out_evicted_slots, int64_t evicted_cap, int64_t *out_num_evicted,
                           int64_t *out_stats, void *stream)
{
    return remap_one(t, identities, metadata, ids, nullptr, n, step, out_slots, out_evicted_slots, evicted_cap,
                     out_num_evicted, out_stats, ResetRows{}, stream);
}

mpzch_status_t mpzch_remap_reset(mpzch_table_t *t, int64_t *identities, int32_t *metadata,
                                 const int64_t *ids, int64_t n, int32_t step,
                                 int64_t *out_slots,
                                 int64_t *out_evicted_slots, int64_t evicted_cap, int64_t *out_num_evicted,
                                 int64_t *out_stats,
                                 void *rows, int64_t num_rows, int64_t row_bytes, int64_t row_stride_bytes,
                                 const void *init_row, void *stream)
{
    if (!rows) return MPZCH_ERR_INVALID_ARG;
    ResetRows rr;
    rr.rows = rows;
    rr.num_rows = num_rows;
    rr.row_bytes = row_bytes;
    rr.row_stride_bytes = row_stride_bytes;
    rr.init_row = init_row;
    return remap_one(t, identities, metadata, ids, nullptr, n, step, out_slots, out_evicted_slots, evicted_cap,
                     out_num_evicted, out_stats, rr, stream);
}

mpzch_status_t mpzch_remap_noalloc(const mpzch_table_t *t, int64_t *identities, int32_t *metadata,
                                   const int64_t *ids, int64_t n, int32_t step,
                                   int64_t *out_slots,
                                   int64_t *out_evicted_slots, int64_t evicted_cap, int64_t *out_num_evicted,
                                   int64_t *out_stats, void *stream)
{
    if (!t || !identities || !metadata || !out_num_evicted) return MPZCH_ERR_INVALID_ARG;
    if (n < 0 || step < 0 || evicted_cap < 0) return MPZCH_ERR_INVALID_ARG;
    if (n > MPZCH_NOALLOC_MAX_BATCH) return MPZCH_ERR_TOO_LARGE;
    if (!layout_ok(t->cfg, identities, metadata)) return MPZCH_ERR_INVALID_ARG;
    if (n > 0 && (!ids || !out_slots)) return MPZCH_ERR_INVALID_ARG;
    if (evicted_cap > 0 && !out_evicted_slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        TRY(fill64(out_num_evicted, 1, 0, s));
        if (out_stats) TRY(fill64(out_stats, MPZCH_STAT_COUNT, 0, s));
        return MPZCH_OK;
    }
    Scratch *sc = nullptr;
    TRY(static_scratch(s, &sc));
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = ids;
    p.n = n;
    p.step = step;
    p.num_tables = 1;
    p.out_slots = out_slots;
    p.t0 = make_desc(t->cfg, identities, metadata, 0, evicted_cap);
    p.out_evicted = out_evicted_slots;
    p.out_num_evicted = out_num_evicted;
    p.out_stats = out_stats;
    Timing off;                                  // never enabled: records nothing, creates no event
    return run_remap(*sc, off, p, windows_of(p.t0), s);
}

mpzch_status_t mpzch_lookup(const mpzch_table_t *t, const int64_t *identities,
                            const int64_t *ids, int64_t n,
                            int64_t *out_slots, uint8_t *out_found, void *stream)
{
    if (!t || !identities_ok(t->cfg, identities)) return MPZCH_ERR_INVALID_ARG;
    if (n < 0 || n > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    if (n == 0) return MPZCH_OK;
    if (!ids || !out_slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    int num_cus = 0;
    TRY(device_cus(&num_cus));
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = ids;
    p.n = n;
    p.num_tables = 1;
    p.out_slots = out_slots;
    p.out_found = out_found;
    p.t0 = make_desc(t->cfg, const_cast<int64_t *>(identities), nullptr, 0, 0);
    if (short_lookup(p, p.t0.P)) {
        TIMED(t->tm, KLookup, s, launch_lookup_short<false>(p, s));
        return MPZCH_OK;
    }
    const int grid = lookup_grid(n, num_cus);
    p.num_segs = grid * kWavesPerBlock;
    p.seg_chunks = (int32_t)(((n + kWave - 1) / kWave + p.num_segs - 1) / p.num_segs);
    TIMED(t->tm, KLookup, s, launch_lookup(p, grid, s));
    return MPZCH_OK;
}

mpzch_status_t mpzch_lookup_stats(mpzch_table_t *t, const int64_t *identities,
                                  const int64_t *ids, int64_t n,
                                  int64_t *out_slots, uint8_t *out_found, int64_t *out_stats, void *stream)
{
    if (!t || !identities_ok(t->cfg, identities) || !out_stats) return MPZCH_ERR_INVALID_ARG;
    if (n < 0 || n > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) return fill64(out_stats, MPZCH_STAT_COUNT, 0, s);
    if (!ids || !out_slots) return MPZCH_ERR_INVALID_ARG;
    TRY(t->sc.query_device());
    Params p;
    std::memset(&p, 0, sizeof p);
    TRY(t->sc.ensure_ctl(&p.ctl));
    p.ids = ids;
    p.n = n;
    p.num_tables = 1;
    p.out_slots = out_slots;
    p.out_found = out_found;
    p.out_stats = out_stats;
    p.t0 = make_desc(t->cfg, const_cast<int64_t *>(identities), nullptr, 0, 0);
    const int grid = grid_for(n, kBlock, t->sc.num_cus, discover_blocks_per_cu());
    p.num_segs = grid * kWavesPerBlock;
    p.seg_chunks = (int32_t)(((n + kWave - 1) / kWave + p.num_segs - 1) / p.num_segs);
    if (!t->tm.begin(KLookup, s)) return MPZCH_ERR_HIP;
    TRY(launch(k_lookup_counting, grid, kBlock, s, p));
    if (!t->tm.end(s)) return MPZCH_ERR_HIP;
    return MPZCH_OK;
}

mpzch_status_t mpzch_reset_rows(const int64_t *slots, const int64_t *num_slots_dev, int64_t slots_cap,
                                void *rows, int64_t num_rows, int64_t row_bytes, int64_t row_stride_bytes,
                                const void *init_row, void *stream)
{
    if (!num_slots_dev || slots_cap < 0 || !rows || num_rows < 1) return MPZCH_ERR_INVALID_ARG;
    if (row_bytes < 4 || row_stride_bytes < row_bytes || (row_bytes & 3) || (row_stride_bytes & 3))
        return MPZCH_ERR_INVALID_ARG;
    if (((uintptr_t)rows & 3) || ((uintptr_t)init_row & 3)) return MPZCH_ERR_INVALID_ARG;
    if (slots_cap == 0) return MPZCH_OK;
    if (!slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const bool wide = !(row_bytes & 15) && !(row_stride_bytes & 15) && !((uintptr_t)rows & 15) &&
                      !((uintptr_t)init_row & 15);
    const int64_t chunks = wide ? row_bytes / 16 : row_bytes / 4;
    if (chunks > 0x7FFFFFFF) return MPZCH_ERR_INVALID_ARG;
    const int grid = row_grid(slots_cap * chunks);
    if (wide)
        TRY(launch(k_reset_rows<u32x4>, grid, kBlock, s, slots, num_slots_dev, slots_cap, (char *)rows, row_mod(num_rows),
                   (int32_t)chunks, row_stride_bytes, (const u32x4 *)init_row));
    else
        TRY(launch(k_reset_rows<uint32_t>, grid, kBlock, s, slots, num_slots_dev, slots_cap, (char *)rows, row_mod(num_rows),
                   (int32_t)chunks, row_stride_bytes, (const uint32_t *)init_row));
    return MPZCH_OK;
}


mpzch_status_t mpzch_reset_rows_multi(const int64_t *slots, const int64_t *num_slots_dev, int64_t slots_cap,
                                      const mpzch_rows_t *tensors, int32_t num_tensors, void *stream)
{
    if (!num_slots_dev || slots_cap < 0 || !tensors || num_tensors < 1 || num_tensors > kMaxResetTensors)
        return MPZCH_ERR_INVALID_ARG;
    RowsDescs ds;
    std::memset(&ds, 0, sizeof ds);
    bool wide = true;
    for (int i = 0; i < num_tensors; ++i) {
        const mpzch_rows_t &t = tensors[i];
        if (!t.rows || t.num_rows < 1) return MPZCH_ERR_INVALID_ARG;
        const RowGeom g = row_geom(t.rows, t.row_bytes, t.row_stride_bytes, t.init_row);
        if (!g.ok) return MPZCH_ERR_INVALID_ARG;
        wide = wide && g.wide;
    }
    int64_t total = 0;
    for (int i = 0; i < num_tensors; ++i) {
        const mpzch_rows_t &t = tensors[i];
        ds.t[i].rows = (char *)t.rows;
        ds.t[i].init_row = t.init_row;
        ds.t[i].mod = row_mod(t.num_rows);
        ds.t[i].row_stride_bytes = t.row_stride_bytes;
        ds.t[i].chunks = (int32_t)(wide ? t.row_bytes / 16 : t.row_bytes / 4);
        total += ds.t[i].chunks;
    }
    if (total > 0x7FFFFFFF) return MPZCH_ERR_INVALID_ARG;
    ds.total_chunks = (int32_t)total;
    if (slots_cap == 0) return MPZCH_OK;
    if (!slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int grid = row_grid(slots_cap * total, kBlock, kMultiBlocks);
    if (wide) TRY(launch(k_reset_rows_multi<u32x4>, grid, kBlock, s, slots, num_slots_dev, slots_cap, ds));
    else TRY(launch(k_reset_rows_multi<uint32_t>, grid, kBlock, s, slots, num_slots_dev, slots_cap, ds));
    return MPZCH_OK;
}

mpzch_status_t mpzch_gather_rows(const int64_t *slots, const int64_t *count_dev, int64_t cap,
                                 const void *rows, int64_t num_rows, int64_t row_bytes, int64_t row_stride_bytes,
                                 void *out_rows, void *stream)
{
    if (cap < 0 || !rows || num_rows < 1 || !out_rows) return MPZCH_ERR_INVALID_ARG;
    const RowGeom g = row_geom(rows, row_bytes, row_stride_bytes, out_rows);
    if (!g.ok) return MPZCH_ERR_INVALID_ARG;
    if (cap == 0) return MPZCH_OK;
    if (!slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int grid = row_grid(cap * g.chunks, kBlock * kPieces, kMoverBlocks);
    if (g.wide)
        TRY(launch(k_gather_rows<u32x4>, grid, kBlock, s, slots, count_dev, cap, (const char *)rows, row_mod(num_rows),
                   (int32_t)g.chunks, row_stride_bytes, (u32x4 *)out_rows));
    else
        TRY(launch(k_gather_rows<uint32_t>, grid, kBlock, s, slots, count_dev, cap, (const char *)rows, row_mod(num_rows),
                   (int32_t)g.chunks, row_stride_bytes, (uint32_t *)out_rows));
    return MPZCH_OK;
}

mpzch_status_t mpzch_lookup_gather(const mpzch_table_t *t, const int64_t *identities,
                                   const int64_t *ids, int64_t n,
                                   const void *rows, int64_t num_rows, int64_t row_bytes, int64_t row_stride_bytes,
                                   void *out_rows, int64_t *out_slots, uint8_t *out_found, void *stream)
{
    if (!t || !identities_ok(t->cfg, identities)) return MPZCH_ERR_INVALID_ARG;
    if (n < 0 || n > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    if (!rows || num_rows < 1 || !out_rows) return MPZCH_ERR_INVALID_ARG;
    const RowGeom g = row_geom(rows, row_bytes, row_stride_bytes, out_rows);
    if (!g.ok || g.chunks > (1 << 20)) return MPZCH_ERR_INVALID_ARG;
    if (n == 0) return MPZCH_OK;
    if (!ids) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    int num_cus = 0;
    TRY(device_cus(&num_cus));
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = ids;
    p.n = n;
    p.num_tables = 1;
    p.out_slots = out_slots;
    p.out_found = out_found;
    p.t0 = make_desc(t->cfg, const_cast<int64_t *>(identities), nullptr, 0, 0);
    p.g_rows = (const char *)rows;
    p.g_out = (char *)out_rows;
    p.g_num_rows = num_rows;
    p.g_stride = row_stride_bytes;
    p.g_chunks = (int32_t)g.chunks;
    p.g_wide = g.wide ? 1 : 0;
    p.g_shift = -1;
    for (int b = 0; b <= 20; ++b)
        if (g.chunks == ((int64_t)1 << b)) p.g_shift = b;
    if (short_lookup(p, p.t0.P)) {
        TIMED(t->tm, KLookup, s, launch_lookup_short<true>(p, s));
        return MPZCH_OK;
    }
    // Seven workgroups of this kernel are resident on a compute unit (22.5 KB of LDS, 68 registers): of eight per unit the
    // last starts when another ends.  Where every wavefront has several chunks anyway, four per unit run in one go and
    // have lines enough under way.  Eight / four per unit, us, rows of 256 bytes: 0.7 M ids 67 / 68, 1 M 103 / 98, 2 M
    // 205 / 194, 4 M 417 / 381 (seven: 67, 104, 205, 389, for a wavefront more or less has one chunk more); rows of 64 bytes
    // 29 / 28, 43 / 42, 89 / 88, 173 / 169.  Right above the line it costs: 530 K ids 43.8 / 46.4 and 22.3 / 21.9.
    const int full = num_cus * discover_blocks_per_cu() * kBlock;
    const int grid = grid_for(n, kBlock, num_cus, n > full ? 4 : discover_blocks_per_cu());
    p.num_segs = grid * kWavesPerBlock;
    p.seg_chunks = (int32_t)(((n + kWave - 1) / kWave + p.num_segs - 1) / p.num_segs);
    if (!t->tm.begin(KLookup, s)) return MPZCH_ERR_HIP;
    TRY(launch(k_lookup_gather, grid, kBlock, s, lookup_args<false, true>(p, p.seg_chunks)));
    if (!t->tm.end(s)) return MPZCH_ERR_HIP;
    return MPZCH_OK;
}

mpzch_status_t mpzch_collect_delta(const mpzch_table_t *t, const int64_t *identities, const int32_t *metadata,
                                   int32_t since_step, int64_t *out_slots, int64_t *out_ids, int64_t cap,
                                   int64_t *out_count, void *stream)
{
    if (!t || !identities || !metadata || !out_count || cap < 0) return MPZCH_ERR_INVALID_ARG;
    if (cap > 0 && (!out_slots || !out_ids)) return MPZCH_ERR_INVALID_ARG;
    if (!layout_ok(t->cfg, identities, metadata)) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    int num_cus = 0;
    TRY(device_cus(&num_cus));
    TRY(fill64(out_count, 1, 0, s));
    // every workgroup scans a whole number of steps
    const int64_t steps = (t->cfg.num_slots + kDeltaSlots - 1) / kDeltaSlots;
    const int64_t most = (int64_t)num_cus * kDeltaBlocksPerCu;
    const int64_t per_block = (steps + most - 1) / most * kDeltaSlots;       // (below 2^32: num_slots <= MPZCH_MAX_SLOTS)
    const int grid = (int)((t->cfg.num_slots + per_block - 1) / per_block);
    if (t->cfg.layout == MPZCH_LAYOUT_RECORDS)
        TRY(launch(k_collect_delta<true>, grid, kDeltaBlock, s, identities, metadata, t->cfg.num_slots, per_block, since_step,
                   out_slots, out_ids, cap, (unsigned long long *)out_count));
    else
        TRY(launch(k_collect_delta<false>, grid, kDeltaBlock, s, identities, metadata, t->cfg.num_slots, per_block, since_step,
                   out_slots, out_ids, cap, (unsigned long long *)out_count));
    return MPZCH_OK;
}

mpzch_status_t mpzch_apply_delta(int64_t *identities, int64_t num_slots,
                                 const int64_t *slots, const int64_t *ids, const int64_t *count_dev, int64_t cap,
                                 void *rows, int64_t num_rows, int64_t row_bytes, int64_t row_stride_bytes,
                                 const void *delta_rows, void *stream)
{
    if (!identities || num_slots < 1 || cap < 0) return MPZCH_ERR_INVALID_ARG;
    RowGeom g{true, false, 1};
    if (rows) {
        if (num_rows < 1 || !delta_rows) return MPZCH_ERR_INVALID_ARG;
        g = row_geom(rows, row_bytes, row_stride_bytes, delta_rows);
        if (!g.ok) return MPZCH_ERR_INVALID_ARG;
    }
    if (cap == 0) return MPZCH_OK;
    if (!slots || !ids) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (rows) {
        const int grid = row_grid(cap * g.chunks, kBlock * kPieces, kMoverBlocks);
        if (g.wide)
            TRY(launch(k_apply_delta_rows<u32x4>, grid, kBlock, s, num_slots, slots, count_dev, cap, (char *)rows,
                       row_mod(num_rows), (int32_t)g.chunks, row_stride_bytes, (const u32x4 *)delta_rows));
        else
            TRY(launch(k_apply_delta_rows<uint32_t>, grid, kBlock, s, num_slots, slots, count_dev, cap, (char *)rows,
                       row_mod(num_rows), (int32_t)g.chunks, row_stride_bytes, (const uint32_t *)delta_rows));
    }
    TRY(launch(k_apply_delta_ids, row_grid(cap), kBlock, s, identities, num_slots, slots, ids, count_dev, cap));
    return MPZCH_OK;
}

mpzch_status_t mpzch_group_create(mpzch_table_t *const *tables, int32_t num_tables, mpzch_group_t **out)
{
    if (!out) return MPZCH_ERR_INVALID_ARG;
    *out = nullptr;
    if (!tables || num_tables < 1 || num_tables > MPZCH_MAX_GROUP_TABLES) return MPZCH_ERR_INVALID_ARG;
    for (int i = 0; i < num_tables; ++i) {
        if (!tables[i]) return MPZCH_ERR_INVALID_ARG;
    }
    mpzch_group *g = new (std::nothrow) mpzch_group();
    if (!g) return MPZCH_ERR_ALLOC;
    for (int i = 0; i < num_tables; ++i) g->cfgs.push_back(tables[i]->cfg);
    *out = g;
    return MPZCH_OK;
}

mpzch_status_t mpzch_group_destroy(mpzch_group_t *g)
{
    if (!g) return MPZCH_OK;
    g->sc.release();
    g->tm.destroy();
    g->train.release();
    g->infer.release();
    g->rows.release();
    delete g;
    return MPZCH_OK;
}

mpzch_status_t mpzch_group_reserve(mpzch_group_t *g, int64_t max_total_values)
{
    if (!g || max_total_values < 0 || max_total_values > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    return g->sc.ensure(max_total_values);
}

mpzch_status_t mpzch_remap_jagged_feature_ttl(mpzch_group_t *g, int64_t *const *identities, int32_t *const *metadata,
                                              const int64_t *values, const int32_t *ttls,
                                              const int64_t *feature_offsets,
                                              int64_t total_values, int32_t step,
                                              int64_t *out_slots,
                                              int64_t *out_evicted_slots, const int64_t *evicted_offsets,
                                              int64_t *out_num_evicted, int64_t *out_stats, void *stream)
{
    if (!g || !identities || !metadata || !feature_offsets || !evicted_offsets || !out_num_evicted)
        return MPZCH_ERR_INVALID_ARG;
    if (total_values < 0 || total_values > MPZCH_MAX_BATCH || step < 0) return MPZCH_ERR_INVALID_ARG;
    if (total_values > 0 && (!values || !out_slots)) return MPZCH_ERR_INVALID_ARG;
    const int T = (int)g->cfgs.size();
    if (ttls) {
        bool any = false;
        for (int f = 0; f < T; ++f) any = any || g->cfgs[f].kind == MPZCH_EVICT_TTL_EXPIRY;
        if (!any) return MPZCH_ERR_INVALID_ARG;          // no table of the group uses retention times
    }
    Windows windows{0, 0};
    bool all_records = true;
    std::vector<TableDesc> descs((size_t)T);
    for (int f = 0; f < T; ++f) {
        if (!identities[f] || !metadata[f]) return MPZCH_ERR_INVALID_ARG;
        if (!layout_ok(g->cfgs[f], identities[f], metadata[f])) return MPZCH_ERR_INVALID_ARG;
        const int64_t cap = evicted_offsets[f + 1] - evicted_offsets[f];
        if (cap < 0 || evicted_offsets[f] < 0) return MPZCH_ERR_INVALID_ARG;
        if (cap > 0 && !out_evicted_slots) return MPZCH_ERR_INVALID_ARG;
        descs[f] = make_desc(g->cfgs[f], identities[f], metadata[f], evicted_offsets[f], cap);
        all_records = all_records && descs[f].sh == 1;
        windows = longest(windows, windows_of(descs[f]));
    }
    hipStream_t s = (hipStream_t)stream;
    if (total_values == 0) {
        TRY(fill64(out_num_evicted, T, 0, s));
        if (out_stats) TRY(fill64(out_stats, (int64_t)T * MPZCH_STAT_COUNT, 0, s));
        return MPZCH_OK;
    }
    TRY(g->sc.ensure(total_values));
    TRY(g->train.put(descs, s));
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = values;
    p.ttls = ttls;
    p.n = total_values;
    p.step = step;
    p.num_tables = T;
    p.out_slots = out_slots;
    p.descs = g->train.dev;
    p.all_records = all_records ? 1 : 0;
    p.offsets = feature_offsets;
    p.t0 = descs[0];
    p.out_evicted = out_evicted_slots;
    p.out_num_evicted = out_num_evicted;
    p.out_stats = out_stats;
    // a group of one table runs the single-table kernels, whose list of evicted slots begins at out_evicted
    if (T == 1 && p.t0.ev_cap > 0) {
        p.out_evicted = out_evicted_slots + p.t0.ev_begin;
        p.t0.ev_begin = 0;
    }
    return run_remap(g->sc, g->tm, p, windows, s);
}

mpzch_status_t mpzch_remap_jagged(mpzch_group_t *g, int64_t *const *identities, int32_t *const *metadata,
                                  const int64_t *values, const int64_t *feature_offsets,
                                  int64_t total_values, int32_t step,
                                  int64_t *out_slots,
                                  int64_t *out_evicted_slots, const int64_t *evicted_offsets,
                                  int64_t *out_num_evicted, int64_t *out_stats, void *stream)
{
    return mpzch_remap_jagged_feature_ttl(g, identities, metadata, values, nullptr, feature_offsets, total_values, step,
                                          out_slots, out_evicted_slots, evicted_offsets, out_num_evicted, out_stats,
                                          stream);
}

mpzch_status_t mpzch_lookup_jagged(mpzch_group_t *g, const int64_t *const *identities,
                                   const int64_t *values, const int64_t *feature_offsets, int64_t total_values,
                                   int64_t *out_slots, uint8_t *out_found, void *stream)
{
    if (!g || !identities || !feature_offsets) return MPZCH_ERR_INVALID_ARG;
    if (total_values < 0 || total_values > MPZCH_MAX_BATCH) return MPZCH_ERR_INVALID_ARG;
    const int T = (int)g->cfgs.size();
    bool there = g->infer.uploaded;              // the descriptors on the device are those of these identities
    for (int f = 0; f < T; ++f) {
        if (!identities_ok(g->cfgs[f], identities[f])) return MPZCH_ERR_INVALID_ARG;
        there = there && g->infer.host[f].I == identities[f];
    }
    if (total_values == 0) return MPZCH_OK;
    if (!values || !out_slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    TRY(g->sc.query_device());
    if (!there) {
        std::vector<TableDesc> descs((size_t)T);
        for (int f = 0; f < T; ++f) descs[f] = make_desc(g->cfgs[f], const_cast<int64_t *>(identities[f]), nullptr, 0, 0);
        TRY(g->infer.put(descs, s));
    }
    const std::vector<TableDesc> &descs = g->infer.host;
    Params p;
    std::memset(&p, 0, sizeof p);
    p.ids = values;
    p.n = total_values;
    p.num_tables = T;
    p.out_slots = out_slots;
    p.out_found = out_found;
    p.descs = g->infer.dev;
    p.offsets = feature_offsets;
    p.t0 = descs[0];
    if (T == 1) p.num_tables = 1;            // a group of one table: the single-table kernel, offsets unused
    int32_t max_p = 1;
    for (const TableDesc &d : descs) max_p = d.P > max_p ? d.P : max_p;
    if (short_lookup(p, max_p)) {
        TIMED(g->tm, KLookup, s, launch_lookup_short<false>(p, s));
        return MPZCH_OK;
    }
    const int grid = lookup_grid(total_values, g->sc.num_cus);
    p.num_segs = grid * kWavesPerBlock;
    p.seg_chunks = (int32_t)(((total_values + kWave - 1) / kWave + p.num_segs - 1) / p.num_segs);
    TIMED(g->tm, KLookup, s, launch_lookup(p, grid, s));
    return MPZCH_OK;
}

mpzch_status_t mpzch_reset_rows_jagged(mpzch_group_t *g, const int64_t *evicted_slots, const int64_t *evicted_offsets,
                                       const int64_t *num_evicted, const mpzch_rows_t *tensors, void *stream)
{
    if (!g || !evicted_offsets || !num_evicted || !tensors) return MPZCH_ERR_INVALID_ARG;
    const int T = (int)g->cfgs.size();
    std::vector<JagRows> descs((size_t)T);
    std::memset(descs.data(), 0, sizeof(JagRows) * (size_t)T);
    bool any = false;
    for (int f = 0; f < T; ++f) {
        const int64_t cap = evicted_offsets[f + 1] - evicted_offsets[f];
        if (cap < 0 || evicted_offsets[f] < 0) return MPZCH_ERR_INVALID_ARG;
        const mpzch_rows_t &t = tensors[f];
        if (!t.rows || cap == 0) continue;                   // this table has no rows to reset
        if (t.num_rows < 1) return MPZCH_ERR_INVALID_ARG;
        const RowGeom geo = row_geom(t.rows, t.row_bytes, t.row_stride_bytes, t.init_row);
        if (!geo.ok) return MPZCH_ERR_INVALID_ARG;
        JagRows &d = descs[f];
        d.rows = (char *)t.rows;
        d.init_row = t.init_row;
        d.mod = row_mod(t.num_rows);
        d.row_stride_bytes = t.row_stride_bytes;
        d.ev_begin = evicted_offsets[f];
        d.ev_cap = cap;
        d.chunks = (int32_t)geo.chunks;
        d.wide = geo.wide ? 1 : 0;
        any = true;
    }
    if (!any) return MPZCH_OK;
    if (!evicted_slots) return MPZCH_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    TRY(g->sc.query_device());
    TRY(g->rows.put(descs, s));
    // (Two / four / eight workgroups per compute unit, whole steps over 26 tables, us: 10 400 values 33.6 / 33.7 / 33.8, 81 K 38.1 / 38.2 / 38.2,
    // 0.64 M 61.2 / 61.4 / 61.5, 2.5 M 131.9 / 131.7 / 131.7, 10.4 M 371.1 / 371.2 / 370.5, 41.6 M 1 238 / 1 237 / 1 237: hardly any difference.  Four,
    // so that rows of several segments are under way in a compute unit, and small steps do not start what they have no use for.)
    TRY(launch(k_reset_rows_jagged, g->sc.num_cus * 4, kBlock, s, evicted_slots, num_evicted, g->rows.dev, T));
    return MPZCH_OK;
}

mpzch_status_t mpzch_set_kernel_timing(mpzch_table_t *t, int32_t enable)
{
    if (!t) return MPZCH_ERR_INVALID_ARG;
    t->tm.set_mode(enable);
    return MPZCH_OK;
}

mpzch_status_t mpzch_kernel_times(mpzch_table_t *t, const char **names, double *ms, int64_t *launches,
                                  int32_t cap, int32_t *count)
{
    if (!t || !names || !ms || !launches || !count || cap < 0) return MPZCH_ERR_INVALID_ARG;
    return t->tm.collect(names, ms, launches, cap, count);
}

mpzch_status_t mpzch_group_set_kernel_timing(mpzch_group_t *g, int32_t enable)
{
    if (!g) return MPZCH_ERR_INVALID_ARG;
    g->tm.set_mode(enable);
    return MPZCH_OK;
}

mpzch_status_t mpzch_group_kernel_times(mpzch_group_t *g, const char **names, double *ms, int64_t *launches,
                                        int32_t cap, int32_t *count)
{
    if (!g || !names || !ms || !launches || !count || cap < 0) return MPZCH_ERR_INVALID_ARG;
    return g->tm.collect(names, ms, launches, cap, count);
}

const char *mpzch_status_string(int32_t status)
{
    switch (status) {
        case MPZCH_OK: return "ok";
        case MPZCH_ERR_INVALID_ARG: return "invalid argument";
        case MPZCH_ERR_ALLOC: return "allocation failed";
        case MPZCH_ERR_HIP: return "HIP runtime error";
        case MPZCH_ERR_UNSUPPORTED: return "unsupported";
        case MPZCH_ERR_TOO_LARGE: return "size beyond the fixed maximum of this entry point";
        default: return "unknown status";
    }
}

}  // extern "C"

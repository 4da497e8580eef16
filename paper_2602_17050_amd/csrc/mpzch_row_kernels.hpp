// Row movers (reset, gather) and the streaming delta.
#pragma once
#include "mpzch_kernels.hpp"

namespace mpzch {

// slot mod num_rows without a division: the quotient by the reciprocal floor((2^64 - 1) / num_rows) is the exact one or
// one less for slots below 2^63.
struct RowMod {
    int64_t num_rows;
    uint64_t inverse;
};
__host__ __device__ inline RowMod row_mod(int64_t num_rows) { return RowMod{num_rows, ~0ull / (uint64_t)num_rows}; }
__device__ __forceinline__ int64_t row_of(const RowMod &m, int64_t slot)
{
    if (slot < m.num_rows) return slot;
    const int64_t r = slot - (int64_t)(__umul64hi((uint64_t)slot, m.inverse) * (uint64_t)m.num_rows);
    return r >= m.num_rows ? r - m.num_rows : r;
}

// The row movers give one piece (16 or 4 bytes) of a row to a lane, so that consecutive lanes move consecutive pieces.  A
// thread takes the pieces first, first + stride, ... of all rows; which row and which piece of it follows by additions
// (no 64-bit division per piece).  kPieces of them are under way at a time: every piece is a chain of two accesses, slot
// and row.
//
// Gather and apply are bound by memory, and what they need not keep goes past the memory-side cache: rows are read and
// written with non-temporal accesses, the payload in between is not, so that the apply that follows finds it there (up to
// 256 MB).  With plain accesses the caches end up full of written rows, whose write-back the next kernel pays for.  A
// delta of 0.6 M rows of 256 bytes out of 50 M slots of records, collect + gather + apply rows + apply ids, us: 243 + 60 +
// 64 + 29 before; non-temporal scan alone 131 + 106 + 76 + 29; rows read that way 131 + 79 + 89 + 32; rows written that
// way too 130 + 65 + 57 + 17; the payload as well 131 + 71 + 75 + 11.  (The gather alone is slower for it where a row is
// half a line: 0.6 M rows of 64 bytes 20 -> 23, and gather + apply 59 -> 50.)  Pieces of 4 bytes go through the caches,
// which put lines together from them: gather + apply of 0.6 M rows of 20 bytes non-temporally 67, plainly 57; 2 M rows
// 241 and 181; 2 M rows of 132 bytes 605 and 519.  (In a table of 600 MB the other way round: 0.6 M rows of 20 bytes 73, 83.)
constexpr int kPieces = 4;
template <typename VEC>
__device__ __forceinline__ VEC load_piece(const VEC *at)
{
    if constexpr (sizeof(VEC) == 16) return __builtin_nontemporal_load(at);
    else return *at;
}
template <typename VEC>
__device__ __forceinline__ void store_piece(VEC v, VEC *at)
{
    if constexpr (sizeof(VEC) == 16) __builtin_nontemporal_store(v, at);
    else *at = v;
}

// How gather and apply share out the pieces of a list: to as many workgroups as have kPieces for each thread, of those that
// the grid has (it is sized for the list's capacity), and in as many turns for all of them alike.  A thread with fewer reads
// the first one again for what is missing: with one each the gather of 28 000 rows of 256 bytes took 7.4 instead of 5.9 us.
// Up to four times as many workgroups as run at a time, or the last ones end late: gather + apply of 2 M rows of 256 bytes
// 552 -> 532 us, of 128 bytes 314 -> 304.  More of them would be there for short lists in large areas, too (1 000 rows of
// 256 bytes, room for 2 M: 10 -> 20 us with four times as many).
// What a workgroup moves in one turn lies side by side, so that all that are under way work on one stretch of the list,
// instead of each on four that are a turn apart: gather + apply of 0.6 M rows of 256 bytes 99 -> 96 us, 2 M 519 -> 497, 4 M
// 1 046 -> 953, 1 M of 512 bytes 484 -> 462, of 64 bytes the same.
// (The resets have no second access to fill with, and the strides that depend on the count cost them more.)
constexpr int64_t kMoverBlocks = 8192;
struct Share {
    int64_t first, turn;         // this thread's first piece; from one turn to the next
    __device__ __forceinline__ explicit Share(int64_t total)
    {
        // (32 bits: 2^32 times 1 024 pieces of four bytes are more than the GPU's memory)
        const uint32_t need = (uint32_t)((total + kBlock * kPieces - 1) / (kBlock * kPieces));
        const uint32_t turns = need > gridDim.x ? (need + gridDim.x - 1) / gridDim.x : 1;
        const int64_t blocks = turns > 1 ? (need + turns - 1) / turns : need;
        turn = blocks * kBlock * kPieces;
        first = (int64_t)blockIdx.x < blocks ? (int64_t)blockIdx.x * kBlock * kPieces + threadIdx.x : total;
    }
};
struct PieceWalk {
    int64_t k, dk;               // row
    uint32_t c, dc, chunks;      // piece of it
    // (first and stride are numbers of threads of a grid, or of their pieces in a turn: 32 bits, which a division takes a tenth
    // of the time of 64)
    __device__ __forceinline__ PieceWalk(uint32_t first, uint32_t stride, int32_t chunks_per_row)
    {
        chunks = (uint32_t)chunks_per_row;
        const uint32_t q = first / chunks, dq = stride / chunks;
        k = q;
        c = first - q * chunks;
        dk = dq;
        dc = stride - dq * chunks;
    }
    // (one division, where there is another turn: lists of one turn are short)
    __device__ __forceinline__ void skip(uint32_t pieces)
    {
        const uint32_t q = pieces / chunks;
        k += q;
        c += pieces - q * chunks;
        if (c >= chunks) {
            c -= chunks;
            ++k;
        }
    }
    __device__ __forceinline__ void next()
    {
        k += dk;
        c += dc;
        if (c >= chunks) {
            c -= chunks;
            ++k;
        }
    }
};

__device__ __forceinline__ int64_t listed(const int64_t *count_dev, int64_t cap)
{
    int64_t count = count_dev ? *count_dev : cap;
    if (count > cap) count = cap;
    return count < 0 ? 0 : count;
}

// rows[(slots[k] mod num_rows)] <- init (or zero bits).  A short list is a chain of round trips, count, slot, store; the
// first slot is requested with the count (12 resets after batches of 20 011, with their remaps: 322.8 -> 320.6 us).
template <typename VEC>
__global__ __launch_bounds__(kBlock) void k_reset_rows(const int64_t *slots, const int64_t *count_dev, int64_t cap,
                                                        char *rows, RowMod mod, int32_t chunks_per_row,
                                                        int64_t row_stride_bytes, const VEC *init_row)
{
    const int64_t first = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    if (first >= cap * chunks_per_row) return;
    PieceWalk at((uint32_t)first, (uint32_t)stride, chunks_per_row);
    int64_t ahead = slots[at.k];                 // (in the list's area, and in the list if the count says so)
    const int64_t total = listed(count_dev, cap) * chunks_per_row;
    for (int64_t i = first; i < total; i += kPieces * stride) {
        int64_t s[kPieces];
        uint32_t c[kPieces];
        s[0] = ahead;
        c[0] = at.c;
        at.next();
#pragma unroll
        for (int u = 1; u < kPieces; ++u) {
            const bool in = i + u * stride < total;
            s[u] = slots[in ? at.k : 0];
            if (!in) s[u] = -1;
            c[u] = at.c;
            at.next();
        }
        if (i + kPieces * stride < total) ahead = slots[at.k];
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            if (s[u] < 0) continue;
            VEC v = VEC(0);
            if (init_row) v = init_row[c[u]];
            __builtin_nontemporal_store(v, reinterpret_cast<VEC *>(rows + row_of(mod, s[u]) * row_stride_bytes) + c[u]);
        }
    }
}

// The same for several tensors at once (embedding weights and optimizer state, Sec. 3.4).  One piece at a time per thread.
// Grid of up to 4 096 workgroups: with 2 048 the last ones end late (two tensors, 0.6 M rows of 256 bytes 81 -> 71 us, of
// 64 bytes 27.5 -> 24.9; 8 192 give 67 and 24.0, but cost a short list in a large area 0.5); four pieces under way gain
// nothing beside that.
constexpr int64_t kMultiBlocks = 4096;
struct RowsDesc {
    char *rows;
    const void *init_row;
    RowMod mod;
    int64_t row_stride_bytes;
    int32_t chunks;          // VEC-sized pieces per row
    int32_t pad_;
};
constexpr int kMaxResetTensors = 4;
struct RowsDescs {
    RowsDesc t[kMaxResetTensors];        // (0 pieces: none)
    int32_t total_chunks;
};

template <typename VEC>
__global__ __launch_bounds__(kBlock) void k_reset_rows_multi(const int64_t *slots, const int64_t *count_dev, int64_t cap,
                                                              RowsDescs ds)
{
    const int64_t first = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    if (first >= cap * ds.total_chunks) return;
    PieceWalk at((uint32_t)first, (uint32_t)stride, ds.total_chunks);
    int64_t ahead = slots[at.k];
    const int64_t total = listed(count_dev, cap) * ds.total_chunks;
    for (int64_t i = first; i < total; i += stride) {
        const int64_t s = ahead;
        uint32_t c = at.c;
        at.next();
        if (i + stride < total) ahead = slots[at.k];
        if (s < 0) continue;
        // (the tensors by number known at compile time: indexed otherwise they are read through memory)
#pragma unroll
        for (int which = 0; which < kMaxResetTensors; ++which) {
            const RowsDesc &t = ds.t[which];
            if (c < (uint32_t)t.chunks) {
                VEC v = VEC(0);
                if (t.init_row) v = reinterpret_cast<const VEC *>(t.init_row)[c];
                __builtin_nontemporal_store(v, reinterpret_cast<VEC *>(t.rows + row_of(t.mod, s) * t.row_stride_bytes) + c);
                break;
            }
            c -= (uint32_t)t.chunks;
        }
    }
}

// Row reset for a group of tables in one launch: table f's evicted slots are
// slots[ev_begin .. ev_begin + min(counts[f], ev_cap)), its rows are reset as in k_reset_rows.
struct JagRows {
    char *rows;               // null: nothing to reset for this table
    const void *init_row;
    RowMod mod;
    int64_t row_stride_bytes;
    int64_t ev_begin;
    int64_t ev_cap;
    int32_t chunks;           // 16-byte (wide) or 4-byte pieces per row
    int32_t wide;
};

// The pieces of all tables are one sequence, shared out evenly.  (One table after the other is a chain of four round
// trips for each, however little there is to do: 26 tables, 50 -> 35 us.)
__global__ __launch_bounds__(kBlock) void k_reset_rows_jagged(const int64_t *slots, const int64_t *counts,
                                                               const JagRows *tables, int num_tables)
{
    __shared__ JagRows s_t[kMaxTables];
    __shared__ int64_t s_begin[kMaxTables + 1];      // first piece of each table
    for (int i = threadIdx.x; i < num_tables * (int)(sizeof(JagRows) / 8); i += kBlock)
        reinterpret_cast<uint64_t *>(s_t)[i] = reinterpret_cast<const uint64_t *>(tables)[i];
    const int64_t mine = (int)threadIdx.x < num_tables ? counts[threadIdx.x] : 0;
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int f = threadIdx.x;
        int64_t pieces = 0;
        if (f < num_tables && s_t[f].rows) {
            int64_t count = mine > s_t[f].ev_cap ? s_t[f].ev_cap : mine;
            if (count < 0) count = 0;
            pieces = count * s_t[f].chunks;
        }
        int64_t upto = pieces;                       // inclusive scan over the lanes
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t below = shfl64(upto, f - o);
            if (f >= o) upto += below;
        }
        s_begin[f + 1] = upto;
        if (f == 0) s_begin[0] = 0;
    }
    __syncthreads();
    const int64_t total = s_begin[num_tables];
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < total; i0 += kPieces * stride) {
        int64_t s[kPieces];
        int32_t c[kPieces];
        int f[kPieces];
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const bool in = i0 + u * stride < total;
            const int64_t i = in ? i0 + u * stride : i0;
            f[u] = find_table(s_begin, num_tables, i);
            const JagRows &t = s_t[f[u]];
            const int64_t k = (i - s_begin[f[u]]) / t.chunks;
            c[u] = (int32_t)(i - s_begin[f[u]] - k * t.chunks);
            s[u] = slots[t.ev_begin + k];
            if (!in) s[u] = -1;
        }
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            if (s[u] < 0) continue;
            const JagRows &t = s_t[f[u]];
            const global_ptr<char> row = (global_ptr<char>)t.rows + row_of(t.mod, s[u]) * t.row_stride_bytes;
            if (t.wide) {
                u32x4 v = u32x4(0);
                if (t.init_row) v = ((global_ptr<const u32x4>)t.init_row)[c[u]];
                __builtin_nontemporal_store(v, (global_ptr<u32x4>)row + c[u]);
            } else {
                uint32_t v = 0u;
                if (t.init_row) v = ((global_ptr<const uint32_t>)t.init_row)[c[u]];
                __builtin_nontemporal_store(v, (global_ptr<uint32_t>)row + c[u]);
            }
        }
    }
}

// out[k, :] <- rows[slots[k] mod num_rows, :], zero bits for a negative slot (dense output rows of chunks * sizeof(VEC)
// bytes)
template <typename VEC>
__global__ __launch_bounds__(kBlock) void k_gather_rows(const int64_t *slots, const int64_t *count_dev, int64_t cap,
                                                         const char *rows, RowMod mod, int32_t chunks,
                                                         int64_t row_stride_bytes, VEC *out)
{
    const int64_t total = listed(count_dev, cap) * chunks;
    const Share share(total);
    if (share.first >= total) return;
    PieceWalk at((uint32_t)share.first, kBlock, chunks);
    for (int64_t i = share.first; i < total; i += share.turn) {
        int64_t s[kPieces];
        uint32_t c[kPieces];
        VEC v[kPieces];
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            s[u] = slots[i + u * kBlock < total ? at.k : 0];
            c[u] = at.c;
            at.next();
        }
#pragma unroll
        for (int u = 0; u < kPieces; ++u)
            v[u] = load_piece(reinterpret_cast<const VEC *>(rows + (s[u] >= 0 ? row_of(mod, s[u]) : 0) * row_stride_bytes) + c[u]);
#pragma unroll
        for (int u = 0; u < kPieces; ++u)
            if (i + u * kBlock < total) out[i + u * kBlock] = s[u] >= 0 ? v[u] : VEC(0);
        if (i + share.turn < total) at.skip((uint32_t)share.turn - kBlock * kPieces);
    }
}

// Streaming delta, receiving side (Sec. 3.8): rows[slots[k] mod num_rows, :] <- delta_rows[k, :] in one launch
// and identities[slots[k]] <- ids[k] in the next one on the same stream, so that every row of the delta
// has landed before any identity points at it (a reader on another stream never finds a new id in
// front of a row that is still partly old).
template <typename VEC>
__global__ __launch_bounds__(kBlock) void k_apply_delta_rows(int64_t num_slots, const int64_t *slots,
                                                              const int64_t *count_dev, int64_t cap,
                                                              char *rows, RowMod mod, int32_t chunks,
                                                              int64_t row_stride_bytes, const VEC *delta_rows)
{
    const int64_t total = listed(count_dev, cap) * chunks;
    const Share share(total);
    if (share.first >= total) return;
    PieceWalk at((uint32_t)share.first, kBlock, chunks);
    for (int64_t i = share.first; i < total; i += share.turn) {
        int64_t s[kPieces];
        uint32_t c[kPieces];
        VEC v[kPieces];
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const bool in = i + u * kBlock < total;
            s[u] = slots[in ? at.k : 0];
            v[u] = delta_rows[in ? i + u * kBlock : 0];
            if (!in) s[u] = -1;
            c[u] = at.c;
            at.next();
        }
#pragma unroll
        for (int u = 0; u < kPieces; ++u)
            if (s[u] >= 0 && s[u] < num_slots)
                store_piece(v[u], reinterpret_cast<VEC *>(rows + row_of(mod, s[u]) * row_stride_bytes) + c[u]);
        if (i + share.turn < total) at.skip((uint32_t)share.turn - kBlock * kPieces);
    }
}

__global__ __launch_bounds__(kBlock) void k_apply_delta_ids(int64_t *identities, int64_t num_slots, const int64_t *slots,
                                                             const int64_t *ids, const int64_t *count_dev, int64_t cap)
{
    const int64_t count = listed(count_dev, cap);
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < count; k += stride) {
        const int64_t s = slots[k];
        const int64_t id = ids[k];
        if (s >= 0 && s < num_slots) __hip_atomic_store(&identities[s], id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Streaming delta, sending side (Sec. 3.8): every occupied slot whose metadata is >= since goes to the
// list (slot, id), order unspecified.  Finds are staged in LDS and appended with one reservation per kDeltaStage finds or
// more (reservations follow each other at 12 ns).
//
// Bound by reading the table: non-temporal loads and few instructions, some 60 for a step of 4 slots per lane.  Records:
// 16 bytes per lane and slot (50 M slots: 217 -> 130 us, 6.1 TB/s, which is the rate of large reads).  Two
// tensors: the metadata decides nearly always, so identities are read only where it lets a slot pass.  The next step is
// requested before this one is looked at, and what a wavefront has found is known to the others by one barrier per
// step: its counts alternate between two places.
constexpr int kDeltaBlock = 512;
constexpr int kDeltaWaves = kDeltaBlock / kWave;
constexpr int kDeltaPerThread = 4;
constexpr int kDeltaSlots = kDeltaBlock * kDeltaPerThread;       // slots of one step
constexpr int kDeltaStage = 1024;
constexpr int kDeltaBlocksPerCu = 4;                             // (147 KB of LDS)
static_assert(kDeltaWaves == 8, "counts are read as two vectors of four");

template <bool REC>
struct DeltaStep {                                               // what a thread has read of one step
    u32x4 rec[REC ? kDeltaPerThread : 1];
    int32_t meta[REC ? 1 : kDeltaPerThread];
    __device__ __forceinline__ void load(const int64_t *identities, const int32_t *metadata, int64_t base, int64_t hi)
    {
        // (past the end of the range: its last slot)
        const int64_t left = hi - base;
        const uint32_t most = left > kDeltaSlots ? (uint32_t)kDeltaSlots - 1u : (uint32_t)left - 1u;
#pragma unroll
        for (int k = 0; k < kDeltaPerThread; ++k) {
            uint32_t o = (uint32_t)(k * kDeltaBlock) + threadIdx.x;
            o = o < most ? o : most;
            if constexpr (REC) rec[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(identities) + base + o);
            else meta[k] = __builtin_nontemporal_load(metadata + base + o);
        }
    }
};

template <bool REC>
__global__ __launch_bounds__(kDeltaBlock, 8) void k_collect_delta(const int64_t *identities, const int32_t *metadata,
                                                                  int64_t num_slots, int64_t per_block, int32_t since,
                                                                  int64_t *out_slots, int64_t *out_ids, int64_t cap,
                                                                  unsigned long long *out_count)
{
    __shared__ int64_t s_id[kDeltaStage + kDeltaSlots];
    __shared__ uint32_t s_at[kDeltaStage + kDeltaSlots];         // slot, from the workgroup's first one
    __shared__ u32x4 s_found[2][2];
    __shared__ unsigned long long s_base;
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < num_slots ? lo + per_block : num_slots;
    uint32_t staged = 0;                                         // the same in all threads
    auto flush = [&]() {                                         // reached by all threads
        __syncthreads();
        if (threadIdx.x == 0 && staged) s_base = atomicAdd(out_count, (unsigned long long)staged);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < staged; i += kDeltaBlock) {
            const int64_t at = (int64_t)s_base + i;
            if (at < cap) {
                out_slots[at] = lo + s_at[i];
                out_ids[at] = s_id[i];
            }
        }
        __syncthreads();
        staged = 0;
    };
    DeltaStep<REC> next;
    if (lo < hi) next.load(identities, metadata, lo, hi);
    int half = 0;
    for (int64_t base = lo; base < hi; base += kDeltaSlots, half ^= 1) {
        const DeltaStep<REC> now = next;
        if (base + kDeltaSlots < hi) next.load(identities, metadata, base + kDeltaSlots, hi);
        const int64_t left = hi - base;
        int64_t id[kDeltaPerThread];
        uint64_t who[kDeltaPerThread];                           // lanes whose slot goes to the list
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kDeltaPerThread; ++k) {
            if constexpr (REC) {
                id[k] = (int64_t)(((uint64_t)now.rec[k].y << 32) | now.rec[k].x);
                who[k] = __ballot((int32_t)now.rec[k].z >= since && (int32_t)now.rec[k].y >= 0);
            } else {
                who[k] = __ballot(now.meta[k] >= since);
            }
            if (left < kDeltaSlots) {
                const int there = (int)left - k * kDeltaBlock - w * kWave;
                who[k] &= there >= kWave ? ~0ull : there > 0 ? (1ull << there) - 1ull : 0ull;
            }
            if constexpr (!REC) {
                id[k] = -1;
                if (who[k] >> lane & 1ull) id[k] = identities[base + k * kDeltaBlock + threadIdx.x];
            }
        }
#pragma unroll
        for (int k = 0; k < kDeltaPerThread; ++k) {
            if constexpr (!REC) who[k] = __ballot(id[k] >= 0);
            sum += (uint32_t)__popcll(who[k]);
        }
        if (lane == 0) reinterpret_cast<uint32_t *>(s_found[half])[w] = sum;
        __syncthreads();
        const u32x4 a = s_found[half][0], b = s_found[half][1];
        const uint32_t total = a.x + a.y + a.z + a.w + b.x + b.y + b.z + b.w;
        if (total == 0) continue;
        if (sum > 0) {
            const uint32_t upto[kDeltaWaves] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            uint32_t at = staged;
#pragma unroll
            for (int i = 0; i < kDeltaWaves; ++i) at += i < w ? upto[i] : 0u;
#pragma unroll
            for (int k = 0; k < kDeltaPerThread; ++k) {
                if (who[k] >> lane & 1ull) {
                    const uint32_t to = at + (uint32_t)__popcll(who[k] & ((1ull << lane) - 1ull));
                    s_id[to] = id[k];
                    s_at[to] = (uint32_t)(base - lo) + (uint32_t)(k * kDeltaBlock) + threadIdx.x;
                }
                at += (uint32_t)__popcll(who[k]);
            }
        }
        staged += total;
        if (staged > kDeltaStage) flush();
    }
    flush();
}

}  // namespace mpzch

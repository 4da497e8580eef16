"""Variants of the kernels that a dispatch rule chooses by size, layout or policy, at the sizes where they can go
wrong, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_17050_amd import binding as mp
from paper_2602_17050_amd import workloads as wl
from gpu_common import Pair

pytestmark = pytest.mark.gpu


def rng_for(key):
    return np.random.Generator(np.random.Philox(key=key))


# ---- Pass 1 over records leaves a slot alone whose metadata is already what the hit would store
@pytest.mark.parametrize("evict", [True, "lru", "expiry", False])
def test_records_refreshed_once(evict):
    """Popular ids many times per batch, batches repeated at the same step (every hit finds its metadata fresh) and
    at later ones; n around multiples of a wavefront and of a workgroup's share."""
    rng = rng_for(901)
    t = Pair(5_000, 16, 2, evict, 11, layout="records")
    for step, n in [(0, 4_000), (0, 4_000), (3, 63), (3, 65), (4, 2_049), (4, 8_191), (9, 20_000), (9, 20_000), (10, 1)]:
        ids = wl.zipf_ids(rng, n, 1.2, 8_000)
        t.step(ids, step)
        t.step(ids, step)
    t.close()


@pytest.mark.parametrize("records", [(0, 1, 2, 3), (1, 3)])
def test_groups_of_records_refreshed_once(records):
    """A group whose tables are all records has a Pass 1 of its own; one with both layouts does not."""
    from test_gpu_jagged import JaggedPair
    rng = rng_for(902)
    specs = [wl.TableSpec(3_000, 16, 1, True, 41), wl.TableSpec(500, 8, 1, True, 42), wl.TableSpec(2_000, 40, 0, False, 43),
             wl.TableSpec(800, 16, 2, "expiry", 44)]
    jp = JaggedPair(specs, records)
    for step in (0, 0, 2, 5, 5):
        counts = rng.integers(0, 5_000, size=len(specs))
        vals = np.concatenate([wl.zipf_ids(rng, int(c), 1.1, 2 * s.num_slots) for s, c in zip(specs, counts)])
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        ttls = rng.integers(0, 6, size=len(vals)).astype(np.int32)
        for tt in (None, ttls):
            jp.step(vals, offsets, step, tt)
    jp.check_state()
    jp.close()


# ---- large batches of a group: whole sixteenths per die from 16 chunks per wavefront on, twice as many wavefronts from
# 2^24 values on
@pytest.mark.parametrize("chunks,more,layout", [(15, 0, "records"), (15, 1, "records"), (15, 1, "separate"), (32, -1, "records"),
                                                (32, 0, "records"), (32, 0, "separate")])
def test_groups_around_the_lines_of_large_batches(chunks, more, layout):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(911)
    n = chunks * torch.cuda.get_device_properties(0).multi_processor_count * 8 * 256 + more
    specs = [wl.TableSpec(1_003, 8, 1, True, 61), wl.TableSpec(50_000, 16, 1, True, 62), wl.TableSpec(7, 3, 1, True, 63),
             wl.TableSpec(2_000_000, 16, 1, True, 64), wl.TableSpec(300_007, 24, 0, False, 65), wl.TableSpec(1_000_000, 16, 1, "expiry", 66)]
    jp = JaggedPair(specs, range(len(specs)) if layout == "records" else ())
    # six features of very different length, one of them empty; what the first, small batch brings in has expired later
    share = np.array([0.21, 0.003, 0.0, 0.4, 0.137, 0.25])
    tot = 0
    for step, size in ((0, 1_000_003), (3, n)):
        counts = (share * size).astype(np.int64)
        counts[-1] = size - counts[:-1].sum()
        vals = np.concatenate([wl.zipf_ids(rng, int(c), 1.05, 2 * s.num_slots) + step for c, s in zip(counts, specs)])
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        tot += sum(s["evictions"] for s in jp.step(vals, offsets, step))
    assert tot > 1_000
    jp.check_state()
    if chunks == 32:
        jp.lookup(vals, offsets)
    jp.close()


# ---- ids with a chosen home slot: the hash is a bijection, so it can be run backwards
def ids_at(homes, num_slots, seed, rng):
    """One valid id per entry of `homes` (int64), hashing to that home slot."""
    homes = np.asarray(homes)
    out = np.empty(homes.size, dtype=np.int64)
    todo = np.arange(homes.size)
    u = np.uint64
    with np.errstate(over="ignore"):
        while todo.size:
            # a random hash value whose high product with num_slots is the home: home * 2^64 / N + a bit less than 2^64 / N
            width = (1 << 64) // num_slots
            h = np.array([-(-(int(x) << 64) // num_slots) for x in homes[todo]], dtype=np.uint64)
            h = h + rng.integers(0, max(1, width - 2), size=todo.size, dtype=np.uint64)

            def unshift(z, s):
                r = z
                for _ in range(64 // s + 1):
                    r = z ^ (r >> u(s))
                return r
            z = unshift(h, 31) * u(pow(0x94D049BB133111EB, -1, 1 << 64))
            z = unshift(z, 27) * u(pow(0xBF58476D1CE4E5B9, -1, 1 << 64))
            z = unshift(z, 30) - u(0x9E3779B97F4A7C15)
            ids = (z ^ u(seed)).astype(np.int64)
            ok = ids >= 0
            out[todo[ok]] = ids[ok]
            todo = todo[~ok]
    return out


def test_ids_at_gives_the_home_asked_for():
    rng = rng_for(903)
    for n_slots in (7, 5_000, 34_000_001):
        homes = rng.integers(0, n_slots, size=200)
        ids = ids_at(homes, n_slots, 99, rng)
        t = Pair(n_slots, 1, 0, True, 99)
        so, fo = t.lookup(ids)                    # an empty table: every lookup returns the home
        assert np.array_equal(so, homes) and not fo.any()
        t.close()


# ---- windows of every length over crowded stretches of the table: shared-out blocks of the later passes, displaced
# claimants, windows that run over the end of the table; blocks aligned (tables beyond 256 MB) or not
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("slots,probe", [(5, 8), (8, 8), (1_000, 9), (4_099, 17), (4_099, 40), (4_099, 65), (4_099, 300),
                                         (34_000_001, 16), (34_000_001, 33), (34_000_001, 130)])
@pytest.mark.parametrize("evict", [True, "expiry", False])
def test_crowded_windows(slots, probe, layout, evict):
    rng = rng_for(904 + slots + probe)
    t = Pair(slots, probe, 1, evict, 5, layout=layout)
    span = min(slots, 700)
    for step, n in [(0, 64), (1, span // 2 + 1), (2, span), (4, span), (5, 3 * span), (7, 9)]:
        # homes within `span` slots around the end of the table, a third of them on a handful of slots
        at = slots - span // 2 + rng.integers(0, span, size=n)
        hot = slots - 3 + rng.integers(0, 5, size=n)
        homes = np.where(rng.random(n) < 0.33, hot, at) % slots
        ids = ids_at(homes, slots, 5, rng)
        if n > 20:
            ids[rng.integers(0, n, size=n // 5)] = ids[rng.integers(0, n, size=n // 5)]      # copies
        t.step(ids, step, check_state=slots < 10_000_000)
        t.lookup(ids)
        t.step(ids[: n // 2 + 1], step, check_state=slots < 10_000_000)
    t.check_state()
    t.close()


# ---- the walk of claims in step: lanes leave a stage before its window is through only in windows of more than 16 slots (one chunk per
# wavefront) or 32 (one workgroup), never in the lists of long calls; windows a slot to either side of those lines, of less than a
# stage, of several, and longer than the table, with far more ids than slots, so that lanes end in every way in one wavefront
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("n", [900, 5_000, 524_289])
@pytest.mark.parametrize("probe", [16, 17, 32, 33, 65, 200])
def test_walks_left_early(n, probe, layout):
    rng = rng_for(990 + probe + n)
    for slots, evict in [(7, True), (n // 6, True), (n // 6, False), (n // 2, "expiry")]:
        if n > 500_000 and slots == 7:
            continue
        t = Pair(slots, probe, 1, evict, 5, layout=layout)
        for step in range(3):
            t.step(rng.integers(0, 1 << 60, size=n), 2 * step)
        t.check_state()
        t.close()


# ---- one workgroup up to 1 024 positions, one chunk per wavefront up to 256 x 8 workgroups of 256 positions (256 compute units); lists beyond that
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("evict,fused", [(True, True), (True, False), ("expiry", False), (False, False)])
def test_batches_around_workgroup_multiples(evict, fused, layout):
    rng = rng_for(905)
    emb = wl.embedding_pattern(7_001, 12, np.float32)
    t = Pair(20_000, 16, 1, evict, 17, emb, layout, fused)
    for step, n in enumerate([1, 63, 64, 65, 255, 256, 257, 511, 513, 1_023, 1_024, 1_025, 4_095, 20_001, 20_000, 7]):
        ids = wl.zipf_ids(rng, n, 1.05, 60_000)
        ids[rng.random(n) < 0.02] = -5
        t.step(ids, 2 * step, init_row=np.full(12, 3.5, np.float32) if step % 2 else None,
               ttls=rng.integers(0, 9, size=n).astype(np.int32) if evict == "expiry" and step % 3 else None)
    t.close()


@pytest.mark.parametrize("n", [524_287, 524_288, 524_289])
def test_batches_around_the_largest_one_chunk_call(n):
    rng = rng_for(906)
    t = Pair(300_000, 24, 0, True, 23, layout="records")
    for step in (0, 1, 2):
        t.step(wl.zipf_ids(rng, n, 1.02, 600_000), step)
    t.close()


# ---- one-chunk calls whose first looks go before the later ones, in tables that the memory-side cache holds: on both sides of each line
@pytest.mark.parametrize("evict", [True, "lru"])
@pytest.mark.parametrize("groups,layout", [(3, "separate"), (4, "separate"), (3, "records"), (4, "records"), (5, "records")])
def test_calls_around_the_lines_of_even_looks(groups, layout, evict):
    """Crowded windows, so that most ids take several looks; n at the line and one position beyond it."""
    rng = rng_for(917)
    n = groups * torch.cuda.get_device_properties(0).multi_processor_count * 256
    slots = n // 2
    t = Pair(slots, 29, 1, evict, 47, layout=layout)
    for step, more in enumerate([0, 1, 0, 1]):
        t.step(rng.integers(0, 2 * slots, size=n + more), step)
    t.close()


def ids_with_home(rng, count, lo, hi, num_slots, seed):
    """Distinct ids >= 0 whose home slots, by the hash of the library, are spread over [lo, hi): the hash undone."""
    want = np.empty(0, dtype=np.int64)
    while want.size < count:
        home = rng.integers(lo, hi, size=3 * count).astype(np.float64) + rng.random(3 * count) * 0.9 + 0.05
        x = (home / num_slots * 2.0 ** 64).astype(np.uint64)
        unxor = lambda x, s: x ^ (x >> np.uint64(s)) ^ (x >> np.uint64(2 * s))
        x = unxor(x, 31) * np.uint64(pow(0x94D049BB133111EB, -1, 1 << 64))
        x = unxor(x, 27) * np.uint64(pow(0xBF58476D1CE4E5B9, -1, 1 << 64))
        x = ((unxor(x, 30) - np.uint64(0x9E3779B97F4A7C15)) ^ np.uint64(seed)).view(np.int64)
        want = np.unique(np.concatenate([want, x[x >= 0]]))
    want = rng.permutation(want)[:count]
    assert all(lo <= oracle.home(int(i), seed, num_slots) < hi for i in want[:100])
    return want


# ---- the same in tables that the cache does not hold
@pytest.mark.parametrize("groups,layout,evict", [(3, "separate", True), (5, "separate", "expiry"), (6, "separate", "lru"),
                                                 (3, "records", "lru"), (4, "records", True), (5, "records", "lru")])
def test_calls_around_the_lines_of_even_looks_beyond_the_cache(groups, layout, evict):
    """Ids whose home slots lie in a small part of the table, so that its windows are crowded and most ids take several looks."""
    rng = rng_for(931)
    n = groups * torch.cuda.get_device_properties(0).multi_processor_count * 256
    slots = 34_000_003 if layout == "separate" else 17_000_003
    pool = ids_with_home(rng, n, 1_000, 1_000 + n // 2, slots, 59)
    t = Pair(slots, 29, 1, evict, 59, layout=layout)
    for step, more in enumerate([0, 1, 0, 1]):
        t.step(rng.choice(pool, size=n + more), step, check_state=step == 3)
    t.close()


# ---- expiry steps: the copies of a popular id agree on their maximum in LDS before they store it
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("n", [3, 64, 100, 257, 20_011, 530_000])
def test_expiry_steps_of_popular_ids(n, layout):
    rng = rng_for(907 + n)
    t = Pair(max(8, n // 2), 16, 3, "expiry", 31, layout=layout)
    for step in (0, 2, 2, 9):
        ids = wl.zipf_ids(rng, n, 1.3, max(4, n))
        ids[rng.random(n) < 0.3] = 77 + step % 2          # one id at a third of the positions, new every other time
        t.step(ids, step, ttls=rng.integers(0, 1_000, size=n).astype(np.int32))
        t.step(ids, step)
    t.close()


# ---- the scan of the streaming delta in steps of 2 048 slots per workgroup, the row movers in pieces
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("slots,rows,dim", [(1, 1, 1), (63, 7, 3), (2_047, 2_047, 4), (2_049, 1_000, 5), (300_001, 299_999, 12),
                                            (2_098_177, 100_003, 20)])
def test_delta_round_trip_at_edges(slots, rows, dim, layout):
    """Collect, gather and apply at sizes around a step, a workgroup's range and a row's pieces (4 and 16 bytes)."""
    rng = rng_for(907)
    ids = np.where(rng.random(slots) < 0.6, rng.integers(0, 1 << 62, size=slots), -1).astype(np.int64)
    meta = rng.integers(-1, 6, size=slots).astype(np.int32)
    ids[-1], meta[-1] = 77, 5                                     # the last slot belongs to every delta
    t = mp.MpzchTable(slots, 8, mp.EVICT_TTL, 1, 5, layout=mp.LAYOUT_RECORDS if layout == "records" else mp.LAYOUT_SEPARATE)
    t.identities.copy_(torch.from_numpy(ids).cuda())
    t.metadata.copy_(torch.from_numpy(meta).cuda())
    emb = torch.from_numpy(wl.embedding_pattern(rows, dim, np.float32)).cuda()
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    for since in (-(1 << 31), 0, 5, 6):
        d_slots = torch.full((slots,), -1, dtype=torch.int64, device="cuda")
        d_ids = torch.full_like(d_slots, -1)
        mp.mpzch_collect_delta(t.handle, t.identities, t.metadata, since, d_slots, d_ids, count)
        want = np.flatnonzero((ids >= 0) & (meta >= since))
        n = int(count.item())
        got = d_slots[:n].cpu().numpy()
        order = np.argsort(got)
        assert np.array_equal(got[order], want) and np.array_equal(d_ids[:n].cpu().numpy()[order], ids[want])
        payload = torch.full((slots, dim), 7.0, dtype=torch.float32, device="cuda")
        mp.mpzch_gather_rows(d_slots, count, emb, payload)
        assert torch.equal(payload[:n], emb[d_slots[:n] % rows]) and bool((payload[n:] == 7.0).all())
        inf_ids = torch.full((slots,), -1, dtype=torch.int64, device="cuda")
        inf_rows = torch.zeros_like(emb)
        mp.mpzch_apply_delta(inf_ids, d_slots, d_ids, count, inf_rows, payload)
        full = np.full(slots, -1, np.int64)
        full[want] = ids[want]
        assert np.array_equal(inf_ids.cpu().numpy(), full)
        touched = torch.zeros(rows, dtype=torch.bool, device="cuda")
        touched[d_slots[:n] % rows] = True
        assert torch.equal(inf_rows, emb * touched[:, None])
        mp.mpzch_reset_rows(d_slots, count, inf_rows)
        assert not bool(inf_rows.any())
        inf_rows.copy_(emb)
        mp.mpzch_reset_rows_multi(d_slots, count, [inf_rows, inf_ids.view(slots, 1).view(torch.float32)])
        assert torch.equal(inf_rows, emb * ~touched[:, None]) and not bool((inf_ids == torch.from_numpy(full).cuda())[d_slots[:n]].any())
    t.close()


# ---- row movers: a list's pieces go to as many workgroups as have work, of a grid sized for its capacity
@pytest.mark.parametrize("dim", [1, 5, 64])
@pytest.mark.parametrize("count,cap", [(0, 1), (1, 1), (63, 64), (64, 100_000), (65, 65), (1_025, 600_000), (262_145, 262_145),
                                       (524_289, 524_289), (524_289, 2_000_000)])
def test_row_movers_share_out_their_pieces(count, cap, dim):
    """Rows of 4, 20 and 256 bytes (pieces of 4 and 16): lists of a few pieces, of a workgroup's share and one more, of all
    that the largest grid takes in one turn and more, each with room for more entries than there are."""
    rng = rng_for(912)
    rows_n, other_n = 600_011, 600_000
    slots = torch.full((cap,), -1, dtype=torch.int64, device="cuda")
    at = torch.from_numpy(rng.permutation(rows_n)[:count]).cuda()          # distinct; a third of them wrap around
    slots[:count] = torch.where(at % 3 == 0, at + rows_n, at)
    slots[count // 2: count // 2 + (count > 9)] = -1                       # one entry that names no slot
    valid = slots[:count] >= 0
    at = at[valid]
    n = torch.tensor([count], dtype=torch.int64, device="cuda")
    src = torch.from_numpy(wl.embedding_pattern(rows_n, dim, np.float32)).cuda()
    out = torch.full((cap, dim), 7.0, device="cuda")
    mp.mpzch_gather_rows(slots, n, src, out)
    want = torch.full((cap, dim), 7.0, device="cuda")
    want[:count] = torch.where(valid[:, None], src[slots[:count].clamp(min=0) % rows_n], torch.zeros((), device="cuda"))
    assert torch.equal(out, want)
    ident, dst = torch.full((2 * rows_n,), -1, dtype=torch.int64, device="cuda"), torch.zeros_like(src)
    mp.mpzch_apply_delta(ident, slots, slots + 5, n, dst, out)
    want = torch.zeros_like(src)
    want[at] = src[at]
    assert torch.equal(dst, want)
    named = slots[:count][valid]
    want = torch.full_like(ident, -1)
    want[named] = named + 5
    assert torch.equal(ident, want)
    a, b = src.clone(), torch.full((other_n, 8), 3.0, device="cuda")
    init = torch.arange(dim, dtype=torch.float32, device="cuda")
    mp.mpzch_reset_rows_multi(slots, n, [a, b], [init, None])
    want = src.clone()
    want[at] = init
    assert torch.equal(a, want)
    other = torch.full((other_n, 8), 3.0, device="cuda")
    other[named % other_n] = 0.0
    assert torch.equal(b, other)
    a = src.clone()
    mp.mpzch_reset_rows(slots, n, a, init)
    assert torch.equal(a, want)


# ---- gather and apply in two and three turns of the largest grid (8 192 workgroups of 1 024 pieces), the last one ragged
@pytest.mark.parametrize("dim,pieces", [(5, 5), (12, 3), (64, 16)])
@pytest.mark.parametrize("turns", [1, 2])
def test_row_movers_take_turns(turns, dim, pieces):
    count = turns * 8_192 * 1_024 // pieces + 77
    rows_n = count + 11
    gen = torch.Generator(device="cuda").manual_seed(914)
    slots = torch.randperm(rows_n, generator=gen, device="cuda")[:count]
    slots[count // 3] = -1
    valid = slots >= 0
    n = torch.tensor([count], dtype=torch.int64, device="cuda")
    src = torch.arange(rows_n * dim, dtype=torch.int32, device="cuda").view(torch.float32).reshape(rows_n, dim)
    out = torch.full((count, dim), 7.0, device="cuda")
    mp.mpzch_gather_rows(slots, n, src, out)
    want = torch.where(valid[:, None], src[slots.clamp(min=0)], torch.zeros((), device="cuda"))
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))
    ident, dst = torch.full((rows_n,), -1, dtype=torch.int64, device="cuda"), torch.zeros_like(src)
    mp.mpzch_apply_delta(ident, slots, slots + 5, n, dst, out)
    want = torch.zeros_like(src)
    want[slots[valid]] = src[slots[valid]]
    assert torch.equal(dst.view(torch.int32), want.view(torch.int32))
    del want


# ---- LRU claims: one group of lanes per claimant, listed per workgroup where every wavefront has one chunk
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("slots,probe", [(3, 8), (700, 1), (900, 8), (3_001, 9), (3_001, 16), (5_003, 31), (5_003, 33), (5_003, 64),
                                         (5_003, 65)])
def test_lru_claims(slots, probe, layout):
    """Batches from one position to several workgroups of claimants that contend for few slots; calls beyond the
    largest one-chunk call too."""
    rng = rng_for(908)
    t = Pair(slots, probe, 0, "lru", 17, layout=layout)
    for step, n in enumerate([1, 63, 257, 300, 1_025, 4_000, 4_000, 20_011, 2]):
        t.step(wl.zipf_ids(rng, n, 1.02, 6 * slots), step)
    t.step(wl.zipf_ids(rng, 530_000, 1.02, 3 * slots), 9)
    t.step(rng.integers(0, 2 * slots, size=2_000), 9)
    t.step(rng.integers(0, 9 * slots, size=2_000), 10)
    t.close()


# displaced claimants whose home slots come from their tags (around the end of the table, in tables hardly longer than a window)
# and slots that are passed over because they were read with a better claim: whole classes of them, in masks of 32 and 64 slots; one chunk
# per wavefront, and lists
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("probe", [7, 8, 9, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("slots,n", [(65, 300), (700, 1_500), (9_000, 12_000), (400_000, 524_289)])
def test_lru_crowded(slots, n, probe, layout):
    rng = rng_for(1_004 + slots + probe)
    t = Pair(slots, probe, 0, "lru", 5, layout=layout)
    for step in range(4):
        ids = rng.integers(0, 1 << 60, size=n)
        if n < 100_000:
            at = rng.random(n) < 0.5
            ids[at] = ids_at((slots - 3 + rng.integers(0, 9, size=int(at.sum()))) % slots, slots, 5, rng)   # homes around the end
        t.step(ids, step + 1)
        t.step(ids[: n // 3 + 1], step + 1)
    t.check_state()
    t.close()


# ... and on both sides of four slots for a position, beyond which no slot is passed over: few windows' homes, so that claims meet there too
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("probe", [8, 9, 32, 64])
@pytest.mark.parametrize("n", [600, 40_000, 140_000])
def test_lru_four_slots_a_position(n, probe, layout):
    rng = rng_for(1_017 + n + probe)
    for slots in (4 * n, 4 * n + 1):
        t = Pair(slots, probe, 0, "lru", 5, layout=layout)
        for step in range(3):
            ids = rng.integers(0, 1 << 60, size=n)
            ids[: n // 8] = ids_with_home(rng, n // 8, slots - 40, slots, slots, 5)
            t.step(ids, step + 1)
        t.check_state()
        t.close()


# ---- LRU claims by workgroups of 1 024, 512 and 256 threads: on both sides of each line, few claimants and mostly claimants
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("groups,probe", [(1, 5), (1, 16), (1, 29), (1, 64), (2, 5), (2, 16), (2, 29), (2, 64), (5, 5), (5, 16)])
def test_lru_claims_around_the_lines_of_their_workgroups(groups, probe, more):
    rng = rng_for(916)
    n = groups * torch.cuda.get_device_properties(0).multi_processor_count * 256 + more
    slots = n // 3
    t = Pair(slots, probe, 0, "lru", 43, layout="records" if more else "separate")
    for step, universe in enumerate([2 * slots, 2 * slots, slots // 2]):
        t.step(rng.integers(0, universe, size=n), step)
    t.close()


# ---- ids that are new and popular at once: copies enter the scratch set once per wavefront
@pytest.mark.parametrize("evict", [True, "lru", False])
@pytest.mark.parametrize("n", [1_025, 4_111, 65_536])
def test_new_ids_with_many_copies(n, evict):
    rng = rng_for(909)
    t = Pair(2_003, 16, 1, evict, 19, layout="records")
    for step in range(4):
        hot = rng.integers(0, 1 << 40, size=5)
        ids = np.where(rng.random(n) < 0.7, hot[rng.integers(0, 5, size=n)], rng.integers(0, 1 << 40, size=n))
        ids[: n // 3] = hot[0]
        t.step(ids[rng.permutation(n)], 2 * step)
    t.close()


# ---- lookups of few ids: as many ids per wavefront as one pass holds the windows of
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("slots,probe", [(5, 8), (300, 8), (300, 16), (4_099, 17), (4_099, 33), (4_099, 65), (4_099, 300)])
def test_lookups_around_the_largest_short_one(slots, probe, layout):
    rng = rng_for(910)
    t = Pair(slots, probe, 1, True, 23, layout=layout)
    for step in range(3):
        t.step(wl.zipf_ids(rng, slots + 7, 1.02, 2 * slots), step)
    shift = 0 if probe <= 8 else 1 if probe <= 16 else 2 if probe <= 32 else 3
    edge = (1 << 18) >> (0 if slots <= 8 else shift)
    rows_np = wl.embedding_pattern(slots, 12, np.float32)
    rows = torch.from_numpy(rows_np).cuda()
    for n in (1, 7, 8, 9, 31, 33, 64, 65, 257, edge - 1, edge, edge + 1):
        q = np.concatenate([wl.zipf_ids(rng, n, 1.02, 3 * slots)[: n - n // 10], rng.integers(-3, 1 << 40, size=n // 10)])
        so, fo = t.o.lookup(q)
        sg, fg = t.g.lookup(torch.from_numpy(q).cuda())
        assert np.array_equal(sg.cpu().numpy(), so) and np.array_equal(fg.cpu().numpy(), fo), n
        out = torch.full((n, 12), -1.0, dtype=torch.float32, device="cuda")
        mp.mpzch_lookup_gather(t.g.handle, t.g.identities, torch.from_numpy(q).cuda(), rows, out)
        assert np.array_equal(out.cpu().numpy(), rows_np[so % slots]), n
    t.close()


# ---- one workgroup makes its claims in a map in LDS of twice as many entries as it has threads: every position new, the
# claimants on as many different slots as there are of them, or all on a few windows
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("evict", [True, "expiry", False])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 500, 1_024])
def test_claims_of_one_workgroup(n, evict, layout):
    rng = rng_for(911 + n)
    t = Pair(30_011, 40, 1, evict, 29, layout=layout)
    for step in range(6):
        homes = rng.integers(0, 30_011, size=n) if step % 2 else (30_000 + rng.integers(0, max(1, n // 30), size=n)) % 30_011
        t.step(ids_at(homes, 30_011, 29, rng), 2 * step)
    t.close()


# ---- the blocks of a probe pass at the edges of small tables (fewer slots than a request is wide; requests moved back from
# the table's end; windows that go on at its start) and of identities that are not aligned to a block
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("slots", [1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 203])
def test_probe_blocks_at_the_edges_of_small_tables(slots, layout):
    rng = rng_for(912 + slots)
    for probe in (1, 5, 8, 13, 32, 64):
        t = Pair(slots, probe, 1, True, 31, layout=layout)
        sizes = [1, max(1, slots // 2), min(1_000, 5 * slots), 1_100] + ([530_000] if slots in (9, 65) and probe == 13 else [])
        for step, n in enumerate(sizes):
            ids = ids_at(rng.integers(0, slots, size=min(n, 3_000)), slots, 31, rng)
            ids = np.concatenate([ids, ids[rng.integers(0, ids.size, size=n - ids.size)]])
            t.step(ids, 2 * step)
            q = np.concatenate([ids[:2_000], ids_at(rng.integers(0, slots, size=70), slots, 31, rng)])
            so, fo = t.lookup(q)
            if layout == "separate":
                for shift in (1, 3, 6):
                    moved = torch.empty(slots + 8, dtype=torch.int64, device="cuda")[shift: shift + slots]
                    moved.copy_(t.g.identities)
                    qg = torch.from_numpy(q).cuda()
                    for count in (q.size, 300_000):                 # a short lookup, and one of whole chunks
                        many = qg.repeat(-(-count // q.size))[:count].contiguous()
                        out = torch.empty_like(many)
                        found = torch.empty(count, dtype=torch.uint8, device="cuda")
                        mp.mpzch_lookup(t.g.handle, moved, many, out, found)
                        assert np.array_equal(out.cpu().numpy(), np.resize(so, count)), (shift, count)
                        assert np.array_equal(found.cpu().numpy(), np.resize(fo, count)), (shift, count)
        t.close()


# ---- lists of one table: new ids alone, with copies in their own wavefront and in others, and with displaced claims (the
# positions stand in any order, so that many a first occurrence comes after a copy; the last table is too small for all)
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("policy", [True, "expiry", False, "lru"])
@pytest.mark.parametrize("slots,copies", [(2_000_003, 1), (700_001, 3), (90_001, 2)])
def test_lists_with_copies_and_displaced_claims(slots, copies, policy, layout):
    rng = rng_for(913 + slots)
    t = Pair(slots, 12, 1, policy, 37, layout=layout)
    n = 524_289
    for step in range(3):
        ids = rng.integers(0, 1 << 50, size=n // copies)
        ids = np.concatenate([ids, ids[rng.integers(0, ids.size, size=n - ids.size)], np.repeat(ids[:40], 64)])
        near = rng.random(ids.size) < 0.5
        t.step(np.where(near, ids, rng.permutation(ids)), 3 * step)
    t.close()


# ---- where lists are kept the allocation counts the outcomes and a workgroup of the last kernel publishes them: every kernel of
# the allocation, calls with and without statistics and counting lookups in turn (what one leaves behind the next would show)
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("policy,probe,n", [(True, 12, 524_289), ("expiry", 24, 524_353), ("lru", 7, 524_289), ("lru", 15, 524_289),
                                            ("lru", 30, 524_290), ("lru", 60, 524_289), ("lru", 70, 1), ("lru", 70, 700), ("lru", 300, 9_000)])
def test_counters_of_lists(policy, probe, n, layout):
    rng = rng_for(921)
    slots = n // 2 + probe
    t = Pair(slots, probe, 1, policy, 43, layout=layout)
    evicted = torch.empty(n, dtype=torch.int64, device="cuda")
    count = torch.empty(1, dtype=torch.int64, device="cuda")
    for step in range(4):
        ids = rng.integers(-1, 3 * slots, size=n)
        if step == 2:
            g = torch.from_numpy(ids).cuda()
            mp.mpzch_remap(t.g.handle, t.g.identities, t.g.metadata, g, 2 * step, torch.empty_like(g), evicted, count, None)
            r = t.o.remap(ids, 2 * step)
            assert np.array_equal(np.sort(evicted[: int(count)].cpu().numpy()), np.sort(r.evicted))
            t.check_state()
        else:
            t.step(ids, 2 * step)
        t.lookup(ids[:5_000])
    t.close()


# ---- ... and calls of many chunks per wavefront, whose outcomes add up, from 2^24 positions on over two segments.  All ids new: into an empty table, then over those of the first call.  The counters are compared with
# what the call has changed in the table.
@pytest.mark.parametrize("n", [9_000_000, (1 << 24) + 65])
@pytest.mark.parametrize("policy,probe,layout", [(mp.EVICT_TTL, 12, "records"), (mp.EVICT_TTL, 12, "separate"), (mp.EVICT_LRU, 7, "records"),
                                                 (mp.EVICT_LRU, 15, "separate"), (mp.EVICT_LRU, 30, "records"), (mp.EVICT_LRU, 60, "separate")])
def test_counters_of_long_lists(policy, probe, layout, n):
    g = mp.MpzchTable(n + n // 8, probe, policy, 1, 53, layout=mp.LAYOUT_RECORDS if layout == "records" else mp.LAYOUT_SEPARATE)
    for call in range(2):
        before = g.identities.clone()
        g.remap(wl.distinct_ids_device(call * n, (call + 1) * n, "cuda", salt=3), 5 * call)
        st = g.stats_dict()
        inserted, changed = (before == -1) & (g.identities >= 0), (before >= 0) & (g.identities != before)
        assert int((g.identities < -1).sum()) == 0
        assert st["miss_pos"] == st["distinct_miss"] == n and st["hit_pos"] == st["invalid_pos"] == 0
        assert st["inserts"] == int(inserted.sum()) and st["evictions"] == int(changed.sum()) == int(g.num_evicted)
        assert st["collisions"] == n - st["inserts"] - st["evictions"]
        assert torch.equal(torch.sort(g.evicted).values, torch.nonzero(changed).flatten())
        assert st["inserts"] > n // 2 if call == 0 else st["evictions"] > n // 2
    g.close()


@pytest.mark.parametrize("kinds", [(True, "lru", False), ("lru", "lru", "expiry")])
@pytest.mark.parametrize("probe", [8, 61, 70])
def test_counters_of_groups(probe, kinds):
    """Features of a handful of values: a wavefront has claimants of many tables, at each of its steps of others."""
    from test_gpu_jagged import JaggedPair
    rng = rng_for(922)
    specs = [wl.TableSpec(40 + 3 * f, probe, 1, kinds[f % 3], 60 + f) for f in range(64)]
    jp = JaggedPair(specs, range(0, 64, 2))
    for step in range(4):
        counts = rng.integers(0, 30, size=64) if step else np.full(64, 3)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        vals = rng.integers(-1, 400, size=int(offsets[-1]))
        if step == 2:
            v = torch.from_numpy(vals).cuda()
            evicted, count = torch.empty_like(v), torch.empty(64, dtype=torch.int64, device="cuda")
            mp.mpzch_remap_jagged(jp.group, jp.I, jp.M, v, torch.from_numpy(offsets).cuda(), 2 * step, torch.empty_like(v), evicted,
                                  offsets.tolist(), count, None)
            _, evs, _ = oracle.remap_jagged(jp.o, vals, offsets, 2 * step, None)
            assert count.tolist() == [len(e) for e in evs]
        else:
            jp.step(vals, offsets, 2 * step)
        jp.check_state()
    jp.close()


# ---- whether the scratch set is read back or the notes decide, on both sides of the lines and with few and many misses
@pytest.mark.parametrize("evict", [True, False])
@pytest.mark.parametrize("n", [32_768, 32_769, 57_344, 57_345, 131_072, 131_073])
def test_first_occurrences_read_back_or_noted(n, evict):
    rng = rng_for(915)
    t = Pair(3 * n, 24, 1, evict, 41, layout="records")
    old = rng.integers(0, 1 << 50, size=n)
    for step, share in enumerate([1.0, 0.4, 0.7]):
        new = rng.integers(0, 1 << 50, size=n)
        ids = np.where(rng.random(n) < share, new, old)
        ids[rng.random(n) < 0.1] = ids[0]
        t.step(rng.permutation(np.concatenate([ids[: n // 2], ids[rng.integers(0, n, size=n - n // 2)]])), step)
        old = ids
    t.close()


# ---- the same in groups: copies are merged within a wavefront and a table, features end inside wavefronts, the same ids are
# new in several of them, and of the copies the one that asks for the latest expiry step counts
@pytest.mark.parametrize("records", [(0, 1, 2, 3, 4), (1, 3)])
@pytest.mark.parametrize("n", [37, 700, 66_000])
def test_new_ids_with_many_copies_in_groups(n, records):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(919)
    specs = [wl.TableSpec(2_003, 16, 1, True, 81), wl.TableSpec(300, 8, 0, "lru", 82), wl.TableSpec(1_501, 24, 2, "expiry", 83),
             wl.TableSpec(5, 3, 1, True, 84), wl.TableSpec(4_000, 16, 0, False, 85)]
    jp = JaggedPair(specs, records)
    for step in range(4):
        counts = n + np.array([0, 1, -5, 30, 7])
        hot = rng.integers(0, 1 << 40, size=5)
        vals = []
        for c in counts:
            v = np.where(rng.random(c) < 0.7, hot[rng.integers(0, 5, size=c)], rng.integers(0, 1 << 40, size=c))
            v[: c // 3] = hot[0]
            vals.append(v[rng.permutation(c)])
        vals = np.concatenate(vals)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        jp.step(vals, offsets, 2 * step, None if step % 2 else rng.integers(0, 6, size=len(vals)).astype(np.int32))
    jp.check_state()
    jp.close()


# ---- groups on both sides of the line at which a second workgroup of the last kernel comes to a compute unit
@pytest.mark.parametrize("more", [0, 1])
def test_groups_around_the_line_of_the_last_kernel(more):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(920)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 16 * 64 + more
    specs = [wl.TableSpec(30_011, 16, 1, True, 91), wl.TableSpec(9_001, 8, 0, "lru", 92), wl.TableSpec(25_000, 24, 2, "expiry", 93)]
    jp = JaggedPair(specs, (0, 2))
    offsets = np.array([0, n // 2 + 7, n // 2 + n // 5, n], dtype=np.int64)
    for step in (0, 3):
        vals = np.concatenate([wl.zipf_ids(rng, int(c), 1.05, 3 * s.num_slots) + step for c, s in zip(np.diff(offsets), specs)])
        jp.step(vals, offsets, step)
    jp.check_state()
    jp.close()


# ---- groups on both sides of the lines at which a wavefront of Pass 1 comes to have a second chunk, and of overlapped inserts: features end inside of
# wavefronts, the same ids are new in all of them, tables of fewer slots than a request is wide, windows around the block sizes
@pytest.mark.parametrize("records", [range(6), (1, 2, 4)], ids=["records", "mixed"])
@pytest.mark.parametrize("chunks,more", [(8, 0), (8, 1), (4, 0), (4, 1)])
def test_groups_around_the_line_of_one_chunk(chunks, more, records):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(923)
    n = torch.cuda.get_device_properties(0).multi_processor_count * chunks * 256 + more
    specs = [wl.TableSpec(120_011, 16, 1, True, 101), wl.TableSpec(50, 64, 1, True, 102), wl.TableSpec(90_001, 9, 0, "lru", 103),
             wl.TableSpec(5, 8, 2, "expiry", 104), wl.TableSpec(150_000, 24, 2, "expiry", 105), wl.TableSpec(80_000, 65, 0, False, 106)]
    jp = JaggedPair(specs, records)
    offsets = np.array([0, n // 3 + 7, n // 3 + 40, n // 2 + 1, n // 2 + 20, n - n // 5, n], dtype=np.int64)
    for step in (0, 3):
        vals = np.concatenate([wl.zipf_ids(rng, int(c), 1.05, 300_000) + 1_000 * step for c in np.diff(offsets)])
        vals[rng.random(n) < 0.01] = -1
        jp.step(vals, offsets, step, None if step else rng.integers(0, 6, size=n).astype(np.int32))
    jp.check_state()
    jp.close()


# ---- groups on both sides of the lines that their longest windows draw for the same kernel (searches that go on beyond its widest
# look, in full tables)
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("chunks,policy,probe,records", [(3, "lru", 33, range(3)), (2, "lru", 65, range(3)), (6, True, 129, range(3)), (6, "lru", 101, (1,)),
                                                         (6, False, 513, range(3)), (3, "lru", 600, ())])
def test_groups_around_the_lines_of_long_windows(chunks, policy, probe, records, more):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(929)
    n = torch.cuda.get_device_properties(0).multi_processor_count * chunks * 256 + more
    specs = [wl.TableSpec(n // 2, 16, 1, True, 121), wl.TableSpec(2_003, probe, 1, policy, 122), wl.TableSpec(n // 3, 24, 2, "expiry", 123)]
    jp = JaggedPair(specs, records)
    offsets = np.array([0, n // 2 + 5, n // 2 + 3_009, n], dtype=np.int64)
    for step in (0, 1, 3):
        vals = np.concatenate([rng.integers(0, 2 * specs[f].num_slots, size=int(c)) + step * 400 for f, c in enumerate(np.diff(offsets))])
        jp.step(vals, offsets, step)
    jp.check_state()
    jp.close()


# ---- claims of groups stand without a look at the table unless a note says that they were displaced: crowded windows, where most
# are, LRU tables (no notes) among the others, copies of new ids, the next call with the notes that this one must not leave behind
@pytest.mark.parametrize("records", [range(5), (0, 3)], ids=["records", "mixed"])
@pytest.mark.parametrize("n", [3_000, 90_001, 1_300_003])
def test_groups_with_displaced_claims(n, records):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(925)
    per = n // 12
    specs = [wl.TableSpec(per, 24, 1, True, 111), wl.TableSpec(per, 16, 0, "lru", 112), wl.TableSpec(per + 1, 64, 2, "expiry", 113),
             wl.TableSpec(per, 7, 0, False, 114), wl.TableSpec(per, 260, 1, True, 115)]
    jp = JaggedPair(specs, records)
    offsets = np.array([0, n // 5, n // 5 + n // 4, n // 2 + 3, n - n // 7, n], dtype=np.int64)
    for step in (0, 2, 4):
        vals = np.concatenate([rng.integers(0, 2 * per, size=int(c)) + step * per // 2 for c in np.diff(offsets)])
        jp.step(vals, offsets, step, rng.integers(0, 4, size=n).astype(np.int32) if step == 2 else None)
        jp.check_state()
    jp.close()


# ---- one-chunk calls whose stores go out beside the scratch set's compare-and-swap: on both sides of each line, with new ids whose
# copies meet within a wavefront and across workgroups, and durations per position
@pytest.mark.parametrize("evict", [True, "expiry", False])
@pytest.mark.parametrize("groups,layout", [(4, "separate"), (3, "separate"), (2, "records")])
def test_calls_around_the_lines_of_overlapped_inserts(groups, layout, evict):
    rng = rng_for(927)
    n = groups * torch.cuda.get_device_properties(0).multi_processor_count * 256
    t = Pair(n, 41, 1, evict, 49, layout=layout)
    for step, more in enumerate([0, 1, 0]):
        ids = wl.zipf_ids(rng, n + more, 1.05, 2 * n) + step * n // 2
        ids[: n // 8] = rng.integers(4 * n, 4 * n + 50, size=n // 8) + 100 * step
        t.step(ids, 2 * step, ttls=rng.integers(0, 5, size=n + more).astype(np.int32) if evict == "expiry" else None)
    t.close()


# ---- the two parts of a feature's region of the scratch set (long calls): features of so few positions that the front part has no entry,
# one or two, each all new, with copies and without; in the last one nearly all positions are new, so that both parts fill up
@pytest.mark.parametrize("layout", ["separate", "records"])
def test_parts_of_the_scratch_set_in_groups(layout):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(931)
    counts = np.array([1, 2, 3, 4, 5, 8, 9, 17, 1 << 23])
    specs = [wl.TableSpec(40, 8, 1, "lru" if f == 4 else True, 130 + f) for f in range(8)] + [wl.TableSpec(2_000_003, 8, 1, True, 139)]
    jp = JaggedPair(specs, range(9) if layout == "records" else ())
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    for step, distinct in ((0, 3), (3, 1 << 40)):
        vals = rng.integers(0, distinct, size=counts.sum()) + step * distinct
        vals[offsets[8]:] = rng.integers(0, 1 << 40, size=counts[8])
        vals[offsets[8] + 5:: 3] = vals[offsets[8]: -5: 3]
        jp.step(vals, offsets, step)
    jp.check_state()
    jp.close()


# ---- ... and of one table, on both sides of the line
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("evict", [True, "lru"])
@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21])
def test_parts_of_the_scratch_set(n, evict, layout):
    rng = rng_for(933)
    t = Pair(700_001, 8, 1, evict, 53, layout=layout)
    for step in (0, 3):
        ids = rng.integers(0, 1 << 40, size=n)
        ids[1000::2] = ids[:-1000:2]
        t.step(ids, step)
    t.close()


# ---- one-chunk calls on both sides of the lines at which windows of 9 to 16 slots are no longer read whole, and the first look is at an
# aligned block: windows that end in its first block and in a later one, reach the table's end and go round it
@pytest.mark.parametrize("evict", [True, "lru", "expiry", False])
@pytest.mark.parametrize("halves,less,layout,probe", [(1, 0, "separate", 16), (1, 0, "records", 9), (2, 256, "records", 9), (2, 256, "records", 30),
                                                      (5, 256, "separate", 8), (5, 256, "separate", 17)])
def test_calls_around_the_lines_of_first_looks(halves, less, layout, probe, evict):
    rng = rng_for(937)
    n = halves * torch.cuda.get_device_properties(0).multi_processor_count * 128 - less
    slots = n // 2 + 5
    t = Pair(slots, probe, 1, evict, 59, layout=layout)
    for step, more in enumerate([0, 1, 0, 1]):
        ids = wl.zipf_ids(rng, n + more, 1.05, 2 * n) + step * n // 8
        ids[: n // 16] = ids_with_home(rng, n // 16, slots - 12, slots, slots, 59)
        t.step(ids, 2 * step, ttls=rng.integers(0, 5, size=n + more).astype(np.int32) if evict == "expiry" else None)
    t.close()


# ---- ... and at which a wavefront looks at the scratch set after a collision: all ids new, copies of them a workgroup and half a call away
@pytest.mark.parametrize("layout,evict", [("separate", False), ("records", True), ("records", "expiry"), ("separate", "lru")])
@pytest.mark.parametrize("more", [-256, -255, 0, 37])
def test_collisions_of_new_ids(layout, evict, more):
    rng = rng_for(941)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 256 + more
    t = Pair(2 * n, 24, 0, evict, 61, layout=layout)
    for step in (0, 2, 4):
        ids = rng.integers(0, 1 << 40, size=n)
        ids[n // 2::3] = ids[: n - n // 2: 3]
        ids[300::7] = ids[:-300:7]
        t.step(ids, step)
    t.close()


# ---- groups whose segments hold the ends of several features: one, two and more of them in a chunk of 64 values, empty ones between, evicted
# slots of many tables in a workgroup
@pytest.mark.parametrize("layout", ["separate", "records"])
@pytest.mark.parametrize("per,empty", [(1, 0), (31, 3), (64, 0), (150, 2), (64 * 16 + 1, 1)])
def test_segments_of_several_features(per, empty, layout):
    from test_gpu_jagged import JaggedPair
    rng = rng_for(947)
    kinds = [True, "lru", "expiry", False]
    specs = [wl.TableSpec(max(9, 2 * per), 8, 0, kinds[f % 4], 150 + f) for f in range(40)]
    jp = JaggedPair(specs, range(40) if layout == "records" else ())
    for step in range(4):
        counts = rng.integers(per // 2, per + 1, size=40)
        counts[rng.permutation(40)[: 5 * empty]] = 0
        vals = rng.integers(0, 6 * per + 1, size=counts.sum()) + step * per
        jp.step(vals, np.concatenate([[0], np.cumsum(counts)]).astype(np.int64), 2 * step)
    jp.check_state()
    jp.close()


# ---- calls of up to one workgroup per compute unit whose windows of 9 to 16 slots are read whole, and those a position, a slot of the table or
# of the window beyond: two tensors from 2^21 slots on, LRU tables of more than 256 MiB.  Homes at the table's end and in one region of it that
# fills up, so that windows go round the end, and are full
@pytest.mark.parametrize("layout,evict,slots,probe", [
    ("separate", True, (1 << 21) - 1, 16), ("separate", True, 1 << 21, 16), ("separate", "expiry", 1 << 21, 9), ("separate", "lru", 1 << 21, 13),
    ("separate", False, 1 << 21, 16), ("separate", "lru", (1 << 25) + 1, 10), ("separate", True, (1 << 25) + 1, 16), ("records", "lru", 1 << 24, 16),
    ("records", "lru", (1 << 24) + 1, 16), ("records", "lru", (1 << 24) + 1, 9)])
def test_calls_around_the_lines_of_whole_windows(layout, evict, slots, probe):
    rng = rng_for(953 + probe)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 256
    t = Pair(slots, probe, 1, evict, 67, layout=layout)
    for step, more in enumerate([0, 1, 0, 1]):
        ids = wl.zipf_ids(rng, n + more, 1.05, 2 * n) + step * n // 8
        ids[: n // 2] = ids_with_home(rng, n // 2, 4_000, 4_000 + n // 2, slots, 67)
        ids[n // 2: n // 2 + 2_000] = ids_with_home(rng, 2_000, slots - 700, slots, slots, 67)
        t.step(ids, 2 * step + 1, check_state=step == 3, ttls=rng.integers(0, 5, size=n + more).astype(np.int32) if evict == "expiry" else None)
    t.close()


# ---- the lines of even looks that windows draw: LRU tables over two tensors beyond the cache, of 16 slots and of one more; in the cache, of 8 and of one
# more, every table
@pytest.mark.parametrize("groups,probe,slots,layout,evict", [(6, 16, (1 << 25) + 1, "separate", "lru"), (5, 17, (1 << 25) + 1, "separate", "lru")] + [
    (3, probe, 1 << 19, layout, evict) for probe in (8, 9) for layout in ("separate", "records") for evict in (True, "lru", "expiry", False)])
def test_calls_around_the_lines_of_even_looks_by_window(groups, probe, slots, layout, evict):
    rng = rng_for(957 + probe)
    n = groups * torch.cuda.get_device_properties(0).multi_processor_count * 256
    t = Pair(slots, probe, 1, evict, 71, layout=layout)
    for step, more in enumerate([0, 1, 0]):
        ids = wl.zipf_ids(rng, n + more, 1.05, 2 * n) + step * n // 8
        ids[: n // 2] = ids_with_home(rng, n // 2, 4_000, 4_000 + n // 2, slots, 71)
        ids[n // 2: n // 2 + 2_000] = ids_with_home(rng, 2_000, slots - 700, slots, slots, 71)
        t.step(ids, 2 * step + 1, check_state=step == 2, ttls=rng.integers(0, 5, size=n + more).astype(np.int32) if evict == "expiry" else None)
    t.close()


def ids_of_hash(hashes, seed):
    """The ids that the library's hash takes to `hashes` (uint64): the hash undone.  Some are negative."""
    unxor = lambda x, s: x ^ (x >> np.uint64(s)) ^ (x >> np.uint64(2 * s))
    with np.errstate(over="ignore"):
        x = unxor(hashes, 31) * np.uint64(pow(0x94D049BB133111EB, -1, 1 << 64))
        x = unxor(x, 27) * np.uint64(pow(0xBF58476D1CE4E5B9, -1, 1 << 64))
        return ((unxor(x, 30) - np.uint64(0x9E3779B97F4A7C15)) ^ np.uint64(seed)).view(np.int64)


# ---- a look at the scratch set that goes round its end: several dozen ids whose first tries are the last entries of it (four for each position, by the
# low word of the hash), spread over wavefronts of new ids, with copies in other workgroups.  They fill the last eight entries and as many at the
# front as are left of them, so that looks begin in each of the last entries, find the rest full, and go on for several steps behind the end
@pytest.mark.parametrize("layout,evict", [("separate", False), ("records", True), ("records", "lru")])
@pytest.mark.parametrize("more,crowd", [(0, 24), (37, 60), (64 * 129 + 1, 250)])
def test_collisions_at_the_end_of_the_scratch_set(layout, evict, more, crowd):
    rng = rng_for(961 + crowd)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 256 + more
    size = 4 * n
    t = Pair(2 * n, 24, 0, evict, 73, layout=layout)
    for step in (0, 2):
        ids = rng.integers(0, 1 << 40, size=n)
        last = np.empty(0, dtype=np.int64)
        while last.size < crowd:
            entry = rng.integers(size - 8, size, size=4 * crowd)
            low = np.array([-(-(int(e) << 32) // size) for e in entry], dtype=np.uint64)      # the first word that leads to the entry
            high = rng.integers(0, 1 << 32, size=4 * crowd, dtype=np.uint64)
            x = ids_of_hash(high << np.uint64(32) | low, 73)
            last = np.unique(np.concatenate([last, x[x >= 0]]))
        last = rng.permutation(last)[:crowd]
        # (what the kernel makes of them)
        low = np.array([(h * size) >> 32 for h in (oracle_hash(int(i), 73) & 0xFFFFFFFF for i in last)])
        assert low.min() >= size - 8 and low.max() < size and len(np.unique(low)) > 4
        at = rng.permutation(n)[: 3 * crowd]
        ids[at] = np.tile(last, 3)
        t.step(ids, step)
    t.close()


def oracle_hash(i, seed):
    """SplitMix64's finalizer over (id xor seed) plus its increment, in whole numbers."""
    m = (1 << 64) - 1
    z = ((i ^ seed) + 0x9E3779B97F4A7C15) & m
    z = (z ^ z >> 30) * 0xBF58476D1CE4E5B9 & m
    z = (z ^ z >> 27) * 0x94D049BB133111EB & m
    return z ^ z >> 31

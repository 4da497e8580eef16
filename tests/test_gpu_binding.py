"""What the binding takes and refuses: the repeated calls are marshalled in native code, and accept what ctypes did."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2602_17050_amd import binding as mp

pytestmark = pytest.mark.gpu
INVALID_ARG = 1


def dev(a, dtype=torch.int64):
    return torch.tensor(a, dtype=dtype, device="cuda")


def refused(status, fn, *args, **kw):
    with pytest.raises(mp.MpzchError) as e:
        fn(*args, **kw)
    assert e.value.status == status


# ---- handles: a ctypes.c_void_p or other pointer, an address, or None (which the library refuses, as for a table that has been closed)
def test_handles_as_pointers_addresses_and_none():
    t = mp.MpzchTable(100, 8, mp.EVICT_TTL, 1, 7, max_batch=64)
    group = mp.mpzch_group_create([t.handle])
    ids = dev([3, 5, 3])
    out, found, stats = torch.empty_like(ids), torch.empty(3, dtype=torch.uint8, device="cuda"), torch.zeros(mp.STAT_COUNT, dtype=torch.int64, device="cuda")
    ev, nev, off = torch.empty_like(ids), torch.zeros(1, dtype=torch.int64, device="cuda"), dev([0, 3])
    rows = torch.ones((100, 4), device="cuda")
    gathered = torch.empty((3, 4), device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    calls = {
        "init_tensors": lambda h, g: mp.mpzch_init_tensors(h, t.identities, t.metadata),
        "remap": lambda h, g: mp.mpzch_remap(h, t.identities, t.metadata, ids, 1, out, ev, nev, stats),
        "noalloc": lambda h, g: mp.mpzch_remap_noalloc(h, t.identities, t.metadata, ids, 1, out, ev, nev, stats),
        "feature_ttl": lambda h, g: mp.mpzch_remap_feature_ttl(h, t.identities, t.metadata, ids, None, 1, out, ev, nev, stats),
        "reset": lambda h, g: mp.mpzch_remap_reset(h, t.identities, t.metadata, ids, 1, out, ev, nev, stats, rows),
        "lookup": lambda h, g: mp.mpzch_lookup(h, t.identities, ids, out, found),
        "lookup_stats": lambda h, g: mp.mpzch_lookup_stats(h, t.identities, ids, out, found, stats),
        "gather": lambda h, g: mp.mpzch_lookup_gather(h, t.identities, ids, rows, gathered, out, found),
        "delta": lambda h, g: mp.mpzch_collect_delta(h, t.identities, t.metadata, 1, out, ev, count),
        "jagged": lambda h, g: mp.mpzch_remap_jagged(g, [t.identities], [t.metadata], ids, off, 1, out, ev, [0, 3], nev, stats),
        "lookup_jagged": lambda h, g: mp.mpzch_lookup_jagged(g, [t.identities], ids, off, out, found),
        "reset_jagged": lambda h, g: mp.mpzch_reset_rows_jagged(g, ev, [0, 3], nev, [rows]),
    }
    for name, call in calls.items():
        call(t.handle, group)
        call(t.handle.value, group.value)
        call(ctypes.cast(t.handle, ctypes.POINTER(ctypes.c_char)), ctypes.cast(group, ctypes.POINTER(ctypes.c_char)))
        refused(INVALID_ARG, call, None, None)
        for other in (1.5, "handle", t):
            with pytest.raises(Exception):
                call(other, other)
    out.fill_(-1)
    mp.mpzch_lookup(t.handle.value, t.identities, ids, out, found)
    assert bool(found.all()) and int(out[0]) == int(out[2])
    mp.mpzch_group_destroy(group)
    t.close()
    refused(INVALID_ARG, t.remap, ids, 2)
    refused(INVALID_ARG, t.lookup, ids)


# ---- initial rows of several tensors: on the device or in pinned host memory; a list may be shorter or longer than the
# tensors (several tensors of one table: refused when shorter; tables of a group: the rest is left alone)
def test_initial_rows_of_several_tensors():
    slots, count = dev([2, 7, 9, 4]), dev([3])
    rows = lambda: torch.arange(80, dtype=torch.float32, device="cuda").view(10, 8).clone()
    pinned = torch.full((8,), 2.5, pin_memory=True)
    init = torch.full((8,), -1.5, device="cuda")
    want = lambda v: torch.stack([torch.full((8,), v) if k in (2, 7, 9) else torch.arange(8 * k, 8 * k + 8).float() for k in range(10)])
    a, b = rows(), rows()
    mp.mpzch_reset_rows_multi(slots, count, [a, b], [pinned, init])
    assert torch.equal(a.cpu(), want(2.5)) and torch.equal(b.cpu(), want(-1.5))
    a, b = rows(), rows()
    mp.mpzch_reset_rows_multi(slots, count, [a, b], [None, init, init])
    assert torch.equal(a.cpu(), want(0.0)) and torch.equal(b.cpu(), want(-1.5))
    refused(INVALID_ARG, mp.mpzch_reset_rows_multi, slots, count, [a, b], [init])
    # a row of another size is refused
    for other in (init[:7], torch.zeros(16, device="cuda"), torch.zeros((8, 2), device="cuda")[:, 0]):
        with pytest.raises(AssertionError):
            mp.mpzch_reset_rows_multi(slots, count, [a], [other])

    tables = [mp.MpzchTable(10, 4, mp.EVICT_TTL, 1, 7) for _ in range(2)]
    group = mp.mpzch_group_create([t.handle for t in tables])
    jagged, counts, at = dev([2, 7, 9, 9, 7, 2]), dev([3, 3]), [0, 3, 6]
    for inits, first, second in [([pinned, init], 2.5, -1.5), ([init], -1.5, None), ([None, pinned, init], 0.0, 2.5)]:
        a, b = rows(), rows()
        mp.mpzch_reset_rows_jagged(group, jagged, at, counts, [a, b], inits)
        assert torch.equal(a.cpu(), want(first))
        assert torch.equal(b.cpu(), rows().cpu() if second is None else want(second))
    mp.mpzch_group_destroy(group)
    for t in tables:
        t.close()


# ---- whole numbers: steps as ctypes takes them, offsets as int() does
def test_steps_and_offsets():
    tables = [mp.MpzchTable(64, 8, mp.EVICT_TTL, 0, 7 + f) for f in range(2)]
    group = mp.mpzch_group_create([t.handle for t in tables])
    I, M = [t.identities for t in tables], [t.metadata for t in tables]
    ids, off = torch.arange(200, dtype=torch.int64, device="cuda"), dev([0, 120, 200])
    out, nev = torch.empty_like(ids), torch.zeros(2, dtype=torch.int64, device="cuda")
    rows = [torch.ones((64, 4), device="cuda") for _ in tables]
    step = 0
    for at in ([0, 120, 200], (0, 120, 200), [0.0, 120.0, 200.0], np.array([0, 120, 200], np.int32), np.array([0.0, 120.0, 200.0]),
               torch.tensor([0, 120, 200]), torch.tensor([0.0, 120.0, 200.0]), off, iter([0, 120, 200])):
        step += 2
        ids += 200
        again = [0, 120, 200] if hasattr(at, "__next__") else at
        ev = torch.full((200,), -7, dtype=torch.int64, device="cuda")
        mp.mpzch_remap_jagged(group, I, M, ids, off, np.int64(step), out, ev, at, nev)
        n = nev.tolist()
        assert step == 2 or min(n) > 0
        assert bool((ev[: n[0]] >= 0).all()) and bool((ev[n[0]: 120] == -7).all())
        assert bool((ev[120: 120 + n[1]] >= 0).all()) and bool((ev[120 + n[1]:] == -7).all())
        for r in rows:
            r.fill_(1.0)
        mp.mpzch_reset_rows_jagged(group, ev, again, nev, rows)
        for f, lo in enumerate((0, 120)):
            want = torch.ones(64, device="cuda")
            want[ev[lo: lo + n[f]]] = 0.0
            assert torch.equal(rows[f], want[:, None].expand(64, 4))
    # one too many is refused; what is left out counts as zero, which the library refuses unless all are
    for fn in (lambda at: mp.mpzch_remap_jagged(group, I, M, ids, off, step, out, ev, at, nev),
               lambda at: mp.mpzch_reset_rows_jagged(group, ev, at, nev, rows)):
        with pytest.raises((ValueError, IndexError)):
            fn([0, 120, 200, 200])
        refused(INVALID_ARG, fn, [0, 120])
        fn([0, 0])
        with pytest.raises(TypeError):
            fn([0, None, 200])
    for bad in (1.0, "1", None):
        with pytest.raises(Exception):
            mp.mpzch_remap(tables[0].handle, I[0], M[0], ids, bad, out, ev, nev)
    mp.mpzch_group_destroy(group)
    for t in tables:
        t.close()


# ---- a tensor that a call cannot do without is not an empty batch
def test_missing_batches_are_refused():
    t = mp.MpzchTable(64, 8, mp.EVICT_TTL, 0, 7, max_batch=64)
    group = mp.mpzch_group_create([t.handle])
    I, M = t.identities, t.metadata
    ids, rows = dev([1, 2, 3]), torch.ones((64, 4), device="cuda")
    out, ev, nev, off, found = torch.empty_like(ids), torch.empty_like(ids), dev([0]), dev([0, 3]), torch.zeros(3, dtype=torch.uint8, device="cuda")
    stats = torch.zeros(mp.STAT_COUNT, dtype=torch.int64, device="cuda")
    for call in (lambda: mp.mpzch_remap(t.handle, I, M, None, 1, out, ev, nev),
                 lambda: mp.mpzch_remap_noalloc(t.handle, I, M, None, 1, out, ev, nev),
                 lambda: mp.mpzch_remap_feature_ttl(t.handle, I, M, None, None, 1, out, ev, nev),
                 lambda: mp.mpzch_remap_reset(t.handle, I, M, None, 1, out, ev, nev, stats, rows),
                 lambda: mp.mpzch_lookup(t.handle, I, None, out, found),
                 lambda: mp.mpzch_lookup_stats(t.handle, I, None, out, found, stats),
                 lambda: mp.mpzch_lookup_gather(t.handle, I, None, rows, torch.empty((0, 4), device="cuda")),
                 lambda: mp.mpzch_remap_jagged(group, [I], [M], None, off, 1, out, ev, [0, 3], nev),
                 lambda: mp.mpzch_lookup_jagged(group, [I], None, off, out, found),
                 lambda: mp.mpzch_reset_rows(None, nev, rows),
                 lambda: mp.mpzch_reset_rows_multi(None, nev, [rows]),
                 lambda: mp.mpzch_collect_delta(t.handle, I, M, 0, None, None, nev),
                 lambda: mp.mpzch_gather_rows(None, nev, rows, torch.empty((0, 4), device="cuda")),
                 lambda: mp.mpzch_apply_delta(I, None, None, nev),
                 lambda: mp.mpzch_apply_delta(None, out, ids, nev)):
        with pytest.raises((AttributeError, TypeError)):
            call()
    # the list of evicted slots and the retention times may be left out
    t.remap(ids, 1)
    mp.mpzch_remap(t.handle, I, M, ids, 2, out, None, nev)
    mp.mpzch_group_destroy(group)
    t.close()


# ---- lists with fewer entries than the group has tables: what is missing is a null pointer, which the library refuses
def test_lists_shorter_than_the_group():
    tables = [mp.MpzchTable(64, 8, mp.EVICT_TTL, 0, 7 + f) for f in range(3)]
    group = mp.mpzch_group_create([t.handle for t in tables])
    I, M = [t.identities for t in tables], [t.metadata for t in tables]
    ids, off, nev = dev([1, 2, 3]), dev([0, 1, 2, 3]), dev([1, 1, 1])
    out, ev, rows = torch.full_like(ids, -7), dev([5, 6, 7]), [torch.ones((64, 4), device="cuda") for _ in tables]
    for n in (0, 1, 2):
        refused(INVALID_ARG, mp.mpzch_remap_jagged, group, I[:n], M[:n], ids, off, 1, out, ev, [0, 1, 2, 3][: n + 1], nev)
        refused(INVALID_ARG, mp.mpzch_lookup_jagged, group, I[:n], ids, off, out)
    refused(INVALID_ARG, mp.mpzch_reset_rows_jagged, group, ev, [0, 1, 2], nev, rows[:2])
    mp.mpzch_reset_rows_jagged(group, ev, [0, 0], nev, rows[:1])
    assert all(bool((r == 1.0).all()) for r in rows) and bool((out == -7).all())
    mp.mpzch_group_destroy(group)
    for t in tables:
        t.close()

"""The work a user of this library has it do, as cases that can be timed and compared.

Every case is one pass through the public entry points (paper_2602_17050_amd.binding) on state that such a
program keeps: a table, its embedding rows, batches that are already in device memory.  The families:

  session   a small or medium table trained from empty: init, an optional bulk load, then `steps` batches.  The
            table is initialised inside the pass, so every pass does the same work.
  stream    one training step on a large table in steady state: `new` of the batch are ids never seen before, the
            rest were new some steps ago (geometric age).  The table carries on from pass to pass.
  load      bulk load of distinct ids with eviction off (long probe ranges, the table filled to the brim),
            through the entry point that allocates nothing.
  lookup    one inference batch on a filled table, with or without the gather of the embedding rows.
  jagged    a keyed jagged batch over several tables, training (with row reset) or inference.
  publish   the streaming delta of a training table carried over to an inference copy.

The batches of a table that carries on must not repeat themselves, or every id would be resident after one round.
A pass therefore moves the ids of the batch it has used forward by a constant (one in-place add on the batch: the
arrival of a later batch in the program's input buffer).  The ids are drawn relative to a running counter, so the
moved batch has the same distribution with respect to the table as the one before.
"""
import math
from types import SimpleNamespace

import torch

from paper_2602_17050_amd import binding as mp
from paper_2602_17050_amd import workloads as wl

DEVICE = "cuda"
MEAN_AGE = 10.0            # steps; how long ago the recurring ids of a stream were new
CHUNK = 1 << 24            # ids per call while a large table is filled before the pass
KINDS = {"ttl": mp.EVICT_TTL, "lru": mp.EVICT_LRU, "expiry": mp.EVICT_TTL_EXPIRY, "none": mp.EVICT_NONE}
DTYPES = {"float32": torch.float32, "bfloat16": torch.bfloat16}


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest training there is: a few thousand slots, 1 024 ids per step, every step a call for the remap
        # and one for the row reset; latency and launches are all that counts
        dict(name="tiny session", family="session", slots=4096, probe=8, policy="ttl", ttl=3, load=0.0, batch=1024,
             steps=8, fresh=0.0, alpha=1.1, universe=16384, rows=4096, dim=16, dtype="float32", layout="separate",
             reset="call"),
        # a medium table that fills from 0.3 to 0.9 over fifty steps of 65 536 ids, rows reset by the remap itself
        dict(name="growing session", family="session", slots=1_000_000, probe=16, policy="ttl", ttl=10, load=0.3,
             batch=65536, steps=50, fresh=0.05, alpha=1.05, universe=2_000_000, rows=1_000_000, dim=64,
             dtype="float32", layout="records", reset="fused"),
        # a table shared by features of different retention (a ttl per position), no size a round number
        dict(name="shared session", family="session", slots=200_003, probe=24, policy="expiry", ttl=5, load=0.5,
             batch=20_011, steps=12, fresh=0.10, alpha=1.1, universe=300_007, rows=50_021, dim=48, dtype="float32",
             layout="separate", reset="call"),
        # collision-free bulk load: as many distinct ids as slots, probe range 64, eviction off
        dict(name="bulk load", family="load", slots=3_000_000, probe=64, ids=3_000_000, per_call=mp.NOALLOC_MAX_BATCH,
             layout="separate"),
        # the largest table: a shard of a billion slots, 4 M ids per step, 10 % of them new
        dict(name="stream 1B records", family="stream", slots=1_000_000_000, probe=16, policy="ttl", ttl=20, load=0.7,
             batch=4_000_000, new=0.10, rows=25_000_000, dim=128, dtype="bfloat16", layout="records", reset="fused"),
        # the same with the two auxiliary tensors apart and the rows reset by a call of their own
        dict(name="stream 500M tensors", family="stream", slots=500_000_000, probe=16, policy="ttl", ttl=20, load=0.9,
             batch=2_000_000, new=0.10, rows=25_000_000, dim=128, dtype="bfloat16", layout="separate", reset="call"),
        # LRU eviction on a nearly full table, weights and optimizer state reset together, ragged sizes
        dict(name="stream 60M lru", family="stream", slots=60_000_001, probe=32, policy="lru", ttl=0, load=0.95,
             batch=300_007, new=0.10, rows=6_000_011, dim=64, dtype="float32", layout="records", reset="multi"),
        # inference on 100 M slots, 1 M ids per batch, 5 % of them unknown
        dict(name="lookup 1M", family="lookup", slots=100_000_000, probe=32, load=0.8, batch=1_000_000, unknown=0.05,
             alpha=1.2, rows=0, dim=0, dtype="bfloat16", layout="separate"),
        # the same fused with the gather of the rows, ragged batch
        dict(name="lookup gather 300K", family="lookup", slots=100_000_000, probe=32, load=0.8, batch=300_007,
             unknown=0.05, alpha=1.2, rows=25_000_000, dim=128, dtype="bfloat16", layout="separate"),
        # one training step of a whole embedding collection: 26 tables of 1 K slots and up, 41 M values
        dict(name="jagged step", family="jagged", train=True, tables=26, total_slots=1_000_000_000, samples=65536,
             load=0.5, dim=16, dtype="bfloat16", layout="records"),
        # a small serving request over the same kind of collection
        dict(name="jagged request", family="jagged", train=False, tables=26, total_slots=100_000_000, samples=16,
             load=0.5, dim=0, dtype="bfloat16", layout="separate"),
        # publishing what changed in the last three steps of a 50 M-slot table
        dict(name="publish", family="publish", slots=50_000_000, probe=16, load=0.8, batch=400_000, new=0.10,
             rows=10_000_000, dim=128, dtype="bfloat16", layout="records"),
    ]


def _log(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm (odd and ragged values come with it)."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    family = rng.choice(["session", "session", "load", "stream", "stream", "lookup", "lookup", "jagged", "jagged", "publish"])
    layout = rng.choice(["separate", "records"])
    if family == "session":
        slots = _log(rng, 2_000, 1_000_000)
        policy = rng.choice(["ttl", "ttl", "expiry", "lru"])
        return dict(family=family, slots=slots, probe=rng.choice([8, 16, 24, 32]), policy=policy, ttl=rng.randint(2, 12),
                    load=rng.choice([0.0, 0.3, 0.5]), batch=_log(rng, 256, 65536), steps=rng.randint(6, 20),
                    fresh=round(rng.uniform(0.0, 0.2), 3), alpha=round(rng.uniform(1.02, 1.2), 3), universe=2 * slots,
                    rows=max(64, slots // rng.choice([1, 3])), dim=rng.choice([16, 24, 48, 64]), dtype="float32",
                    layout=layout, reset="call" if policy == "expiry" else rng.choice(["call", "fused", "multi"]))
    if family == "load":
        slots = _log(rng, 100_000, 3_000_000)
        return dict(family=family, slots=slots, probe=rng.choice([8, 16, 64, 256, 512]),
                    ids=int(slots * rng.uniform(0.5, 1.0)), per_call=_log(rng, 65536, mp.NOALLOC_MAX_BATCH), layout=layout)
    if family == "stream":
        slots = _log(rng, 20_000_000, 600_000_000)
        policy = rng.choice(["ttl", "ttl", "lru"])
        return dict(family=family, slots=slots, probe=rng.choice([8, 16, 32, 64]), policy=policy,
                    ttl=rng.randint(5, 30) if policy == "ttl" else 0, load=round(rng.uniform(0.6, 0.95), 3),
                    batch=_log(rng, 65536, 3_000_000), new=round(rng.uniform(0.02, 0.2), 3),
                    rows=_log(rng, 2_000_000, 10_000_000), dim=rng.choice([32, 64, 128]), dtype="bfloat16",
                    layout=layout, reset=rng.choice(["fused", "call", "multi"]))
    if family == "lookup":
        gather = rng.random() < 0.5
        return dict(family=family, slots=_log(rng, 1_000_000, 100_000_000), probe=rng.choice([16, 32, 64]),
                    load=round(rng.uniform(0.5, 0.9), 3), batch=_log(rng, 1_000, 2_000_000),
                    unknown=round(rng.uniform(0.0, 0.2), 3), alpha=round(rng.uniform(1.05, 1.3), 3),
                    rows=_log(rng, 1_000_000, 20_000_000) if gather else 0, dim=rng.choice([32, 64, 128]) if gather else 0,
                    dtype="bfloat16", layout=layout)
    if family == "jagged":
        train = rng.random() < 0.5
        return dict(family=family, train=train, tables=rng.randint(4, 26), total_slots=_log(rng, 2_000_000, 200_000_000),
                    samples=_log(rng, 512, 16384) if train else _log(rng, 8, 16384), load=round(rng.uniform(0.3, 0.7), 3),
                    dim=16 if train else 0, dtype="bfloat16", layout=layout if not train else "records")
    return dict(family=family, slots=_log(rng, 5_000_000, 50_000_000), probe=16, load=round(rng.uniform(0.5, 0.9), 3),
                batch=_log(rng, 20_000, 400_000), new=round(rng.uniform(0.05, 0.2), 3), rows=_log(rng, 1_000_000, 10_000_000),
                dim=rng.choice([64, 128]), dtype="bfloat16", layout=layout)


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 7919 + wl.DATA_SEED)
    return g


def _origin(seed):
    """Where a seed's ids begin: far from those of other seeds, room for 2^32 ids on either side."""
    return (1 << 40) + ((int(seed) % (1 << 20)) << 34) + (1 << 33)


def _zipf(gen, n, alpha, universe):
    """n ranks in [1, universe], popularity ~ rank^-alpha: the inverse CDF of workloads.zipf_ranks, on the device."""
    top = float(universe + 1) ** (1.0 - alpha)
    u = torch.rand(n, dtype=torch.float64, device=DEVICE, generator=gen)
    x = u.mul_(top - 1.0).add_(1.0).pow_(1.0 / (1.0 - alpha))
    return x.floor_().clamp_(max=float(universe)).to(torch.int64)


def _stream_batch(gen, n, m, origin, index):
    """Step `index` of a stream: m ids of its own, the other n - m were new some steps ago."""
    first = origin + index * m
    age = torch.empty(n - m, dtype=torch.float64, device=DEVICE).geometric_(1.0 / MEAN_AGE, generator=gen).clamp_(max=100.0)
    old = first - age.to(torch.int64) * m + torch.randint(0, m, (n - m,), device=DEVICE, generator=gen)
    ids = torch.cat([torch.arange(first, first + m, dtype=torch.int64, device=DEVICE), old])
    return ids[torch.randperm(n, device=DEVICE, generator=gen)].contiguous()


def _layout(case):
    return mp.LAYOUT_RECORDS if case["layout"] == "records" else mp.LAYOUT_SEPARATE


def _table(case, policy, ttl, max_batch):
    return mp.MpzchTable(case["slots"], case["probe"], KINDS[policy], ttl, wl.HASH_SEED_BASE + 7, max_batch=max_batch,
                         layout=_layout(case))


def _state_of(t):
    return [t.records] if t.layout == mp.LAYOUT_RECORDS else [t.identities, t.metadata]


def _fill(t, lo, hi, out, step_of=None):
    """Inserts the ids [lo, hi), CHUNK per call; step_of(k): the step of the k-th call (0 when not given)."""
    for k, a in enumerate(range(lo, hi, CHUNK)):
        b = min(a + CHUNK, hi)
        t.remap(torch.arange(a, b, dtype=torch.int64, device=DEVICE), step_of(k) if step_of else 0, out[: b - a])


def _rows(case, gen, count=1):
    return [torch.empty((case["rows"], case["dim"]), dtype=DTYPES[case["dtype"]], device=DEVICE).uniform_(0.5, 1.5, generator=gen)
            for _ in range(count)]


def prepare(case, seed):
    return _PREPARE[case["family"]](case, _generator(seed), _origin(seed))


def run(s):
    return s.run(s)


def _prepare_session(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_session)
    n, steps = case["batch"], case["steps"]
    prefill = int(case["load"] * case["slots"])
    s.table = _table(case, case["policy"], case["ttl"], max(n, prefill))
    s.rows = _rows(case, gen, 2 if case["reset"] == "multi" else 1)
    s.prefill = torch.arange(prefill, dtype=torch.int64, device=DEVICE) + (origin + (1 << 32)) if prefill else None
    s.ids = origin + _zipf(gen, n * steps, case["alpha"], case["universe"]).view(steps, n)
    fresh = int(case["fresh"] * n)
    if fresh:
        for k in range(steps):
            at = torch.randperm(n, device=DEVICE, generator=gen)[:fresh]
            s.ids[k, at] = torch.arange(fresh, dtype=torch.int64, device=DEVICE) + (origin - (1 << 32) + k * fresh)
    s.ttls = None
    if case["policy"] == "expiry":
        kinds = torch.tensor([1, case["ttl"], 4 * case["ttl"]], dtype=torch.int32, device=DEVICE)
        s.ttls = kinds[torch.randint(0, 3, (steps, n), device=DEVICE, generator=gen)].contiguous()
    s.out = torch.empty((steps, n), dtype=torch.int64, device=DEVICE)
    s.out_prefill = torch.empty(max(prefill, 1), dtype=torch.int64, device=DEVICE)
    return s


def _run_session(s):
    t, reset = s.table, s.case["reset"]
    mp.mpzch_init_tensors(t.handle, t.identities, t.metadata)
    if s.prefill is not None:
        t.remap(s.prefill, 0, s.out_prefill)
    for k in range(s.case["steps"]):
        if reset == "fused":
            t.remap_reset(s.ids[k], k + 1, s.rows[0], out_slots=s.out[k])
            continue
        t.remap(s.ids[k], k + 1, s.out[k], ttls=None if s.ttls is None else s.ttls[k])
        if reset == "multi":
            mp.mpzch_reset_rows_multi(t._evicted, t.num_evicted, s.rows)
        else:
            t.reset_rows(s.rows[0])
    return [s.out, t.num_evicted, t.stats, s.rows] + _state_of(t)


def _prepare_load(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_load)
    s.table = _table(case, "none", 0, 0)
    s.ids = origin + torch.randperm(2 * case["ids"], device=DEVICE, generator=gen)[: case["ids"]]
    s.out = torch.empty_like(s.ids)
    calls = -(-case["ids"] // case["per_call"])
    s.num_evicted = torch.zeros((calls, 1), dtype=torch.int64, device=DEVICE)
    s.stats = torch.zeros((calls, mp.STAT_COUNT), dtype=torch.int64, device=DEVICE)
    return s


def _run_load(s):
    t, step = s.table, s.case["per_call"]
    mp.mpzch_init_tensors(t.handle, t.identities, t.metadata)
    for k, lo in enumerate(range(0, s.case["ids"], step)):
        mp.mpzch_remap_noalloc(t.handle, t.identities, t.metadata, s.ids[lo: lo + step], 1 + k, s.out[lo: lo + step], None,
                               s.num_evicted[k], s.stats[k])
    return [s.out, s.stats] + _state_of(t)


RING = 4                   # batches a stream keeps; each is moved on by RING steps when it has been used


def _prepare_stream(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_stream)
    n = case["batch"]
    s.new = max(1, int(case["new"] * n))
    s.table = t = _table(case, case["policy"], case["ttl"], CHUNK)
    out = torch.empty(CHUNK, dtype=torch.int64, device=DEVICE)
    # what has been seen before the stream goes on: under TTL all of it expired, under LRU of different age
    _fill(t, origin - int(case["load"] * case["slots"]), origin, out, (lambda k: k) if case["policy"] == "lru" else None)
    s.step = 200
    s.rows = _rows(case, gen, 2 if case["reset"] == "multi" else 1)
    s.ring = [_stream_batch(gen, n, s.new, origin, k) for k in range(RING)]
    s.out = torch.empty(n, dtype=torch.int64, device=DEVICE)
    s.evicted = torch.empty(n, dtype=torch.int64, device=DEVICE)
    s.num_evicted = torch.zeros(1, dtype=torch.int64, device=DEVICE)
    s.stats = torch.zeros(mp.STAT_COUNT, dtype=torch.int64, device=DEVICE)
    return s


def _run_stream(s):
    t, reset = s.table, s.case["reset"]
    ids = s.ring[s.step % RING]
    if reset == "fused":
        mp.mpzch_remap_reset(t.handle, t.identities, t.metadata, ids, s.step, s.out, s.evicted, s.num_evicted, s.stats, s.rows[0])
    else:
        mp.mpzch_remap(t.handle, t.identities, t.metadata, ids, s.step, s.out, s.evicted, s.num_evicted, s.stats)
        if reset == "multi":
            mp.mpzch_reset_rows_multi(s.evicted, s.num_evicted, s.rows)
        else:
            mp.mpzch_reset_rows(s.evicted, s.num_evicted, s.rows[0])
    ids.add_(RING * s.new)          # the next batch of this buffer
    s.step += 1
    return [s.out, s.num_evicted, s.stats, s.rows] + _state_of(t)


def _prepare_lookup(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_lookup, at=0)
    n, resident = case["batch"], int(case["load"] * case["slots"])
    s.table = t = _table(case, "none", 0, 0)
    out = torch.empty(CHUNK, dtype=torch.int64, device=DEVICE)
    _fill(t, origin, origin + resident, out)
    unknown = int(case["unknown"] * n)
    s.ring = []
    for _ in range(RING):
        # popular ids lie anywhere in the order in which the ids came
        known = origin + (_zipf(gen, n - unknown, case["alpha"], resident) * 2654435761 + 12345) % resident
        other = torch.randint(0, 1 << 62, (unknown,), device=DEVICE, generator=gen)
        s.ring.append(torch.cat([known, other])[torch.randperm(n, device=DEVICE, generator=gen)].contiguous())
    s.out = torch.empty(n, dtype=torch.int64, device=DEVICE)
    s.found = torch.empty(n, dtype=torch.uint8, device=DEVICE)
    s.rows = s.out_rows = None
    if case["rows"]:
        s.rows = _rows(case, gen)[0]
        s.out_rows = torch.empty((n, case["dim"]), dtype=s.rows.dtype, device=DEVICE)
    return s


def _run_lookup(s):
    t, ids = s.table, s.ring[s.at % RING]
    s.at += 1
    if s.rows is None:
        mp.mpzch_lookup(t.handle, t.identities, ids, s.out, s.found)
        return [s.out, s.found]
    mp.mpzch_lookup_gather(t.handle, t.identities, ids, s.rows, s.out_rows, s.out, s.found)
    return [s.out_rows, s.out, s.found]


def _collection(case):
    return wl.c5_spec(total_slots_cap=case["total_slots"], samples=case["samples"], num_tables=case["tables"])


TAIL = 1 << 32             # how far the ids of a feature's tail lie from those of its head


def _head(table):
    return max(1, table.num_slots // 4)


class _Group:
    """A group handle that goes when the state goes."""

    def __init__(self, handles):
        self.handle = mp.mpzch_group_create(handles)

    def __del__(self):
        mp.mpzch_group_destroy(self.handle)


def _prepare_jagged(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_jagged_train if case["train"] else _run_jagged_lookup)
    spec = _collection(case)
    s.tables = [mp.MpzchTable(t.num_slots, t.max_probe, mp.EVICT_TTL, t.ttl, t.hash_seed, layout=_layout(case)) for t in spec.tables]
    s.identities = [t.identities for t in s.tables]
    s.metadata = [t.metadata for t in s.tables]
    s.owner = _Group([t.handle for t in s.tables])
    s.group = s.owner.handle
    out = torch.empty(CHUNK, dtype=torch.int64, device=DEVICE)
    for t in s.tables:
        head = _head(t)
        _fill(t, origin - head, origin, out)
        _fill(t, origin + TAIL - int(case["load"] * t.num_slots), origin + TAIL - head, out)
        t.close()                           # gives its scratch back; the group keeps what it needs
    # the popular quarter of a feature's ids stays, the long tail behind it moves on from step to step
    s.ring = []
    for k in range(2):
        sizes = wl.rng_for(5, 1000 + k)
        counts = [int(sizes.integers(0, 2 * p + 1, size=spec.samples).sum()) for p in spec.pooling]
        ranks = [_zipf(gen, c, 1.05, 2 * t.num_slots) for c, t in zip(counts, spec.tables)]
        tail = torch.cat([r > _head(t) for r, t in zip(ranks, spec.tables)])
        values = torch.cat([origin - r for r in ranks]) + tail * (TAIL + k)
        offsets = torch.tensor([sum(counts[:f]) for f in range(len(counts) + 1)], dtype=torch.int64, device=DEVICE)
        s.ring.append((values, offsets, torch.empty_like(values), tail.to(torch.int8) * 2))
    total = max(r[0].numel() for r in s.ring)
    s.step = 20
    if case["train"]:
        mp.mpzch_group_reserve(s.group, total)
        cap = [max(1, int(spec.samples * p * 1.5)) for p in spec.pooling]
        s.evicted_offsets = [sum(cap[:f]) for f in range(len(cap) + 1)]
        s.evicted = torch.empty(s.evicted_offsets[-1], dtype=torch.int64, device=DEVICE)
        s.num_evicted = torch.zeros(len(cap), dtype=torch.int64, device=DEVICE)
        s.stats = torch.zeros((len(cap), mp.STAT_COUNT), dtype=torch.int64, device=DEVICE)
        s.rows = [torch.ones((t.num_slots, case["dim"]), dtype=DTYPES[case["dtype"]], device=DEVICE) for t in spec.tables]
        for _ in range(4):
            _run_jagged_train(s)
    else:
        s.found = torch.empty(total, dtype=torch.uint8, device=DEVICE)
    return s


def _run_jagged_train(s):
    values, offsets, out, move = s.ring[s.step % 2]
    mp.mpzch_remap_jagged(s.group, s.identities, s.metadata, values, offsets, s.step, out, s.evicted, s.evicted_offsets,
                          s.num_evicted, s.stats)
    mp.mpzch_reset_rows_jagged(s.group, s.evicted, s.evicted_offsets, s.num_evicted, s.rows)
    values.add_(move)               # the next batch of this buffer
    s.step += 1
    return [out, s.num_evicted, s.stats, s.rows, [t.records for t in s.tables]]


def _run_jagged_lookup(s):
    values, offsets, out, _ = s.ring[s.step % 2]
    found = s.found[: values.numel()]
    s.step += 1
    mp.mpzch_lookup_jagged(s.group, s.identities, values, offsets, out, found)
    return [out, found]


def _prepare_publish(case, gen, origin):
    s = SimpleNamespace(case=case, run=_run_publish)
    n, m = case["batch"], max(1, int(case["new"] * case["batch"]))
    s.table = t = _table(case, "ttl", 20, 0)
    out = torch.empty(CHUNK, dtype=torch.int64, device=DEVICE)
    _fill(t, origin - int(case["load"] * case["slots"]), origin, out)
    s.copy_identities = t.identities.clone().contiguous()       # the inference side as it was last published
    s.since = 100
    for k in range(3):
        t.remap(_stream_batch(gen, n, m, origin, k), s.since + k, out[:n])
    s.rows = _rows(case, gen)[0]
    s.copy_rows = torch.zeros_like(s.rows)
    cap = 3 * n
    s.slots = torch.empty(cap, dtype=torch.int64, device=DEVICE)
    s.ids = torch.empty(cap, dtype=torch.int64, device=DEVICE)
    s.count = torch.zeros(1, dtype=torch.int64, device=DEVICE)
    s.payload = torch.empty((cap, case["dim"]), dtype=s.rows.dtype, device=DEVICE)
    return s


def _run_publish(s):
    t = s.table
    mp.mpzch_collect_delta(t.handle, t.identities, t.metadata, s.since, s.slots, s.ids, s.count)
    mp.mpzch_gather_rows(s.slots, s.count, s.rows, s.payload)
    mp.mpzch_apply_delta(s.copy_identities, s.slots, s.ids, s.count, s.copy_rows, s.payload)
    return [s.count, s.copy_identities, s.copy_rows]            # (the order of the delta's entries is free)


_PREPARE = {"session": _prepare_session, "load": _prepare_load, "stream": _prepare_stream, "lookup": _prepare_lookup,
            "jagged": _prepare_jagged, "publish": _prepare_publish}


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _zipf_distinct(n, alpha, universe, first=1):
    """Expected number of distinct ranks >= first among n draws (sum of 1 - exp(-n p_k), in bins of the logarithm)."""
    total, lo = 0.0, float(first)
    top = (universe + 1.0) ** (1.0 - alpha) - 1.0
    while lo <= universe:
        hi = min(universe + 1.0, max(lo + 1.0, lo * 1.1))
        share = (hi ** (1.0 - alpha) - lo ** (1.0 - alpha)) / top
        total += (hi - lo) * -math.expm1(-n * share / (hi - lo))
        lo = hi
    return total


def _stream_distinct(n, m):
    """(distinct recurring ids, new ids) of a stream batch: the draws of one age spread over the m ids of that age."""
    p = 1.0 / MEAN_AGE
    return sum(m * -math.expm1(-(n - m) / m * p * (1.0 - p) ** (a - 1)) for a in range(1, 101)), m


def _row_bytes(case):
    return case["dim"] * (4 if case["dtype"] == "float32" else 2)


def _train_bytes(n, known, new, evictions, row_bytes):
    """ids in, slots out; an identity read and a metadata word written per distinct id; what is placed is written; the
    evicted rows are written."""
    return 16.0 * n + 12.0 * (known + new) + 8.0 * new + evictions * row_bytes


def work(case):
    return {"bytes": _BYTES[case["family"]](case), "flops": 0.0}


def _bytes_session(case):
    n, slots = case["batch"], case["slots"]
    prefill, fresh = int(case["load"] * slots), int(case["fresh"] * n)
    per = _zipf_distinct(n - fresh, case["alpha"], case["universe"])
    ever = _zipf_distinct((n - fresh) * case["steps"], case["alpha"], case["universe"]) + fresh * case["steps"]
    evictions = min(max(0.0, prefill + ever - slots), ever)
    tensors = 2 if case["reset"] == "multi" else 1
    total = (16.0 if case["layout"] == "records" else 12.0) * slots + _train_bytes(prefill, 0, prefill, 0, 0)
    known = case["steps"] * (per + fresh) - ever
    return total + _train_bytes(n * case["steps"], max(0.0, known), ever, evictions, tensors * _row_bytes(case))


def _bytes_load(case):
    return (16.0 if case["layout"] == "records" else 12.0) * case["slots"] + _train_bytes(case["ids"], 0, case["ids"], 0, 0)


def _bytes_stream(case):
    n = case["batch"]
    m = max(1, int(case["new"] * n))
    known, new = _stream_distinct(n, m)
    tensors = 2 if case["reset"] == "multi" else 1
    return _train_bytes(n, known, new, new * case["load"], tensors * _row_bytes(case))


def _bytes_lookup(case):
    n = case["batch"]
    unknown = int(case["unknown"] * n)
    distinct = _zipf_distinct(n - unknown, case["alpha"], int(case["load"] * case["slots"])) + unknown
    total = 17.0 * n + 8.0 * distinct
    if case["rows"]:
        total += (n + distinct) * _row_bytes(case)
    return total


def _bytes_jagged(case):
    spec, total = _collection(case), 0.0
    for t, pooling in zip(spec.tables, spec.pooling):
        n = spec.samples * pooling
        distinct = _zipf_distinct(n, 1.05, 2 * t.num_slots)
        if case["train"]:
            new = _zipf_distinct(n, 1.05, 2 * t.num_slots, 1 + int(case["load"] * t.num_slots))
            total += _train_bytes(n, distinct - new, new, new * case["load"], _row_bytes(case))
        else:
            total += 17.0 * n + 8.0 * distinct
    return total


def _bytes_publish(case):
    n, m = case["batch"], max(1, int(case["new"] * case["batch"]))
    known, new = _stream_distinct(n, m)
    changed = known + 3 * new
    scan = (16.0 if case["layout"] == "records" else 12.0) * case["slots"]
    # the scan; slot and id of an entry out; its row read, and written on the other side with its identity
    return scan + changed * (16.0 + 2.0 * _row_bytes(case) + 8.0)


_BYTES = {"session": _bytes_session, "load": _bytes_load, "stream": _bytes_stream, "lookup": _bytes_lookup,
          "jagged": _bytes_jagged, "publish": _bytes_publish}


def tolerance(case):
    return "exact"             # whole numbers and bytes throughout

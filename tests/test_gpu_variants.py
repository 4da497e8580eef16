"""Variants of the kernels that a dispatch rule chooses by size, layout or policy, at the sizes where they can go
wrong, against the oracle."""
import numpy as np
import pytest
import torch

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

"""The binned record against the direct record (the whole table: keys and edge
bits; the junctions) where its bins change shape: a block to a bucket, buckets
split by block, the last bucket partly filled, several passes; k-mers of many
copies, whose items find no room and spill, and more of them than the spill
holds (the record then runs directly)."""
import numpy as np
import pytest

import synth
from helpers import to_genomes

pytestmark = pytest.mark.gpu

SINGLE, BLOCKED = 1, 4


def genomes(k, units):
    r = synth.rng(97, k, units)
    base = synth.random_bases(r, 300_000)
    out = [base]
    for _ in range(2):
        x = base.copy()
        x[r.integers(0, x.size, 9000)] = r.integers(0, 5, 9000)  # 4: cut in strings
        out.append(x)
    # one k-mer after another base every time, `units` times
    motif = synth.random_bases(r, k + 3)
    out.append(np.concatenate([np.concatenate([motif, synth.random_bases(r, 1)])
                               for _ in range(units)] + [base[:k]]))
    return out


# table_load sets the table's size: 0.9 some 60 to 120 blocks, 0.05 more than 512
@pytest.mark.parametrize("k, load, passes, units, flags", [
    (25, 0.9, 0, 10, BLOCKED), (25, 0.05, 0, 10, BLOCKED), (25, 0.05, 3, 10, BLOCKED | SINGLE),
    (27, 0.05, 0, 10, 0), (15, 0.9, 2, 10, BLOCKED), (25, 0.05, 0, 3_000, BLOCKED),
    (25, 0.05, 0, 20_000, BLOCKED)])
def test_binned_record_equals_direct(k, load, passes, units, flags):
    import paper_1602_05856_amd as tp
    plan = tp.Plan(to_genomes(genomes(k, units)), k, 2**18, 3, flags)
    d_in = plan.upload()
    got = []
    for mode in (1, 2):
        plan.config = {"record_binned": mode, "table_shape": 2, "table_load": load,
                       "record_passes": passes}
        for _ in range(2):  # the second run's scratch holds the first one's items
            plan.run(d_in)
            st = plan.stats()
        if mode == 1:
            assert st["record_passes"] == 0
        elif units < 20_000:
            assert st["record_passes"] >= max(1, passes)
        keys, masks = plan.debug_table()
        o = np.argsort(keys[:, 0])
        assert len(o) == st["table_keys"]
        got.append((keys[o, 0], masks[o], st["junctions"], st["table_capacity"]))
    blocks = (got[0][3] - 4096) // 8192
    assert blocks > 512 if load < 0.1 else 1 < blocks <= 512
    assert got[0][2:] == got[1][2:]
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    plan.close()

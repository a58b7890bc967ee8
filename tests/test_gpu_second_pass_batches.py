"""The second pass over batches of tiles: thousands of one-tile genomes in sets
of one to thousands, so that batches of four tiles, batches cut by a set's end
and walks that end inside a batch all occur, against the oracle and against a
grid wide enough that every batch is one tile."""
import numpy as np
import pytest

import synth
from helpers import oracle_run, to_genomes

pytestmark = pytest.mark.gpu

BLOCKED = 4


def related(r, n, size):
    base = synth.random_bases(r, size)
    out = []
    for i in range(n):
        g = synth.substitute(r, base[: size - int(r.integers(0, size // 2))], 0.02)
        if i % 7 == 3:
            g[g.size // 3:g.size // 3 + 2] = 4  # two strings
        out.append(g)
    return out


@pytest.mark.parametrize("k", [15, 31, 40, 70])
def test_batches_of_tiles(k):
    import paper_1602_05856_amd as tp
    r = synth.rng(97, k)
    sets = [related(r, n, s) for n, s in ((1, 300), (3, 2500), (700, 160), (2, 200), (3100, 220),
                                          (1, 90), (1300, 300))]
    b = 1 << 14
    want = None
    for wg, queue in ((0, 1), (1, 1), (1, 0)):
        for slabs in (0, 2, 3, 4, 7):
            plan = tp.Plan.batch([(to_genomes(gs), b) for gs in sets], k, 3, BLOCKED)
            plan.config = {"wg_per_cu": [wg] * 4, "tile_queue": queue, "pass2_slabs": slabs}
            d_in = plan.upload()
            plan.run(d_in)
            res = plan.download()
            got = (res.junction_offset, res.junction_pos, res.vertex, res.strand, res.edges)
            if want is None:
                want = [np.copy(x) for x in got]
                first = 0
                for gs in sets:
                    o, junctions, _, _ = oracle_run(gs, k, b, 3, BLOCKED)
                    for g in range(len(gs)):
                        assert np.array_equal(res.junctions(first + g), junctions[g])
                    first += len(gs)
            assert all(np.array_equal(x, y) for x, y in zip(got, want)), (wg, queue, slabs)
            plan.close()

"""The standard query's table of decided windows: thousands of one-tile related
genomes in a few sets (batches of up to 8 tiles, cut where a set ends), against
the oracle and against a grid so wide that every tile is decided by itself."""
import numpy as np
import pytest

import synth
from helpers import oracle_run, to_genomes

pytestmark = pytest.mark.gpu

SINGLE = 1


def related(r, n, size):
    base = synth.random_bases(r, size)
    out = []
    for i in range(n):
        g = synth.substitute(r, base[: size - int(r.integers(0, size // 3))], 0.02)
        if i % 5 == 2:
            g[g.size // 2] = 4
        if i % 7 == 3:
            g = synth.reverse_complement(g)
        out.append(g)
    return out


@pytest.mark.parametrize("k", [11, 31, 63, 64, 127])
def test_windows_decided_once(k):
    import paper_1602_05856_amd as tp
    r = synth.rng(99, k)
    sets = [related(r, n, s) for n, s in ((1, 400), (2300, 350), (3, 2100), (1900, 280),
                                          (1500, 300))]
    b, h, flags = 1 << 13, 3, SINGLE if k == 11 else 0
    want = None
    for wg, queue, rounds in ((0, 1, 1), (1, 1, 1), (1, 0, 1), (0, 1, 2), (1, 1, 2)):
        plan = tp.Plan.batch([(to_genomes(gs), b) for gs in sets], k, h, flags)
        plan.rounds = rounds
        plan.config = {"wg_per_cu": [wg] * 4, "tile_queue": queue}
        d_in = plan.upload()
        plan.run(d_in)
        c1 = plan.debug_candidates()
        if want is None:
            first, per_genome = 0, plan.bitmap_positions(c1)
            for gs in sets:
                o, _, _, _ = oracle_run(gs, k, b, h, flags)
                for g in range(len(gs)):
                    assert np.array_equal(per_genome[first + g], o.c1[g])
                first += len(gs)
        if want is None or (rounds == 2 and wg == 0):
            want = c1
        assert np.array_equal(c1, want), (wg, queue, rounds)
        plan.close()

"""The binned fill against the atomic fill (filter words, popcount, C1) where
its bins change shape: one region, 1024 regions, the larger regions of a
2^30-bit pool, buckets split by region; items without room (a homopolymer
fills one bucket); tiles of many strings; pools of several filters; rounds."""
import numpy as np
import pytest

import synth
from helpers import to_genomes

pytestmark = pytest.mark.gpu

SINGLE, BLOCKED = 1, 4


def genomes(k):
    r = synth.rng(93, k)
    base = synth.random_bases(r, 50_000)
    cut = base.copy()
    cut[r.integers(0, cut.size, 900)] = 4  # many strings to a tile, some shorter than k
    return [base, cut, np.zeros(300_000, np.uint8),  # every edge the same: no room for most
            np.tile(synth.random_bases(r, 3), 9000), synth.random_bases(r, 2048 * 3 + 1)]


def fills(make, rounds=1):
    import paper_1602_05856_amd as tp
    got = []
    for mode in (1, 2):
        plan = make(tp)
        plan.rounds = rounds
        plan.config = {"fill_binned": mode}
        d_in = plan.upload()
        plan.run(d_in)
        plan.run(d_in)  # the second run fills the same pool again
        st = plan.stats()
        assert (st["fill_chunks"] > 0) == (mode == 2)
        got.append(([plan.debug_bloom(s) for s in range(plan.n_sets)], plan.debug_candidates(),
                    [plan.stats(s)["bloom_popcount"] for s in range(plan.n_sets)],
                    st["junctions"]))
        plan.close()
    a, b = got
    assert all(np.array_equal(x, y) for x, y in zip(a[0], b[0]))
    assert np.array_equal(a[1], b[1])
    assert a[2:] == b[2:]


@pytest.mark.parametrize("k", [25, 40, 100])
@pytest.mark.parametrize("log2b", [6, 19, 26, 29, 30, 31])
def test_bins_of_one_filter(k, log2b):
    flags = BLOCKED | (SINGLE if log2b == 26 else 0)
    gs = to_genomes(genomes(k))
    fills(lambda tp: tp.Plan(gs, k, 1 << log2b, 3, flags))


def test_bins_over_several_filters():
    # filter starts inside regions, one filter over many regions, rounds
    sets = [(to_genomes([g]), 1 << b) for g, b in zip(genomes(31), (10, 22, 25, 16, 30))]
    for rounds in (1, 3):
        fills(lambda tp: tp.Plan.batch(sets, 31, 4, BLOCKED), rounds)


@pytest.mark.parametrize("k", [25, 40, 100])
@pytest.mark.parametrize("log2b, h", [(5, 3), (19, 1), (26, 16), (28, 5), (30, 4)])
def test_bins_of_a_standard_filter(k, log2b, h):
    gs = to_genomes(genomes(k))
    fills(lambda tp: tp.Plan(gs, k, 1 << log2b, h, SINGLE if log2b == 26 else 0))


def test_bins_over_several_standard_filters():
    sets = [(to_genomes([g]), 1 << b) for g, b in zip(genomes(31), (5, 22, 25, 16, 30))]
    for rounds in (1, 3):
        fills(lambda tp: tp.Plan.batch(sets, 31, 4, 0), rounds)

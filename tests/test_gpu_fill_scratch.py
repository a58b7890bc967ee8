"""The binned fill's scratch is optional: where it is refused, moved or cut the
results are those of the atomic fill."""
import numpy as np
import pytest

import synth
from helpers import to_genomes

pytestmark = pytest.mark.gpu

BLOCKED = 4


def related(seed, n, genomes):
    return to_genomes(synth.genome_set(synth.rng(seed, n), n, genomes))


def run_plan(gs, k, b, h, flags, rounds=1, **cfg):
    import paper_1602_05856_amd as tp
    plan = tp.Plan(gs, k, b, h, flags)
    plan.rounds = rounds
    plan.config = cfg
    d_in = plan.upload()
    plan.run(d_in)
    got = plan.stats(), plan.debug_bloom(), plan.debug_candidates(), plan.download()
    plan.close()
    return got


def test_refused_scratch_counts_the_filter_bits():
    """A server's budget admits the job but not 16 items of 4 bytes a position:
    the fill runs with atomics, and the job's filter popcount is the filter's."""
    import paper_1602_05856_amd as tp
    gs, b, h = related(31, 1_000_000, 4), 1 << 26, 16
    st, bloom, _, want = run_plan(gs, 25, b, h, 0, fill_binned=1)
    bits = int(np.unpackbits(bloom.view(np.uint8)).sum())
    assert st["bloom_popcount"] == bits > 0
    srv = tp.Server(hbm_budget=200 << 20, workers=1, max_batch=1)
    res, _ = srv.wait(srv.submit(gs, 25, b, h, 0))
    srv.close()
    assert res.stats["fill_chunks"] == 0, "the scratch was not refused"
    assert res.stats["bloom_popcount"] == bits
    assert res.stats["candidates"] == want.stats["candidates"]
    assert np.array_equal(res.junction_pos, want.junction_pos)

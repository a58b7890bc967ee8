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


@pytest.mark.parametrize("h, flags", [(4, BLOCKED), (1, 0)])
def test_scratch_moved_by_a_rounds_table(h, flags):
    """The items lie in the exact table's buffer.  Where every position is a
    candidate a round's table outgrows them and moves the buffer, and the next
    round's fill has to follow."""
    r = synth.rng(32, h)
    gs = to_genomes([synth.random_bases(r, 1_000_003) for _ in range(3)])
    a = run_plan(gs, 25, 1 << 22, h, flags, rounds=3, fill_binned=1)
    b = run_plan(gs, 25, 1 << 22, h, flags, rounds=3, fill_binned=2)
    st = b[0]
    assert st["fill_chunks"] == 1 and a[0]["fill_chunks"] == 0
    items = 4 * (1 if flags else h) * 2.5 / 3 * 1.1 * st["positions"]
    assert 8 * st["table_capacity"] > items, "the table did not outgrow the items"
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
    assert st["bloom_popcount"] == a[0]["bloom_popcount"]
    for f in ("junction_pos", "vertex", "strand", "edges"):
        assert np.array_equal(getattr(a[3], f), getattr(b[3], f)), f


def random_set(seed, n, genomes):
    """`genomes` copies of one random genome (few candidates), without N."""
    import paper_1602_05856_amd as tp
    pk = np.random.default_rng(seed).integers(0, 256, (n + 3) // 4, dtype=np.uint8)
    return [tp.Genome(packed=pk, n_bases=n, n_runs=np.zeros((0, 2), np.uint64))] * genomes


def test_admission_asks_for_what_the_atomic_fill_needs():
    """100 Mbp with a 128 MiB filter in a budget of 512 MiB."""
    import paper_1602_05856_amd as tp
    gs = random_set(33, 50_000_000, 2)
    st, _, _, want = run_plan(gs, 25, 1 << 30, 4, BLOCKED, fill_binned=1)
    srv = tp.Server(hbm_budget=512 << 20, workers=1, max_batch=1)
    res, _ = srv.wait(srv.submit(gs, 25, 1 << 30, 4, BLOCKED))
    peak = srv.stats()["peak_held_bytes"]
    srv.close()
    assert peak <= 512 << 20
    assert res.stats["candidates"] == st["candidates"]
    assert np.array_equal(res.junction_pos, want.junction_pos)


def test_scratch_is_not_waited_for():
    """A small job whose scratch does not fit beside a running large one fills
    with atomics and ends first."""
    import time
    import paper_1602_05856_amd as tp
    n, b = 800_000_000, 1 << 34
    large, small = random_set(34, n, 1), related(35, 1_000_000, 4)
    room = n // 4 + b // 8 + 3 * n // 8 + 20 * (n // 2048)
    srv = tp.Server(hbm_budget=room + (300 << 20), workers=2, max_batch=1, wg_per_cu=2)
    a = srv.submit(large, 25, b, 16, 0)
    while not srv.stats()["running"]:
        time.sleep(0.001)
    c = srv.submit(small, 25, 1 << 26, 16, 0)
    res, small_info = srv.wait(c)
    _, large_info = srv.wait(a)
    srv.close()
    assert res.stats["fill_chunks"] == 0
    assert large_info["start_s"] < small_info["start_s"]
    assert small_info["end_s"] < large_info["end_s"]


def test_scratch_takes_a_quarter_of_the_free_memory():
    """13 GB of items where 20 GiB are free: smaller chunks, the same filter."""
    import torch
    import paper_1602_05856_amd as tp
    gs, b, h = random_set(36, 50_000_000, 2), 1 << 31, 16
    _, bloom, c1, _ = run_plan(gs, 25, b, h, 0, fill_binned=1)
    plan = tp.Plan(gs, 25, b, h, 0)
    d_in = plan.upload()
    torch.cuda.empty_cache()
    rest = torch.empty(torch.cuda.mem_get_info()[0] - (20 << 30), dtype=torch.uint8, device="cuda")
    free = torch.cuda.mem_get_info()[0]
    plan.run(d_in)
    used = free - torch.cuda.mem_get_info()[0]
    plan.run(d_in)
    st = plan.stats()
    got = plan.debug_bloom(), plan.debug_candidates()
    plan.close()
    del rest
    torch.cuda.empty_cache()
    assert st["fill_chunks"] > 1
    assert used < free / 4 + (1 << 30)  # and the filter, the bitmaps, the outputs
    assert np.array_equal(got[0], bloom) and np.array_equal(got[1], c1)


@pytest.mark.parametrize("log2b, n, binned", [(12, 2_000_000, 0), (18, 6_000_000, 0),
                                              (18, 2_000_000, 1), (21, 40_000_000, 1),
                                              (14, 100_000, 0), (16, 100_000, 1)])
@pytest.mark.parametrize("flags", [BLOCKED, 0])
def test_filters_of_few_regions_are_filled_atomically(log2b, n, binned, flags):
    import paper_1602_05856_amd as tp
    gs = random_set(37, n, 1)
    for cfg in ({}, {"fill_binned": 2}):
        st, bloom, _, _ = run_plan(gs, 25, 1 << log2b, 4, flags | tp.TP_FLAG_PASS1_ONLY, **cfg)
        assert (st["fill_chunks"] > 0) == bool(binned or cfg)
        want = bloom if not cfg else want
        assert np.array_equal(bloom, want)

"""The binned record by default, and where it is given up."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

BLOCKED = 4


def genome(codes):
    import paper_1602_05856_amd as tp
    pk, runs = synth.pack(codes)
    return tp.Genome(packed=pk, n_bases=codes.size, n_runs=runs)


def motif_units(r, k, units):
    """`units` copies of one motif, a random base after each: some hundred
    k-mers make up all of it, each with several pairs of bases around it."""
    x = np.tile(np.append(synth.random_bases(r, k + 3), np.uint8(0)), units)
    x[k + 3::k + 4] = r.integers(0, 4, units)
    return x


def mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


@pytest.fixture(scope="module")
def repetitive():
    r = synth.rng(51)
    return [genome(synth.random_bases(r, 13_000_000)), genome(motif_units(r, 25, 400_000))]


def test_direct_record_keeps_the_power_of_two(repetitive):
    """More items than the scratch takes: the record runs directly, in the table
    a direct record takes (home slot: the hash's low bits)."""
    import paper_1602_05856_amd as tp
    plan = tp.Plan(repetitive, 25, 1 << 20, 4, BLOCKED)  # every position a candidate
    plan.run(plan.upload())
    st = plan.stats()
    keys, _ = plan.debug_table()
    plan.close()
    assert st["record_passes"] == 0 and st["table_keys"] == len(keys) > 12_000_000
    cap = st["table_capacity"] - 4096
    assert cap & (cap - 1) == 0 and cap * 8 >= 128 << 20
    home = mix64(keys[:, 0] ^ np.uint64(0x082EFA98EC4E6C89)) & np.uint64(cap - 1)
    # in slot order the home slots rise, but for a probe's length here and there
    # (and the last ones' wrap to the table's start)
    late = home[4096:].astype(np.int64) < np.maximum.accumulate(home[4096:].astype(np.int64)) - 4096
    assert late.sum() == 0


def test_a_record_given_up_is_not_tried_again(repetitive):
    import paper_1602_05856_amd as tp
    plan = tp.Plan(repetitive, 25, 1 << 20, 4, BLOCKED)
    d_in = plan.upload()
    got = []
    for attempts in (2, 1, 1):
        plan.run(d_in)
        st = plan.stats()
        assert (st["table_attempts"], st["record_passes"]) == (attempts, 0)
        got.append((st["table_keys"], plan.download().junction_pos))
    plan.config = {"record_binned": 1}
    plan.run(d_in)
    assert plan.stats()["table_attempts"] == 1
    want = plan.download().junction_pos
    for keys, pos in got:
        assert keys == plan.stats()["table_keys"] and np.array_equal(pos, want)
    plan.config = {"record_binned": 2, "table_shape": 2}  # as asked: tried every time
    for _ in range(2):
        plan.run(d_in)
        assert plan.stats()["table_attempts"] == 2
    plan.close()


@pytest.mark.parametrize("units, attempts", [(3_000, 1), (20_000, 2)])
def test_items_without_room_spill_or_give_up(units, attempts):
    """A motif's k-mers, `units` items each and one block's, against that block's
    room (its share of the candidates, six standard deviations and 64): some
    spill, and of the larger number more than the spill takes."""
    import paper_1602_05856_amd as tp
    from helpers import to_genomes
    from test_gpu_record_bins import genomes
    plan = tp.Plan(to_genomes(genomes(25, units)), 25, 2**18, 3, BLOCKED)
    plan.config = {"record_binned": 2, "table_shape": 2, "table_load": 0.05}
    plan.run(plan.upload())
    st = plan.stats()
    plan.close()
    blocks = (st["table_capacity"] - 4096) // 8192
    mean = st["candidates"] / blocks
    assert blocks > 512 and units > 1.02 * mean + 6 * (4 * mean) ** 0.5 + 80
    assert st["table_attempts"] == attempts and (st["record_passes"] > 0) == (attempts == 1)

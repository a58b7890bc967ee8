"""The exact table of reference words (k >= 28: a slot names the position
where the sequence reads its key) at the k where it starts and where the
value width changes, on inputs that make its compare decide: k-mers read on
both strands, even-k palindromes, keys in the last bases of the input."""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_parity, to_genomes

pytestmark = pytest.mark.gpu

SINGLE, BLOCKED = 1, 4


def genomes(k):
    base = synth.random_bases(synth.rng(91, k), 3000)
    other = base.copy()
    other[np.arange(40, 3000, 97)] = (other[np.arange(40, 3000, 97)] + 1) % 4
    half = synth.random_bases(synth.rng(91, k, 1), k // 2)
    pal = np.concatenate([half, synth.reverse_complement(half)])  # even k: its own complement
    ends = np.concatenate([pal, other[:700], pal])
    # the last genome ends on a tile boundary, on a k-mer shared with the others
    last = np.concatenate([synth.random_bases(synth.rng(91, k, 2), 2048 - 700), other[:700]])
    return [base, synth.reverse_complement(other), ends, last]


@pytest.mark.parametrize("k", [28, 31, 32, 63, 64, 127])
@pytest.mark.parametrize("shape", [1, 2])
def test_reference_words_match_the_oracle(k, shape):
    for load, flags in ((0.7, BLOCKED), (0.7, SINGLE), (8.0, BLOCKED)):
        # a small filter makes most positions candidates; load 8 regrows
        assert_parity(genomes(k), k, 2**13, 3, flags=flags, label="reference words",
                      config={"table_shape": shape, "table_load": load})


@pytest.mark.parametrize("k", [28, 63, 100])
def test_table_keys_outlive_the_input(k):
    """tp_debug_table reads the keys of the last run after the caller has
    overwritten its input buffer."""
    import paper_1602_05856_amd as tp
    gs = genomes(k)
    plan = tp.Plan(to_genomes(gs), k, 2**13, 3, BLOCKED)
    d_in = plan.upload()
    plan.run(d_in)
    d_in.zero_()
    keys, masks = plan.debug_table()
    got = {sum(int(x) << (64 * i) for i, x in enumerate(row)): int(m)
           for row, m in zip(keys, masks)}
    vals = sorted(got)
    inm, outm, _ = oracle.vertex_masks(gs, k, vals, single_strand=False)
    assert len(got) == plan.stats()["table_keys"]
    assert [got[v] for v in vals] == [int(i) | int(o) << 4 for i, o in zip(inm, outm)]
    plan.close()

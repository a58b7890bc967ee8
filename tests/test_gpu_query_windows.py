"""The standard query's table of decided windows at its full batch of 32 tiles,
and with rounds (a window's verdict is of the round's class): every candidate
position against the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from helpers import to_genomes

pytestmark = pytest.mark.gpu


def related(r, n, size, bases):
    """n genomes of up to `size` bases, a tile each, from a few base sequences."""
    base = [synth.random_bases(r, size) for _ in range(bases)]
    out = []
    for i in range(n):
        g = synth.substitute(r, base[i % bases][: size - i % 11], 0.004)
        if i % 5 == 2:
            g[g.size // 2] = 4
        out.append(synth.reverse_complement(g) if i % 7 == 3 else g)
    return out


# 33,000 tiles over 256 workgroups, 4 batches each and more: 32 tiles to a batch
@pytest.mark.parametrize("k, n, size, rounds", [(15, 33_000, 45, 1), (63, 33_000, 95, 1),
                                                (127, 33_000, 160, 1), (25, 33_000, 55, 2),
                                                (70, 4_500, 250, 3)])
def test_candidates_match_the_oracle(k, n, size, rounds):
    import paper_1602_05856_amd as tp
    gs = related(synth.rng(98, k), n, size, 9)
    b = 1 << 20
    if rounds == 1:
        want = oracle.twopass(gs, k, b, 3)
    else:
        want = oracle.rounds(gs, k, b, 3, rounds)
    plan = tp.Plan(to_genomes(gs), k, b, 3)
    plan.rounds = rounds
    plan.run(plan.upload())
    got = plan.bitmap_positions(plan.debug_candidates())
    st = plan.stats()
    plan.close()
    assert len(got) == n and all(np.array_equal(x, y) for x, y in zip(got, want.c1))
    marked = sum(x.size for x in want.c1)
    assert 0.02 * st["positions"] < marked < 0.98 * st["positions"]

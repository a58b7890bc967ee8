"""The blocked query's pair tests where a middle is its own reverse complement
(each of its edges then takes its own orientation), with every pair of bases
around it, and at the k whose windows fill their words."""
import numpy as np
import pytest

import synth
from helpers import assert_parity

pytestmark = pytest.mark.gpu

SINGLE, BLOCKED = 1, 4


@pytest.mark.parametrize("k", [1, 3, 5, 25, 31, 33, 63, 65, 127])
def test_palindromic_middles(k):
    r = synth.rng(95, k)
    half = synth.random_bases(r, (k - 1) // 2)
    pal = np.concatenate([half, synth.reverse_complement(half)])  # k - 1 bases
    parts = []
    for x in range(4):
        for y in range(4):
            parts += [synth.random_bases(r, 140 + k), np.array([x], np.uint8), pal,
                      np.array([y], np.uint8)]
    g = np.concatenate(parts + [synth.random_bases(r, 200)])
    for b, flags in ((2**12, BLOCKED), (2**20, BLOCKED), (2**12, BLOCKED | SINGLE)):
        assert_parity([g, synth.reverse_complement(g), g[: g.size // 2]], k, b, 3, flags=flags,
                      label="palindromes")

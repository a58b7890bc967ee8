"""The distinct-count sketch against its definition: of every candidate
position's 64-bit hash (blocked filter: the sum of the G values of the k-mer's
two middles; standard: its table hash) the top 12 bits choose a register, the
leading zeros of the other 52 give the rank.  The estimate has to be equal."""
import math

import numpy as np
import pytest

import synth
from helpers import to_genomes

pytestmark = pytest.mark.gpu

BLOCKED = 4
S0, S2, S3 = (np.uint64(x) for x in (0x243F6A8885A308D3, 0xA4093822299F31D0, 0x082EFA98EC4E6C89))


def mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def normalised(codes, at, n, words):
    """The normalised n-mers at positions `at`, most significant word first."""
    def value(digit):
        w = [np.zeros(at.size, np.uint64) for _ in range(words)]
        for t in range(n):
            place = n - 1 - t
            w[words - 1 - place // 32] |= digit(t).astype(np.uint64) << np.uint64(2 * (place % 32))
        return w
    f = value(lambda t: codes[at + t])
    r = value(lambda t: 3 - codes[at + n - 1 - t])
    less, same = np.zeros(at.size, bool), np.ones(at.size, bool)
    for a, b in zip(r, f):
        less |= same & (a < b)
        same &= a == b
    return [np.where(less, a, b) for a, b in zip(r, f)]


def fold(words):
    x = words[0]
    for w in words[1:]:
        x = mix64(x ^ S0) ^ w
    return x


def estimate(hashes):
    reg = (hashes >> np.uint64(52)).astype(np.int64)
    rest = hashes & np.uint64((1 << 52) - 1)
    # leading zeros of the 52 bits (exact in a double), plus one
    rank = np.where(rest == 0, 53, 53 - np.frexp(rest.astype(np.float64))[1])
    hll = np.zeros(4096, np.int64)
    np.maximum.at(hll, reg, rank)
    z, zeros, m = float(np.sum(0.5 ** hll)), int((hll == 0).sum()), 4096.0
    e = 0.7213 / (1 + 1.079 / m) * m * m / z
    return m * math.log(m / zeros) if e <= 2.5 * m and zeros else e


@pytest.mark.parametrize("k, n, log2b, flags", [
    (25, 12_000_003, 22, BLOCKED),  # ranks that need more than 32 of the hash's bits
    (31, 60_000, 16, BLOCKED), (40, 60_000, 16, BLOCKED), (100, 60_000, 16, BLOCKED),
    (25, 4_000_003, 20, 0), (100, 60_000, 16, 0)])
def test_estimate_is_the_sketch_of_64_bit_hashes(k, n, log2b, flags):
    import paper_1602_05856_amd as tp
    codes = synth.random_bases(synth.rng(41, k, n), n)
    plan = tp.Plan(to_genomes([codes]), k, 1 << log2b, 4, flags)
    plan.run(plan.upload())
    at = np.asarray(plan.bitmap_positions(plan.debug_candidates())[0], np.int64)
    got = plan.stats()["distinct_estimate"]
    plan.close()
    assert at.size > n // 2
    words = 1 if k <= 31 else 2 if k <= 63 else 4
    hashes = np.zeros(at.size, np.uint64)
    for a in range(0, at.size, 1 << 20):
        p = at[a:a + (1 << 20)]
        if flags & BLOCKED:
            h = sum(mix64(fold(normalised(codes, p + o, k - 1, words)) ^ S2) for o in (0, 1))
        else:
            h = mix64(fold(normalised(codes, p, k, words)) ^ S3)
        hashes[a:a + p.size] = h
    assert got == int(estimate(hashes))

"""Coefficients whose row norms leave the double range (from 2^1023 on): the prime
count still covers the result, which equals the oracle's from host and device
memory."""

import random

import pytest

import paper_1201_1548_amd as br
from oracle.resultant import bi_transpose, discriminant_y, resultant_y

CASES = {
    "one": ([[1 << 1100], [3, 1]], [[5, 2], [1, 7]]),
    "negative": ([[-(1 << 1100), 5], [3, 1], [1 << 1050]], [[5, 2], [1, 7], [4]]),
    "sum": ([[1 << 1023] * 9, [3, -1]], [[5, 2], [1, 7]]),
    "edge": ([[(1 << 1024) - 1, 1 - (1 << 1024)], [3, -1]], [[5, -(1 << 1023)], [1, 7]]),
    "both": ([[1 << 2000, 3], [-(1 << 1500), 7]], [[5, 1 << 1999], [1, 7 << 1700], [9]]),
}


def wide(seed, m, n, bits):
    rng = random.Random(seed)
    draw = lambda: rng.getrandbits(rng.choice([3, 40, bits])) * rng.choice([1, -1])  # noqa: E731
    return [[draw() for _ in range(4)] for _ in range(m + 1)], [[draw() for _ in range(3)] for _ in range(n + 1)]


@pytest.mark.parametrize("name", CASES)
def test_the_prime_count_covers_the_result(name):
    F, G = CASES[name]
    D, P, log2_bound = br.plan(F, G)
    R = resultant_y(F, G)
    assert len(R) <= D
    top = max(abs(c).bit_length() for c in R)
    assert log2_bound >= top - 1 and P * 31 > top


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_results(name):
    F, G = CASES[name]
    assert br.resultant(F, G) == resultant_y(F, G)
    b = br.DeviceBatch([("res", F, G, "y"), ("res", bi_transpose(F), bi_transpose(G), "x")])
    for _ in range(3):
        b.run()
        assert b.results() == [resultant_y(F, G)] * 2


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [1000, 1030, 1400])
def test_random_sizes(bits):
    jobs, want = [], []
    for i in range(6):
        F, G = wide(100 * bits + i, 1 + i % 4, 2 + i % 3, bits)
        F[-1][0] = F[-1][0] or 1
        G[-1][0] = G[-1][0] or 1
        jobs.append(("res", F, G, "y"))
        want.append(resultant_y(F, G))
        if len(F) > 2:
            jobs.append(("disc", F, None, "y"))
            want.append(discriminant_y(F))
    got, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs) and got == want
    b = br.DeviceBatch(jobs)
    b.run()
    assert b.results() == want

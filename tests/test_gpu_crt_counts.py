"""The explicit CRT over the range of prime counts: every class edge, the counts
around 128 and those whose operands no longer fit (Garner's digits), on
results whose limbs make carries run through whole segments.  The pairs are
f = y + f_0 (f_0 constant) and g = q f + t, so R = g(x, -f_0) = t(x) coefficient
by coefficient, while the size of f_0 and the degree of q set the prime count."""

import random

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth
from tests.test_gpu_interp_nodes import det2

pytestmark = pytest.mark.gpu


EDGE = [0, 1, -1, 2, -(1 << 31), 1 << 32, -(1 << 32), (1 << 32) - 1, -(1 << 64), 1 << 128, -(1 << 128),
        (1 << 128) - 1, 1 - (1 << 128), -(1 << 256), (1 << 256) - 1, 1 << 96, -(1 << 96) - 1]


def planted(P, n):
    """A pair needing P primes and the n coefficients of its resultant t(x)."""
    rng = random.Random(P)
    ny = 1 + 30 * P // 400
    c0 = int(30.415 * P / (ny + 1))
    for c in range(max(1, c0 - 34), c0 + 10):
        f0 = rng.getrandbits(c) | 1 << (c - 1)
        t = [EDGE[i] if i < len(EDGE) and abs(EDGE[i]) < 1 << c else rng.getrandbits(rng.randint(1, c)) *
             rng.choice([1, -1]) for i in range(n)]
        t[-1] = t[-1] or 1
        q = [[rng.getrandbits(4) - 8 for _ in range(n)] for _ in range(ny)]
        for e in range(0, 61, 5):
            q[-1] = [1 << e] * n
            G = [[(f0 * q[j][i] if j < ny else 0) + (q[j - 1][i] if j else 0) + (t[i] if j == 0 else 0)
                  for i in range(n)] for j in range(ny + 1)]
            if br.plan([[f0], [1]], G)[1] == P:
                return [[f0], [1]], G, t
    raise AssertionError("no pair with %d primes" % P)


@pytest.mark.parametrize("P", [1, 2, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 127, 128, 129, 135, 136, 137, 200, 256,
                               301, 500])
@pytest.mark.parametrize("n", [31, 33, 70])
def test_prime_counts_and_carries(P, n):
    F, G, t = planted(P, n)
    assert br.resultant(F, G) == t


@pytest.mark.parametrize("P", [640, 700, 760, 1025])
def test_counts_around_the_operand_limit(P):
    F, G, t = planted(P, 40)
    assert br.resultant(F, G) == t


def test_mixed_counts_in_one_batch():
    jobs, want = [], []
    for i, P in enumerate([3, 20, 40, 60, 90, 120, 128, 129, 180, 260, 400, 800, 10, 50]):
        F, G, t = planted(P, 20 + 5 * i)
        jobs.append(("res", F, G, "y"))
        want.append(t)
    res, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    assert res == want
    b = br.DeviceBatch(jobs)
    b.run()
    assert b.results() == want


def test_mixed_classes_beyond_one_round():
    # more blocks than run at once: one launch per class
    jobs, want = [], []
    for i in range(40):
        bits = 30 + 37 * (i % 13)
        F, G = synth.random_rect(4000 + i, 1, 900, 1, 900 + i, bits)
        jobs.append(("res", F, G, "y"))
        want.append(det2(F, G))
    res, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    assert res == want

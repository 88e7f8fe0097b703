"""The block gcd over F_p at the edges of its rounds (63, 64 and 31-step
multiples), with degree gaps, sparse remainder sequences and planted common
factors: bit-exact against the oracle or, at sizes it is too slow for, against
the planted factor (the cofactors are coprime modulo a 61-bit prime)."""

import random

import pytest

import paper_1201_1548_amd as br
from oracle import zx
from oracle.gcd import gcd_mod_p, gcd_zx

pytestmark = pytest.mark.gpu
Q61 = (1 << 61) - 1


def rpoly(rng, d, bits):
    a = [rng.randint(-(1 << bits), 1 << bits) for _ in range(d + 1)]
    a[-1] = a[-1] or 1
    return a


def primitive(a):
    from math import gcd
    g = 0
    for c in a:
        g = gcd(g, c)
    g = -g if a[-1] < 0 else g
    return [c // g for c in a]


@pytest.mark.parametrize("da,db,dc", [(62, 61, 0), (63, 62, 1), (64, 63, 0), (65, 64, 2), (95, 94, 3), (96, 95, 0),
                                      (126, 125, 40), (127, 126, 0), (160, 159, 64), (64, 64, 0), (130, 40, 20),
                                      (200, 5, 1), (33, 1, 30), (500, 499, 100), (300, 260, 150),
                                      (200, 199, 560)])
def test_degrees_at_round_edges(da, db, dc):
    rng = random.Random(1000 * da + db)
    A, B = rpoly(rng, da, 12), rpoly(rng, db, 12)
    C = primitive(rpoly(rng, dc, 12)) if dc else [1]
    # with gcd(A, B) = 1 modulo a prime that does not divide the leading coefficients, gcd(A C, B C) = C
    assert A[-1] % Q61 and B[-1] % Q61 and gcd_mod_p(A, B, Q61) == [1]
    a, b = zx.mul(primitive(A), C), zx.mul(primitive(B), C)
    assert br.gcd(a, b) == C
    assert br.gcd(b, a) == C


@pytest.mark.parametrize("n,k", [(96, 1), (100, 36), (130, 65), (128, 96)])
def test_sparse_sequences_with_gaps(n, k):
    # x^n - 1 and x^k - 1 (remainders with long runs of zeros), times planted
    # factors: the gcd is x^gcd(n, k) - 1
    from math import gcd
    x = lambda m: [-1] + [0] * (m - 1) + [1]  # noqa: E731
    assert br.gcd(x(n), x(k)) == x(gcd(n, k))
    rng = random.Random(n)
    A, B = rpoly(rng, 70, 10), rpoly(rng, 70, 10)
    a, b = zx.mul(x(n), A), zx.mul(x(k), B)
    assert br.gcd(a, b) == gcd_zx(a, b)


def test_degree_gap_after_several_normal_steps():
    # built backwards: a remainder sequence whose degrees drop by one except
    # for one gap of five in the middle (not at a multiple of the rounds)
    rng = random.Random(3)
    lo, hi = [1], [rng.randint(1, 3), 1]
    for i in range(120):
        quo = [rng.randint(-2, 2) for _ in range(6 if i == 47 else 1)] + [1]
        lo, hi = hi, zx.add(zx.mul(quo, hi), lo)
    assert br.gcd(hi, lo) == [1]
    C = primitive(rpoly(rng, 9, 20))
    assert br.gcd(zx.mul(hi, C), zx.mul(lo, C)) == C


def test_squarefree_with_long_factors():
    rng = random.Random(9)
    a1, a2 = primitive(rpoly(rng, 140, 20)), primitive(rpoly(rng, 70, 20))
    assert gcd_mod_p(a1, a2, Q61) == [1]
    u, f = br.squarefree(zx.scale(zx.mul(a1, zx.mul(a2, a2)), -6))
    assert u == -6 and f == [a1, a2]

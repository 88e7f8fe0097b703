"""Reduction of coefficients of several limbs modulo the primes: extreme values
of each length, at prime counts that leave remainders of the groups of 4 and 16
primes, for f, g and derivatives, in launches small and large enough for both
splits of the primes."""

import pytest

import paper_1201_1548_amd as br
from oracle import zx
from oracle.resultant import discriminant_y
from oracle.subresultants import polar_resultant_y

pytestmark = pytest.mark.gpu


def extremes(L, k):
    top = 1 << (32 * L - 1)
    v = [top - 1, -top, 1 - top, (top >> 1) + 0x80000000, -(1 << (32 * (L - 1))), (1 << (32 * (L - 1))) - 1, -1, 0]
    return v[k % 8:] + v[: k % 8]


@pytest.mark.parametrize("L", [2, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("copies", [1, 300])
def test_extreme_values_of_each_length(L, copies):
    F, G = [extremes(L, 0), extremes(L, 3)], [extremes(L, 5)[:3], extremes(L, 1)[:5]]
    res, status = br.resultant_batch([("res", F, G, "y")] * copies)
    assert status == [0] * copies
    want = zx.sub(zx.mul(F[1], G[0]), zx.mul(F[0], G[1]))
    assert all(r == want for r in res)
    H = [extremes(L, 2)[:4], extremes(L, 4)[:4], [3 - (1 << (32 * L - 1)), 1, 0, 0]]
    assert br.discriminant(H) == discriminant_y(H)
    assert br.polar_resultant(H) == polar_resultant_y(H)

"""Principal subresultant coefficients along the normal sequence in registers
(degrees that differ by at most one, below 68) at the edges of its tiles and
chains, sampled against the determinants over F_p, with points where the
sequence is not normal, and next to the general kernel's shapes."""

import pytest

import paper_1201_1548_amd as br
from oracle import zx
from oracle.subresultants import psc_at_mod
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def check(F, G, p, samples):
    _, rows = br.psc(F, G, prime=p)
    for a in samples:
        got = [zx.evaluate(r, a) % p if r else 0 for r in rows]
        assert got == psc_at_mod(F, G, a, p), a


@pytest.mark.parametrize("m,n", [(1, 1), (2, 1), (1, 2), (2, 2), (15, 15), (16, 15), (15, 16), (17, 17), (22, 21), (23, 22),
                                 (22, 23), (24, 24), (30, 31), (32, 32), (39, 40), (47, 48), (66, 66), (67, 66), (66, 67),
                                 (67, 67), (68, 67), (9, 7), (5, 9)])
def test_degrees_at_tile_and_chain_edges(m, n):
    F, G = synth.random_rect(77 * m + n, m, 2, n, 1, 30)
    p = br.primes(3)[m % 3]
    check(F, G, p, [0, 1, 5, p - 2] if max(m, n) < 40 else [3])


@pytest.mark.parametrize("m,n", [(4, 3), (4, 4), (3, 4)])
def test_blocks_that_leave_the_normal_sequence(m, n):
    # lc(F) vanishes at x = 4, lc(G) at x = 2; F and G share a root in y at x = 8
    F, G = synth.random_rect(m * 10 + n, m, 60, n, 1, 12)
    F[m] = [-4, 1] + [0] * 59
    G[n] = [-2, 1]
    p = br.primes(1)[0]
    check(F, G, p, [0, 1, 2, 4, 8, 16, 12345])
    H = [[-8, 1], [3, 0], [0, 0], [1, 0]]  # y^3 + 3 y + x - 8
    I = [[8, -1], [5, 0], [1, 0]]
    check(H, I, p, [1, 2, 8, 9])

"""Interpolation on the geometric nodes 2^i at the edges of its column tiles
(256 outputs), windows (64 inputs), tile pairs and launch classes, and the
evaluation there: degree-1 pairs in y, whose resultant is the 2 x 2 determinant
f_1 g_0 - f_0 g_1, and pairs whose leading coefficient or remainder vanishes at
a node."""

import pytest

import paper_1201_1548_amd as br
from oracle import zx
from oracle.resultant import discriminant_y, resultant_y
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def det2(F, G):
    a, b = zx.mul(F[1], G[0]), zx.mul(F[0], G[1])
    return zx.sub(a, b)


@pytest.mark.parametrize("D", [1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 300, 511, 512, 513, 767, 1023, 1024, 1025,
                               1281, 1537, 2049, 4097, 8096])
def test_points_at_tile_and_class_edges(D):
    dxf = (D - 1) // 3
    F, G = synth.random_rect(900 + D, 1, dxf, 1, D - 1 - dxf, 40)
    assert br.plan(F, G)[0] == D
    assert br.resultant(F, G) == det2(F, G)


def test_mixed_classes_in_one_batch():
    jobs, want = [], []
    for i, D in enumerate([1, 3, 200, 256, 257, 400, 600, 1024, 1100, 1600, 40, 513]):
        F, G = synth.random_rect(1700 + i, 1, D // 2, 1, D - 1 - D // 2, 8 + 20 * i)
        jobs.append(("res", F, G, "y"))
        want.append(det2(F, G))
    res, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    assert res == want


@pytest.mark.parametrize("node", [1, 2, 4, 64])
def test_vanishing_leading_coefficient_and_remainder_at_a_node(node):
    # lc_y f vanishes at x = node; f and g share a root in y there
    F, G = synth.random_rect(77 + node, 5, 4, 4, 3, 20)
    F[5] = [-node, 1, 0, 0, 0]
    assert br.resultant(F, G) == resultant_y(F, G)
    H = [[-node, 1], [0, 3], [5, 1], [1]]  # H(node, y) = y (3 node + ...): a degree drop along the remainders
    assert br.resultant(F, H) == resultant_y(F, H)
    assert br.discriminant(H) == discriminant_y(H)


@pytest.mark.parametrize("prime", [0, 1, 40])
def test_subresultants_at_another_table_prime(prime):
    F, G = synth.random_rect(5, 4, 3, 3, 5, 30)
    p = br.primes(prime + 1)[prime]
    _, rows = br.psc(F, G, prime=p)
    R = [c % p for c in resultant_y(F, G)]
    while R and R[-1] == 0:
        R.pop()
    assert rows[0] == R

"""Contents in the gcd and the square-free decomposition where the gcd of the
outer coefficients is not the content: one, several or all inner coefficients
lack a factor that both ends share, with trailing zero bits and limbs."""

import random

import pytest

import paper_1201_1548_amd as br
from oracle import zx
from oracle.gcd import gcd_zx
from oracle.squarefree import squarefree_yun

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("outer", [1, 6, 1 << 40, 3 << 64, (1 << 130) - 5])
@pytest.mark.parametrize("lacking", ["none", "first", "last", "all"])
def test_outer_coefficients_share_more_than_the_content(outer, lacking):
    rng = random.Random(outer % 1009)
    n, cont = 9, 35 << 33
    C = [rng.randint(1, 1 << 70) * 2 + 1 for _ in range(n + 1)]
    lack = {"none": [], "first": [1], "last": [n - 1], "all": list(range(1, n))}[lacking]
    C = [c * cont * (1 if i in lack else outer) for i, c in enumerate(C)]
    A, B = zx.mul(C, [3, 0, outer]), zx.mul(C, [outer, -5])
    assert br.gcd(A, B) == gcd_zx(A, B)
    assert br.gcd(C, zx.scale(C, -outer)) == C
    R = zx.mul(C, zx.mul([3, outer], [3, outer]))
    u, factors = br.squarefree(R)
    assert (u, factors) == squarefree_yun(R)

"""The gcd kernels at the ends of their ranges: degrees up to the largest that is
taken (8000, four arrays of it in LDS), and the degree chain of the N^- / N^+
test with inputs too long for its second buffers."""

import random

import numpy as np
import pytest

import paper_1201_1548_amd as br
from oracle import zx
from paper_1201_1548_amd import synth
from tests.test_gpu_gcd_rounds import primitive, rpoly

pytestmark = pytest.mark.gpu
P31 = (1 << 31) - 1


def gcd_degree_mod(a, b, p=P31):
    """deg gcd(a, b) mod p by Euclid with vector steps (products below 2^62)."""
    x, y = np.array([c % p for c in a], dtype=np.int64), np.array([c % p for c in b], dtype=np.int64)
    while len(y):
        inv = pow(int(y[-1]), -1, p)
        while len(x) >= len(y):
            c = int(x[-1]) * inv % p
            x[len(x) - len(y):] = (x[len(x) - len(y):] - c * y) % p
            nz = np.flatnonzero(x)
            x = x[:nz[-1] + 1] if len(nz) else x[:0]
        x, y = y, x
    return len(x) - 1


@pytest.mark.parametrize("da,db,dc", [(8000, 7999, 41), (8000, 8000, 0), (7990, 3, 2), (6000, 5999, 3000)])
def test_largest_degrees(da, db, dc):
    rng = random.Random(da + db)
    A, B = primitive(rpoly(rng, da - dc, 12)), primitive(rpoly(rng, db - dc, 12))
    assert A[-1] % P31 and B[-1] % P31 and gcd_degree_mod(A, B) == 0
    C = primitive(rpoly(rng, dc, 12)) if dc else [1]
    assert br.gcd(zx.mul(A, C), zx.mul(B, C)) == C


def test_beyond_the_largest_degree():
    with pytest.raises(br.BiresError):
        br.gcd([1] * 8002, [1, 2, 1])


@pytest.mark.parametrize("extra", [9000, 11000])
def test_fiber_bounds_without_second_buffers(extra):
    # R* h for an h without common factors with the subresultants or Q modulo p:
    # deg S_0 grows by deg h, every later gcd and the common part stay
    F = synth.singular_curve_deg40(1, dg=6, dh=4, dk=4, bits=6, square_k=True)
    R = br.discriminant(F)
    Rs = [1]
    for a in br.squarefree(R)[1]:
        Rs = zx.mul(Rs, a)
    ny = 12
    assert any(F[ny]) and not any(any(r) for r in F[ny + 1:])
    nm, npl, flags = br.fiber_bounds(F, Rs, len(R) - 1)
    rng = random.Random(extra)
    h = [rng.randint(-9, 9) for _ in range(extra)] + [1]
    nm2, npl2, flags2 = br.fiber_bounds(F, zx.mul(Rs, h), len(R) - 1)
    assert (nm2, npl2, flags2) == (nm + (ny - 1) * extra, npl + ny * extra, flags)

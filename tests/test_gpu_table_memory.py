"""Device memory that calls leave behind as tables: a prime count whose launch does
not take the explicit CRT builds none of its tables, and subresultants modulo a late
table prime build that prime's alone."""

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth
from tests.test_gpu_crt_counts import planted
from tests.test_gpu_interp_nodes import det2

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_counts_beyond_the_operand_limit_leave_no_tables():
    # a table of 700 primes takes about 10 MB; the buffers of every call come
    # from the pools that the first, largest one has filled
    counts = [711, 700, 702, 704, 706, 708, 710]
    jobs = [planted(P, 40) for P in counts]
    assert br.resultant(*jobs[0][:2]) == jobs[0][2]
    before = free_bytes()
    for F, G, t in jobs[1:]:
        assert br.resultant(F, G) == t
    assert before - free_bytes() < 16 * MIB


@pytest.mark.parametrize("index", [2047, 900, 1])
def test_subresultants_build_the_tables_of_their_prime_alone(index):
    # degrees 1 and 1 in y: sr_0 is the 2 x 2 determinant; 1561 points
    F, G = synth.random_rect(61 + index, 1, 700, 1, 860, 30)
    assert br.plan(F, G)[0] == 1561
    R = det2(F, G)
    ps = br.primes(index + 1)
    for p in (ps[0], ps[index]):
        before = free_bytes()
        _, rows = br.psc(F, G, prime=p)
        assert rows[0] == [c % p for c in R]
    assert before - free_bytes() < 8 * MIB

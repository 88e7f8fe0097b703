"""Device memory that calls leave behind as tables: a prime count whose launch does
not take the explicit CRT builds none of its tables."""

import pytest

import paper_1201_1548_amd as br
from tests.test_gpu_crt_counts import planted

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

"""Batches large enough for the stored powers of the evaluation points: rows up
to and beyond the stored 32 powers, on the nodes 2^i and, for jobs that share
point and prime counts, 0..D-1, growing and shrinking counts in turn, against
the general kernel."""

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx", [30, 31, 32, 70, 15])
@pytest.mark.parametrize("same", [True, False])
def test_stored_powers_against_the_general_kernel(dx, same):
    jobs = []
    for i in range(40):
        m, n = (22, 21) if same else (4 + i % 27, 3 + i % 5)
        F, G = synth.random_rect(4000 + 50 * dx + i, m, dx, n, dx - (0 if same else i % 3), 60 if same else 20 + i)
        jobs.append(("res", F, G, "y"))
    got, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    try:
        br.set_eval_kernel("lds")
        want, status = br.resultant_batch(jobs)
    finally:
        br.set_eval_kernel("auto")
    assert status == [0] * len(jobs)
    assert got == want

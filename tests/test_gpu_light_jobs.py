"""Jobs of small degrees and short rows (the general kernel's in calls that they
fill) at the edges of the rule that picks them: degree 8 and rows of 16, 24, 32
and 48 coefficients, on the nodes 2^a and (jobs that share point and prime
counts) 0, 1, .., alone, as the smaller part of a batch, and with leading
coefficients that vanish at nodes, against the general kernel for all."""

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def against_general(jobs):
    got, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    try:
        br.set_eval_kernel("lds")
        want, _ = br.resultant_batch(jobs)
    finally:
        br.set_eval_kernel("auto")
    assert got == want


@pytest.mark.parametrize("m,n", [(1, 1), (2, 1), (1, 2), (3, 3), (6, 5), (7, 8), (8, 8), (9, 8)])
@pytest.mark.parametrize("row", [1, 2, 16, 17, 24, 25, 33, 49])
@pytest.mark.parametrize("same", [True, False])
def test_edges_of_the_rule(m, n, row, same):
    # (one pair, and enough of them for the rule of full launches)
    count = max(40, 70000 // (3 * (m + n) * row)) if m + n < 14 else 40
    jobs = []
    for i in range(min(count, 400)):
        F, G = synth.random_rect(3000 + 10 * m + n + i, m, row - 1, n, max(0, row - 1 - (0 if same else i % 3)), 20)
        jobs.append(("res", F, G, "y"))
    against_general(jobs[:1])
    against_general(jobs)


def test_vanishing_leads_and_mixed_batches():
    light = []
    for i in range(300):
        F, G = synth.random_rect(4000 + i, 3 + i % 4, 5, 3 + i % 3, 5, 20)
        if i % 5 == 0:
            F[-1] = [-(1 << (i % 7)), 1] + [0] * 4  # vanishes at the node 2^(i % 7)
        if i % 7 == 0:
            G[-1] = [-(i % 9), 1] + [0] * 4
        if i % 11 == 0:
            F = [r if j % 2 == 0 else [0] * 6 for j, r in enumerate(F)]
        light.append(("res", F, G, "y"))
    heavy = [("res",) + synth.random_rect(5000 + i, 20, 30, 19, 30, 40) + ("y",) for i in range(12)]
    against_general(light)
    against_general(light[:40] + heavy)
    against_general(light + heavy[:2])
    against_general([("disc", F, None, "y") for _, F, _, _ in light if len(F) > 2 and any(any(r) for r in F[1:])])

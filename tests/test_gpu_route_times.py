"""Evaluation times of the default route against the general kernel's where the
registers have least to offer: it may lose what their attempt costs, no more."""

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def evaluation_time(b, kernel):
    """Milliseconds of the evaluation and elimination launches, best of twenty calls."""
    try:
        br.set_eval_kernel(kernel)
        b.run()
        b.run()
        best = 1e30
        for _ in range(20):
            br.set_timing(True)
            b.run()
            ms, launches = br.kernel_time()
            br.set_timing(False)
            best = min(best, ms / launches)
        return best, b.results()
    finally:
        br.set_timing(False)
        br.set_eval_kernel("auto")


@pytest.mark.parametrize("m,n", [(64, 62), (66, 64)])
def test_sequences_that_are_not_normal(m, n):
    # even in y: every remainder skips a degree, every block is recomputed
    F, G = synth.random_rect(2, m, 10, n, 10, 30)
    F, G = ([r if j % 2 == 0 else [0] * len(r) for j, r in enumerate(P)] for P in (F, G))
    b = br.DeviceBatch([("res", F, G, "y")] * 20)
    general, want = evaluation_time(b, "lds")
    registers, got = evaluation_time(b, "auto")
    assert got == want
    # the attempt is one evaluation and a step of a chain: a tenth measured, 3.3 times
    # with a quarter of the blocks that the general kernel has at once
    assert registers < 1.5 * general


@pytest.mark.parametrize("count,degree,row", [(3000, 1, 4), (3000, 2, 4), (3000, 4, 5), (1, 1, 4)])
def test_small_degrees(count, degree, row):
    # capacity 24 took 2.2, 1.6, 1.4 and 1.9 times the general kernel's time
    b = br.DeviceBatch([("res",) + synth.random_rect(100 + i % 5, degree, row - 1, degree, row - 1, 20) + ("y",)
                        for i in range(count)])
    general, want = evaluation_time(b, "lds")
    default, got = evaluation_time(b, "auto")
    assert got == want
    assert default < 1.25 * general

"""Row statistics of inputs in device memory at the edges of the lanes that share
a row (4 to 64, longer rows in pieces), for one and several limbs, sparse and zero
rows and extreme values, through the results they plan, against the same calls
on host memory."""

import random

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limbs", [1, 2, 3, 5])
def test_row_lengths_and_values(limbs):
    rng = random.Random(limbs)
    top = 1 << (32 * limbs - 1)
    jobs = []
    for nx in [0, 1, 3, 4, 7, 8, 9, 15, 16, 31, 32, 33, 62, 63, 64, 65, 127, 128, 130]:
        for ny in (1, 2, 3):
            F, G = synth.random_rect(97 * nx + ny, ny, nx, 2, max(nx - 2, 0), 32 * limbs, zero_frac=0.4)
            F[0] = [rng.choice([0, -1, 1, top - 1, -top, -(top >> 1)]) for _ in F[0]]
            F[ny][nx // 2] = -top
            G[2][0] = 1
            G[1] = [0] * len(G[1])
            jobs.append(("res", F, G, "y"))
    for rows in (63, 64, 65):  # more rows than a block of the scan holds
        F, G = synth.random_rect(rows, rows, 3, 1, 2, 32 * limbs)
        jobs.append(("res", F, G, "y"))
    want, status = br.resultant_batch(jobs)
    assert status == [0] * len(jobs)
    b = br.DeviceBatch(jobs)
    b.run()
    assert b.results() == want

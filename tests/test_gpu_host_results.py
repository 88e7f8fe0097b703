"""Results in host memory: every row and limb of the caller's buffer is written
(zeros above the degree, sign extension), whatever its capacities and contents."""

import ctypes

import numpy as np
import pytest

import paper_1201_1548_amd as br
from oracle import zx
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def limbs(rows, L):
    a = [[(c >> (32 * l)) & 0xFFFFFFFF for l in range(L)] for r in rows for c in r]
    return np.array(a, dtype=np.uint32).reshape(len(rows), len(rows[0]), L)


@pytest.mark.parametrize("rows_more,limbs_more", [(0, 0), (3, 0), (0, 1), (1, 2), (700, 40)])
def test_every_word_of_larger_buffers_is_written(rows_more, limbs_more):
    pairs = [synth.random_rect(60 + i, 1, 5 + 20 * i, 1, 3 + i, 30 + 31 * i) for i in range(6)]
    n = len(pairs)
    f, g, out = (br.Bipoly * n)(), (br.Bipoly * n)(), (br.Upoly * n)()
    keep, bufs = [], []
    for i, (F, G) in enumerate(pairs):
        for d, X in ((f, F), (g, G)):
            w = limbs(X, (30 + 31 * i) // 32 + 1)
            keep.append(w)
            d[i] = br.Bipoly(w.shape[0] - 1, w.shape[1] - 1, w.shape[2], w.ctypes.data)
        D, L = br.bounds(F, G)
        b = np.full((D + 1 + rows_more, L + limbs_more), 0xDEADBEEF, dtype=np.uint32)
        bufs.append(b)
        out[i] = br.Upoly(b.shape[0] - 1, b.shape[1], b.ctypes.data)
    kinds, variables, status = (ctypes.c_int32 * n)(), (ctypes.c_int32 * n)(*[1] * n), (ctypes.c_int32 * n)()
    assert br.lib().bires_resultant_batch(n, f, g, kinds, variables, out, status, br.MEM_HOST, None) == 0
    for i, (F, G) in enumerate(pairs):
        want = zx.sub(zx.mul(F[1], G[0]), zx.mul(F[0], G[1]))
        assert out[i].degree == len(want) - 1
        want = want + [0] * (bufs[i].shape[0] - len(want))
        assert np.array_equal(bufs[i], limbs([want], bufs[i].shape[1])[0]), i

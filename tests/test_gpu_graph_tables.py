"""Graph replay and the tables that launches take by value: two batches alike in
every block count, size and offset, whose degree-20 pairs need 256 and 256
primes in one and 192 and 320 in the other, so that only the stored powers of
the points differ between their launch sequences; and point counts that grow
from call to call, each with tables that take the place of the former ones."""

import functools

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def pair_of(P, seed):
    """A dense degree-20 pair that needs P primes at 401 points."""
    for bits in range(7 * P // 10, 9 * P // 10):
        F, _ = synth.random_dense(seed, 20, bits)
        for more in range(4):
            _, G = synth.random_dense(seed, 20, bits + more)
            if br.plan(F, G)[:2] == (401, P):
                return "res", F, G, "y"
    raise AssertionError("no pair with %d primes" % P)


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
def test_a_replayed_graph_reads_its_own_tables(order, monkeypatch):
    import torch
    monkeypatch.setattr(br, "DeviceBipoly", functools.partial(br.DeviceBipoly, limbs=9))
    large = ("res",) + synth.random_dense(3, 32, 170) + ("y",)  # sets the largest degree and prime count of both
    counts = [(256, 256), (192, 320)]
    batches = [br.DeviceBatch([pair_of(P, 20 + i) for i, P in enumerate(c)] + [large]) for c in counts]
    assert br.plan(large[1], large[2])[1] > 320
    br.set_plan_cache(False)
    try:
        br.set_graphs(True)
        got = []
        for rep in range(3):
            for i in order:
                for t in batches[i].out_tensors:
                    t.fill_(-1)
                torch.cuda.synchronize()
                batches[i].run()
                got.append((i, batches[i].results()))
    finally:
        br.set_graphs(False)
        br.set_plan_cache(True)
    want = []
    for b in batches:
        b.run()
        want.append(b.results())
    for i, r in got:
        assert r == want[i]


def test_outgrown_tables_and_their_graphs():
    # 16 sizes up to 7936 points, each replayed, then all again on the last tables
    batches = [br.DeviceBatch([("res",) + synth.random_rect(71 + k, 1, 5, 1, 256 + 512 * k - 6, 40) + ("y",)])
               for k in range(16)]
    br.set_plan_cache(False)
    try:
        br.set_graphs(True)
        got = []
        for b in [b for b in batches for _ in range(3)] + batches:
            for t in b.out_tensors:
                t.fill_(-1)
            b.run()
            got.append(b.results())
    finally:
        br.set_graphs(False)
        br.set_plan_cache(True)
    try:
        br.set_eval_kernel("lds")
        for i, b in enumerate(batches):
            b.run()
            assert got[3 * i:3 * i + 3] + [got[48 + i]] == [b.results()] * 4
    finally:
        br.set_eval_kernel("auto")

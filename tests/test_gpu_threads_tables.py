"""Tables of the geometric nodes that go, because a larger one takes their place,
while calls of other threads read them."""

import threading

import pytest

import paper_1201_1548_amd as br
from paper_1201_1548_amd import synth

pytestmark = pytest.mark.gpu


def test_tables_that_go_while_other_threads_read_them():
    # 20 sizes up to 6086 points (and 40 primes: tables that no smaller call
    # leaves) in growing order, dealt to four threads with a stream each
    batches = [br.DeviceBatch([("res",) + synth.random_rect(171 + k, 1, 5, 1, 1900 + 220 * k, 600) + ("y",)])
               for k in range(20)]
    import torch
    torch.cuda.synchronize()
    got, errors = [None] * 20, []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            for k in range(t, 20, 4):
                for _ in range(3):
                    batches[k].run(stream)
                stream.synchronize()
                got[k] = batches[k].results()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    try:
        br.set_eval_kernel("lds")
        for k, b in enumerate(batches):
            b.run()
            assert got[k] == b.results(), k
    finally:
        br.set_eval_kernel("auto")

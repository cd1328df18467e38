"""The device blocks that the library keeps between calls: results stay those of
a first call with several threads on one stream, a stream per thread, sizes
that come and go, and after the blocks are given back."""
import threading

import numpy as np
import pytest
import torch

from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu

SIZES = (300, 5000, 1000, 20011, 64)


def _pass(x, q, stream):
    t = kdt.build(x, leaf_size=16, stream=stream)
    idx, d2 = t.knn(q, 8, stream=stream)
    cnt, off, lists = t.range(q, 0.05, lists=True, stream=stream)
    lab = t.fof(0.01, stream=stream)
    stream.synchronize()
    return [to_host(a).copy() for a in (idx, d2, cnt, off, lists, lab)]


def _case(seed):
    n = SIZES[seed % len(SIZES)]
    return to_dev(workloads.clustered(n, seed)), to_dev(workloads.uniform(500, 3, seed + 50))


@pytest.mark.parametrize("streams", (1, 4))
def test_threads_share_the_kept_blocks(streams):
    dev()
    s = [torch.cuda.Stream() for _ in range(streams)]
    data = [_case(k) for k in range(20)]
    torch.cuda.synchronize()
    want = [_pass(x, q, s[0]) for x, q in data]
    got = [[None] * len(data) for _ in range(4)]
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(s[k % streams]):
                for j in range(len(data)):
                    i = (j + 5 * k) % len(data)
                    got[k][i] = _pass(*data[i], s[k % streams])
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(4):
        for i, w in enumerate(want):
            for a, b in zip(got[k][i], w):
                np.testing.assert_array_equal(a, b)
        say(f"thread {k} of {streams} stream(s): equal")
    for st in s:
        kdt.stream_release(st)


def test_blocks_come_back_after_a_release():
    dev()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        x, q = _case(3)
        torch.cuda.synchronize()
        want = _pass(x, q, st)
        for _ in range(3):
            kdt.stream_release(st)
            for a, b in zip(_pass(x, q, st), want):
                np.testing.assert_array_equal(a, b)
    kdt.stream_release(st)

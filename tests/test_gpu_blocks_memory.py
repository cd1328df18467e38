"""Device memory that the library keeps: every idle block goes back before a request
fails for lack of memory, whatever its size and kind, and streams may be destroyed with blocks
kept for them -- a later stream, even one with the same handle, gets the results of a
first call."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2609_18316_amd import kdt, workloads
from tests.gpu_util import dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu
LARGE = 3_000_000  # records of 48 MB: the list scratch and the tree pass 128 MiB


def _warm(x, q):
    t = kdt.build(x, leaf_size=16)
    t.knn(q, 8)
    t.range(q, 0.05, lists=True)
    t.close()
    torch.cuda.synchronize()


def _calls():
    x, q = to_dev(workloads.clustered(20011, 5)), to_dev(workloads.uniform(3000, 3, 6))
    big = to_dev(workloads.uniform(LARGE, 8, 7))
    off = np.array([0, 900, 6000, 20011], np.int64)
    t = kdt.build(x, leaf_size=16)
    more = to_dev(workloads.uniform(70001, 3, 8))

    def small():
        kdt.stream_release()  # nothing idle has these sizes: the pool is asked
        return t.knn(more, 8)

    def large():
        b = kdt.build(big, leaf_size=64, check_finite=False)
        i = b.knn(big[:1000].contiguous(), 1)
        b.close()
        return i

    def plan():
        p = kdt.BatchPlan(off, 3, 4, leaf_size=16)
        r = p.launch(x, torch.full((3,), 0.01, device=x.device))
        r = [a.clone() for a in r]
        p.close()
        return r

    return x, q, {"small": small, "large": large, "plan": plan}


def test_idle_blocks_go_back_before_memory_runs_out():
    dev()
    x, q, calls = _calls()
    side = torch.cuda.Stream()
    for name, call in calls.items():
        want = [to_host(a).copy() for a in call()]
        for after in (1, 2, 5):
            _warm(x, q)
            with torch.cuda.stream(side):
                _warm(x, q)
            assert kdt.kept_bytes() > 0 and kdt.kept_bytes(side) > 0
            before = kdt.kept_bytes(every=True)
            kdt.fail_memory(after)
            got = call()
            kdt.fail_memory(0)
            torch.cuda.synchronize()
            say(f"{name}, request {after} finds no memory: {before} bytes kept before, "
                f"{kdt.kept_bytes(side)} for the other stream after")
            for a, b in zip(got, want):
                np.testing.assert_array_equal(to_host(a), b)
            if after == 1:
                assert kdt.kept_bytes(side) == 0, name


def test_streams_destroyed_without_a_release():
    dev()
    hip = kdt.load()  # (its own dependencies' symbols are found through it)
    x, q = to_dev(workloads.clustered(20011, 5)), to_dev(workloads.uniform(3000, 3, 6))
    t = kdt.build(x, leaf_size=16)
    want = [to_host(a).copy() for a in t.range(q, 0.05, lists=True)]
    torch.cuda.synchronize()
    handles, most = set(), 0
    for i in range(40):
        h = C.c_void_p()
        assert hip.hipStreamCreate(C.byref(h)) == 0
        handles.add(h.value)
        s = torch.cuda.ExternalStream(h.value)
        tree = kdt.build(x, leaf_size=16, stream=s)
        got = tree.range(q, 0.05, lists=True, stream=s)
        tree.close()
        assert hip.hipStreamSynchronize(h) == 0
        assert hip.hipStreamDestroy(h) == 0
        most = max(most, kdt.kept_bytes(every=True))
        if i == 4:
            early = most
        for a, b in zip(got, want):
            np.testing.assert_array_equal(to_host(a), b)
    say(f"40 streams, {len(handles)} handles, {early} bytes kept after 5, {most} at most")
    # blocks of streams that are gone are used again, not kept beside new ones
    assert most <= early
    t.close()

"""The wait for a build's status: a kernel writes it to a page of host memory
that the waiting thread polls."""
import os
import subprocess
import sys
import time

import numpy as np
import pytest

import oracle
from tests._util import dev, workload

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def bht():
    import paper_2108_07232_amd
    return paper_2108_07232_amd


def table_for(n, seed):
    p = oracle.params_for("bcht", n, 0.8, seed)
    return p, bht().Table(p.m * p.b, p.b, "bcht", p.a, p.c, rng_seed=p.rng_seed)


def builds_and_waits():
    """Statuses and the longest of 40 waits, good and refused builds in turn."""
    import torch
    B = bht()
    good, bad = workload(40000, 71), workload(40000, 72)
    bad[0][123] = 0xFFFFFFFF
    data = [(dev(k), dev(v)) for k, v in (good, bad)]
    _, t = table_for(40000, 7100)
    t.build(*data[0])
    torch.cuda.synchronize()
    worst = 0.0
    for i in range(40):
        t0 = time.perf_counter()
        st = t.build(*data[i % 2])
        worst = max(worst, time.perf_counter() - t0)
        assert st == (B.BHT_ERR_SENTINEL_KEY if i % 2 else B.BHT_OK)
    t.close()
    return worst


def test_wait_does_not_depend_on_the_environment():
    """With host memory that is not coherent unless asked for, statuses
    arrive as they do by default: well before the 2 s after which a wait stops
    polling."""
    code = ("import sys; sys.path.insert(0, %r); from tests.test_gpu_status import *; "
            "print('worst', builds_and_waits())" % ROOT)
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100,
                         env=dict(os.environ, HIP_HOST_COHERENT="0"))
    assert out.returncode == 0, out.stderr
    assert float(out.stdout.split("worst")[1]) < 1.0
    assert builds_and_waits() < 1.0


def test_wait_in_a_capture_is_refused_at_once():
    """Waiting for a build in a stream that is being captured fails without
    waiting and leaves the capture as it is: the graph builds the table when
    it is launched."""
    import torch
    B = bht()
    keys, vals = workload(5000, 73)
    dk, dv = dev(keys), dev(vals)
    p, t = table_for(5000, 7300)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.bht_build_async(t.handle, dk, dv, stream=side)
        t0 = time.perf_counter()
        for _ in range(3):
            with pytest.raises(B.BhtError) as e:
                B.bht_build_wait(t.handle, stream=side)
            assert e.value.status == B.BHT_ERR_HIP
        took = time.perf_counter() - t0
    assert took < 0.5
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert B.bht_build_wait(t.handle) == B.BHT_OK
        assert oracle.check32(p, t.download(), keys, vals) == (0, "ok")
    t.close()

"""Builds captured into HIP graphs, with the table's workspace at hand or not:
a graph may be replayed after any later build of the same table."""
import numpy as np
import pytest

import datagen
import oracle
from tests._util import dev, host_u32, host_u8, workload

pytestmark = pytest.mark.gpu


def bht():
    import paper_2108_07232_amd
    return paper_2108_07232_amd


def table_for(scheme, n, lf, seed, b=16):
    """Parameters and table for n pairs (iceberg: two levels, t = b)."""
    p = oracle.params_for(scheme, n, lf, seed, b=b, max_chain=512)
    if scheme == "iht":
        p.threshold, p.b2, p.m2 = b, 8, max(1, p.m * b // 64)
    t = bht().Table(p.m * b, b, scheme, p.a, p.c, rng_seed=p.rng_seed, max_chain=512,
                    iht_threshold=p.threshold, iht_secondary_b=p.b2, iht_secondary_m=p.m2)
    return p, t


def check(t, p, keys, vals, seed=7):
    import torch
    code, msg = oracle.check32(p, t.download(), keys, vals)
    assert code == 0, msg
    q = datagen.mixed_queries(len(keys), min(2 * len(keys), 1 << 20), 0.5, seed)
    v, f = t.find(dev(q))
    torch.cuda.synchronize()
    ev, ef = oracle.brute_find32(keys, vals, q)
    np.testing.assert_array_equal(host_u8(f), ef)
    np.testing.assert_array_equal(host_u32(v), ev)


def capture(t, dk, dv):
    import torch
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        bht().bht_build_async(t.handle, dk, dv, stream=side)
    return graph


@pytest.mark.parametrize("scheme,n", [("bcht", 40000), ("cht1", 140000), ("iht", 20000),
                                      ("bp2ht", 20000)])
def test_captured_small_build_keeps_no_workspace(scheme, n):
    """Sizes that take the table's workspace when it is at hand: a captured
    build does not, so the graph holds after a larger build has replaced it."""
    import torch
    B = bht()
    b = 1 if scheme == "cht1" else 16
    many, few = workload(9 * n // 8, 61), workload(n, 62)
    dk, dv = dev(few[0]), dev(few[1])
    p, t = table_for(scheme, 9 * n // 8, 0.82, 6100, b=b)
    assert t.build(dk, dv) == B.BHT_OK                 # the workspace is at hand
    graph = capture(t, dk, dv)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
    assert B.bht_build_wait(t.handle) == B.BHT_OK
    assert not B.bht_build_stats(t.handle)[0]
    check(t, p, *few)
    assert t.build(dev(many[0]), dev(many[1])) == B.BHT_OK     # a larger one
    check(t, p, *many)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        check(t, p, *few)
    t.close()


def test_captured_iceberg_build_asks_for_no_more_than_is_at_hand():
    """A two-level iceberg build of nearly 2^24 pairs, captured after a build
    that left a workspace for the pairs but not for the secondary counts."""
    import torch
    B = bht()
    most = (1 << 24) + 4096                            # past the counted sizes
    keys, vals = workload(most, 63)
    dk, dv = dev(keys), dev(vals)
    p, t = table_for("iht", most, 0.7, 6300)
    like = B.Table(p.m * p.b, p.b, "bcht", p.a, p.c)   # the same plan for the pairs
    at_hand = B.bht_build_workspace_bytes(like.handle, most)
    n = next(n for n in range(1 << 24, 1 << 23, -(1 << 16))
             if B.bht_build_workspace_bytes(like.handle, n) <= at_hand)
    assert B.bht_build_workspace_bytes(like.handle, n) + 64 * p.m2 > at_hand
    like.close()
    assert t.build(dk, dv) == B.BHT_OK
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        B.bht_build_async(t.handle, dk, dv, n=n, stream=side)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
    assert B.bht_build_wait(t.handle) == B.BHT_OK
    check(t, p, keys[:n], vals[:n])
    t.close()


def test_captured_workspace_outlives_a_larger_build():
    """From 2^18 pairs a captured build uses the table's workspace, which
    stays allocated when a larger build replaces it."""
    import torch
    B = bht()
    n, more = 1 << 18, 1 << 20
    few, many = workload(n, 64), workload(more, 65)
    dk, dv, dk2, dv2 = dev(few[0]), dev(few[1]), dev(many[0]), dev(many[1])
    for last in (False, True):                         # the first time loads the kernels
        p, t = table_for("bcht", more, 0.8, 6400)
        assert t.build(dk, dv) == B.BHT_OK
        graph = capture(t, dk, dv)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        assert t.build(dk2, dv2) == B.BHT_OK
        taken = before - torch.cuda.mem_get_info()[0]
        if not last:
            t.close()
    assert taken >= B.bht_build_workspace_bytes(t.handle, more)     # nothing was freed for it
    check(t, p, *many)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        check(t, p, *few)
    assert t.build(dk2, dv2) == B.BHT_OK
    check(t, p, *many)
    t.close()

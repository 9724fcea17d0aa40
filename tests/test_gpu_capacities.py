"""Steps over graphs of one size and different arc capacities.

The launch shape of a step is captured once; capacities go into it rounded, so
that graphs that differ in their arc counts share the captured shapes, and the
last launch of a step places every arc whatever the rounding.
"""
from __future__ import annotations

import time

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def updates(g, k, w_max):
    return W.mixed_stream(g, k, w_max, g.n + k, 0.5, 0.5, 4)


@pytest.mark.parametrize("caps", [(1023, 1024, 1025), (2047, 2048, 3071, 3072, 3073), (70000, 5000, 1300)])
def test_arc_capacities_around_the_chunks(caps):
    """E* as large as the capacity allows in the smallest, far from it in the largest."""
    say(f"capacities: {caps}")
    graphs = [W.directed_out_degree(130, 7, 50, c) for c in caps]
    ctx = make_ctx(130, slots=16)
    grs = [ctx.load_graph(g, arc_capacity=c, estar_capacity=c) for g, c in zip(graphs, caps)]
    ups = [updates(g, 4, 50) for g in graphs]
    for k in range(4):
        ctx.enqueue([(gr, u[k]) for gr, u in zip(grs, ups)])
        while ctx.step(max_jobs=1 + k % 2):
            pass
        graphs = [W.apply_update(g, u[k]) for g, u in zip(graphs, ups)]
    ctx.sync()
    for gr, g in zip(grs, graphs):
        check_full(gr, g, str(caps), dags=(0, 64))
    ctx.close()


def test_steps_share_their_captured_shapes():
    """One step on each of 96 graphs: with a capacity each, hardly more time than with one for all
    (half as much again when every capacity is captured by itself)."""
    def steps(caps):
        g = W.directed_out_degree(300, 8, 100, 5)
        up = updates(g, 1, 100)[0]
        ctx = make_ctx(g.n, slots=64)
        grs = [ctx.load_graph(g, arc_capacity=c, estar_capacity=c) for c in caps]
        ctx.sync()
        ctx.enqueue([(gr, up) for gr in grs])
        t0 = time.perf_counter()
        while ctx.step(max_jobs=1):
            pass
        ctx.sync()
        t = time.perf_counter() - t0
        want = grs[0].scores()
        for gr in grs[1:]:
            assert np.allclose(gr.scores(), want, rtol=1e-10, atol=1e-10)
        ctx.close()
        return t

    steps([3000] * 8)
    same, each = (min(steps(c) for _ in range(4)) for c in ([64000] * 96, [33000 + 320 * i for i in range(96)]))
    say(f"capacities: one for all {same * 1e3:.1f} ms, one each {each * 1e3:.1f} ms")
    assert each < 1.3 * same

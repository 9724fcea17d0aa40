"""The static pass where a source has more DAG arcs than its list holds.

Equal weights and many arcs per vertex: three and more DAG arcs a vertex, which the
static pass walks vertex by vertex.  Mean degrees go over every number of lanes
per vertex, sizes over every workgroup size, with a chain behind the dense part (as
many frontiers as the chain is long) and hubs that hold most of the arcs; path
counts up to and past 2^64 - 1.
"""
from __future__ import annotations

import time

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def with_tail(core: W.Graph, tail: int) -> W.Graph:
    """core, and a chain of `tail` more vertices from its vertex 0 back to its vertex 1."""
    t = np.arange(core.n, core.n + tail)
    src = np.concatenate([core.src, [0], t[:-1], t[-1:]])
    dst = np.concatenate([core.dst, t[:1], t[1:], [1]])
    w = np.concatenate([core.w, np.ones(tail + 1, np.int64)])
    return W.Graph(core.n + tail, core.directed, src.astype(np.int32), dst.astype(np.int32), w)


def joined(layers: int, width: int) -> W.Graph:
    """Complete joins between consecutive layers, unit weights."""
    l, i, j = np.meshgrid(np.arange(layers - 1), np.arange(width), np.arange(width), indexing="ij")
    src, dst = (l * width + i).ravel(), ((l + 1) * width + j).ravel()
    return W.Graph(layers * width, True, src.astype(np.int32), dst.astype(np.int32), np.ones(src.size, np.int64))


def hubs(n: int, count: int) -> W.Graph:
    """`count` hubs joined both ways to every other vertex, unit weights: two hops
    between any two others, by every hub."""
    h, v = (x.ravel() for x in np.meshgrid(np.arange(count), np.arange(count, n), indexing="ij"))
    return W.Graph(n, False, h.astype(np.int32), v.astype(np.int32), np.ones(h.size, np.int64))


GRAPHS = {
    "64 threads, 16 lanes": lambda: with_tail(W.directed_out_degree(120, 50, 1, 1), 31),
    "64 threads, a wave a vertex": lambda: with_tail(W.directed_out_degree(300, 200, 2, 2), 5),
    "128 threads, 8 lanes": lambda: with_tail(W.directed_out_degree(600, 22, 1, 3), 60),
    "128 threads, a wave a vertex": lambda: W.directed_out_degree(700, 300, 1, 4),
    "256 threads, 4 lanes": lambda: with_tail(W.directed_out_degree(2100, 16, 1, 5), 9),
    "512 threads, 8 lanes": lambda: with_tail(W.directed_out_degree(4200, 20, 1, 6), 3),
    "undirected": lambda: with_tail(W.gnp_undirected(513, 30.0, 2, 7), 40),
    "hubs": lambda: hubs(520, 5),
    "more hubs": lambda: with_tail(hubs(1030, 40), 17),
    "the largest path count": lambda: joined(14, 40),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_more_dag_arcs_than_the_list_holds(name):
    g = GRAPHS[name]()
    arcs = g.m if g.directed else 2 * g.m
    say(f"ties: {name}, n={g.n}, arcs={arcs}")
    ctx = make_ctx(g.n)
    gr = ctx.load_graph(g, arc_capacity=arcs + 16, estar_capacity=arcs + 16)
    dags = sorted({0, 1, g.n // 2, g.n - 1})
    check_full(gr, g, name, dags=dags, deltas=dags[:1])
    gr.recompute_estar()  # the slots are not cleared in between
    check_full(gr, g, name + ", over E*", dags=dags)
    ctx.close()


def test_path_count_past_64_bits():
    from paper_1311_2147_amd import bcinc

    g, good = joined(15, 40), with_tail(W.directed_out_degree(550, 40, 1, 8), 10)  # 40^12 fits, 40^13 does not
    say(f"ties: sigma overflow, n={g.n}")
    ctx = make_ctx(g.n)
    with pytest.raises(bcinc.BcError) as e:
        ctx.load_graph(g, arc_capacity=g.m, estar_capacity=g.m)
    assert e.value.name == "BC_ERR_SIGMA_OVERFLOW"
    gr = ctx.load_graph(good, arc_capacity=good.m + 16, estar_capacity=good.m + 16)
    check_full(gr, good, "after an overflow", dags=(0, 1))
    ctx.close()


def test_time_does_not_grow_with_arcs_times_levels():
    """A dense part of 1024 vertices and a chain of 1000 against a chain of as many vertices: both
    have 1000 levels or more.  A pass over all arcs per level takes fifty times the chain's time."""
    def best(g):
        ctx = make_ctx(g.n)
        gr = ctx.load_graph(g, arc_capacity=g.m + 16, estar_capacity=g.m + 16)
        t = []
        for _ in range(3):
            ctx.sync()
            t0 = time.perf_counter()
            gr.recompute()
            t.append(time.perf_counter() - t0)
        ctx.close()
        return min(t)

    dense = best(with_tail(W.directed_out_degree(1024, 64, 1, 9), 1000))
    chain = best(W.path_graph(2024, directed=True))
    say(f"ties: {dense * 1e3:.1f} ms, chain {chain * 1e3:.1f} ms")
    assert dense < 10 * chain

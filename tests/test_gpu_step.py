"""Edges of an update step's launches.

E* sizes around one and two times the 1024 arcs a workgroup places at a time, the keep masks
scanned by their own launch (an E* capacity above 2^20 arcs), graphs up to and
past the size where a source can be deferred, and 8 and 64 arcs per direction
(loads go out eight at a time), on directed and undirected graphs.  Plain and
batched steps are both compared with the oracle.
"""
from __future__ import annotations

import pytest

from gpu_util import check_full, check_sampled, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(g, ups, label, **kw):
    say(f"step: {label}, n={g.n}, m={g.m}, {len(ups)} updates")
    ctx = make_ctx(g.n, slots=64)
    plain, batched = ctx.load_graph(g, **kw), ctx.load_graph(g, **kw)
    for up in ups:
        plain.update(up)
    ctx.submit([(batched, up) for up in ups])
    ctx.sync()
    for up in ups:
        g = W.apply_update(g, up)
    for gr, how in ((plain, "plain"), (batched, "batched")):
        check_full(gr, g, f"{label}, {how}", dags=(0, g.n - 1))
    ctx.close()


@pytest.mark.parametrize("n", [1022, 1023, 1024, 1025, 2046, 2047, 2048, 2049])
def test_estar_around_the_placing_chunks(n):
    g = W.cycle_graph(n, directed=True)
    _run(g, [W.Update("edge", u=0, v=n // 2, w=3), W.Update("edge", u=n // 2, v=0, w=2)], f"cycle {n}")


@pytest.mark.parametrize("cap", [1 << 20, (1 << 20) + 1])
def test_capacity_that_scans_the_masks(cap):
    g = W.random_small(700, 0.02, 9, seed=21)
    _run(g, W.mixed_stream(g, 6, 9, 5, 0.4, 0.3, 6), f"capacity {cap}", arc_capacity=cap, estar_capacity=cap)


@pytest.mark.parametrize("n", [511, 512, 513])
@pytest.mark.parametrize("directed", [True, False])
def test_sizes_around_the_first_deferral(n, directed):
    g = W.random_small(n, 0.012, 4, seed=n, directed=directed)
    _run(g, W.mixed_stream(g, 5, 4, n, 0.4, 0.3, 5), f"n {n}")


@pytest.mark.parametrize("k", [7, 8, 9, 63, 64, 65, 130])
@pytest.mark.parametrize("directed", [True, False])
def test_arcs_per_update(k, directed):
    g = W.random_small(150, 0.9, 50, seed=k, directed=directed)
    cap = 2 * 150 * 150
    _run(g, W.vertex_stream(g, 2, k, 50, k), f"{k} arcs", arc_capacity=cap, estar_capacity=cap)


@pytest.mark.parametrize("gap", [15, 16, 17, 400])
def test_runs_of_heads_without_arcs(gap):
    """E* arcs into every gap-th vertex only: more long runs per chunk than are listed, and none."""
    n = 1600
    heads = W.np.arange(gap, n, gap)
    src = W.np.concatenate([W.np.zeros(heads.size), heads[:-1]]).astype(W.np.int32)
    dst = W.np.concatenate([heads, heads[1:]]).astype(W.np.int32)
    g = W.Graph(n, True, src, dst, W.np.full(src.size, 5, W.np.int64))
    _run(g, [W.Update("edge", u=0, v=int(heads[0]), w=1), W.Update("edge", u=int(heads[0]), v=1, w=2),
             W.Update("edge", u=0, v=n - 1, w=1)], f"gap {gap}")


def test_nothing_to_merge_into():
    g = W.Graph(300, True, *(W.np.zeros(0, t) for t in (W.np.int32, W.np.int32, W.np.int64)))
    _run(g, [W.Update("edge", u=5, v=299, w=1), W.Update("edge", u=299, v=0, w=1), W.Update("edge", u=0, v=5, w=4)],
         "empty graph")


@pytest.mark.parametrize("n", [4095, 4097, 8191, 8193])
def test_whole_rows_that_are_no_quads(n):
    """Sizes around one and two trips of a workgroup over a row read pair by pair."""
    g = W.cycle_graph(n, directed=True)
    ups = [W.Update("edge", u=0, v=n // 3, w=1), W.Update("vertex", v=n // 2, edges=[(5, n // 2, 1), (n // 2, 9, 2)])]
    say(f"step: rows of {n}")
    ctx = make_ctx(n, slots=64)
    gr = ctx.load_graph(g)
    for up in ups:
        gr.update(up)
        g = W.apply_update(g, up)
    check_sampled(gr, g, [0, 1, 5, 9, n // 3 - 1, n // 3, n // 2, n - 1], f"rows of {n}")
    ctx.close()

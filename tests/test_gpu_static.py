"""The static pass at the edges of its paths.

Values in LDS (up to 18432 vertices), the distance row only (up to 36864) or
nothing; the list of DAG arcs against sweeps over E* (more than three DAG arcs
per vertex); level counts in LDS (below 2048 levels) or in the slot; the search's
queue and its list of heavy vertices full.  Small
graphs are compared with the oracle in full.  Large ones are many small
components, so that the oracle can give a component's betweenness by itself,
and the device's state check covers distances, counts and predecessors.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import BC_TOL, bc_err, check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def layered(layers: int, width: int) -> W.Graph:
    """Complete joins between consecutive layers, unit weights."""
    l, i, j = np.meshgrid(np.arange(layers - 1), np.arange(width), np.arange(width), indexing="ij")
    src = (l * width + i).ravel().astype(np.int32)
    dst = ((l + 1) * width + j).ravel().astype(np.int32)
    return W.Graph(layers * width, True, src, dst, np.ones(src.size, np.int64))


def hub_row(hubs: int, degree: int, n: int) -> W.Graph:
    """Vertex 0 reaches `hubs` vertices at distance 1, each with `degree` out-arcs: the
    search expands them all at once (queue of 256 at these sizes, 256 chunks of heavy
    vertices, 256 arcs per chunk)."""
    rs = np.random.default_rng(hubs * 1000 + degree)
    src, dst = [np.zeros(hubs, np.int64)], [np.arange(1, hubs + 1)]
    for h in range(1, hubs + 1):
        others = rs.permutation(np.delete(np.arange(1, n), h - 1))[:degree]
        src.append(np.full(others.size, h))
        dst.append(others)
    src, dst = np.concatenate(src), np.concatenate(dst)
    w = rs.integers(1, 60, src.size)
    w[:hubs] = 1
    return W.Graph(n, True, src.astype(np.int32), dst.astype(np.int32), w.astype(np.int64))


SMALL = {
    "one vertex": lambda: W.Graph(1, True, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int64)),
    "two": lambda: W.path_graph(2),
    "512 in one wave per 8": lambda: W.random_small(512, 0.02, 5, seed=3),
    "513": lambda: W.random_small(513, 0.02, 5, seed=4, directed=False),
    "list full to the brim and past it": lambda: W.random_small(150, 0.5, 2, seed=5),
    "sweeps": lambda: layered(4, 40),
    "2048 levels": lambda: W.path_graph(2048),
    "2049 levels": lambda: W.path_graph(2049, directed=True),
    "2500 levels": lambda: W.path_graph(2500),
    "more hubs than the queue holds": lambda: hub_row(300, 64, 700),
    "65 arcs a hub": lambda: hub_row(300, 65, 700),
    "heaviest hubs taken with others": lambda: hub_row(200, 256, 700),
    "lightest hubs in chunks, list full": lambda: hub_row(130, 257, 700),
    "more chunks than the heavy list holds": lambda: hub_row(200, 400, 700),
    "no arc at all": lambda: W.Graph(130, True, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int64)),
    "one heavy weight": lambda: W.Graph(3, True, np.array([0, 1, 0], np.int32), np.array([1, 2, 2], np.int32),
                                        np.array([1, 2, 2 ** 31 - 2], np.int64)),
    "unit weights": lambda: W.chung_lu_directed(1201, 2.5, 16.0, 1, 9),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_graphs_against_the_oracle(name):
    g = SMALL[name]()
    say(f"static pass: {name}, n={g.n}, m={g.m}")
    ctx = make_ctx(g.n)
    arcs = g.m if g.directed else 2 * g.m
    gr = ctx.load_graph(g, arc_capacity=arcs + 16, estar_capacity=arcs + 16)  # ties can put every arc in E*
    dags = sorted({0, g.n // 2, g.n - 1})
    check_full(gr, g, name, dags=dags, deltas=dags[:1])
    gr.recompute()  # the slots are not cleared in between
    check_full(gr, g, name + ", recomputed", dags=dags)
    gr.recompute_estar()
    check_full(gr, g, name + ", over E*", dags=dags)
    ctx.close()


@pytest.mark.parametrize("n", [18432, 18433, 36864, 36865, 65537])
def test_large_graphs_by_component(n):
    size, dense = 60, layered(3, 190)  # the dense component's sources take the sweeps at the two smaller sizes
    blocks, at, parts = [], 0, []
    while n - at >= max(size, 0) and at < 60 * 40:
        blocks.append((at, W.random_small(size, 0.08, 3, seed=n + at)))
        at += size
    blocks.append((at, dense))
    at += dense.n
    for off, b in blocks:
        parts.append((b.src + off, b.dst + off, b.w))
    g = W.Graph(n, True, *(np.concatenate(x) for x in zip(*parts)))
    g.src, g.dst = g.src.astype(np.int32), g.dst.astype(np.int32)
    say(f"static pass by component: n={n}, m={g.m}")
    ctx = make_ctx(n, slots=300)
    gr = ctx.load_graph(g)
    gr.check()
    bc = gr.scores()
    for off, b in (blocks[0], blocks[17], blocks[-1]):
        ref = oracle.brandes(b)
        assert bc_err(bc[off:off + b.n], ref["bc"]) <= BC_TOL
        D, S = gr.rows(off, 2)
        assert np.array_equal(S[:, off:off + b.n], ref["sigma"][:2])
        assert np.array_equal(D[:, off:off + b.n], ref["D"][:2])
    assert not bc[at:].any()
    ctx.close()

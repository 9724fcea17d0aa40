"""Arcs read back from clones that share the loaded arc list.

New weights are kept beside the shared list, inserted arcs behind it: the arcs
of the graph and of each clone are its own, in the order of the list, and reading
them costs the same whether weights have changed or not.
"""
from __future__ import annotations

import time

import numpy as np
import pytest

from gpu_util import make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def sorted_arcs(g):
    o = np.lexsort((g.dst, g.src))
    return [np.asarray(x)[o].astype(np.int64) for x in (g.src, g.dst, g.w)]


@pytest.mark.parametrize("directed", [True, False])
def test_arcs_of_a_graph_and_its_clones(directed):
    g = W.directed_out_degree(90, 6, 200, 3) if directed else W.gnp_undirected(90, 8.0, 200, 3)
    say(f"clone arcs: directed {directed}")
    ctx = make_ctx(g.n, slots=16)
    pairs = [[ctx.load_graph(g), g]]
    for k in range(3):  # the graph and two clones, each with a stream of its own
        for i, p in enumerate(pairs):
            # the lowest and the highest arc of the list among the changes
            order = np.lexsort((p[1].dst, p[1].src))
            ends = [W.Update("edge", u=int(p[1].src[e]), v=int(p[1].dst[e]), w=int(p[1].w[e]) - 1)
                    for e in (order[0], order[-1]) if p[1].w[e] > 1]
            for up in ends + W.mixed_stream(p[1], 5, 200, 10 * k + i, 0.4, 0.6, 4):
                if up.kind == "edge" and ends and (up.u, up.v) in {(e.u, e.v) for e in ends} and up not in ends:
                    continue
                p[0].update(up)
                p[1] = W.apply_update(p[1], up)
        for gr, cur in pairs:
            a = gr.arcs()
            assert all(np.array_equal(x, y) for x, y in zip(sorted_arcs(a), sorted_arcs(cur)))
        if k < 2:
            pairs.append([pairs[k][0].clone(), pairs[k][1]])
    ctx.close()


def test_time_to_read_arcs_of_a_clone():
    n = 2048
    g = W.complete_undirected(n, n * n, 1)
    ctx = make_ctx(n)
    gr = ctx.load_graph(g)
    clone = gr.clone()

    def best(x):
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            x.arcs()
            t.append(time.perf_counter() - t0)
        return min(t)

    plain = best(gr)
    for up in W.mixed_stream(g, 8, n * n, 3, 0.0, 0.5, 32):
        clone.update(up)
    changed = best(clone)
    say(f"clone arcs: {plain * 1e3:.2f} ms, with new weights {changed * 1e3:.2f} ms")
    assert changed < 2 * plain
    ctx.close()

"""Errors that no call has read before the work slots are used again.

An update overflows, and the next static pass comes before any call reads the
graph's status: of the same graph once its state fits again, or of another graph
on the same context, or after the failed graph is gone.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu

SIDE = 35  # C(68, 34) paths between the corners of a 35 x 35 grid: more than 2^64 - 1


def grid() -> tuple[W.Graph, W.Update, W.Update]:
    """Arcs right and down, the last one too heavy to count; the update that lowers it, and one
    that makes every count fit again."""
    i = np.arange(SIDE * SIDE).reshape(SIDE, SIDE)
    src = np.concatenate([i[:, :-1].ravel(), i[:-1, :].ravel()]).astype(np.int32)
    dst = np.concatenate([i[:, 1:].ravel(), i[1:, :].ravel()]).astype(np.int32)
    w = np.ones(src.size, np.int64)
    n = SIDE * SIDE
    last = (src == n - 1 - SIDE) & (dst == n - 1)
    w[last] = 2
    g = W.Graph(n, True, src, dst, w)
    return g, W.Update("edge", u=n - 1 - SIDE, v=n - 1, w=1), W.Update("edge", u=0, v=n - 1, w=1)


@pytest.mark.parametrize("via", ["plain", "submit"])
def test_recomputed_before_the_error_is_read(via):
    g, over, fits = grid()
    say(f"unread error: recompute, {via}")
    ctx = make_ctx(g.n, slots=16)
    gr = ctx.load_graph(g)
    for up in (over, fits):
        gr.update(up) if via == "plain" else ctx.submit([(gr, up)])
        g = W.apply_update(g, up)
    gr.recompute()
    check_full(gr, g, "recomputed", dags=(0, 1))
    more = W.Update("edge", u=2, v=g.n - 1, w=1)
    gr.update(more)
    check_full(gr, W.apply_update(g, more), "and updated", dags=(0, 2))
    ctx.close()


@pytest.mark.parametrize("freed", [False, True])
@pytest.mark.parametrize("n", [300, 1500])  # below and above the failed graph's size
def test_another_graph_loaded_before_the_error_is_read(n, freed):
    g, over, _ = grid()
    other = W.directed_out_degree(n, 16, 1, 3)
    say(f"unread error: load of {n}, freed {freed}")
    ctx = make_ctx(max(g.n, n), slots=16)
    gr = ctx.load_graph(g)
    gr.update(over)
    if freed:
        gr.free()
    o = ctx.load_graph(other)
    check_full(o, other, "loaded", dags=(0, n - 1))
    up = W.Update("vertex", v=3, edges=[(a, 3, 1) for a in (5, 9, 11) if (a, 3) not in
                                        set(zip(other.src.tolist(), other.dst.tolist()))])
    o.update(up)
    check_full(o, W.apply_update(other, up), "and updated", dags=(0, 5))
    ctx.close()

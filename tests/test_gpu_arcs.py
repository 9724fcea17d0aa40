"""The host's arc lists: loads from arcs in any order, and the list a graph
shares with its clones while both are updated (new weights beside the list,
inserted arcs, a recompute that folds them in, the clone freed)."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, make_ctx
from paper_1311_2147_amd import bcinc
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def _arcs(x):
    a, b, w = np.asarray(x.src), np.asarray(x.dst), np.asarray(x.w)
    if not x.directed:
        a, b = np.minimum(a, b), np.maximum(a, b)
    return sorted(zip(a.tolist(), b.tolist(), w.tolist()))


@pytest.mark.parametrize("directed", [True, False])
def test_loads_from_arcs_in_any_order(directed):
    g = W.random_small(90, 0.3, 40, seed=8, directed=directed)
    order = np.random.default_rng(1).permutation(g.m)
    src, dst = g.src[order], g.dst[order]
    if not directed:  # an edge may name its ends in either order
        src, dst = np.where(order % 2, dst, src), np.where(order % 2, src, dst)
    ctx = make_ctx(90)
    gr = ctx.load_graph(W.Graph(90, directed, src.astype(np.int32), dst.astype(np.int32), g.w[order]))
    check_full(gr, g, "permuted arcs")
    assert _arcs(gr.arcs()) == _arcs(g)
    twice = W.Graph(90, directed, np.append(src, dst[0] if not directed else src[0]).astype(np.int32),
                    np.append(dst, src[0] if not directed else dst[0]).astype(np.int32), np.append(g.w, 5))
    with pytest.raises(bcinc.BcError) as e:
        ctx.load_graph(twice)
    assert e.value.name == "BC_ERR_DUPLICATE_EDGE"
    ctx.close()


@pytest.mark.parametrize("directed", [True, False])
def test_a_list_shared_with_clones(directed):
    g0 = W.random_small(80, 0.2, 40, seed=2, directed=directed)
    ctx = make_ctx(80)
    gr = ctx.load_graph(g0)
    twin = gr.clone()
    state = {gr: g0, twin: g0}

    def step(x, seed):
        for up in W.mixed_stream(state[x], 6, 40, seed, 0.3, 0.4, 5):
            x.update(up)
            state[x] = W.apply_update(state[x], up)
        assert _arcs(x.arcs()) == _arcs(state[x])

    step(gr, 1)
    step(twin, 2)
    third = twin.clone()  # of a list with new weights beside it
    state[third] = state[twin]
    step(third, 3)
    step(twin, 4)
    twin.recompute()  # folds its own changes into a list of its own
    step(twin, 5)
    with pytest.raises(bcinc.BcError) as e:  # not below the current weight, which only the overlay holds
        a, b, w = next(iter(zip(state[gr].src, state[gr].dst, state[gr].w)))
        gr.update_edge(int(a), int(b), int(w))
    assert e.value.name == "BC_ERR_NOT_INCREMENTAL"
    third.free()
    step(gr, 6)
    for x in (gr, twin):
        check_full(x, state[x], "after the stream")
        x.recompute()
        check_full(x, state[x], "recomputed")
    ctx.close()

"""Changed targets' new predecessors (Alg 2) for updates with several in-arcs
and out-arcs: vertex updates and undirected arcs, where the row of v'' is formed
from the rows of the out-arcs' heads and v may get its new in-arcs from one or
several tails.  Ties (weights 1 and 2) and spread weights, sources kept in LDS
and sent through the wide kernel (paired and whole); every stored predecessor is
compared with the oracle's DAGs after each update.
"""
from __future__ import annotations

import pytest

from gpu_util import check_full, check_preds, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sch", [{}, {"big_b": 1, "wide_stage": 1, "wide_block": 1024, "block": 128, "table": 128}])
@pytest.mark.parametrize("w_max", [2, 1000])
@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("k", [2, 9])
def test_predecessors_of_vertex_updates(directed, w_max, k, sch):
    g = W.random_small(130, 0.05, w_max, seed=17 + k, directed=directed)
    ups = W.mixed_stream(g, 10, w_max, k, 0.2, 0.2, k)
    say(f"alg2: directed={directed} w_max={w_max} k={k} {sch}")
    ctx = make_ctx(g.n, slots=16)
    if sch:
        ctx.set_schedule(**sch)
    gr = ctx.load_graph(g)
    for i, up in enumerate(ups):
        gr.update(up)
        g = W.apply_update(g, up)
        check_preds(gr, g, range(g.n), f"#{i}")
    check_full(gr, g, "end", dags=(0, g.n - 1))
    ctx.close()

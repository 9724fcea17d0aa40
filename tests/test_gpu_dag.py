"""The DAG kernel's paths by the size of a source's sub-DAG.

A chain into one or two hubs with many leaves: lowering or inserting an arc in
front of a hub changes the hub and its leaves for every source on the chain.
Leaf counts go over the union walk's bound (3/8 of the table's slots), the
table's vertex capacity, and with the chain over what the accumulation in LDS
holds (about 650 vertices with the 128-slot table, 1300 with the 256-slot one);
two hubs give every leaf two DAG in-arcs.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def broom(chain: int, hubs: int, leaves: int) -> W.Graph:
    """0 -> 1 -> ... -> chain-1, each arc of weight 2, then `hubs` hubs at weight 9,
    each with an arc of weight 1 to every leaf."""
    src, dst, w = list(range(chain - 1)), list(range(1, chain)), [2] * (chain - 1)
    for h in range(chain, chain + hubs):
        src.append(chain - 1)
        dst.append(h)
        w.append(9)
        for x in range(leaves):
            src.append(h)
            dst.append(chain + hubs + x)
            w.append(1)
    n = chain + hubs + leaves
    return W.Graph(n, True, np.array(src, np.int32), np.array(dst, np.int32), np.array(w, np.int64))


@pytest.mark.parametrize("table", [128, 256])
@pytest.mark.parametrize("hubs", [1, 2])
@pytest.mark.parametrize("chain,leaves", [(6, 40), (6, 47), (6, 48), (6, 94), (6, 95), (6, 96), (30, 191), (4, 630),
                                          (4, 660), (300, 990), (330, 990)])
def test_changed_targets_below_a_hub(chain, leaves, hubs, table):
    g = broom(chain, hubs, leaves)
    last, h = chain - 1, list(range(chain, chain + hubs))
    ups = [W.Update("edge", u=last, v=h[0], w=7),  # one hub nearer: with two hubs the ties go
           W.Update("edge", u=max(0, chain - 3), v=h[-1], w=9),  # a shortcut to the last hub
           W.Update("vertex", v=last, edges=[(last, x, 5) for x in h]),  # equal again
           W.Update("edge", u=0, v=h[0], w=1, insert=True)]
    say(f"dag: chain {chain}, {hubs} hubs, {leaves} leaves, table {table}")
    ctx = make_ctx(g.n, slots=16)
    ctx.set_schedule(big_b=1024, table=table, block=128 if table == 128 else 256)
    gr = ctx.load_graph(g)
    for i, up in enumerate(ups):
        gr.update(up)
        g = W.apply_update(g, up)
        if g.n < 300 or i == len(ups) - 1:
            check_full(gr, g, f"update {i}", dags=(0, last, h[0]))
    ctx.sync()
    ctx.close()

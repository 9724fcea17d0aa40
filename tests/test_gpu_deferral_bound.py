"""How many sources of a step go to the wide kernel before the threshold.

Sources with more than 256 changed targets and at most big_b are deferred while
places last: 128 in a step, whichever of its graphs they belong to, and again in
the next step.  Past the threshold a source is deferred without a place.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu

PLACES = 128


def chain_to_hub(chain: int, leaves: int) -> W.Graph:
    """Every vertex of the chain reaches the hub and its leaves through the chain's end."""
    n = chain + 1 + leaves
    src = list(range(chain)) + [chain] * leaves
    dst = list(range(1, chain + 1)) + list(range(chain + 1, n))
    return W.Graph(n, True, np.array(src, np.int32), np.array(dst, np.int32), np.full(len(src), 9, np.int64))


def lowered(chain: int, w: int) -> W.Update:
    return W.Update("edge", u=chain - 1, v=chain, w=w)


@pytest.mark.parametrize("chain,leaves,want", [(127, 400, 127), (128, 400, 128), (129, 400, 128), (900, 300, 128),
                                               (900, 256, 128), (900, 255, 0), (300, 511, 128), (300, 512, 300)])
def test_one_graph(chain, leaves, want):
    g = chain_to_hub(chain, leaves)  # leaves + 1 changed targets for every source of the chain
    say(f"deferral: {chain} sources, {leaves + 1} targets")
    ctx = make_ctx(g.n)
    gr = ctx.load_graph(g)
    for w in (5, 3):
        gr.update(lowered(chain, w))
        assert gr.stats()["deferred_sources"] == want
        g = W.apply_update(g, lowered(chain, w))
    check_full(gr, g, f"{chain} {leaves}", dags=(0, chain))
    ctx.close()


@pytest.mark.parametrize("shapes", [[(200, 320), (150, 400)], [(100, 300), (20, 500), (300, 280)],
                                    [(60, 300), (50, 480)], [(60, 300), (50, 300)]])
def test_graphs_of_a_step_share_the_places(shapes):
    graphs = [chain_to_hub(*s) for s in shapes]
    say(f"deferral: {shapes} in one step")
    ctx = make_ctx(max(g.n for g in graphs))
    grs = [ctx.load_graph(g) for g in graphs]
    for w in (6, 4, 2):
        ctx.wait(ctx.submit([(gr, lowered(c, w)) for gr, (c, _) in zip(grs, shapes)]))
        deferred = [gr.stats()["deferred_sources"] for gr in grs]
        # a step whose graphs have no more vertices than big_b has no wide kernel
        places = PLACES if max(g.n for g in graphs) > 512 else 0
        assert sum(deferred) == min(places, sum(c for c, _ in shapes)), deferred
        graphs = [W.apply_update(g, lowered(c, w)) for g, (c, _) in zip(graphs, shapes)]
    for gr, g, (c, _) in zip(grs, graphs, shapes):
        check_full(gr, g, str(shapes), dags=(0, c))
    ctx.close()

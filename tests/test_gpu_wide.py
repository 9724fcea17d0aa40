"""Passes of deferred sources: over all of DAG(s) (from an eighth of the row) and
walked back from the changed targets.

Small graphs send every affected source to the wide kernel: a star of changed
targets of every share of the row around the eighth, with the row staged in LDS
or read from memory, with ties (several in-arcs per vertex) up to more DAG arcs
than the record of four per vertex holds.  Large ones lie on both sides of the
size up to which the dependency fits in LDS beside the counts.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, check_sampled, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sch", [{"wide_stage": 1, "wide_block": 1024}, {"wide_stage": 2, "wide_block": 256}])
@pytest.mark.parametrize("n,p,w_max", [(31, 0.2, 3), (64, 0.06, 500), (200, 0.5, 1), (257, 0.03, 1), (700, 0.01, 40)])
def test_every_affected_source_deferred(n, p, w_max, sch):
    g = W.random_small(n, p, w_max, seed=n, directed=True)
    ups = W.mixed_stream(g, 6, w_max, n, 0.5, 0.0, 7)
    say(f"wide: n={n} p={p} w_max={w_max} {sch}")
    ctx = make_ctx(n, slots=16)
    ctx.set_schedule(big_b=1, **sch)
    gr = ctx.load_graph(g, arc_capacity=n * n, estar_capacity=n * n)
    deferred = 0
    for up in ups:
        gr.update(up)
        deferred += gr.stats()["deferred_sources"]
        g = W.apply_update(g, up)
    assert deferred > 0
    check_full(gr, g, f"n={n}", dags=range(0, n, 7))
    ctx.close()


@pytest.mark.parametrize("leaves", [63, 64, 65, 300])
def test_share_of_the_row(leaves):
    """A chain into a hub in a row of 512: from an eighth of it whole-DAG passes."""
    n, chain = 512, 40
    src = list(range(chain)) + [chain] * leaves + list(range(chain + leaves + 1, n - 1))
    dst = list(range(1, chain + 1)) + list(range(chain + 1, chain + 1 + leaves)) + list(range(chain + leaves + 2, n))
    g = W.Graph(n, True, np.array(src, np.int32), np.array(dst, np.int32), np.full(len(src), 3, np.int64))
    say(f"wide: {leaves} leaves of {n}")
    ctx = make_ctx(n, slots=16)
    ctx.set_schedule(big_b=1)
    gr = ctx.load_graph(g)
    for up in [W.Update("edge", u=chain - 1, v=chain, w=1),
               W.Update("vertex", v=chain, edges=[(5, chain, 1), (chain, n - 1, 2)])]:
        gr.update(up)
        g = W.apply_update(g, up)
        check_full(gr, g, f"{leaves} leaves", dags=(0, 5, chain))
    ctx.close()


@pytest.mark.parametrize("n", [11000, 11500])
def test_dependency_in_lds_and_out_of_it(n):
    g = W.directed_out_degree(n, 4, 20, seed=n)
    hub = W.Update("vertex", v=7, edges=[(a, 7, 1) for a in range(100, 110)] + [(7, b, 1) for b in range(200, 230)])
    say(f"wide: n={n}")
    ctx = make_ctx(n)
    gr = ctx.load_graph(g)
    have = set(zip(g.src.tolist(), g.dst.tolist()))
    hub.edges = [e for e in hub.edges if e[:2] not in have]
    gr.update(hub)
    st = gr.stats()
    g = W.apply_update(g, hub)
    assert st["deferred_sources"] > 0
    check_sampled(gr, g, [7, 100, 101, 109, 0, n - 1], f"n={n}")
    ctx.close()


@pytest.mark.parametrize("chain,leaves", [(200, 320), (100, 500), (330, 256), (330, 255)])
def test_sources_deferred_before_the_threshold(chain, leaves):
    """A chain into a hub: every source on it gets leaves + 1 changed targets, more than 256 and
    fewer than big_b; of these at most about 128 go to the wide kernel, with the rest listed."""
    n = chain + 1 + leaves
    src = list(range(chain)) + [chain] * leaves
    dst = list(range(1, chain + 1)) + list(range(chain + 1, n))
    g = W.Graph(n, True, np.array(src, np.int32), np.array(dst, np.int32), np.full(len(src), 9, np.int64))
    say(f"wide: {chain} sources with {leaves + 1} changed targets")
    ctx = make_ctx(n, slots=16)
    gr = ctx.load_graph(g)
    for up in [W.Update("edge", u=chain - 1, v=chain, w=4),
               W.Update("vertex", v=chain, edges=[(chain - 1, chain, 3), (chain, n - 1, 2)])]:
        gr.update(up)
        deferred = gr.stats()["deferred_sources"]
        g = W.apply_update(g, up)
        check_full(gr, g, f"{chain} {leaves}", dags=(0, chain - 1, chain))
        if n > 512:
            assert (0 < deferred <= chain) if leaves + 1 > 256 else deferred == 0
    ctx.close()

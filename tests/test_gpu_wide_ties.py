"""Deferred sources whose DAG has more arcs than a whole-DAG pass records.

A chain leads into a core with many ties and, by an arc that the updates lower, to
a hub with leaves: the changed targets are the hub and its leaves, shares of the
row on both sides of an eighth and of a half, while the core's arcs fill the
record of four per vertex, overfill it by a little or by far, with E* on both
sides of sixteen arcs per vertex (from there a sample decides whether the record
is begun).
"""
from __future__ import annotations

import time

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def comet(chain: int, core: int, degree: int, leaves: int, w_max: int) -> W.Graph:
    """core vertices, then the chain, the hub and the leaves."""
    g = W.directed_out_degree(core, degree, w_max, core + degree)
    c = np.arange(core, core + chain)
    hub = core + chain
    src = np.concatenate([g.src, c[:-1], [c[-1], c[-1]], np.full(leaves, hub)])
    dst = np.concatenate([g.dst, c[1:], [0, hub], np.arange(hub + 1, hub + 1 + leaves)])
    w = np.concatenate([g.w, np.full(chain - 1, 2), [1, 900], np.full(leaves, 3)])
    return W.Graph(hub + 1 + leaves, True, src.astype(np.int32), dst.astype(np.int32), w.astype(np.int64))


def lowered(chain: int, core: int, count: int):
    return [W.Update("edge", u=core + chain - 1, v=core + chain, w=893 - 7 * i) for i in range(count)]


@pytest.mark.parametrize("sch", [{"wide_stage": 1, "wide_block": 256}, {"wide_stage": 2, "wide_block": 512}])
@pytest.mark.parametrize("core,degree,w_max", [(700, 40, 1), (700, 14, 1), (900, 30, 12), (300, 60, 1)])
@pytest.mark.parametrize("share", [(1, 8, -1), (1, 8, 0), (1, 3, 0), (1, 2, -1), (1, 2, 0), (2, 3, 0)])
def test_record_overfilled(share, core, degree, w_max, sch):
    chain = 21
    p, q, more = share
    # hub and leaves: nb = leaves + 1 of n = core + chain + nb
    nb = -(-(core + chain) * p // (q - p)) + more
    g = comet(chain, core, degree, nb - 1, w_max)
    if more <= 0 and share != (2, 3, 0):
        assert (nb * q >= g.n * p) == (more == 0)
    say(f"wide ties: core {core}/{degree}/{w_max}, {nb} of {g.n}, {sch}")
    ctx = make_ctx(g.n, slots=16)
    ctx.set_schedule(big_b=1, **sch)
    gr = ctx.load_graph(g)
    for i, up in enumerate(lowered(chain, core, 2)):
        gr.update(up)
        assert gr.stats()["deferred_sources"] == chain
        g = W.apply_update(g, up)
    check_full(gr, g, f"{nb} of {g.n}", dags=(core, core + chain - 1))
    ctx.close()


def test_time_does_not_follow_the_core():
    """Updates that change a quarter of the row, far from the core: a dense core costs no more than a
    thin one by much (with a sweep over all of E* per source it takes eleven times as long)."""
    def best(degree):
        chain, core = 300, 3000
        g = comet(chain, core, degree, 1024, 1)
        ctx = make_ctx(g.n)
        gr = ctx.load_graph(g)
        t = []
        for _ in range(4):
            copy = gr.clone()
            ctx.sync()
            t0 = time.perf_counter()
            for up in lowered(chain, core, 8):
                copy.update(up)
            ctx.sync()
            t.append(time.perf_counter() - t0)
            copy.free()
        ctx.close()
        return min(t)

    dense, thin = best(64), best(3)
    say(f"wide ties: dense core {dense * 1e3:.1f} ms, thin core {thin * 1e3:.1f} ms")
    assert dense < 5 * thin

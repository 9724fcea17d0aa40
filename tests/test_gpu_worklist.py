"""How a step's sources are shared out over the persistent workgroups.

Each workgroup's first source is dealt by its index, the others come from a
counter, and the segments (one or two per job) are looked up 64 at a time.
The cases cross those edges: fewer and more workgroups than sources, more than
64 and more than 128 segments, and deferred sources that run as pairs of units
up to the number of item regions.  Every graph is compared with the oracle.
"""
from __future__ import annotations

import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots,count,big_b", [(1, 70, 512), (2, 70, 1), (5, 3, 1), (300, 130, 1), (0, 70, 512)])
def test_sources_of_many_jobs_are_all_taken(slots, count, big_b):
    say(f"worklist: slots {slots}, {count} graphs, deferral above {big_b}")
    ctx = make_ctx(32, slots=slots)
    ctx.set_schedule(big_b=big_b)
    graphs = [W.random_small(17 + i % 13, 0.2, 6, seed=1000 + i, directed=i % 3 != 0) for i in range(count)]
    streams = [W.mixed_stream(g, 2, 6, 50 + i, 0.4, 0.3, 3) for i, g in enumerate(graphs)]
    loaded = [ctx.load_graph(g) for g in graphs]
    ctx.submit([(gr, up) for gr, ups in zip(loaded, streams) for up in ups])
    ctx.sync()
    for i, (gr, g, ups) in enumerate(zip(loaded, graphs, streams)):
        for up in ups:
            g = W.apply_update(g, up)
        check_full(gr, g, f"graph {i}", dags=(0,))
    ctx.close()

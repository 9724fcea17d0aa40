"""A clone takes over what outlives a call: sizes whose ranges end inside one
thread's 16 bytes, one workgroup's loads or none, and one past the size from
which the copy goes around the caches.  The clone and its source are compared
right after, then updated apart, recomputed and compared with the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, check_sampled, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 63, 65, 513, 2897])
def test_clone_matches_and_goes_its_own_way(n):
    g = W.cycle_graph(n, directed=True) if n < 5 else W.random_small(n, min(0.3, 6.0 / n), 30, seed=n, directed=True)
    say(f"clone: n={n}")
    ctx = make_ctx(n, slots=16)
    gr = ctx.load_graph(g)
    first = None
    if n > 5:
        first = W.mixed_stream(g, 2, 30, n, 0.5, 0.0, 4)
        for up in first:
            gr.update(up)
            g = W.apply_update(g, up)
    twin = gr.clone()
    for a, b in zip(gr.rows(0, min(n, 64)), twin.rows(0, min(n, 64))):
        assert np.array_equal(a, b)
    assert np.array_equal(gr.scores(), twin.scores())
    assert all(np.array_equal(a, b) for a, b in zip(gr.estar(), twin.estar()))
    if n > 5:
        h = g
        for up in W.mixed_stream(g, 3, 30, n + 1, 0.5, 0.0, 4):
            twin.update(up)
            h = W.apply_update(h, up)
        (check_full if n < 1000 else check_sampled)(twin, h, *([] if n < 1000 else [[0, 1, n - 1]]), "the clone")
        twin.recompute()
        (check_full if n < 1000 else check_sampled)(twin, h, *([] if n < 1000 else [[0, 1, n - 1]]), "recomputed")
    (check_full if n < 1000 else check_sampled)(gr, g, *([] if n < 1000 else [[0, 1, n - 1]]), "the source")
    ctx.close()

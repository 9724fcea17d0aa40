"""The union walk's accumulation where one push completes several vertices.

Layers of equal weights, every vertex of one with an arc to every vertex of the
next: all vertices of a layer are complete at once, so the lanes of every wave
list vertices for the next round while other waves start on this one.  Waves of
one workgroup have to agree on where the round ends, hence the block sizes.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import check_full, make_ctx, say
from paper_1311_2147_amd import workloads as W

pytestmark = pytest.mark.gpu


def layers(chain: int, count: int, width: int) -> W.Graph:
    """0 -> ... -> chain-1 by arcs of weight 2, the last to every vertex of the first layer by
    weight 7, then `count` layers of `width` vertices joined by arcs of weight 3."""
    src, dst, w = list(range(chain - 1)), list(range(1, chain)), [2] * (chain - 1)
    for x in range(width):
        src.append(chain - 1)
        dst.append(chain + x)
        w.append(7)
    for k in range(count - 1):
        for a in range(width):
            for b in range(width):
                src.append(chain + k * width + a)
                dst.append(chain + (k + 1) * width + b)
                w.append(3)
    return W.Graph(chain + count * width, True, np.array(src, np.int32), np.array(dst, np.int32),
                   np.array(w, np.int64))


@pytest.mark.parametrize("block", [64, 128, 192, 256])
@pytest.mark.parametrize("count,width", [(2, 2), (3, 9), (4, 11), (2, 20), (7, 4)])
def test_many_vertices_complete_at_once(count, width, block):
    chain = 12
    g = layers(chain, count, width)
    first = chain
    ups = [W.Update("edge", u=chain - 1, v=first, w=5),
           W.Update("vertex", v=chain - 1, edges=[(chain - 1, first + x, 4) for x in range(width)]),
           W.Update("vertex", v=g.n - 1, edges=[(chain - 4, g.n - 1, 6 + 4 + 3 * (count - 1)), (0, g.n - 1, 1)]),
           W.Update("edge", u=0, v=chain - 1, w=1, insert=True)]
    say(f"union: {count} layers of {width}, block {block}")
    ctx = make_ctx(g.n, slots=16)
    ctx.set_schedule(table=256, block=block)
    gr = ctx.load_graph(g)
    for i, up in enumerate(ups):
        gr.update(up)
        g = W.apply_update(g, up)
        check_full(gr, g, f"update {i}", dags=(0, chain - 1, first))
    ctx.sync()
    ctx.close()

"""The heightfield's height range, which bounds the walk of its cells, formed
by one workgroup (up to 64x64 heights) or in parts (more): a flat pass first,
then heights with a plateau or a pit at one end of the array, against the FP64
oracle.  Rays miss whatever a range left out."""
import numpy as np
import pytest

from gpu_common import GpuRun, matched_paths, maxrel
from oracle import oracle as O
from paper_2609_32920_amd import lt
from test_gpu_heightfield import hf_only_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [2, 3, 64, 65, 200])
@pytest.mark.parametrize("end", ["first", "last"])
@pytest.mark.parametrize("level", [0.15, -0.15])
def test_ends_of_the_heights_are_in_the_range(G, end, level):
    sc = hf_only_scene(G=G, width=24, height=24)
    h = np.zeros((G, G))
    rows = max(1, G // 8)  # an eighth of the surface: 6% of the paths and more meet it
    h[:rows] = level
    if end == "last":
        h = h[::-1]
    sc = dict(sc, heights=np.ascontiguousarray(h).reshape(-1))
    g = GpuRun(sc)
    g.set_params(heights=np.zeros(G * G))
    g.trace(3, 4096, 2)
    g.set_params(heights=sc["heights"])
    n, depth = 1 << 14, 2
    mask, ids, mismatch = matched_paths(sc, g, 7, n, depth)
    assert mismatch <= 2e-3  # a path a side of a cell's edge, as in the other heightfield tests
    got, want = g.trace(7, n, depth, mask=mask)["image"], O.render(sc, 7, n, depth, path_list=ids)["image"]
    assert maxrel(got, want) <= 1e-4


def test_range_of_every_part_in_a_batch():
    """Instances above and below the size at which the range is formed in parts, in one table."""
    import torch
    insts, runs = [], []
    for G in (16, 64, 65, 130):
        h = np.zeros((G, G))
        h[-(G // 8):] = 0.15
        g = GpuRun(dict(hf_only_scene(G=G, width=24, height=24), heights=h.reshape(-1)))
        new = lambda *s: torch.zeros(s, device=g.dev)
        insts.append(dict(ctx=g.ctx, seed=7, n_paths=20000, depth=2, attached=False, albedo=g.albedo, Le=g.Le,
                          heights=g.heights, guide=None, target=new(24, 24, 3), image=new(24, 24, 3), d_image=new(24, 24, 3),
                          loss=new(1), g_albedo=torch.zeros_like(g.albedo), g_Le=torch.zeros_like(g.Le), g_heights=None))
        runs.append(g)
    b = lt.Batch(0)
    for graph in (False, True, True):
        b.step(insts, use_graph=graph)
        torch.cuda.synchronize()
        for q, g in zip(insts, runs):
            want = GpuRun(g.sc).trace(7, 20000, 2)["image"]
            assert maxrel(q["image"].cpu().numpy(), want) <= 1e-5  # the same terms in another order


@pytest.mark.parametrize("G", [64, 96])
def test_range_follows_the_heights_in_a_graph(G):
    """A captured forward replayed after its heights have changed in place,
    lower and higher, with eager passes between."""
    import torch
    g = GpuRun(hf_only_scene(G=G, width=24, height=24))
    n = 20000
    con, img = torch.zeros(n, device=g.dev), torch.zeros((24, 24, 3), device=g.dev)
    a, p = g.ctx.args(7, n, 2, contrib=con), g.params()
    g.ctx.trace(a, p, img)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.ctx.trace(a, p, img)
    for level in (0.2, -0.2, 0.0, 0.3):
        h = torch.zeros((G, G), device=g.dev)
        h[: G // 8] = level
        h[-(G // 8):] = -0.5 * level
        g.heights.copy_(h.reshape(g.heights.shape))
        con.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        fresh = GpuRun(dict(g.sc, heights=h.cpu().numpy().astype(np.float64).reshape(-1)))
        want = torch.zeros(n, device=g.dev)
        fresh.ctx.trace(fresh.ctx.args(7, n, 2, contrib=want), fresh.params(), img)
        torch.cuda.synchronize()
        assert torch.equal(con, want) and float(want.max()) > 0.0
        g.trace(5, 4096, 2)

"""The heightfield's slopes, differenced once a pass, against a normal map that
holds the same differences: every path the same, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import GpuRun
from paper_2609_32920_amd import lt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [2, 3, 17, 64])
def test_slopes_of_the_heights(G):
    sc = scenes.caustic_scene(G=G, width=24, height=20)
    h = np.random.default_rng(G).uniform(-0.02, 0.02, size=(G, G)).astype(np.float32)
    dx = np.float32(sc["hf"]["dx"])
    at = np.arange(G)
    lo, hi = np.maximum(at - 1, 0), np.minimum(at + 1, G - 1)
    step = (hi - lo).astype(np.float32) * dx
    nm = np.stack([(h[:, hi] - h[:, lo]) / step[None, :], (h[hi] - h[lo]) / step[:, None]], axis=-1)
    g = GpuRun(sc)
    heights = torch.as_tensor(h, device=g.dev).reshape(g.heights.shape)
    nmap = torch.as_tensor(np.ascontiguousarray(nm, np.float32), device=g.dev)

    def contrib(m):
        con = torch.full((20000,), -1.0, device=g.dev)
        img = torch.empty((20, 24, 3), device=g.dev)
        g.ctx.trace(g.ctx.args(5, 20000, 5, 0, contrib=con), g.ctx.params(g.albedo, g.Le, heights, normal_map=m), img)
        torch.cuda.synchronize()
        return con

    with_map, without = contrib(nmap), contrib(None)
    assert torch.equal(with_map, without)
    assert float(without.max()) > 0.0

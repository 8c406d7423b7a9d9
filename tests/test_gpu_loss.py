"""The loss and its adjoint around the size from which it takes more workgroups."""
import pytest
import torch

from gpu_common import GpuRun
from paper_2609_32920_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(20 << 20) - 1, (20 << 20) + 1, 40000003])
def test_large_loss(n):
    g = GpuRun(scenes.box_scene(8, 8))
    gen = torch.Generator(device=g.dev).manual_seed(n)
    for _ in range(2):
        i, t = (torch.rand(n, device=g.dev, generator=gen) for _ in range(2))
        d, loss = torch.full_like(i, 9.0), torch.empty(1, device=g.dev)
        g.ctx.loss_l2(i, t, d, loss)
        torch.cuda.synchronize()
        x = i.double() - t.double()
        want = float((x * x).mean())
        assert abs(float(loss) - want) <= 1e-7 * want  # FP64 sums, one rounding to FP32
        assert torch.equal(d, (2.0 * x / n).float())

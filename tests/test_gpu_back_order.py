"""2D batches of 224 MiB and more whose column tiles run backwards: every image
against the oracle, with whole and broken rounds of tiles, both directions."""
import numpy as np
import pytest

import oracle
from gpu_util import TOL_FP32, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,batch", [(1024, 28), (1024, 29), (128, 227)])
def test_large_batches(nx, batch):
    import torch

    import paper_1203_4938_amd as dp
    g = torch.Generator(device="cuda").manual_seed(nx + batch)
    x = torch.view_as_complex(torch.rand(batch, 1024, nx, 2, generator=g, device="cuda") * 2 - 1)
    p = dp.Plan(shape=(1024, nx), batch=batch, rank=2)
    y = p.exec(x)
    z = p.exec(y, inverse=True)
    ey = ez = 0.0
    for i in range(batch):
        h = x[i : i + 1].cpu().numpy()
        ey = max(ey, oracle.rel_l2_f32(y[i : i + 1].cpu().numpy(), oracle.fft2d(h)).max())
        ez = max(ez, oracle.rel_l2_f32(z[i : i + 1].cpu().numpy(), h.astype(np.complex128)).max())
    say(f"[back] {p.describe()} forward {ey:.3e} round trip {ez:.3e}")
    assert ey <= TOL_FP32 and ez <= TOL_FP32

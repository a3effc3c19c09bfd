"""Long real signals whose four-step passes pair the bins in their tiles: every
split the planner makes (512 and 1024-point paired lines, equal and unequal
sides), batches whose tiles fill the persistent grid unevenly, both ways of reading
the intermediate (from 128 MiB on: 129 x 2^18, 65 x 2^20), both directions
against the oracle, and the imaginary parts of bins 0 and N/2 ignored."""
import numpy as np
import pytest

import oracle
from gpu_util import TOL_FP32, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lg,batch", [(18, 17), (19, 8), (19, 11), (20, 5), (21, 3), (22, 1), (22, 2),
                                      (18, 129), (20, 65)])
def test_paired_passes(lg, batch):
    import torch

    import paper_1203_4938_amd as dp
    n = 1 << lg
    x = np.random.default_rng(lg * 100 + batch).uniform(-1, 1, (batch, n)).astype(np.float32)
    p = dp.Plan(n, batch, real=True)
    say("[real paired]", p.describe().replace("\n", " | "))
    assert p.num_steps() == 2 and "pairing in the tiles" in p.describe()
    spec = p.exec(torch.from_numpy(x).cuda())
    ref = oracle.fft_batch(x.astype(np.complex64))[:, : n // 2 + 1]
    ef = oracle.rel_l2_f32(spec.cpu().numpy(), ref)
    half = torch.from_numpy(ref.astype(np.complex64)).cuda()
    torch.view_as_real(half)[:, 0, 1] = 3.0
    torch.view_as_real(half)[:, n // 2, 1] = -2.0
    back = p.exec(half, inverse=True)
    eb = oracle.rel_l2_f32(back.cpu().numpy().astype(np.complex64), x.astype(np.complex128))
    say(f"   forward max {ef.max():.3e} inverse max {eb.max():.3e}")
    assert ef.max() <= TOL_FP32 and eb.max() <= TOL_FP32


@pytest.mark.parametrize("lg,batch", [(17, 64), (23, 1)])
def test_other_lengths_keep_the_pairing_launch(lg, batch):
    import paper_1203_4938_amd as dp
    p = dp.Plan(1 << lg, batch, real=True)
    assert p.num_steps() == 3 and "real_pairs:" in p.describe()

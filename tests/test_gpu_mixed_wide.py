"""GPU parity of the wide runtime-radix passes (radices 6, 10, 12, 14, 15, 18,
20, 21, 24, 25) alone, in every position and with partly idle threads; of the
four-step twiddles after each kind of last pass; and of the real rows that
pair their bins in LDS.  Against the FP64 oracle, rel L2 <= 1e-5 per signal."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL_FP32, max_rel, run_plan, say, to_dev

pytestmark = pytest.mark.gpu

#: each radix alone; two passes of near-equal and of very different radices;
#: three and four passes; lengths around the 256-thread limit
ROWS = [10, 14, 18, 20, 21, 24, 30, 42, 50, 150, 196, 225, 245, 250, 252, 400, 441, 500, 576, 625,
        720, 735, 960, 1500, 1890, 3000, 3750, 4050, 4200, 5000, 9261, 10584, 13824, 16200]


@pytest.mark.parametrize("order", [0, 1])
def test_rows(order, monkeypatch):
    import paper_1203_4938_amd as dp
    monkeypatch.setenv("DPFFT_FORCE_PLAN", f"o={order}")
    for n in ROWS:
        batch = 13
        x = synth.uniform_complex(synth.BASE_SEED + 520 + n % 89, n, batch)
        p = dp.Plan(n, batch)
        xd = to_dev(x)
        for inv in (False, True):
            e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(),
                        oracle.fft_batch(x, inverse=inv))
            say(f"[wide rows] {p.describe().splitlines()[1].strip()} inverse={inv}: {e:.3e}")
            assert e <= TOL_FP32, (n, inv, e)


@pytest.mark.parametrize("n,batch", [
    (20000, 3), (30870, 2), (59049, 2), (75000, 2), (117649, 1), (300000, 1), (1000000, 1),
    (4000000, 1), (11573604, 1),
])
@pytest.mark.parametrize("order", [0, 1])
def test_four_step(n, batch, order, monkeypatch):
    """Order 1 ends every line with its largest radix (up to 25)."""
    import paper_1203_4938_amd as dp
    monkeypatch.setenv("DPFFT_FORCE_PLAN", f"o={order}")
    x = synth.uniform_complex(synth.BASE_SEED + 620, n, batch)
    p = dp.Plan(n, batch)
    say("[wide four-step]", p.describe().replace("\n", " | "))
    xd = to_dev(x)
    for inv in (False, True):
        e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(), oracle.fft_batch(x, inverse=inv))
        say(f"   inverse={inv}: {e:.3e}")
        assert e <= TOL_FP32, (n, inv, e)


@pytest.mark.parametrize("ny,nx,b", [(3, 2, 5), (5, 4, 3), (7, 6, 3), (9, 50, 4), (6, 1250, 3),
                                     (5, 1920, 3), (1080, 18, 2), (2160, 30, 1), (3, 32400, 2)])
def test_real_rows(ny, nx, b):
    """Half rows of one point, odd lengths (no self-paired middle bin), even
    ones, several lines per workgroup with a ragged last one, the longest."""
    import torch

    import paper_1203_4938_amd as dp
    g = np.random.default_rng(ny * 7919 + nx)
    x = g.uniform(-1, 1, (b, ny, nx)).astype(np.float32)
    p = dp.Plan(shape=(ny, nx), batch=b, rank=2, real=True)
    say("[real rows]", p.describe().replace("\n", " | "))
    spec = p.exec(torch.from_numpy(x).cuda())
    back = p.exec(spec, inverse=True)
    torch.cuda.synchronize()
    ref = oracle.fft2d(x.astype(np.complex64))[:, :, : nx // 2 + 1]
    ef = oracle.rel_l2_f32(spec.cpu().numpy(), ref)
    eb = oracle.rel_l2_f32(back.cpu().numpy().astype(np.complex64), x.astype(np.complex128))
    say(f"   forward max {ef.max():.3e} round trip max {eb.max():.3e}")
    assert ef.max() <= TOL_FP32 and eb.max() <= TOL_FP32


@pytest.mark.parametrize("n", [6, 14, 18, 70, 250, 1000, 9450, 30000, 32400])
def test_real_signals(n):
    """7-smooth real signals, batches from which the bins are paired in LDS."""
    import torch

    import paper_1203_4938_amd as dp
    for batch in (4, 37):
        x = np.random.default_rng(n).uniform(-1, 1, (batch, n)).astype(np.float32)
        p = dp.Plan(n, batch, real=True)
        say("[real signals]", p.describe().replace("\n", " | "))
        assert p.num_steps() == 1 and p.workspace_bytes == 0
        spec = p.exec(torch.from_numpy(x).cuda())
        back = p.exec(spec, inverse=True)
        torch.cuda.synchronize()
        ref = oracle.fft_batch(x.astype(np.complex64))[:, : n // 2 + 1]
        ef = oracle.rel_l2_f32(spec.cpu().numpy(), ref)
        eb = oracle.rel_l2_f32(back.cpu().numpy().astype(np.complex64), x.astype(np.complex128))
        assert ef.max() <= TOL_FP32 and eb.max() <= TOL_FP32, (n, batch, ef.max(), eb.max())


def test_ragged_every_column_length():
    """Four-step signals whose column and row lines take every compile-time
    length, their intermediate rows padded to whole lines."""
    import paper_1203_4938_amd as dp
    lines = [n for n in synth.smooth_sizes(125, 256)]
    sizes = [a * b for a, b in zip(lines, lines[1:] + lines[:1])] + [a * a for a in lines]
    sizes = [n for n in sizes if n > 16384]
    flat, offs = synth.uniform_ragged(synth.BASE_SEED + 805, sizes)
    p = dp.Plan(ragged_sizes=sizes)
    x = to_dev(flat)
    for inv in (False, True):
        y = p.exec(x, inverse=inv).cpu().numpy()
        ref = oracle.fft_ragged(flat, sizes, offs, inverse=inv)
        for n, o in zip(sizes, offs):
            e = np.linalg.norm(y[o:o + n] - ref[o:o + n]) / np.linalg.norm(ref[o:o + n])
            assert e <= TOL_FP32, (n, inv, e)

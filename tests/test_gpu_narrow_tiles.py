"""Few-tile launches: narrow column and transposed-row tiles, as the planner
picks them for small batches and forced on every width, against the oracle
(rel L2 <= 1e-5 per signal or image, both directions)."""
import re

import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL_FP32, max_rel, run_plan, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lg", range(15, 23))
@pytest.mark.parametrize("force", ["", "c0=8 c1=8", "c0=4 c1=4", "c0=2 c1=2"])
def test_four_step(lg, force, monkeypatch):
    import paper_1203_4938_amd as dp
    n, batch = 1 << lg, 1 if lg > 18 else 3
    if force:
        monkeypatch.setenv("DPFFT_FORCE_PLAN", force)
    try:
        p = dp.Plan(n, batch)
    except dp.FftError:
        pytest.skip("no instance of that width")
    say("[narrow]", p.describe().replace("\n", " | "))
    if not force and batch * n < 1 << 20:  # the planner narrows its tiles
        assert all(int(c) <= 8 for c in re.findall(r" C=(\d+)", p.describe()))
    x = synth.uniform_complex(synth.BASE_SEED + 640 + lg, n, batch)
    xd = to_dev(x)
    for inv in (False, True):
        e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(), oracle.fft_batch(x, inverse=inv))
        say(f"   inverse={inv}: {e:.3e}")
        assert e <= TOL_FP32, (n, force, inv, e)


@pytest.mark.parametrize("ny,nx", [(128, 64), (256, 256), (512, 128), (1024, 32), (2048, 16)])
@pytest.mark.parametrize("width", [0, 8, 4])
@pytest.mark.parametrize("real", [False, True])
def test_images(ny, nx, width, real, monkeypatch):
    """2D column tiles; real images end with a tile of one column."""
    import torch

    import paper_1203_4938_amd as dp
    if width:
        # the real inverse runs its columns as its first launch
        monkeypatch.setenv("DPFFT_FORCE_PLAN", f"c1={width} c0={width}" if real else f"c1={width}")
    g = np.random.default_rng(ny + nx)
    try:
        p = dp.Plan(shape=(ny, nx), batch=2, rank=2, real=real)
    except dp.FftError:
        pytest.skip("no instance of that width")
    x = g.uniform(-1, 1, (2, ny, nx)).astype(np.float32)
    if not real:
        x = (x + 1j * g.uniform(-1, 1, x.shape)).astype(np.complex64)
    y = p.exec(torch.from_numpy(x).cuda())
    z = p.exec(y, inverse=True)
    torch.cuda.synchronize()
    ref = oracle.fft2d(x.astype(np.complex64))
    ey = oracle.rel_l2_f32(y.cpu().numpy(), ref[:, :, : nx // 2 + 1] if real else ref)
    ez = oracle.rel_l2_f32(z.cpu().numpy().astype(np.complex64), x.astype(np.complex128))
    say(f"[narrow 2d] {p.describe()} forward {ey.max():.3e} round trip {ez.max():.3e}")
    assert ey.max() <= TOL_FP32 and ez.max() <= TOL_FP32

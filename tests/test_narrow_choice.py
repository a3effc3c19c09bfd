"""When a launch of few tiles takes narrower ones, and what that may cost."""
import re

import numpy as np
import pytest

import synth


def _tiles(**kw):
    """(lines per tile, threads, tiles) of each launch of a plan for 256 CUs."""
    import paper_1203_4938_amd as dp
    d, keep = dp.make_desc(**kw)
    st, text = dp.fft_plan_dry(d)
    assert st == dp.FFT_OK, text
    return [tuple(int(v) for v in m) for m in
            re.findall(r" C=(\d+) threads=(\d+) (?:.*?tiles=|grid=)(\d+)", text)]


@pytest.mark.parametrize("n", [1 << lg for lg in range(15, 22)])
def test_four_step_tiles(n):
    for batch in range(1, 17):
        for C, threads, tiles in _tiles(n=n, batch=batch):
            # narrower than the 16 (2048 points: 8) only while no CU gets two
            if C < (8 if threads // C >= 128 else 16):
                assert tiles <= 256 and threads >= 64, (n, batch, C, threads, tiles)
    for C, threads, tiles in _tiles(n=n, batch=1):  # and as narrow as that allows
        assert C <= 8 or 2 * tiles > 256


@pytest.mark.parametrize("ny,nx,batch,C", [
    (128, 16, 1, 16), (128, 64, 1, 16), (256, 16, 6, 16),  # fewer short columns' tiles than XCDs
    (128, 64, 2, 8), (512, 16, 1, 4), (256, 256, 1, 4), (256, 512, 3, 8),
    (2048, 256, 4, 4), (2048, 256, 6, 8), (2048, 512, 3, 8), (1024, 512, 5, 16),
])
def test_column_tiles(ny, nx, batch, C):
    assert _tiles(rank=2, shape=(ny, nx), batch=batch)[1][0] == C


@pytest.mark.gpu
@pytest.mark.parametrize("lg", [15, 16, 17, 18, 19, 20, 21])
def test_error_of_narrow_signals(lg, monkeypatch):
    """Narrow tiles are as accurate as the wide ones: the same radices (or
    fewer, larger ones in the wide tile) and twiddles that are table entries.
    The error over 2^15 random points and more varies by less than 1%."""
    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import run_plan, say, to_dev
    n = 1 << lg
    x = synth.uniform_complex(synth.BASE_SEED + 870 + lg, n, 2 if lg < 18 else 1)
    xd, ref = to_dev(x), oracle.fft_batch(x)

    def err(force):
        if force:
            monkeypatch.setenv("DPFFT_FORCE_PLAN", force)
        y = run_plan(dp.Plan(n, len(x)), xd).cpu().numpy()
        monkeypatch.delenv("DPFFT_FORCE_PLAN", raising=False)
        return float(np.linalg.norm(y - ref) / np.linalg.norm(ref))

    wide = "c0=16 p0=0 t0={} c1={} p1=0"
    T = 1 << (lg // 2 - 4)  # threads per line of the columns
    narrow, full = err(""), err(wide.format(16 * T, 8 if lg == 21 else 16))
    say(f"[narrow error] 2^{lg}: {narrow:.4e}, wide tiles {full:.4e}")
    assert narrow <= 1.015 * full


@pytest.mark.gpu
@pytest.mark.parametrize("ny,wide", [(128, 16), (256, 16), (512, 16), (1024, 16), (2048, 8)])
def test_error_of_narrow_columns(ny, wide, monkeypatch):
    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import run_plan, say, to_dev
    nx, b = 256, 1
    x = synth.uniform_complex(synth.BASE_SEED + 880, ny * nx, b).reshape(b, ny, nx)
    xd, ref = to_dev(x), oracle.fft2d(x)

    def err(force):
        if force:
            monkeypatch.setenv("DPFFT_FORCE_PLAN", force)
        y = run_plan(dp.Plan(shape=(ny, nx), batch=b, rank=2), xd).cpu().numpy()
        monkeypatch.delenv("DPFFT_FORCE_PLAN", raising=False)
        return float(np.linalg.norm(y - ref) / np.linalg.norm(ref))

    narrow, full = err(""), err(f"c1={wide}")
    say(f"[narrow error] {ny} x {nx}: {narrow:.4e}, wide tiles {full:.4e}")
    assert narrow <= 1.015 * full

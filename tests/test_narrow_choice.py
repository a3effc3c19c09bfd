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

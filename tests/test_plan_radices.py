"""Radix plans of every 7-smooth line length the runtime-radix kernels take:
the passes multiply to the length, every pass's butterflies are owned by the
line's threads, and the workgroup and its LDS fit."""
import re

import pytest

import synth

#: butterflies a thread may own in a pass of each radix
QMAX = {2: 8, 3: 6, 4: 4, 5: 4, 6: 3, 7: 3, 8: 2, 9: 2, 10: 2, 12: 2, 14: 1, 15: 1, 16: 1, 18: 1,
        20: 1, 21: 1, 24: 1, 25: 1}


def _dry(**kw):
    import paper_1203_4938_amd as dp
    d, keep = dp.make_desc(**kw)
    st, text = dp.fft_plan_dry(d)
    assert st == dp.FFT_OK, text
    return text


def _check(line):
    m = re.search(r"L=(\d+) radices=(\S*) passes=(\S*) .*?C=(\d+) threads=(\d+) .*lds=(\d+)B", line)
    L, C, th, lds = (int(m.group(i)) for i in (1, 4, 5, 6))
    for part in (2, 3):
        prod = 1
        for r in filter(None, m.group(part).split("x")):
            prod *= int(r)
        assert prod == L, line
    assert th % C == 0 and th <= 1024 and lds <= 160 * 1024, line
    for r in filter(None, m.group(3).split("x")):
        assert L // int(r) <= th // C * QMAX[int(r)], line


def _lengths():
    return [n for n in synth.smooth_sizes(3, 16384) if n & (n - 1)]


@pytest.mark.parametrize("order", [0, 1])
def test_row_plans(order, monkeypatch):
    monkeypatch.setenv("DPFFT_FORCE_PLAN", f"o={order}")
    for n in _lengths():
        _check(_dry(n=n, batch=7).splitlines()[1])


def test_column_and_real_row_plans():
    import paper_1203_4938_amd as dp
    for n in _lengths():
        for ln in _dry(rank=2, shape=(n, 48), batch=2).splitlines()[1:]:
            _check(ln)
        text = _dry(rank=2, shape=(48, 2 * n), batch=2, flags=dp.FFT_F_REAL)
        for ln in text.splitlines()[1:]:
            if "passes=" in ln:
                _check(ln)


def test_four_step_workspace():
    """The intermediate's rows take whole 128-byte lines, except where only the
    dense one fits the 64 MiB that execution without a workspace offers."""
    for n, n2 in ((59049, 243), (46080, 240), (1000000, 1000), (300000, 600)):
        dense, pad = 8 * n, 8 * (n // n2) * ((n2 + 15) // 16 * 16)
        for b in (1, (64 << 20) // pad, (64 << 20) // dense, (64 << 20) // dense + 1):
            want = dense if b * dense <= 64 << 20 < b * pad else pad
            assert f"workspace={b * want}B" in _dry(n=n, batch=b), (n, b)


def test_ragged_workspace():
    for n, pad in ((59049, 243 * 256), (46080, 46080)):
        for b in (1, (8 << 20) // pad, (8 << 20) // n, (8 << 20) // n + 1):
            want = n if b * n <= 8 << 20 < b * pad else pad
            assert f"workspace={8 * b * want}B" in _dry(ragged_sizes=[n] * b), (n, b)


def test_real_signals_cover_the_batch_once():
    """Real signals of a power of two: one workgroup per C signals."""
    import paper_1203_4938_amd as dp
    for n, batch in ((2, 1000), (128, 19912), (2048, 1447), (32768, 7)):
        text = _dry(n=n, batch=batch, flags=dp.FFT_F_REAL)
        for m in re.finditer(r"real_(?:forward|inverse): .*? C=(\d+) threads=\d+ grid=(\d+)", text):
            assert int(m.group(2)) == -(-batch // int(m.group(1))), text

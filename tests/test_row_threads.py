"""Threads and lines of short rows: no line of 10 or more points on one thread,
whole 256-thread workgroups for batches beyond the last-level cache, and the
rows of images without gaps tiled as one list; then the same plans' results."""
import re

import numpy as np
import pytest

import synth

SHORT = [n for n in synth.smooth_sizes(3, 360) if n & (n - 1)]


def _rows(**kw):
    """(points, lines per workgroup, threads, grid) of the plan's first launch."""
    import paper_1203_4938_amd as dp
    d, keep = dp.make_desc(**kw)
    st, text = dp.fft_plan_dry(d)
    assert st == dp.FFT_OK, text
    m = re.search(r"L=(\d+) .*?C=(\d+) threads=(\d+) grid=(\d+)", text.splitlines()[1])
    return tuple(int(v) for v in m.groups())


def test_threads_of_short_rows():
    for n in SHORT:
        most = 9 if n < 10 else 12 if n <= 48 else 10 if n <= 96 else 14 if n <= 120 else 20
        L, C, threads, _ = _rows(n=n, batch=1000)
        assert L == n and threads % C == 0 and n <= most * (threads // C), n


def test_lines_beyond_the_cache():
    for n in SHORT:
        for points in (1 << 24, (1 << 24) + n):  # 256 MiB in and out, and one line more
            L, C, threads, grid = _rows(n=n, batch=points // n)
            T = threads // C
            large = n * (points // n) > 1 << 24
            assert grid == -(-(points // n) // C)
            if large and T <= 12:
                assert C == 256 // T, (n, C, T)


def test_rows_of_dense_images_are_one_list():
    for ny, nx, b in ((64, 45, 100), (7, 18, 9), (64, 120, 300), (3, 1000, 5)):
        L, C, _, grid = _rows(rank=2, shape=(ny, nx), batch=b)
        assert grid == -(-ny * b // C), (ny, nx, b)
        L, C, _, grid = _rows(rank=2, shape=(ny, nx), batch=b, dist=ny * nx + 3)
        assert grid == b * -(-ny // C), (ny, nx, b)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 9, 10, 12, 14, 15, 18, 20, 21, 24, 25, 27, 28, 48, 49, 56, 60, 96,
                               98, 105, 120, 126, 144, 288, 360])
def test_short_rows(n, monkeypatch):
    """A ragged last workgroup, with the lines of small and of large batches."""
    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import TOL_FP32, max_rel, run_plan, say, to_dev
    batch = 517
    x = synth.uniform_complex(synth.BASE_SEED + 830 + n, n, batch)
    xd = to_dev(x)
    _, C, threads, _ = _rows(n=n, batch=batch)
    for c in (C, 256 // (threads // C)):
        monkeypatch.setenv("DPFFT_FORCE_PLAN", f"c0={c}")
        p = dp.Plan(n, batch)
        for inv in (False, True):
            e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(), oracle.fft_batch(x, inverse=inv))
            say(f"[short rows] n={n} C={c} inverse={inv}: {e:.3e}")
            assert e <= TOL_FP32, (n, c, inv, e)


@pytest.mark.gpu
@pytest.mark.parametrize("ny,nx,b", [(5, 45, 9), (64, 18, 3), (7, 120, 4), (3, 1000, 2)])
@pytest.mark.parametrize("gap", [0, 5])
def test_rows_of_images(ny, nx, b, gap):
    import torch

    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import TOL_FP32
    x = synth.uniform_complex(synth.BASE_SEED + 840 + nx, ny * nx, b)
    D = ny * nx + gap
    buf = torch.zeros(b * D, dtype=torch.complex64, device="cuda")
    for i in range(b):
        buf[i * D:i * D + ny * nx] = torch.from_numpy(x[i]).cuda()
    d, keep = dp.make_desc(rank=2, shape=(ny, nx), batch=b, dist=D if gap else 0)
    st, h = dp.fft_plan(d)
    assert st == dp.FFT_OK, dp.fft_last_error()
    try:
        for inv in (False, True):
            out = torch.full_like(buf, 3.0)
            st = dp.fft_exec(h, buf.data_ptr(), out.data_ptr(),
                             dp.FFT_INVERSE if inv else dp.FFT_FORWARD)
            assert st == dp.FFT_OK, dp.fft_last_error()
            torch.cuda.synchronize()
            y = out.cpu().numpy()
            ref = oracle.fft2d(x.reshape(b, ny, nx), inverse=inv)
            for i in range(b):
                got = y[i * D:i * D + ny * nx].reshape(ny, nx)
                e = np.linalg.norm(got - ref[i]) / np.linalg.norm(ref[i])
                assert e <= TOL_FP32, (inv, i, e)
                if gap and i + 1 < b:
                    assert (y[i * D + ny * nx:(i + 1) * D] == 3.0).all()
    finally:
        dp.fft_destroy(h)


FOUR = [16807, 17496, 21609, 28125, 49000, 59049, 84035, 98415, 117649, 174960, 177147, 300000]


def test_threads_of_transposed_rows():
    """Whole 128-byte lines of the intermediate where the threads are few."""
    import paper_1203_4938_amd as dp
    for n in FOUR:
        for real in (False, True):
            if real and n % 2 == 0:
                continue
            d, keep = dp.make_desc(n=2 * n if real else n, batch=3, flags=dp.FFT_F_REAL if real else 0)
            st, text = dp.fft_plan_dry(d)
            assert st == dp.FFT_OK
            rows = re.findall(r"rows_transposed\S*: L=\d+ .*?C=(\d+) threads=(\d+)", text)
            assert rows
            for C, threads in rows:
                T = int(threads) // int(C)
                assert T >= 64 or T % 16 == 0, (n, T)


@pytest.mark.gpu
@pytest.mark.parametrize("n", FOUR)
def test_transposed_rows(n):
    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import TOL_FP32, max_rel, run_plan, to_dev
    x = synth.uniform_complex(synth.BASE_SEED + 850, n, 3)
    p, xd = dp.Plan(n, 3), to_dev(x)
    for inv in (False, True):
        e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(), oracle.fft_batch(x, inverse=inv))
        assert e <= TOL_FP32, (n, inv, e)


LONG = [n for n in synth.smooth_sizes(3600, 16384) if n & (n - 1)]


def test_threads_of_long_rows():
    """At most four waves to 4096 points; beyond, 16 points per thread where the
    plan of fewer or more threads leaves no more workgroups on a CU."""
    for n in LONG:
        _, C, threads, _ = _rows(n=n, batch=50)
        T = threads // C
        assert T <= 256 or n > 4096, n
        assert T <= 1024
    for n, T in ((3920, 245), (5103, 319), (6561, 411), (7203, 451), (7875, 493), (12005, 751)):
        assert _rows(n=n, batch=50)[1:3] == (1, T)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [3920, 4050, 4116, 5103, 6561, 6912, 7203, 7875, 8000, 10240,
                               12005, 12288, 15309, 16200])
def test_long_rows(n):
    import torch

    import oracle
    import paper_1203_4938_amd as dp
    from gpu_util import TOL_FP32, max_rel, run_plan, to_dev
    x = synth.uniform_complex(synth.BASE_SEED + 860, n, 3)
    p, xd = dp.Plan(n, 3), to_dev(x)
    for inv in (False, True):
        e = max_rel(run_plan(p, xd, inverse=inv).cpu().numpy(), oracle.fft_batch(x, inverse=inv))
        assert e <= TOL_FP32, (n, inv, e)
    r = np.random.default_rng(n).uniform(-1, 1, (5, 2 * n)).astype(np.float32)
    q = dp.Plan(2 * n, 5, real=True)
    spec = q.exec(torch.from_numpy(r).cuda())
    back = q.exec(spec, inverse=True)
    torch.cuda.synchronize()
    ref = oracle.fft_batch(r.astype(np.complex64))[:, : n + 1]
    assert oracle.rel_l2_f32(spec.cpu().numpy(), ref).max() <= TOL_FP32
    assert oracle.rel_l2_f32(back.cpu().numpy().astype(np.complex64), r.astype(np.complex128)).max() <= TOL_FP32

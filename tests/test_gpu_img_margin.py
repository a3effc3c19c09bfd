"""Nearest codewords of vectors with full 24-bit significands whose BF16 pieces
err in favour of the wrong one: the assignment ranks by BF16 products and has
to notice when these do not decide.  The pairs' distances differ by more than
the FP32 products can round, so the FP32 decision is the exact one."""
import numpy as np
import pytest

from gpu_util import say

U = 2.0 ** -24


def _bf16(x):
    """Round to nearest even to 8 significant bits (float32 in and out)."""
    b = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    b = (b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000
    return b.astype(np.uint32).view(np.float32)


def _pieces(x):
    hi = _bf16(x)
    lo = _bf16(x - hi)
    return hi.astype(np.float64), lo.astype(np.float64)


def _mantissas(g, n, sign, lim=3):
    """(n, 15) values 1 + m 2^-7 + sign (2^-8 - t): the high pieces err by
    almost 2^-8, the low ones by up to 2^-17, all in one direction per row."""
    t = g.choice([-2.0 ** -17, -2.0 ** -22, 0.0, 2.0 ** -22, 2.0 ** -17 - 2.0 ** -22, 2.0 ** -17,
                  2.0 ** -17 + 2.0 ** -22, 2.0 ** -16], (n, 1))
    return 1.0 + g.integers(0, lim, (n, 15)) * 2.0 ** -7 + sign * (2.0 ** -8 - t)


def _by_pieces(v, c):
    """D of both codewords from the three products hi hi, hi lo and lo hi."""
    (vh, vl), (ch, cl) = _pieces(v), _pieces(c)
    d = (vh[:, None] * ch + vh[:, None] * cl + vl[:, None] * ch).sum(2)
    return d - 0.5 * (c.astype(np.float64) ** 2).sum(2)


def _pairs(seed, take, a, b):
    """v (take, 16) about a, c (take, 2, 16) about b, both float32: c[:, 0] is
    the nearer one by a sweep of gaps from the FP32 roundings upwards."""
    g = np.random.default_rng(seed)
    count = 10 * take
    f32 = lambda x: np.asarray(x, dtype=np.float32)
    sv, sc = (g.choice([-1, 1], (count, 1)) for _ in range(2))
    v = f32(a * np.concatenate([_mantissas(g, count, sv), g.choice([0.25, 1.0], (count, 1))], 1))
    c = np.empty((count, 2, 16), np.float32)
    # low pieces of opposite signs in the two codewords: the dropped products
    # take from the one what they give to the other; the rest is the same
    m = g.integers(0, 3, (count, 15)) * 2.0 ** -7
    c[:, 0, :15] = f32(b * (m + _mantissas(g, count, sc, 1)))
    c[:, 1, :15] = f32(b * (m + _mantissas(g, count, -sc, 1)))
    # neighbouring or equal high pieces
    c[:, 1, :15] += f32(b * sc * 2.0 ** -7 * g.integers(0, 2, (count, 1)))
    c[:, :, 15] = f32(b * g.choice([0.0625, 0.25, 1.0], (count, 1)))
    v64, c64 = v.astype(np.float64), c.astype(np.float64)
    dist = lambda c64: (v64[:, None] * c64).sum(2) - 0.5 * (c64 * c64).sum(2)
    norm = np.sqrt((c64 * c64).sum(2)).max(1)
    S = np.sqrt((v64 * v64).sum(1)) * norm + 0.5 * norm * norm
    gap = S * U * np.exp(g.uniform(np.log(85.0), np.log(800.0), count))
    # the last component of the second codeword sets its distance
    want = dist(c64)[:, 0] - gap
    part = (v64[:, :15] * c64[:, 1, :15]).sum(1) - 0.5 * (c64[:, 1, :15] ** 2).sum(1)
    z = v64[:, 15]
    with np.errstate(over="ignore", invalid="ignore"):  # (where there is none, no such pair)
        for _ in range(60):  # z c - c^2 / 2 = want - part
            c[:, 1, 15] = f32((want - part + 0.5 * c[:, 1, 15].astype(np.float64) ** 2) / z)
        d = dist(c.astype(np.float64))
    # 17 roundings of each D and 17 of each h, twice over
    norm = np.sqrt((c.astype(np.float64) ** 2).sum(2)).max(1)
    S = np.sqrt((v64 * v64).sum(1)) * norm + 0.5 * norm * norm
    with np.errstate(invalid="ignore"):
        keep = np.flatnonzero(d[:, 0] - d[:, 1] > 80 * U * S)
    # three in four of the pairs: those that the pieces misjudge the most
    p = _by_pieces(v[keep], c[keep])
    worst = np.argsort((p[:, 0] - p[:, 1]) / S[keep], kind="stable")
    pick = keep[np.concatenate([worst[: 3 * take // 4], g.permutation(len(keep))[: take // 4]])]
    return v[pick], c[pick]


def test_pieces_bound():
    """The bounds that the assignment's margin is made of."""
    g = np.random.default_rng(3)
    x = np.concatenate([_mantissas(g, 300, 1).ravel(), _mantissas(g, 300, -1).ravel(),
                        g.uniform(1, 2, 200000)])
    x = x.astype(np.float32)
    hi, lo = _pieces(x)
    x64 = x.astype(np.float64)
    assert (np.abs(x64 - hi) <= 2.0 ** -8 * x64).all() and (np.abs(lo) <= 2.0 ** -8 * x64).all()
    assert (np.abs(x64 - hi - lo) <= 2.0 ** -17 * x64).all()
    assert np.abs(lo / x64).max() > 0.98 * 2.0 ** -8
    assert np.abs((x64 - hi - lo) / x64).max() > 0.98 * 2.0 ** -17


@pytest.mark.gpu
@pytest.mark.parametrize("k", [2, 28, 64])
@pytest.mark.parametrize("a,b", [(256.0, 1.0), (8.0, 1.0), (2.0 ** 20, 8.0), (2.0 ** -9, 2.0 ** -12)])
def test_undecided_pairs(k, a, b):
    _check_pairs(k, a, b)


def _check_pairs(k, a, b):
    import torch

    import paper_1203_4938_amd as dp
    v, c = _pairs(int(k + a + 1 / b), 6000, a, b)
    n = len(v)
    assert n == 6000 and (_by_pieces(v, c)[:, 0] < _by_pieces(v, c)[:, 1]).sum() > 1000
    g = np.random.default_rng(k)
    at = np.stack([g.permutation(k)[:2] for _ in range(n)])  # the pair's places
    cb = np.zeros((n, k, 16), np.float32)
    cb[np.arange(n)[:, None], at] = c
    # one block per image (the other codewords, zero, are far)
    code = dp.img_encode(torch.from_numpy(v.reshape(n, 1, 16)).cuda(),
                         torch.ones(n, 1, device="cuda"), torch.from_numpy(cb).cuda(), 4, 4, 0.5)
    torch.cuda.synchronize()
    bad = int((code.cpu().numpy()[:, 0] != 1 + at[:, 0]).sum())
    # for the record: what the three products alone would take
    d = _by_pieces(v, c)
    say(f"[margin] k={k} a={a:g} b={b:g}: {n} pairs, {int((d[:, 1] > d[:, 0]).sum())} misjudged by "
        f"the pieces, {bad} wrong codes")
    assert bad == 0


@pytest.mark.gpu
@pytest.mark.parametrize("a,b", [(256.0, 2.0 ** -80), (1.0, 2.0 ** -72), (2.0 ** 30, 2.0 ** -70)])
def test_tiny_codewords(a, b):
    """Codewords whose squared norm is zero in FP32."""
    _check_pairs(33, a, b)

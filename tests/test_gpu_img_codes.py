"""Nearest-codeword decisions at the edges of the assignment kernel: codebooks
around its groups of 32 and 64 codewords, block counts that leave rounds and
workgroups partly empty, ties, near ties and magnitudes at which the BF16
ranking decides nothing.  Small integer vectors (times a power of two) make
every product and sum exact in FP32, so the codes must equal the integer
decision, ties to the lower index, without any tolerance."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _codes(dev, act, cb, tau):
    """1 + first maximiser of 2 v.c - |c|^2 (int64), 0 below tau."""
    out = np.zeros(dev.shape[:2], dtype=np.int32)
    for b in range(dev.shape[0]):
        d = 2 * dev[b] @ cb[b].T - (cb[b] * cb[b]).sum(1)
        out[b] = np.where(act[b] >= tau, 1 + d.argmax(1), 0)
    return out


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 128, 129, 255, 256])
@pytest.mark.parametrize("h,w", [(4, 4), (36, 28), (64, 68), (128, 132), (260, 260)])
def test_integer_decisions(k, h, w):
    import torch

    import paper_1203_4938_amd as dp
    g = np.random.default_rng(1000 * k + h)
    nb, B, tau = (h // 4) * (w // 4), 2, 0.25
    for lim, dup, scale in ((9, False, 1.0), (3, True, 1.0), (9, False, 2.0 ** 52),
                            (9, True, 2.0 ** -55)):
        dev = g.integers(-lim, lim + 1, (B, nb, 16)).astype(np.int64)
        cb = g.integers(-lim, lim + 1, (B, k, 16)).astype(np.int64)
        if dup and k > 2:
            cb[:, k // 2:] = cb[:, : k - k // 2]  # every codeword twice
        act = g.uniform(0, 1, (B, nb)).astype(np.float32)
        got = dp.img_encode(torch.from_numpy((dev * scale).astype(np.float32)).cuda(),
                            torch.from_numpy(act).cuda(),
                            torch.from_numpy((cb * scale).astype(np.float32)).cuda(), h, w, tau)
        torch.cuda.synchronize()
        want = _codes(dev, act, cb, tau)
        bad = int((got.cpu().numpy() != want).sum())
        say(f"[codes] k={k} {h}x{w} lim={lim} dup={dup} scale={scale:g}: {bad} differ")
        assert bad == 0


@pytest.mark.parametrize("k,h,w", [(1, 8, 4), (16, 36, 28), (33, 128, 132), (65, 260, 260),
                                   (200, 256, 260)])
def test_cluster_means(k, h, w):
    """One Lloyd iteration on blocks of integer deviations: the means of the
    clusters are quotients of exact integer sums."""
    import torch

    import paper_1203_4938_amd as dp
    g = np.random.default_rng(77 * k + h)
    rgb = np.repeat(g.integers(0, 256, (2, h, w, 1)), 3, axis=3).astype(np.uint8)
    one = dp.img_compress(torch.from_numpy(rgb).cuda(), k, 1, 8.0)
    none = dp.img_compress(torch.from_numpy(rgb).cuda(), k, 0, 8.0)
    torch.cuda.synchronize()
    dev, code = none["dev"].cpu().numpy().astype(np.float64), none["code"].cpu().numpy()
    seeds, means = none["codebook"].cpu().numpy(), one["codebook"].cpu().numpy()
    for b in range(2):
        for c in range(k):
            m = dev[b][code[b] == c + 1]
            want = m.mean(0) if len(m) else seeds[b, c]
            # a sum of n FP32 values of at most 256 rounds by n 2^-24 256 n per term
            tol = max(len(m), 1) * 256 * 2.0 ** -23
            assert np.abs(means[b, c] - want).max() <= tol, (b, c, len(m))

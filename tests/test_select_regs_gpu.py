"""Selection with the keys in registers at the edges of its four prefix classes
(4096, 8192, 16384 and 32768 positions), odd row strides, plateaus, bins with
more keys than are ranked directly, and one to all but one position kept; the
positions are whole numbers and equal the oracle's."""
import numpy as np
import pytest
import torch

from paper_2512_21859_amd import _lib

pytestmark = pytest.mark.gpu


def _scores(kind, shape, rng):
    x = rng.standard_normal(shape).astype(np.float32)
    if kind == "skewed":
        return np.exp(3 * x)
    if kind == "plateau":                # runs of equal keys, as max-pooling makes
        return np.maximum.reduce([np.roll(np.abs(x), s, axis=-1) for s in range(-3, 4)])
    if kind == "three":                  # thousands of keys in one bin
        return np.round(x).clip(-1, 1).astype(np.float32)
    if kind == "narrow":                 # keys that differ in their lowest bits only
        return (np.float32(1.0) + np.abs(x) * np.float32(2.0 ** -18)).astype(np.float32)
    return x                             # signed


@pytest.mark.parametrize("kind", ["signed", "skewed", "plateau", "three", "narrow"])
@pytest.mark.parametrize("L,Lmax", [
    ([2, 66, 300], 301), ([4096 + 16, 4097 + 16, 5], 4118), ([8192 + 16, 8193 + 16], 8212),
    ([16384 + 16, 16385 + 16], 16404), ([32768 + 16, 32767, 100], 32785), ([32768 + 16, 20001], 32784),
])
def test_positions(kind, L, Lmax):
    w = 1 if min(L) <= 16 else 16
    rng = np.random.default_rng(Lmax + len(kind))
    B, Hkv = len(L), 2
    sc = _scores(kind, (B, Hkv, Lmax), rng)
    dev = torch.from_numpy(sc).cuda()
    for alpha in (0.02, 0.5, 0.97, 1.0):
        keep = torch.full((B, Hkv, Lmax), -1, dtype=torch.int32, device="cuda")
        al = [min(alpha, 1.0 - (w + 1.5) / n) if alpha == 1.0 else alpha for n in L]
        al = [max(a, 0.0) for a in al]
        n_keep = _lib.tb_select_topk(dev, L, w, al, keep)
        got = keep.cpu().numpy()
        for b, n in enumerate(L):
            want = n_keep[b] - w
            for g in range(Hkv):
                order = np.argsort(-sc[b, g, :n - w].astype(np.float64), kind="stable")[:want]
                ref = np.concatenate([np.sort(order), np.arange(n - w, n)])
                assert np.array_equal(got[b, g, :n_keep[b]], ref), (alpha, b, g)
                assert (got[b, g, n_keep[b]:] == -1).all()

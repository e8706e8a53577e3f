"""Prefill attention where two waves share a row tile (and its neighbours in
the choice of the block shape): prompts at the edges of its 128-key stages and
64-row blocks, ragged batches, both head sizes, against float64 on the CPU."""
import math

import pytest
import torch

from paper_2512_21859_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d,L,w", [
    (4, 2, 64, [192], 16), (4, 2, 64, [193, 1], 1), (7, 1, 128, [256, 64, 65], 33), (4, 2, 128, [257, 64, 129], 16),
    (8, 8, 64, [257, 200], 32), (2, 1, 128, [639], 64), (4, 4, 64, [1000, 129, 128], 16),
    (6, 3, 128, [1024], 32), (4, 2, 64, [1025], 32), (2, 1, 64, [2049, 300], 32), (2, 2, 128, [1025], 16),
])
def test_split(Hq, Hkv, d, L, w):
    g = torch.Generator().manual_seed(Hq * 100 + d + max(L))
    B, Lmax = len(L), max(L) + 7
    q, k, v = (torch.randn((B, h, Lmax, d), generator=g).bfloat16() for h in (Hq, Hkv, Hkv))
    k[:, :, ::50] *= 4                       # heavy keys, met at any time of a row's chain
    _check(q, k, v, L, min(w, min(L)))


@pytest.mark.parametrize("low", [-math.inf, float(torch.finfo(torch.bfloat16).min), -1e30])
@pytest.mark.parametrize("first,last", [(64, 96), (64, 128), (70, 400)])
@pytest.mark.parametrize("Hq,Hkv,d,L", [(4, 2, 64, [193, 100]), (2, 1, 128, [400]), (2, 2, 128, [200])])
def test_masked_keys(Hq, Hkv, d, L, first, last, low):
    """Keys that one channel takes to the lowest logits have no weight, also
    where they are all that one wave of a row tile sees (first or throughout)."""
    g = torch.Generator().manual_seed(Hq * 100 + d + max(L) + last)
    B, Lmax = len(L), max(L) + 7
    q, k, v = (torch.randn((B, h, Lmax, d), generator=g).bfloat16() for h in (Hq, Hkv, Hkv))
    q[..., 0] = 1.0
    k[:, :, first:last, 0] = low
    _check(q, k, v, L, 16)


def _check(q, k, v, L, w):
    B, Hq, Lmax, d = q.shape
    G = Hq // k.shape[1]
    out = torch.full((B, Hq, Lmax, d), -7.0, dtype=torch.bfloat16, device="cuda")
    stats = torch.zeros((B, Hq, w, 2), device="cuda")
    _lib.tb_prefill_attn(q.cuda(), k.cuda(), v.cuda(), L, out, w, stats)
    out, stats = out.cpu().double(), stats.cpu().double()
    for b, n in enumerate(L):
        for h in range(Hq):
            s = q[b, h, :n].double() @ k[b, h // G, :n].double().T / math.sqrt(d)
            s.masked_fill_(torch.ones(n, n, dtype=torch.bool).triu(1), -math.inf)
            m = s.max(dim=-1, keepdim=True).values
            p = torch.exp(s - m)
            z = p.sum(dim=-1, keepdim=True)
            ref = p @ v[b, h // G, :n].double() / z
            # P and the output are rounded to bf16 (2^-9 each): of values under
            # max |v| < 5, at most 5 * 2^-8; 2^-9 relative in the mean
            err = (out[b, h, :n] - ref).abs()
            assert float(err.max()) <= 5 * 2.0 ** -8, (b, h, float(err.max()))
            assert float(err.norm() / ref.norm()) <= 2.0 ** -8
            # fp32 logits (d products, |s| < 80: 1e-5) and sums
            assert float((stats[b, h, :, 0] - m[n - w:, 0]).abs().max()) <= 5e-5
            assert float(((stats[b, h, :, 1] - z[n - w:, 0]) / z[n - w:, 0]).abs().max()) <= 1e-4
        assert bool((out[b, :, n:] == -7.0).all())

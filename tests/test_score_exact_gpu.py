"""bf16 window and H2O scores at the edges of the digit kernels: row counts on
both sides of every wave, block and chunk boundary, prompts around the 64-key
tiles, and values the digits can and cannot hold (float64 products), against
float64."""
import math

import pytest
import torch

from paper_2512_21859_amd import _lib
from paper_2512_21859_amd.pipeline import Evictor

pytestmark = pytest.mark.gpu

# fp32 exponential (1 ulp of the hardware exp2 + half an ulp of its argument),
# its fp32 sum of four, and the fp32 rounding of the score: under 5 * 2^-24
REL = 3e-7


def _values(kind, shape, g):
    x = torch.randn(shape, generator=g)
    if kind == "outlier":            # one channel far above the rest, as attention keys have
        x[..., 3] *= 300.0
    elif kind == "wide":             # magnitudes over 2^-40 .. 1: below every digit of the row
        x = torch.sign(x) * torch.exp2(-40.0 * torch.rand(shape, generator=g)) * 8
    elif kind == "mixed":            # some tiles only
        x[..., 64:128, 0] = 2.0 ** -30
        x[..., 128:192, :] = 0.0
    elif kind == "tiny":             # bf16 subnormals among them
        x = x * 2.0 ** -127
    return x.to(torch.bfloat16)


def _raw64(q, k, L, w, scale):
    """Column sums of the window softmax in float64."""
    B, Hq, _, d = q.shape
    Hkv = k.shape[1]
    G = Hq // Hkv
    out = torch.zeros((B, Hkv, k.shape[2]), dtype=torch.float64)
    for b, n in enumerate(L):
        at = torch.arange(n - w, n)
        for h in range(Hq):
            s = q[b, h].double() @ k[b, h // G, :n].double().T * scale
            s.masked_fill_(torch.arange(n)[None, :] > at[:, None], -math.inf)
            out[b, h // G, :n - w] += torch.softmax(s, dim=-1).sum(dim=0)[:n - w]
    return out


@pytest.mark.parametrize("kind", ["normal", "outlier", "wide", "mixed", "tiny"])
@pytest.mark.parametrize("G,w,d,L", [
    (1, 1, 128, [65, 2, 64]), (1, 32, 64, [129, 33]), (1, 33, 128, [200]), (3, 32, 64, [777]),
    (4, 32, 128, [63, 512]), (5, 32, 128, [300]), (7, 32, 128, [1024, 999]), (7, 32, 64, [321]),
    (8, 32, 128, [450, 64]), (7, 40, 128, [257]), (8, 128, 64, [193]),
])
def test_raw_scores(kind, G, w, d, L):
    g = torch.Generator().manual_seed(len(L) * 1000 + G * 100 + w + d)
    B, Hkv, Lmax = len(L), 2, max(L) + 5
    q = _values(kind if kind in ("wide", "normal") else "normal", (B, G * Hkv, w, d), g)
    k = _values(kind, (B, Hkv, Lmax, d), g)
    _check_raw(q, k, L, w)


@pytest.mark.parametrize("value", [math.nan, math.inf, -math.inf])
def test_not_finite(value):
    """A NaN or infinite key spoils its own column and the rows whose logit with
    it is NaN or +inf, which then count nowhere; rows that see it at -inf give it
    no weight.  The other tiles are still computed, and no score is left
    unwritten."""
    g = torch.Generator().manual_seed(5)
    q, k = _values("normal", (1, 4, 16, 128), g), _values("normal", (1, 1, 300, 128), g)
    k[0, 0, 70, 5] = value
    ev = Evictor(1, 300, 4, 1, 128, 16, 1)
    ev.scores.fill_(-1.0)
    ev.score(q.cuda(), k.cuda(), [300])
    s = ev.scores[0, 0, :284].cpu().double()
    logits = q[0].reshape(64, 128).double() @ k[0, 0].double().T / math.sqrt(128)
    logits.masked_fill_(torch.arange(300)[None, :] > torch.arange(284, 300).repeat(4)[:, None], -math.inf)
    counts = logits[:, 70] == -math.inf
    ref = torch.softmax(logits[counts], dim=-1).sum(dim=0)[:284]
    assert torch.isnan(s[70])
    keep = torch.arange(284) != 70
    assert bool(((s - ref)[keep].abs() <= REL * ref[keep]).all())
    assert 16 < int(counts.sum()) < 48 or math.isnan(value)


def _check_raw(q, k, L, w):
    ref = _raw64(q, k, L, w, 1.0 / math.sqrt(q.shape[-1]))
    B, Hq, Hkv, d, Lmax = q.shape[0], q.shape[1], k.shape[1], q.shape[3], k.shape[2]
    ev = Evictor(B, Lmax, Hq, Hkv, d, w, 1)
    ev.scores.fill_(-1.0)
    ev.score(q.cuda(), k.cuda(), L)
    got = ev.scores.cpu().double()
    for b, n in enumerate(L):
        err = (got[b, :, :n - w] - ref[b, :, :n - w]).abs() / ref[b, :, :n - w].clamp_min(1e-37)
        assert float(err.max()) <= REL, (b, float(err.max()))


@pytest.mark.parametrize("big", [1.0, 2.0 ** 12])
@pytest.mark.parametrize("shift", [-1000.0, -100000.0, 1000.0])
@pytest.mark.parametrize("w,d,L", [(32, 128, [130, 65]), (32, 64, [161]), (64, 128, [700, 66])])
def test_far_logits(w, d, L, shift, big):
    """Every logit far from 0, also where rows of the window see no key of the
    last tile; `big` takes the products to float64."""
    g = torch.Generator().manual_seed(w + d + len(L))
    q = torch.randn((len(L), 4, w, d), generator=g).bfloat16()
    k = torch.randn((len(L), 2, max(L) + 5, d), generator=g).bfloat16()
    q[..., 6], q[..., 7] = 32.0, 1.0
    k[..., 6] = shift * math.sqrt(d) / 32.0
    q[..., 8], k[..., 8], q[..., 9], k[..., 9] = big, big, big, -big     # cancels, and widens both rows
    _check_raw(q, k, L, w)


@pytest.mark.parametrize("masked", [[70], range(64, 128), range(0, 64), range(0, 120), [5, 66, 150]])
@pytest.mark.parametrize("w,d", [(16, 128), (32, 64)])
def test_masked_keys(w, d, masked):
    """Keys at -inf have no weight, also where they fill a tile."""
    g = torch.Generator().manual_seed(w + d + len(masked))
    q, k = torch.randn((1, 6, w, d), generator=g).bfloat16(), torch.randn((1, 2, 200, d), generator=g).bfloat16()
    q[..., 5] = 1.0
    k[:, :, list(masked), 5] = -math.inf
    _check_raw(q, k, [200], w)


@pytest.mark.parametrize("Hq,Hkv,w,d,L", [(64, 8, 32, 128, 8250), (64, 8, 32, 64, 8250), (64, 32, 16, 128, 8200),
                                          (64, 32, 32, 64, 8200), (64, 16, 32, 128, 8200)])
def test_float64_runs(Hq, Hkv, w, d, L):
    """Blocks of several tiles whose keys leave the digits' range for a while, for
    one tile or a few, at the start and at the end of a prompt."""
    g = torch.Generator().manual_seed(Hkv + w + d)
    q, k = torch.randn((1, Hq, w, d), generator=g).bfloat16(), torch.randn((1, Hkv, L, d), generator=g).bfloat16()
    for lo, hi in ((0, 70), (300, 301), (900, 2100), (2300, 2400), (4000, 4064), (L - 200, L)):
        k[:, :, lo:hi, 3] *= 300
    k[:, ::2, 5000:6000, 3] *= 300
    k[:, 1::2, 6100:6101, 3] = 2.0 ** -40    # truncated: one tile past the bound, but not far
    _check_raw(q, k, [L], w)


def _h2o_ref(q, k, n):
    """Column sums of the causal softmax of one sequence in float64 (NaN where a
    row without a finite logit reaches)."""
    Hq, Hkv = q.shape[0], k.shape[0]
    ref = torch.zeros((Hkv, n), dtype=torch.float64)
    later = torch.ones(n, n, dtype=torch.bool).triu(1)
    for h in range(Hq):
        s = q[h, :n].double() @ k[h // (Hq // Hkv), :n].double().T / math.sqrt(q.shape[-1])
        s.masked_fill_(later, -math.inf)
        ref[h // (Hq // Hkv)] += torch.softmax(s, dim=-1).masked_fill(later, 0.0).sum(dim=0)
    return ref


@pytest.mark.parametrize("kind", ["normal", "outlier", "wide", "mixed", "tiny"])
@pytest.mark.parametrize("Hq,Hkv,d,L", [
    (2, 2, 128, [1, 64, 65]), (6, 2, 64, [127, 129, 16]), (4, 1, 128, [257, 300]),
    (28, 4, 128, [700]), (64, 8, 64, [1030, 520]),
])
def test_h2o_scores(kind, Hq, Hkv, d, L):
    g = torch.Generator().manual_seed(Hq * 1000 + d + max(L))
    B, Lmax = len(L), max(L) + 3
    q = _values("wide" if kind == "wide" else "normal", (B, Hq, Lmax, d), g)
    k = _values(kind, (B, Hkv, Lmax, d), g)
    ev = Evictor(B, Lmax, Hq, Hkv, d, 1, 1, scorer="h2o")
    ev.scores.fill_(-1.0)
    ev.score(q.cuda(), k.cuda(), L)
    got = ev.scores.cpu().double()
    for b, n in enumerate(L):
        ref = _h2o_ref(q[b], k[b], n)
        # terms under 2^-126 are fp32 subnormals, each within 2^-150: a sum of
        # up to 4 * 1030 * 8 of them is REL-exact from 1e-35 on
        err = (got[b, :, :n] - ref).abs() / ref.clamp_min(1e-35)
        assert float(err.max()) <= REL, (b, float(err.max()))
        assert bool((got[b, :, n:] == -1.0).all())


@pytest.mark.parametrize("shift", [0.0, -1000.0])
@pytest.mark.parametrize("masked", [[70], range(64, 128), range(0, 64), range(0, 200), [5, 66, 250]])
@pytest.mark.parametrize("Hq,Hkv,d,L", [(4, 2, 128, 300), (28, 4, 64, 264)])
def test_h2o_masked(Hq, Hkv, d, L, masked, shift):
    """Keys at -inf have no weight, whatever part of a row or a tile they are,
    and the other keys' logits may lie far below 0."""
    g = torch.Generator().manual_seed(Hq + d + len(masked))
    q, k = (torch.randn((1, h, L, d), generator=g).bfloat16() for h in (Hq, Hkv))
    q[..., 5], q[..., 6] = 1.0, 32.0
    k[..., 6] = shift * math.sqrt(d) / 32.0
    k[:, :, list(masked), 5] = -math.inf
    ev = Evictor(1, L, Hq, Hkv, d, 1, 1, scorer="h2o")
    ev.scores.fill_(-1.0)
    ev.score(q.cuda(), k.cuda(), [L])
    got, ref = ev.scores[0].cpu().double(), _h2o_ref(q[0], k[0], L)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    err = (got - ref).abs() / ref.clamp_min(1e-35)
    assert float(err[~torch.isnan(ref)].max()) <= REL


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("at", [3, 40, 130])
@pytest.mark.parametrize("Hq,Hkv,d,L", [(4, 2, 128, 300), (28, 4, 64, 264)])
def test_h2o_huge_key(Hq, Hkv, d, L, at, sign):
    """One finite key with logits past 2^31 in base 2: it takes all (or none) of
    the weight of every row that sees it, also from tiles of ordinary keys."""
    g = torch.Generator().manual_seed(Hq + d + at)
    q, k = (torch.randn((1, h, L, d), generator=g).bfloat16() for h in (Hq, Hkv))
    q[..., 7] = 1.0
    k[:, :, at, 7] = sign * 2.0 ** 36
    ev = Evictor(1, L, Hq, Hkv, d, 1, 1, scorer="h2o")
    ev.scores.fill_(-1.0)
    ev.score(q.cuda(), k.cuda(), [L])
    got, ref = ev.scores[0].cpu().double(), _h2o_ref(q[0], k[0], L)
    assert float(((got - ref).abs() / ref.clamp_min(1e-35)).max()) <= REL


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 2, 9])
def test_h2o_few_keys(L, d):
    """Rows of a few keys, whose rounding does not average out; a row of one key
    gives exactly 1."""
    B, H = 16, 64
    g = torch.Generator().manual_seed(L + d)
    q, k = (torch.randn((B, H, L, d), generator=g).bfloat16() for _ in range(2))
    ev = Evictor(B, L, H, H, d, 1, 1, scorer="h2o")
    ev.score(q.cuda(), k.cuda(), [L] * B)
    got = ev.scores.cpu().double()
    ref = torch.stack([_h2o_ref(q[b], k[b], L) for b in range(B)])
    if L == 1:
        assert bool((got == 1.0).all())
    # fp32 rounding of the score: 2^-24 / sqrt(3) at mantissa 1, 2.5e-8 over all;
    # of the terms beside the row's largest, which is exact: 2.5e-8 of at most
    # half the weight.  Together 2.8e-8, and 3.0e-8 allows for 1024 samples; with
    # the largest term rounded as well it is 3.5e-8 and more
    assert float(((got - ref) / ref).pow(2).mean().sqrt()) <= 3.0e-8

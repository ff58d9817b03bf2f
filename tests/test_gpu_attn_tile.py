"""GPU parity of the attention tile step (both contractions on the matrix cores, lazily raised
softmax maximum) where it can go wrong: scores that grow from tile to tile (the maximum is raised
again and again), shrink, or jump late by hundreds of binary orders, every padding of the query
heads into the score tile's columns, both head dims, and tails of one to sixteen rows.

Tolerance: a bf16 output is off by at most 2^-9 of its value, and an fp32 logit of up to 2^9
(log2 domain) by a few 2^-15, i.e. a weight by some 1e-4 of itself; with |v| <= 4 that leaves
|o - o_ref| <= 2^-8 |o_ref| + 2e-3.
"""
import math

import numpy as np
import pytest
import torch

from gpu_helpers import D
from oracle import delta_oracle as O
from paper_2510_09883_amd import synth

pytestmark = pytest.mark.gpu

LENS = [1, 15, 16, 17, 64, 83, 305]


def _pattern(kind, s, d, g):
    """Keys [s, d] whose scores against a query of ones follow `kind`."""
    t = torch.arange(s, dtype=torch.float32)
    level = {"rising": 0.05 * t, "falling": -0.05 * t, "spike": torch.where(t == s - 1, 30.0, -2.0),
             "flat": 0 * t, "steps": 8.0 * (t // 16 % 3)}[kind]
    return level[:, None] + 0.1 * torch.randn((s, d), generator=g)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 3, 4, 5, 8])
def test_tile_step_matches_float64(G, d):
    dd, hkv = D(), 2
    hq = hkv * G
    g = torch.Generator().manual_seed(100 * G + d)
    for kind in ("rising", "falling", "spike", "flat", "steps"):
        n = [(s + 15) // 16 for s in LENS]
        pt = torch.zeros((len(LENS), max(n)), dtype=torch.int32)
        k = torch.full((sum(n), hkv, 16, d), float("nan"), dtype=torch.bfloat16)
        v = torch.full_like(k, float("nan"))     # rows past a sequence's end stay NaN
        off = 0
        for b, s in enumerate(LENS):
            pt[b, :n[b]] = torch.arange(off, off + n[b])
            for h in range(hkv):
                for cache, x in ((k, _pattern(kind, s, d, g)),
                                 (v, torch.randn((s, d), generator=g).clamp(-4, 4))):
                    rows = torch.full((16 * n[b], d), float("nan"), dtype=torch.bfloat16)
                    rows[:s] = x.to(torch.bfloat16)
                    cache[off:off + n[b], h] = rows.view(-1, 16, d)
            off += n[b]
        q = (1 + 0.3 * torch.randn((len(LENS), hq, d), generator=g)).to(torch.bfloat16)
        shape = dd.make_shape(len(LENS), hq, hkv, d, max(n), max(LENS))
        dev = [x.cuda() for x in (k, v, pt, torch.tensor(LENS, dtype=torch.int32), q)]
        out = torch.full_like(dev[4], float("nan"))
        dd.delta_full_attn(shape, dd.make_kv(*dev[:4]), dev[4], out, dd.alloc_workspace(shape))
        torch.cuda.synchronize()
        for b, s in enumerate(LENS):
            K = O.gather_tokens(synth.bits(k), pt[b].numpy(), s)
            V = O.gather_tokens(synth.bits(v), pt[b].numpy(), s)
            o, _ = O.full_attention(O.bf16_bits_to_f64(synth.bits(q[b])), K, V, O.default_scale(d))
            err = np.abs(out[b].float().cpu().numpy() - o) - (2.0 ** -8 * np.abs(o) + 2e-3)
            assert err.max() <= 0, f"{kind} G {G} d {d} length {s}: over tolerance by {err.max():.3g}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 4, 5, 7, 8])
def test_infinite_values_stay_infinite(G, d):
    """A weight times an infinite value is infinite, also where the weight is a power of two, i.e.
    its lower bf16 terms are zero (one token has weight one); other columns are not touched."""
    dd = D()
    g = torch.Generator().manual_seed(7 * G + d)
    n = [(s + 15) // 16 for s in LENS]
    pt = torch.zeros((len(LENS), max(n)), dtype=torch.int32)
    k = (0.1 * torch.randn((sum(n), 1, 16, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((sum(n), 1, 16, d), generator=g).clamp(-4, 4).to(torch.bfloat16)
    off = 0
    for b, s in enumerate(LENS):
        pt[b, :n[b]] = torch.arange(off, off + n[b])
        last = off + (s - 1) // 16
        v[off, 0, 0, 3] = float("inf")
        v[last, 0, (s - 1) % 16, 20] = -float("inf")
        v[last, 0, (s - 1) % 16, d - 1] = float("inf")
        off += n[b]
    q = torch.randn((len(LENS), G, d), generator=g).to(torch.bfloat16)
    shape = dd.make_shape(len(LENS), G, 1, d, max(n), max(LENS))
    dev = [x.cuda() for x in (k, v, pt, torch.tensor(LENS, dtype=torch.int32), q)]
    out = torch.full_like(dev[4], float("nan"))
    dd.delta_full_attn(shape, dd.make_kv(*dev[:4]), dev[4], out, dd.alloc_workspace(shape))
    torch.cuda.synchronize()
    finite = torch.ones(d, dtype=torch.bool)
    finite[[3, 20, d - 1]] = False
    for b, s in enumerate(LENS):
        o = out[b].float().cpu()
        assert (o[:, 3] == float("inf")).all() and (o[:, d - 1] == float("inf")).all(), (s, o[:, 3])
        assert (o[:, 20] == -float("inf")).all(), (s, o[:, 20])
        K = O.gather_tokens(synth.bits(k), pt[b].numpy(), s)
        V = np.where(np.isinf(V := O.gather_tokens(synth.bits(v), pt[b].numpy(), s)), 0.0, V)
        ref, _ = O.full_attention(O.bf16_bits_to_f64(synth.bits(q[b])), K, V, O.default_scale(d))
        err = (np.abs(o.numpy() - ref) - (2.0 ** -8 * np.abs(ref) + 2e-3))[:, finite.numpy()]
        assert err.max() <= 0, f"length {s}: over tolerance by {err.max():.3g}"


def _one_head(K, V, G, lens, q_value=1.0):
    """Outputs [batch, G, d] of queries of `q_value` over one KV head's keys and values: lists of
    [s, d] per sequence, one page run each; rows past a sequence's end stay NaN."""
    dd, d = D(), K[0].shape[1]
    n = [(s + 15) // 16 for s in lens]
    pt = torch.zeros((len(lens), max(n)), dtype=torch.int32)
    k = torch.full((sum(n), 1, 16, d), float("nan"), dtype=torch.bfloat16)
    v = torch.full_like(k, float("nan"))
    off = 0
    for b, s in enumerate(lens):
        pt[b, :n[b]] = torch.arange(off, off + n[b])
        for cache, x in ((k, K[b]), (v, V[b])):
            rows = torch.full((16 * n[b], d), float("nan"), dtype=torch.bfloat16)
            rows[:s] = x.to(torch.bfloat16)
            cache[off:off + n[b], 0] = rows.view(-1, 16, d)
        off += n[b]
    q = torch.full((len(lens), G, d), q_value, dtype=torch.bfloat16)
    shape = dd.make_shape(len(lens), G, 1, d, max(n), max(lens))
    dev = [x.cuda() for x in (k, v, pt, torch.tensor(lens, dtype=torch.int32), q)]
    out = torch.full_like(dev[4], float("nan"))
    dd.delta_full_attn(shape, dd.make_kv(*dev[:4]), dev[4], out, dd.alloc_workspace(shape))
    torch.cuda.synchronize()
    return out.float().cpu()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 4, 5, 8])
def test_huge_scores_choose_one_token(G, d):
    """Scores of 2^13 to 2^97, every token's at least 2^-8 of itself from the next: the highest
    one has weight 1 and all others 0, so the output is its value, bit for bit."""
    g = torch.Generator().manual_seed(G + d)
    for e in (7, 20, 48):
        mant = torch.stack([1 + torch.arange(128) / 128.0, 2 + torch.arange(128) / 64.0]).flatten()
        lens = [s for s in LENS if s <= 256]
        level = [2.0 ** e * mant[torch.randperm(256, generator=g)[:s]] for s in lens]
        V = [torch.randn((s, d), generator=g).to(torch.bfloat16).float() for s in lens]
        out = _one_head([x[:, None].expand(-1, d) for x in level], V, G, lens, 2.0 ** e)
        for b, s in enumerate(lens):
            want = V[b][level[b].argmax()]
            assert torch.equal(out[b], want.expand(G, d)), f"2^{e} length {s}: {out[b][0]} for {want}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 8])
def test_output_is_the_rounded_quotient(G, d):
    """Equal keys, half of the values one bf16 step above the other half: the sum is exact in fp32
    and the mean lies half way between the two, so the output is the even one of them."""
    lens = [2, 14, 30, 94]
    a = 1 + torch.arange(d) / 128.0
    V = [torch.where((torch.arange(s) % 2 == 0)[:, None], a, a + 2.0 ** -7) for s in lens]
    out = _one_head([torch.ones((s, d)) for s in lens], V, G, lens)
    want = torch.where((torch.arange(d) % 2 == 0), a, a + 2.0 ** -7)     # 128 + j even, or the next
    for b, s in enumerate(lens):
        assert torch.equal(out[b], want.expand(G, d)), f"length {s}: {(out[b] != want).sum()} differ"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 4, 5, 8])
def test_large_finite_values_stay_finite(G, d):
    """Values up to bf16's largest, 3.3e38, under one token's weight; and 1e38 under weights that
    rise by 2^6 from one of a wave's pages to the next (2^1.5 a page), so that a maximum raised
    late, or a term counted twice, would pass fp32's range, which the sums themselves stay below.
    Tolerance: bf16 rounding, and weights off by 5e-4 of themselves (logits below 2^7)."""
    g = torch.Generator().manual_seed(3 * G + d)
    sign = torch.where(torch.rand((d,), generator=g) < 0.5, -1.0, 1.0)
    for big in (3.3e38, 1e38):
        K, V = [], []
        for s in LENS:
            t = torch.arange(s)
            top = (t == s - 1) if big > 2e38 else (t % 16 == 0)
            level = torch.where(top, 1.5 * (t // 16), -80.0)         # log2 of a weight
            K.append((level * math.log(2) / math.sqrt(d))[:, None].expand(-1, d))
            V.append(torch.where(top[:, None], big * sign, torch.randn((s, d), generator=g)))
        out = _one_head(K, V, G, LENS)
        for b, s in enumerate(LENS):
            k = K[b].to(torch.bfloat16).double()
            v = V[b].to(torch.bfloat16).double()
            ref = torch.softmax(k.sum(1) / math.sqrt(d), 0) @ v
            err = (out[b].double() - ref).abs() - (2.0 ** -8 * ref.abs() + 5e-4 * big)
            assert torch.isfinite(out[b]).all() and err.max() <= 0, f"{big:.1e} length {s}: {out[b][0]}"

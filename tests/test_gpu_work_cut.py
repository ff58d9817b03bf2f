"""GPU parity of the ways an attention launch's work is cut: one sequence far below the host's
length bound, few pairs in more than 16 splits, more workgroups than CUs for sparse layers over
pages and over tokens (some selections shorter than the budget), and pieces longer than the
kernel's page list.  Full and Delta layers must give the same output bits.

Tolerance: as in test_gpu_attn_tile.py, |o - o_ref| <= 2^-8 |o_ref| + 2e-3 (bf16 outputs of fp32
sums; logits stay below 2^9); the reference is float64 torch.
"""
import pytest
import torch

import balanced_cases as BC
from gpu_helpers import D

pytestmark = pytest.mark.gpu


def _inputs(lens, hq, hkv, d, bound, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = [-(-s // 16) for s in lens]
    pt = torch.zeros((len(lens), -(-bound // 16)), dtype=torch.int32, device="cuda")
    order = torch.randperm(sum(n), generator=g, device="cuda", dtype=torch.int32)
    off = 0
    for b, x in enumerate(n):
        pt[b, :x] = order[off:off + x]
        off += x
    k = torch.empty((sum(n), hkv, 16, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    v = torch.empty_like(k).normal_(generator=g)
    for b, s in enumerate(lens):
        if s % 16:
            k[pt[b, s // 16].long(), :, s % 16:] = float("nan")
            v[pt[b, s // 16].long(), :, s % 16:] = float("nan")
    q = torch.empty((len(lens), hq, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    return pt, torch.tensor(lens, dtype=torch.int32, device="cuda"), k, v, q


def _reference(pt, k, v, q, b, tokens, head, G):
    t = tokens.long()
    K = k[pt[b].long()[t // 16], head, t % 16].double()
    V = v[pt[b].long()[t // 16], head, t % 16].double()
    w = torch.softmax(q[b, head * G:(head + 1) * G].double() @ K.t().contiguous() / q.shape[2] ** 0.5, -1)
    return w @ V, w


def _close(out, ref, what):
    err = (out.double() - ref).abs() - (2.0 ** -8 * ref.abs() + 2e-3)
    assert float(err.max()) <= 0, f"{what}: over tolerance by {float(err.max()):.3g}"


@pytest.mark.parametrize("lens,hq,hkv,d,bound,check", [
    ([700], 8, 2, 64, 9000, [(0, 0), (0, 1)]),                  # far below the bound
    ([5000], 7, 1, 128, 5000, [(0, 0)]),                        # 32 splits of one pair
    ([4999, 300, 33], 5, 1, 128, 8000, [(0, 0), (1, 0), (2, 0)]),
    (BC.SHORT_PIECES, 16, 8, 64, max(BC.SHORT_PIECES), [(0, 0), (7, 7), (8, 1), (30, 4), (47, 7)]),
] + [(lens, hkv, hkv, 64, max(lens), check) for hkv, lens, _, check in BC.LONG_PIECES])
def test_full_and_delta_layers(lens, hq, hkv, d, bound, check):
    dd = D()
    pt, sl, k, v, q = _inputs(lens, hq, hkv, d, bound, len(lens))
    shape, sel = dd.make_shape(len(lens), hq, hkv, d, pt.shape[1], bound), dd.make_select(256, 32, delta_path=1)
    ws = dd.alloc_workspace(shape, sel)
    kv = dd.make_kv(k, v, pt, sl)
    full, delta = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    scores = torch.zeros((len(lens), pt.shape[1]), device="cuda")
    idx = torch.empty((len(lens), 16), dtype=torch.int32, device="cuda")
    cnt = torch.empty((len(lens),), dtype=torch.int32, device="cuda")
    for _ in range(2):   # the counters are re-armed
        dd.delta_full_attn(shape, kv, q, full, ws)
        dd.delta_delta_attn_select(shape, kv, q, delta, sel, idx, cnt, scores, ws)
    torch.cuda.synchronize()
    assert torch.equal(full.view(torch.int16), delta.view(torch.int16))
    G = hq // hkv
    for b, head in check:
        ref, _ = _reference(pt, k, v, q, b, torch.arange(lens[b], device="cuda"), head, G)
        _close(full[b, head * G:(head + 1) * G], ref, f"sequence {b} head {head}")
    if hkv <= 2:   # every head of the sequence: the page scores too (fp32 sums of 16 weights)
        for b, s in enumerate(lens):
            w = torch.cat([_reference(pt, k, v, q, b, torch.arange(s, device="cuda"), h, G)[1] for h in range(hkv)])
            m = torch.nn.functional.pad(w.max(0).values, (0, -s % 16)).view(-1, 16).sum(1)
            torch.testing.assert_close(scores[b, :m.numel()].double(), m, rtol=2e-5, atol=1e-9)


@pytest.mark.parametrize("unit", [16, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_sparse_layers_of_more_pairs_than_cus(unit, d):
    dd, B, hkv = D(), 48, 8
    lens = [600 if b % 5 else 97 + b for b in range(B)]
    pt, sl, k, v, q = _inputs(lens, hkv, hkv, d, 600, unit)
    K = 256 // unit
    g = torch.Generator().manual_seed(3)
    idx = torch.full((B, K), -1, dtype=torch.int32)
    cnt = torch.zeros((B,), dtype=torch.int32)
    for b, s in enumerate(lens):
        n = -(-s // unit)
        pick = torch.randperm(n, generator=g)[:K].sort().values
        pick[-1] = n - 1          # the partial last unit
        cnt[b] = pick.numel()
        idx[b, :pick.numel()] = pick
    idx, cnt = idx.cuda(), cnt.cuda()
    shape, sel = dd.make_shape(B, hkv, hkv, d, pt.shape[1], 600), dd.make_select(256, 16, unit)
    ws = dd.alloc_workspace(shape, sel)
    u = idx.clamp(min=0).long()
    phys = pt.gather(1, u) if unit == 16 else pt.gather(1, u // 16) * 16 + (u % 16).to(torch.int32)
    phys = torch.where(idx < 0, idx, phys).contiguous()
    outs = []
    for p in (None, phys, None):
        out = torch.full_like(q, float("nan"))
        dd.delta_sparse_attn(shape, dd.make_kv(k, v, pt, sl), q, out, sel, idx, cnt, ws, sel_phys=p)
        outs.append(out)
    torch.cuda.synchronize()
    assert all(torch.equal(o.view(torch.int16), outs[0].view(torch.int16)) for o in outs)
    for b in range(0, B, 3):
        t = (idx[b, :int(cnt[b]), None].long() * unit + torch.arange(unit, device="cuda")).flatten()
        t = t[t < lens[b]]
        for head in (0, b % hkv, hkv - 1):
            _close(outs[0][b, head:head + 1], _reference(pt, k, v, q, b, t, head, 1)[0], f"sequence {b} head {head}")


@pytest.mark.parametrize("unit", [16, 1])
def test_sparse_bits_depend_on_the_own_sequence_only(unit):
    """160 pairs: other sequences with fewer selected units, or none, leave a sequence's bits."""
    dd, B, hkv, hq, d = D(), 20, 8, 32, 128
    lens = [1100] * B
    pt, sl, k, v, q = _inputs(lens, hq, hkv, d, 1100, 5)
    K = 1024 // unit
    g = torch.Generator().manual_seed(7)
    idx = torch.stack([torch.randperm(-(-1100 // unit), generator=g)[:K].sort().values for _ in range(B)])
    idx = idx.to(torch.int32).cuda()
    shape, sel = dd.make_shape(B, hq, hkv, d, pt.shape[1], 1100), dd.make_select(1024, 16, unit)
    ws, kv = dd.alloc_workspace(shape, sel), dd.make_kv(k, v, pt, sl)
    kept = [0, 3, 9, 10, 19]
    want = None
    for others in (K, K // 3, 1, 0):
        cnt = torch.full((B,), others, dtype=torch.int32)
        cnt[kept] = K
        out = torch.full_like(q, float("nan"))
        dd.delta_sparse_attn(shape, kv, q, out, sel, idx, cnt.cuda(), ws)
        got = out[kept].view(torch.int16)
        want = got if want is None else want
        assert torch.equal(got, want), others
    for b in kept:
        t = (idx[b, :, None].long() * unit + torch.arange(unit, device="cuda")).flatten()
        t = t[t < lens[b]]
        _close(out[b, :4], _reference(pt, k, v, q, b, t, 0, 4)[0], f"sequence {b}")


@pytest.mark.parametrize("B,hkv,budget,d,unit", [(*c[:4], 1) for c in BC.LONG_TOKEN_PIECES]
                         + [(*c[:3], 64, c[3]) for c in BC.SPARSE_SPLITS])
def test_sparse_pieces(B, hkv, budget, d, unit):
    """Pieces of single tokens that are listed in parts, and the edges of the sparse split rule; some
    selections shorter than the budget and not whole groups, with and without stored locations."""
    dd, s, K = D(), budget + 100, budget // unit
    pt, sl, k, v, q = _inputs([s] * B, 2 * hkv, hkv, d, s, budget)
    g = torch.Generator(device="cuda").manual_seed(B)
    idx = torch.full((B, K), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((B,), K, dtype=torch.int32)
    for b in range(B):
        if b % 3 == 1:
            cnt[b] = [K - 5, 17, K // 2 + 1, 1][b // 3 % 4]
        n = int(cnt[b])
        idx[b, :n] = torch.randperm(-(-s // unit), generator=g, device="cuda")[:n].sort().values.to(torch.int32)
    u = idx.clamp(min=0).long()
    phys = pt.gather(1, u) if unit == 16 else pt.gather(1, u // 16) * 16 + (u % 16).to(torch.int32)
    phys = torch.where(idx < 0, idx, phys).contiguous()
    shape, sel = dd.make_shape(B, 2 * hkv, hkv, d, pt.shape[1], s), dd.make_select(budget, 16, unit)
    ws, kv = dd.alloc_workspace(shape, sel), dd.make_kv(k, v, pt, sl)
    outs = []
    for p in (None, phys):
        out = torch.full_like(q, float("nan"))
        dd.delta_sparse_attn(shape, kv, q, out, sel, idx, cnt.cuda(), ws, sel_phys=p)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    for b in sorted({*range(min(B, 14)), B - 1}):
        t = (idx[b, :int(cnt[b]), None].long() * unit + torch.arange(unit, device="cuda")).flatten()
        t = t[t < s]
        for head in (0, b % hkv, hkv - 1):
            ref, _ = _reference(pt, k, v, q, b, t, head, 2)
            _close(outs[0][b, 2 * head:2 * head + 2], ref, f"sequence {b} head {head}")

"""The selection kernel at the edges of its launch widths (256, 512 and 1024 threads, one to eight
candidates per thread), with distinct scores and with long runs of equal ones: the chosen units
must be exactly the recency window and the highest of the device's own unit scores, equal scores
lower index first, ascending, with their physical locations."""
import numpy as np
import pytest
import torch

from gpu_helpers import D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("unit,cands", [(1, c) for c in (255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4097, 8192)]
                         + [(16, c) for c in (256, 513, 1025, 2049)])
def test_selection_is_exact(unit, cands, ties):
    dd, d, recent = D(), 64, 16
    L = -(-recent // unit)
    s = unit * (cands + L) - (3 if unit == 16 else 0)      # a partial last page
    lens = [s, max(1, s // 3), s - unit]
    n = [-(-x // 16) for x in lens]
    g = torch.Generator(device="cuda").manual_seed(cands + unit)
    pt = torch.zeros((3, max(n)), dtype=torch.int32, device="cuda")
    order = torch.randperm(sum(n), generator=g, device="cuda", dtype=torch.int32)
    for b in range(3):
        pt[b, :n[b]] = order[sum(n[:b]):sum(n[:b + 1])]
    k = torch.empty((sum(n), 1, 16, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    if ties:    # five kinds of page
        k = k[torch.randint(0, 5, (sum(n),), generator=g, device="cuda")].contiguous()
        k[:] = k[:, :, :1]
    v = torch.empty_like(k).normal_(generator=g)
    q = torch.empty((3, 2, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    K = max(32, cands // 5)
    shape, sel = dd.make_shape(3, 2, 1, d, max(n), s), dd.make_select(K * unit, recent, unit)
    idx = torch.full((3, K), -7, dtype=torch.int32, device="cuda")
    phys, cnt = torch.full_like(idx, -7), torch.zeros((3,), dtype=torch.int32, device="cuda")
    scores = torch.zeros((3, -(-s // unit)), device="cuda")
    out = torch.empty_like(q)
    dd.delta_delta_attn_select(shape, dd.make_kv(k, v, pt, torch.tensor(lens, dtype=torch.int32, device="cuda")),
                               q, out, sel, idx, cnt, scores, dd.alloc_workspace(shape, sel), sel_phys=phys)
    torch.cuda.synchronize()
    for b in range(3):
        n_u = -(-lens[b] // unit)
        S = scores[b, :n_u].cpu().numpy()
        if n_u <= K:
            want = np.arange(n_u)
        else:
            old = np.argsort(-S[:n_u - L], kind="stable")[:K - L]
            want = np.concatenate([np.sort(old), np.arange(n_u - L, n_u)])
        got = idx[b].cpu().numpy()
        assert int(cnt[b]) == len(want)
        np.testing.assert_array_equal(got[:len(want)], want)
        assert np.all(got[len(want):] == -1)
        p = pt[b].cpu().numpy()
        loc = p[want] if unit == 16 else p[want // 16] * 16 + want % 16
        np.testing.assert_array_equal(phys[b].cpu().numpy()[:len(want)], loc)
        if ties and n_u > 64:
            assert len(np.unique(S)) < n_u // 2

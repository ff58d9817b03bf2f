"""The binding's buffer check decides what passes by whole-shape comparisons: it accepts and
refuses the same tensors as the rule entry by entry (None entries of a shape are free)."""
import pytest
import torch

from gpu_helpers import D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want", [None, (3,), (None,), (2, 3), (None, 3), (2, None), (None, None),
                                  (None, 2, 3), (None, 2, None)])
def test_buffer_check_follows_the_rule(want):
    dev = D()._dev
    have = [(), (0,), (3,), (2, 3), (3, 2), (0, 3), (5, 2, 3), (1, 2, 3), (2, 3, 1), (2, 2, 4)]
    tensors = [torch.empty(h, dtype=t, device="cuda") for h in have for t in (torch.bfloat16, torch.int32)]
    tensors += [torch.empty((3, 2), device="cuda", dtype=torch.bfloat16).t(),
                torch.empty((2, 6), device="cuda", dtype=torch.bfloat16)[:, ::2],
                torch.nn.Parameter(torch.empty((2, 3), device="cuda", dtype=torch.bfloat16)),
                torch.empty((2, 3), dtype=torch.bfloat16)]
    for t in tensors:
        fits = want is None or (t.dim() == len(want) and
                                all(w is None or w == d for w, d in zip(want, t.shape)))
        ok = t.is_cuda and t.dtype == torch.bfloat16 and t.is_contiguous() and fits
        if ok:
            assert dev("x", t, torch.bfloat16, want) is t
        else:
            with pytest.raises(ValueError, match="^x: "):
                dev("x", t, torch.bfloat16, want)

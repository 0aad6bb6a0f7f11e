"""Active-row lists and streamed reductions whose arrays start at any address: the four-at-a-time loads of the row
compaction and of the KL sums against the same call on aligned copies, around the sizes of a group of four tokens, a
wavefront and a block."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _shifted(t, by):
    """a contiguous copy that starts `by` elements into its buffer"""
    out = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)[by:].view(t.shape)
    return out.copy_(t)


@pytest.mark.parametrize("B,T", [(1, 1), (3, 2), (5, 7), (2, 1023), (3, 2049), (2, 16385)])
@pytest.mark.parametrize("with_mask", [True, False])
def test_kl_sums_at_any_alignment(lib, B, T, with_mask):
    g = torch.Generator(device="cuda").manual_seed(B * T)
    lp = torch.randn(B, T, generator=g, device="cuda")
    base = lp + 0.1 * torch.randn(B, T, generator=g, device="cuda")
    m = (torch.rand(B, T, generator=g, device="cuda") < 0.6).to(torch.uint8) if with_mask else None
    r = torch.randn(B, generator=g, device="cuda")
    dirty = lp if m is None else torch.where(m.bool(), lp, torch.full_like(lp, float("nan")))
    shaped, kl = lib.kl_shaped_rewards(r, dirty, base, m, 0.05)
    d = lp.double() - base.double()
    rkl = d.sum(1) if m is None else torch.where(m.bool(), d, torch.zeros_like(d)).sum(1)
    assert float((kl.double() - rkl).abs().max()) <= 2.0 ** -23 * float(rkl.abs().max()) + 1e-12     # one fp32 rounding
    assert float((shaped.double() - (r.double() - 0.05 * rkl)).abs().max()) <= 2.0 ** -23 * (float(r.abs().max()) + float(rkl.abs().max()))
    for by in (1, 2):
        s2, k2 = lib.kl_shaped_rewards(r, _shifted(dirty, by), base, None if m is None else _shifted(m, by), 0.05)
        assert torch.equal(shaped, s2) and torch.equal(kl, k2)

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


@pytest.mark.parametrize("N", [1, 3, 4, 5, 255, 257, 4095, 4096, 4097, 8191, 12289])
def test_compaction_at_any_alignment(lib, N):
    g = torch.Generator(device="cuda").manual_seed(N)
    H = torch.randn(N, 8, generator=g, device="cuda").bfloat16()
    W = torch.randn(20, 8, generator=g, device="cuda").bfloat16()
    t = torch.randint(-1, 21, (N,), generator=g, device="cuda").int()          # some out of range
    m = (torch.rand(N, generator=g, device="cuda") < 0.6).to(torch.uint8)
    logp, lse = lib.token_logprobs(H, W, t, m)
    ok = (m != 0) & (t >= 0) & (t < 20)
    z = H.double() @ W.double().T
    rlse = torch.logsumexp(z, dim=1)
    rlogp = z.gather(1, t.long().clamp(0, 19)[:, None])[:, 0] - rlse
    zero = torch.zeros_like(rlse)
    assert float((lse.double() - torch.where(ok, rlse, zero)).abs().max()) <= 1e-5
    assert float((logp.double() - torch.where(ok, rlogp, zero)).abs().max()) <= 1e-5
    l2, s2 = lib.token_logprobs(H, W, _shifted(t, 1), _shifted(m, 3))
    assert torch.equal(logp, l2) and torch.equal(lse, s2)
    a = lib.token_logprobs_partial(H, W, t, 0, 20, m)
    b = lib.token_logprobs_partial(H, W, _shifted(t, 3), 0, 20, _shifted(m, 1))
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    assert bool((a[0][~ok] == -float("inf")).all()) and not bool(a[1][~ok].any())
    coef = torch.where(ok, torch.randn(N, generator=g, device="cuda"), torch.zeros(N, device="cuda"))
    tc = t.clamp(0, 19)
    dH, dW = lib.offpolicy_loss_bwd(H, W, tc, lse, coef)
    dH2, dW2 = lib.offpolicy_loss_bwd(H, W, _shifted(tc, 1), lse, _shifted(coef, 1))
    assert torch.equal(dH, dH2) and torch.equal(dW, dW2) and not bool(dH[~ok].any())


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


# A launch has fewer than 2^32 threads: larger batches take several.
def _room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip("needs %d GiB of device memory" % gib)


@pytest.mark.parametrize("B,T", [(1 << 22, 2049), ((1 << 24) + 5, 3), ((1 << 20) + 7, 2)])
def test_kl_sums_of_many_generations(lib, B, T):
    _room(8 * B * T // 2 ** 30 + 4)
    lp = torch.full((B, T), 0.25, device="cuda")
    base = torch.zeros(B, T, device="cuda")
    r = torch.arange(B, device="cuda", dtype=torch.float32)
    shaped, kl = lib.kl_shaped_rewards(r, lp, base, None, 0.5)
    ok = bool((kl == 0.25 * T).all()), torch.equal(shaped, (r.double() - 0.125 * T).float())
    assert all(ok)                                                  # (pytest would print the tensors)
    del lp, base
    torch.cuda.empty_cache()


@pytest.mark.parametrize("B", [(1 << 20) + 7, (1 << 24) + 5])
def test_loss_of_many_generations(lib, B):
    T = 2
    t = torch.arange(B, device="cuda")
    mask = torch.stack([torch.ones_like(t), t % 3 == 0], dim=1).to(torch.uint8).contiguous()      # lengths 2, 1, 1, 2, ..
    logp = torch.full((B * T,), -1.0, device="cuda")
    loss, coef, stats = lib.offpolicy_loss_fwd(logp, logp, torch.ones(B, device="cuda"), mask, B, T, norm_mode=lib.NORM_SEQ_MEAN)
    per = torch.where(t % 3 == 0, 0.5, 1.0).double()[:, None] / B * mask.double()
    assert float((coef.double().view(B, T) + per).abs().max()) <= 2.0 ** -22 / B
    assert abs(float(loss) - 1.0) <= 1e-6 and float(stats[0]) == float(mask.sum().float()) and float(stats[4]) == 0


@pytest.mark.parametrize("P", [(1 << 22) + 3, (1 << 26) + 3])
def test_advantages_of_many_prompts(lib, P):
    r = torch.arange(2 * P, device="cuda").remainder(1 << 20).float()
    adv = lib.group_advantages(r, 2)
    d = (r.view(P, 2)[:, 0] - r.view(P, 2)[:, 1]) / 2
    ok = torch.equal(adv.view(P, 2), torch.stack([d, -d], dim=1))
    assert ok


@pytest.mark.parametrize("N", [(1 << 28) + 257, (1 << 32) + 257])
def test_merge_of_many_tokens(lib, N):
    _room(22 * N // 2 ** 30 + 4)
    m = torch.full((1, N), -2.0, device="cuda")
    s = torch.ones(1, N, device="cuda")
    zt = torch.full((1, N), -3.0, device="cuda")
    logp, lse = lib.merge_partials(m, s, zt)
    ok = bool((lse == -2.0).all()), bool((logp == -1.0).all())
    assert all(ok)
    del m, s, zt, logp, lse
    torch.cuda.empty_cache()

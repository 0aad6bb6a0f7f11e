"""The loss forward at the sizes where its launches change: one workgroup (up to 8192 tokens and 1024 generations; the
second half of them in a second group of four a thread) against several, generation lengths that no group of four tokens
or wavefront lines up with, the grid's stride."""
import numpy as np
import pytest
import torch

from oracle import aipo_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T", [(1, 1), (1, 3), (3, 1), (1024, 1), (1025, 1), (5, 7), (1000, 3), (63, 65), (4, 255), (3, 257),
                                 (1, 4096), (1, 4097), (3, 2049), (63, 67), (7, 1170), (1000, 8), (1, 8191), (1, 8192),
                                 (2, 4096), (1024, 8), (1, 8193), (1025, 7), (1, 16383),
                                 (1, 16384), (16, 1024), (7, 2341), (2, 8193), (1024, 17), (5, 4099),
                                 (2, 1100001)])
@pytest.mark.parametrize("norm,clip,per_token,with_mask,with_targets",
                         [(0, 0, False, True, True), (1, 1, True, True, False), (2, 0, True, False, False),
                          (1, 0, False, False, True)])
def test_loss_sizes(lib, B, T, norm, clip, per_token, with_mask, with_targets):
    rng = np.random.default_rng(B * 7919 + T)
    N, V = B * T, 50
    logp = (-2.0 * rng.exponential(size=N)).astype(np.float32)
    mu = (logp + 0.3 * rng.standard_normal(N)).astype(np.float32)
    adv = rng.standard_normal(N if per_token else B).astype(np.float32)
    mask = (rng.random((B, T)) < 0.7).astype(np.uint8) if with_mask else np.ones((B, T), np.uint8)
    targets = rng.integers(-2, V + 2, size=N).astype(np.int32) if with_targets else None
    dev = lambda x: None if x is None else torch.from_numpy(x).cuda()
    args = (dev(logp), dev(mu), dev(adv), dev(mask) if with_mask else None, B, T)
    kw = dict(rho=1.1, norm_mode=norm, clip_mode=clip, targets=dev(targets), V=V)
    loss, coef, stats = lib.offpolicy_loss_fwd(*args, **kw)
    ok = mask.reshape(-1).astype(bool)
    bad = 0
    if with_targets:
        out = (targets < 0) | (targets >= V)
        bad = int((ok & out).sum())
        ok = ok & ~out
    m = ok.reshape(B, T).astype(np.uint8)
    ref = orc.offpolicy_loss_fwd(logp.astype(np.float64), mu.astype(np.float64), adv.reshape((B, T) if per_token else B),
                                 m, 1.1, norm, clip, 0.2, 0.2)
    rloss, rcoef, rstats = ref["loss"], np.asarray(ref["coef"]).reshape(-1), ref["stats"]
    c = coef.double().cpu().numpy()
    off = np.abs(c - rcoef) > 1e-6 * max(np.abs(rcoef).max(), 1e-30)               # a few fp32 roundings
    assert off.sum() <= (2 if clip == 1 else 0)     # PPO's coef jumps where the ratio is within rounding of a bound
    assert abs(float(loss) - rloss) <= 1e-6 * np.abs(rcoef * logp).sum() + 1e-6 * abs(rloss) + 1e-30 + \
        (1e-6 * np.abs(adv).max() if clip == 1 else 0.0)
    s = stats.double().cpu().numpy()
    n = max(1, int(m.sum()))
    assert s[0] == m.sum() and s[4] == bad
    assert abs(s[1] - rstats[1]) <= 1e-6 * max(1.0, abs(rstats[1])) and abs(s[3] - rstats[3]) <= 1e-6
    assert abs(s[2] - rstats[2]) <= 2.0 / n + 1e-7          # a ratio within rounding of the bound counts on either side
    l2, c2, s2 = lib.offpolicy_loss_fwd(*args, **kw)
    assert torch.equal(loss, l2) and torch.equal(coef, c2) and torch.equal(stats, s2)

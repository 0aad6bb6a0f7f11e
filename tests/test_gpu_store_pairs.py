"""dH and dW in one launch (both on tiles of 128 or 64): each pairing of tile edges and output forms, ragged sizes, split and
whole tiles on either side, in one pass and in row passes; entry by entry against float64."""
import pytest
import torch

from tile_util import loops

pytestmark = pytest.mark.gpu


# (N, V, d, active share), (dH, dW) edges
SIZES = [
    ("bf16", 37, 130, 72, 1.0, ("64", "64")), ("bf16", 1, 70, 8, 1.0, ("64", "64")), ("bf16", 500, 1000, 264, 0.6, ("64", "64")),
    ("bf16", 300, 9001, 264, 0.8, ("64", "128")), ("bf16", 300, 9001, 1032, 0.8, ("128", "128")),
    ("bf16", 1041, 5003, 520, 0.7, ("128", "128")), ("bf16", 2050, 130, 1032, 0.5, ("128", "64")),
    ("bf16", 2048, 130, 1032, 0.9, ("128", "64")), ("bf16", 2049, 130, 1032, 0.9, ("128", "64")),       # H^T by either kernel
    ("f32", 37, 130, 72, 1.0, ("64", "64")), ("f32", 1, 70, 4, 1.0, ("64", "64")), ("f32", 1000, 3000, 516, 0.7, ("64", "64")),
    ("f32", 300, 16400, 260, 0.8, ("64", "128")), ("f32", 500, 5003, 1032, 0.7, ("128", "128")),
    ("f32", 700, 3000, 1032, 0.9, ("128", "64")),
]


@pytest.mark.parametrize("dt,N,V,d,share,edges", SIZES)
@pytest.mark.parametrize("form", ["plain", "accumulate", "fp32", "fp32 accumulate", "no rows"])
def test_pair(lib, dt, N, V, d, share, edges, form):
    assert loops(N, V, d, dt == "bf16")[2:] == edges
    _check_pair(lib, dt, N, V, d, share, form)


# ... in passes of R rows, which pick their tiles by R: the first full, the second partly filled and added to the first's dW, the
# third empty
@pytest.mark.parametrize("dt,N,V,d,R,edges", [
    ("bf16", 552, 130, 264, 256, ("64", "64")), ("bf16", 552, 9001, 264, 256, ("64", "128")),
    ("bf16", 2088, 1000, 2056, 1024, ("128", "128")), ("bf16", 2088, 130, 2056, 1024, ("128", "64")),
    ("f32", 552, 1000, 264, 256, ("64", "64")), ("f32", 552, 9001, 520, 256, ("64", "128")),
    ("f32", 552, 9001, 1032, 256, ("128", "128")), ("f32", 1576, 3000, 1032, 768, ("128", "64")),
])
@pytest.mark.parametrize("form", ["fp32", "fp32 accumulate"])
def test_pair_in_passes(lib, dt, N, V, d, R, edges, form):
    assert loops(R, V, d, dt == "bf16")[2:] == edges
    _check_pair(lib, dt, N, V, d, 0.7, form, R)


def _check_pair(lib, dt, N, V, d, share, form, rows_per_pass=None):
    bf16 = dt == "bf16"
    store = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N + V + d)
    H = torch.randn(N, d, generator=g, device="cuda").to(store)
    W = (torch.randn(V, d, generator=g, device="cuda") * d ** -0.5).to(store)
    y = torch.randint(0, V, (N,), generator=g, device="cuda")
    coef = torch.randn(N, generator=g, device="cuda") / N
    coef[torch.rand(N, generator=g, device="cuda") >= (0.0 if form == "no rows" else share)] = 0.0
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, dim=1)
    dz = -torch.exp(z - lse[:, None])
    dz[torch.arange(N, device="cuda"), y] += 1.0
    dz *= coef.double()[:, None]
    rdH, rdW = dz @ W.double(), dz.T @ H.double()
    old = torch.randn(V, d, generator=g, device="cuda") * rdW.std().float()
    kw = {}
    if "fp32" in form:
        kw["dW_dtype"] = torch.float32
    if "accumulate" in form:
        kw.update(dW=old.to(torch.float32 if "fp32" in form else store), accumulate_dW=True)
        rdW = rdW + kw["dW"].double()
    if rows_per_pass:
        assert rows_per_pass < int((coef != 0).sum()) <= 2 * rows_per_pass
        kw["max_rows_per_pass"] = rows_per_pass
    dH, dW = lib.offpolicy_loss_bwd(H, W, y.int(), lse.float(), coef, **kw)
    # An entry is a sum of K products.  bf16: each dz is rounded once, by up to 2^-8 of it (8 significant bits); the stored result once more.  In both types
    # exp(z - lse) carries the logits' and lse's own rounding, |z| <= 8: 8 sqrt(d) 2^-24 and 10 2^-24, below 2^-15, and the
    # sum's order sqrt(K) 2^-24.  (dz * 1 + tiny: coef * (1 - p) of the target cancels only where p is near 1.)
    each, result = (2.0 ** -8 + 2.0 ** -14, 2.0 ** -8) if bf16 else (2.0 ** -14, 2.0 ** -22)
    for name, got, ref, bound in (("dH", dH, rdH, dz.abs() @ W.double().abs()), ("dW", dW, rdW, dz.abs().T @ H.double().abs())):
        rounds = 2.0 ** -22 if got.dtype == torch.float32 else result
        assert bool(((got.double() - ref).abs() <= each * bound + rounds * ref.abs()).all()), name
    assert not bool(dH[coef == 0].any())


@pytest.mark.parametrize("dt,N,V,d,share,edges", [c for c in SIZES if c[1] >= 300])
def test_the_call_that_records_events_runs_the_same_kernels(lib, dt, N, V, d, share, edges):
    g = torch.Generator(device="cuda").manual_seed(N + V + d)
    store = torch.bfloat16 if dt == "bf16" else torch.float32
    H = torch.randn(N, d, generator=g, device="cuda").to(store)
    W = (torch.randn(V, d, generator=g, device="cuda") * d ** -0.5).to(store)
    y = torch.randint(0, V, (N,), generator=g, device="cuda").int()
    coef = torch.randn(N, generator=g, device="cuda") / N
    coef[torch.rand(N, generator=g, device="cuda") >= share] = 0.0
    lse = lib.token_logprobs(H, W, y)[1]
    events = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
    for e in events:
        e.record()
    plain = lib.offpolicy_loss_bwd(H, W, y, lse, coef)
    timed = lib.offpolicy_loss_bwd(H, W, y, lse, coef, phase_events=[e.cuda_event for e in events])
    assert all(torch.equal(a, b) for a, b in zip(plain, timed))       # other parts of K would be another order of the sums
    torch.cuda.synchronize()
    between = [a.elapsed_time(b) for a, b in zip(events, events[1:])]
    assert min(between) >= 0 and between[4] > between[2]


# bf16's dH reads W, so this is no pair: dW is written when dH is done
@pytest.mark.parametrize("dt,N,V,d,share,edges", [c for c in SIZES if c[1] >= 300])
def test_weights_updated_in_place(lib, dt, N, V, d, share, edges):
    g = torch.Generator(device="cuda").manual_seed(N + V + d)
    store = torch.bfloat16 if dt == "bf16" else torch.float32
    H = torch.randn(N, d, generator=g, device="cuda").to(store)
    W = (torch.randn(V, d, generator=g, device="cuda") * d ** -0.5).to(store)
    y = torch.randint(0, V, (N,), generator=g, device="cuda").int()
    coef = torch.randn(N, generator=g, device="cuda") / N
    coef[torch.rand(N, generator=g, device="cuda") >= share] = 0.0
    lse = lib.token_logprobs(H, W, y)[1]
    dH, dW = lib.offpolicy_loss_bwd(H, W, y, lse, coef, dW_dtype=torch.float32)
    updated = W.clone()
    got, _ = lib.offpolicy_loss_bwd(H, updated, y, lse, coef, dW=updated, accumulate_dW=True)
    # Both dH are sums of the same products, their K cut into other parts: fp32 sums of up to 2^14 terms in another order, below
    # 2^-17 of their largest.  That can put them on either side of the middle between two bf16 numbers, which are up to 2^-7 of
    # the smaller one apart (eight significant bits); one rounding of a sum is half of that.
    apart = 2.0 ** -7 if dt == "bf16" else 0.0
    assert bool(((got.double() - dH.double()).abs() <= apart * dH.double().abs() + 2.0 ** -17 * dH.double().abs().max()).all())
    want = W.double() + dW.double()
    assert bool(((updated.double() - want).abs() <= (apart / 2 + 2.0 ** -23) * want.abs() + 2.0 ** -17 * dW.double().abs().max()).all())

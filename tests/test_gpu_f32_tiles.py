"""fp32 contractions on 128 x 128 and 64 x 64 tiles with operands split into three bf16 parts: sizes at the edges of
the tiles, of a K slab (32) and of the rule that picks the tile, against float64; values that cannot be split."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(N, V, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn(N, d, generator=g, device="cuda")
    W = torch.randn(V, d, generator=g, device="cuda") * d ** -0.5
    t = torch.randint(0, V, (N,), generator=g, device="cuda").int()
    coef = torch.randn(N, generator=g, device="cuda") / N
    return H, W, t, coef


def _reference(H, W, t, coef):
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, dim=1)
    logp = z.gather(1, t.long()[:, None])[:, 0] - lse
    dz = -torch.exp(z - lse[:, None])
    dz[torch.arange(t.numel(), device="cuda"), t.long()] += 1.0
    dz *= coef.double()[:, None]
    return logp, lse, dz @ W.double(), dz.T @ H.double()


def _rel(a, b):
    return float((a.double() - b).norm() / b.norm())


def _worst(a, b):
    """relative error of the worst row or column: almost all of dW's norm sits in its few target rows, and a tile that
    was lost elsewhere does not show in the norm of the whole.  (Of 32 entries or more: fewer can cancel all together.)"""
    diff, out = a.double() - b, 0.0
    for dim in (0, 1):
        if b.shape[dim] < 32:
            continue
        n, e = b.norm(dim=dim), diff.norm(dim=dim)
        assert not bool(e[n == 0].any())             # rows of tokens without gradient are exactly zero
        if bool((n > 0).any()):
            out = max(out, float((e[n > 0] / n[n > 0]).max()))
    return out


# a sum of K products, each rounded to 2^-24 of a partial sum no larger than sqrt(K) standard products, in any order:
# relative error of the result's norm below sqrt(K) 2^-24; the logits feed dz through exp(z - lse), |z| <= 8 here
@pytest.mark.parametrize("N,V,d", [
    (1, 64, 4), (64, 64, 32), (65, 63, 36), (63, 129, 28), (127, 1025, 64), (128, 128, 256), (129, 257, 260),
    (384, 8064, 68), (385, 8193, 100),          # 189 and 260 tiles of 128: either side of the logits rule
    (500, 512, 512), (512, 3000, 480),          # dH on 64-tiles, split along K
    (700, 4100, 516), (1100, 4097, 516),        # dW and dH on either tile
])
def test_tile_edges(lib, N, V, d):
    H, W, t, coef = _inputs(N, V, d, 7 * N + V + d)
    logp, lse = lib.token_logprobs(H, W, t)
    rlogp, rlse, rdH, rdW = _reference(H, W, t, coef)
    bound = 2.0 ** -24 * d ** 0.5
    assert float((lse.double() - rlse).abs().max()) <= 8 * bound + 2e-6
    assert float((logp.double() - rlogp).abs().max()) <= 16 * bound + 2e-6
    dH, dW = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    tol = 2.0 ** -24 * (max(V, N, d) ** 0.5 + 16)
    assert _rel(dH, rdH) <= tol and _rel(dW, rdW) <= tol
    assert _worst(dH, rdH) <= tol and _worst(dW, rdW) <= tol


@pytest.mark.parametrize("N,V,d", [(200, 33000, 260), (300, 40000, 512)])      # dH in up to 32 parts: 64- and 128-tiles
def test_many_parts(lib, N, V, d):
    test_tile_edges(lib, N, V, d)


# the last slab of 32 up to one 16-byte chunk, half of it (a lane's first chunk) and past that, alone and after another
@pytest.mark.parametrize("N,V", [(65, 129), (400, 8200)])                      # 64- and 128-tiles
@pytest.mark.parametrize("d", [4, 16, 20, 44, 48])
def test_last_slab(lib, N, V, d):
    test_tile_edges(lib, N, V, d)


@pytest.mark.parametrize("N,V,d", [(130, 300, 40), (400, 9000, 40)])      # 64- and 128-tiles
def test_values_that_cannot_be_split(lib, N, V, d):
    # a constant-one column makes W[:, 0] a bias; -inf there bans a token, and 3.4e38 (infinity in bf16) times
    # 1e-38 is an ordinary number: both are what fp32 arithmetic gives
    H, W, t, _ = _inputs(N, V, d, 5)
    H[:, 0] = 1.0
    H[:, 1] = 3.4e38
    W[:, 1] = 1e-38 * W[:, 2]
    banned = torch.tensor([3, V - 1], device="cuda")
    W[banned, 0] = -float("inf")
    t = torch.where((t == 3) | (t == V - 1), torch.zeros_like(t), t)
    logp, lse = lib.token_logprobs(H, W, t)
    z = H.double() @ torch.where(torch.isinf(W), torch.zeros_like(W), W).double().T
    z[:, banned] = -float("inf")
    rlse = torch.logsumexp(z, dim=1)
    rlogp = z.gather(1, t.long()[:, None])[:, 0] - rlse
    assert float((lse.double() - rlse).abs().max()) <= 2e-5
    assert float((logp.double() - rlogp).abs().max()) <= 2e-5
    # a NaN row stays in its own row (its maximum ignores NaN, so lse is -inf rather than NaN: fmax semantics)
    H[17, 4] = float("nan")
    logp2, lse2 = lib.token_logprobs(H, W, t)
    assert not bool(torch.isfinite(lse2[17])) and bool(torch.isnan(logp2[17]))
    ok = torch.arange(N, device="cuda") != 17
    assert float((lse2[ok].double() - rlse[ok]).abs().max()) <= 2e-5


def test_every_tile_contracted_twice(lib):
    # 1105 tiles of 128, two or three a workgroup, and in each a value that cannot be split: what a tile's second pass leaves in LDS,
    # and the flag that asks for it, must not reach the next tile
    test_values_that_cannot_be_split(lib, 2100, 8200, 40)


def _no_smaller_than(x, low):
    """x with every magnitude below `low` replaced by one in [low, 2 low) of as many bits"""
    small = x.abs() < low
    return torch.where(small, torch.copysign(low * (1 + x.abs() / low), x), x)


def _split(x):
    h = x.bfloat16().float()
    m = (x - h).bfloat16().float()
    return h, m, x - h - m


@pytest.mark.parametrize("N,V,d", [(100, 300, 64), (400, 9000, 64)])      # 64- and 128-tiles
@pytest.mark.parametrize("shift", [-100, -60, 60, 100])
def test_scaling_by_a_power_of_two_changes_no_bit(lib, N, V, d, shift):
    # At +-100 most of the smaller operand's values lie in [2^-109, 2^-108) and their third parts, down to 2^-133, are
    # subnormal: parts that were flushed would take up to 2^-17 of their values along.
    H, W, t, _ = _inputs(N, V, d, 9)
    if shift > 0:
        H = _no_smaller_than(H * 2.0 ** -9, 2.0 ** -9)
    else:
        W = _no_smaller_than(W * 2.0 ** -6, 2.0 ** -9)
    Hs, Ws = H * 2.0 ** -shift, W * 2.0 ** shift
    low = Hs if shift > 0 else Ws
    part = _split(low)[2].abs()
    assert torch.equal(part.bfloat16().float(), part)
    assert abs(shift) < 100 or float(((part > 0) & (part < 2.0 ** -126)).float().mean()) > 0.5
    a = lib.token_logprobs(H, W, t)
    b = lib.token_logprobs(Hs, Ws, t)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def _full_mantissas(g, exponent, *shape):
    """fp32 numbers in [2^exponent, 2^(exponent+1)) with random 24-bit significands"""
    x = 1.0 + torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)
    return torch.ldexp(x, torch.tensor(exponent, device="cuda")).float()


def _ulps(got, exact):
    """distance in units of the last place of an fp32 number of exact's size"""
    ulp = torch.ldexp(torch.ones_like(exact), (torch.frexp(exact)[1] - 24).clamp(min=-149))
    return float(((got.double() - exact).abs() / ulp).max())


# Sums with one product that is not zero: the bare arithmetic of a product, in all three contractions.  The five bf16
# products of orders 2^-8 and 2^-16 and the last two of 2^-25 meet in one fp32 sum below 2^-6 of the factors' leading
# powers of two: its roundings (2^-32 + 2^-31 and smaller ones) and the product left out (2^-34) are below 2^-7 ulp of the
# result, the final addition is half an ulp.
@pytest.mark.parametrize("N,V,d", [(130, 300, 4), (2000, 512, 64), (4096, 8192, 260)])      # 64-, 64- and 128-tiles
@pytest.mark.parametrize("ex,ey", [(0, 0), (40, -70), (-100, 55), (60, -108),                    # sums of 2 ey stay finite
                                   (-111, 55), (-114, 55), (-126, 55), (-135, 55), (50, -120), (100, -108)])  # bits below 2^-133
def test_single_products(lib, N, V, d, ex, ey):
    g = torch.Generator(device="cuda").manual_seed(N + ex)
    rows = torch.arange(N, device="cuda")
    x, W = _full_mantissas(g, ex, N), _full_mantissas(g, ey, V, d)
    H = torch.zeros(N, d, device="cuda")
    H[rows, rows % d] = x                                           # one-hot rows: a logit is one product
    t = (rows * 37 % V).int()
    _, _, zt = lib.token_logprobs_partial(H, W, t, 0, V)
    assert _ulps(zt, x.double() * W[t.long(), rows % d].double()) <= 0.5 + 2.0 ** -7
    # lse = inf: dz is coef at the target and zero elsewhere; distinct targets
    n = min(N, V)
    t = torch.randperm(V, generator=g, device="cuda")[:n]
    H, coef = _full_mantissas(g, ey, n, d), x[:n].contiguous()
    dH, dW = lib.offpolicy_loss_bwd(H, W, t.int(), torch.full((n,), float("inf"), device="cuda"), coef)
    assert _ulps(dH, coef.double()[:, None] * W[t].double()) <= 0.5 + 2.0 ** -7
    assert _ulps(dW[t], coef.double()[:, None] * H.double()) <= 0.5 + 2.0 ** -7


@pytest.mark.parametrize("N,V,d", [(100, 300, 64), (2100, 8100, 64)])      # 64- and 128-tiles
def test_gradient_of_a_very_unlikely_row(lib, N, V, d):
    # H[:, 0] = 1 makes W[:, 0] a bias: -82 nats on two rows, whose dz is 2^-118 .. 2^-124 and has fp32 numbers' 24 bits
    H, W, t, _ = _inputs(N, V, d, 11)
    g = torch.Generator(device="cuda").manual_seed(12)
    coef = torch.rand(N, generator=g, device="cuda") / 64 + 1.0 / 64
    rows = torch.tensor([5, V - 3], device="cuda")
    H[:, 0] = 1.0
    W[:, 0] = 0.0
    W[rows] *= 0.125
    W[rows, 0] = -82.0 + torch.logsumexp(H.double() @ W.double().T, dim=1).float().mean()
    t = torch.where((t[:, None] == rows).any(1), torch.zeros_like(t), t)
    _, lse = lib.token_logprobs(H, W, t)
    _, _, _, rdW = _reference(H, W, t, coef)
    _, dW = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    assert float(rdW[rows].abs().max()) < 2.0 ** -107
    # z and lse of about 82 are rounded to 2^-18 each, which is the relative error of p = exp(z - lse) they leave
    for r in rows.tolist():
        assert _rel(dW[r], rdW[r]) <= 2.0 ** -16


def test_backward_of_a_head_with_more_transpose_tiles_than_a_launch_holds_blocks(lib):
    # 16385 x 256 tiles of 64 x 64 for W^T: one 1024-thread block each would be 2^32 threads and more
    V, d = 1048640, 16384
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 215 << 30:
        pytest.skip("needs 207 GB of device memory: W, its transpose and dW")
    W = torch.zeros(V, d, device="cuda")
    W[-1] = torch.arange(d, device="cuda") % 7
    H = torch.zeros(1, d, device="cuda")
    H[0, :64] = torch.arange(64, device="cuda") / 64
    t = torch.tensor([V - 1], device="cuda").int()
    dH, dW = lib.offpolicy_loss_bwd(H, W, t, torch.full((1,), float("inf"), device="cuda"), torch.full((1,), 2.0, device="cuda"))
    assert torch.equal(dH[0], 2.0 * W[-1]) and torch.equal(dW[-1], 2.0 * H[0])        # dz = 2 at the target, 0 elsewhere
    assert all(not bool(dW[i:i + 65536].any()) for i in range(0, V - 65536, 65536))
    del W, dW
    torch.cuda.empty_cache()

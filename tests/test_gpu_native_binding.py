"""The marshalling in C++: what it accepts, what it refuses and with which error, the caller's buffers and streams."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _head(N=70, V=900, d=64):
    g = torch.Generator(device="cuda").manual_seed(5)
    H = torch.randn(N, d, generator=g, device="cuda").bfloat16()
    W = (torch.randn(V, d, generator=g, device="cuda") * d ** -0.5).bfloat16()
    return H, W, torch.randint(0, V, (N,), generator=g, device="cuda").int()


def test_refusals_raise_the_bindings_error(lib):
    H, W, y = _head()
    coef = lse = torch.zeros(70, device="cuda")
    for args in [(H.float(), W, y), (H, W[:, :32], y), (H, W, y.long()), (H, W, y[:-1]), (H.t(), W, y), (H.half(), W.half(), y),
                 (H.cpu(), W, y), (H, W, y, torch.ones(69, dtype=torch.uint8, device="cuda"))]:
        with pytest.raises(lib.LlamarlError) as e:
            lib.token_logprobs(*args)
        assert e.value.status == lib.ERR_INVALID_ARG
    with pytest.raises(lib.LlamarlError) as e:
        lib.token_logprobs(H, W, y, ws=torch.empty(64, dtype=torch.uint8, device="cuda"))
    assert e.value.status == lib.ERR_WORKSPACE and "needed" in str(e.value)
    for kw in [dict(dW_dtype=torch.float16), dict(accumulate_dW=True), dict(grad_loss=float("nan")), dict(max_rows_per_pass=-1)]:
        with pytest.raises(lib.LlamarlError):
            lib.offpolicy_loss_bwd(H, W, y, lse, coef, **kw)
    with pytest.raises(lib.LlamarlError):
        lib.group_advantages(coef, 9)
    with pytest.raises(lib.LlamarlError):
        lib.merge_partials(coef, coef, coef)
    with pytest.raises(TypeError):
        lib.token_logprobs([1.0], W, y)


def test_callers_buffers_and_streams(lib):
    H, W, y = _head()
    logp, lse = lib.token_logprobs(H, W, y)
    coef = torch.linspace(-1, 1, 70, device="cuda")
    dH, dW = lib.offpolicy_loss_bwd(H, W, y, lse, coef)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    ws = torch.empty(lib.workspace_bytes(70, 64, 900, lib.BF16, lib.PASS_LOSS_BWD), dtype=torch.uint8, device="cuda")
    out = torch.full_like(W, float("nan")), torch.full_like(H, float("nan"))
    with torch.cuda.stream(s):
        on_current = lib.token_logprobs(H, W, y)
    given = lib.token_logprobs(H, W, y, stream=s)
    got = lib.offpolicy_loss_bwd(H, W, y, lse, coef, dW=out[0], dH=out[1], ws=ws, stream=s)
    torch.cuda.synchronize()
    assert got[0] is not None and got[0].data_ptr() == out[1].data_ptr() and got[1].data_ptr() == out[0].data_ptr()
    assert torch.equal(out[1], dH) and torch.equal(out[0], dW)
    for a in (on_current, given):
        assert torch.equal(a[0], logp) and torch.equal(a[1], lse)

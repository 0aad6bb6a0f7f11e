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


def _segment_stream(ptr):
    """stream whose pool the memory at an address belongs to"""
    for seg in torch.cuda.memory_snapshot():
        if seg["address"] <= ptr < seg["address"] + seg["total_size"]:
            return seg["stream"]


def test_what_a_call_on_a_given_stream_allocates_is_that_streams(lib):
    # From the current stream's pool, the workspace would be given to that stream's next allocation while the kernels of the
    # call still use it.
    N, d, V = 8192, 64, 60000               # workspaces of 10 MB and more, which the allocator gives a segment of their own
    H, W, y = _head(N, V, d)
    s = torch.cuda.Stream()
    many = torch.zeros(1 << 21, device="cuda")
    coef = torch.linspace(-1, 1, N, device="cuda")
    lse = torch.zeros(N, device="cuda")
    ones = torch.ones(2, N, device="cuda")
    torch.cuda.synchronize()
    here = torch.cuda.current_stream().cuda_stream
    assert s.cuda_stream != here
    g = torch.ones((), device="cuda")
    events = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
    for e in events:
        e.record()
    calls = [lambda: lib.token_logprobs(H, W, y, stream=s), lambda: lib.token_logprobs_partial(H, W, y, 0, V, stream=s),
             lambda: lib.merge_partials(ones, ones, ones, stream=s),
             lambda: lib.offpolicy_loss_fwd(many, many, many, None, 512, 4096, stream=s),
             lambda: lib.offpolicy_loss_bwd(H, W, y, lse, coef, stream=s),
             lambda: lib.offpolicy_loss_bwd(H, W, y, lse, coef, stream=s, max_rows_per_pass=256),
             lambda: lib.offpolicy_loss_bwd(H, W, y, lse, coef, stream=s, phase_events=[e.cuda_event for e in events]),
             lambda: lib.offpolicy_loss_bwd_slice(H, W, y, 0, lse, coef, stream=s),
             lambda: lib.offpolicy_loss_bwd_device_scale(H, W, y, lse, coef, g, stream=s),
             lambda: (lib.group_advantages(coef, 8, stream=s),), lambda: lib.kl_shaped_rewards(coef, lse, lse, None, 0.1, stream=s)]
    for call in calls:
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        before = torch.cuda.memory_stats()["reserved_bytes.all.current"]
        mine = sum(seg["total_size"] for seg in torch.cuda.memory_snapshot() if seg["stream"] == here)
        out = call()
        assert all(_segment_stream(t.data_ptr()) == s.cuda_stream for t in out)
        # nothing, the workspace neither, came out of the current stream's pool
        assert mine == sum(seg["total_size"] for seg in torch.cuda.memory_snapshot() if seg["stream"] == here)
        assert torch.cuda.memory_stats()["reserved_bytes.all.current"] > before
        assert torch.cuda.current_stream().cuda_stream == here
        torch.cuda.synchronize()
        del out
    # the caller's own buffers stay where they are, and the stream is the current one again after an error
    dW = torch.empty_like(W)
    assert lib.offpolicy_loss_bwd(H, W, y, lse, coef, dW=dW, stream=s)[1].data_ptr() == dW.data_ptr()
    with pytest.raises(lib.LlamarlError):
        lib.token_logprobs(H, W, y, ws=torch.empty(64, dtype=torch.uint8, device="cuda"), stream=s)
    assert torch.cuda.current_stream().cuda_stream == here
    torch.cuda.synchronize()

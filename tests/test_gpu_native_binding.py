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


def test_arrays_too_small_for_the_head_are_refused(lib):
    # the kernels take their sizes from H and W: each of these would be read or written past its end
    H, W, y = _head()
    N, d, V = 70, 64, 900
    f = torch.zeros(N, device="cuda")
    m = torch.ones(N, dtype=torch.uint8, device="cuda")
    g = torch.ones((), device="cuda")
    events = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
    for e in events:
        e.record()
    phases = dict(phase_events=[e.cuda_event for e in events])
    ws = torch.empty(lib.workspace_bytes(N, d, V, lib.BF16, lib.PASS_LOSS_BWD), dtype=torch.uint8, device="cuda")
    refused = []
    for args in [(H, W[:, :32].contiguous(), y, f, f), (H, W, y[:-1], f, f), (H, W, y, f[:-1], f), (H, W, y, f, f[:-1])]:
        refused += [lambda a=args: lib.offpolicy_loss_bwd(*a), lambda a=args: lib.offpolicy_loss_bwd(*a, **phases),
                    lambda a=args: lib.offpolicy_loss_bwd(*a, max_rows_per_pass=256),
                    lambda a=args: lib.offpolicy_loss_bwd_slice(*a[:3], 0, *a[3:]),
                    lambda a=args: lib.offpolicy_loss_bwd_device_scale(*a, g)]
    for kw in [dict(dW=W[:-1].clone()), dict(dH=H[:-1].clone()), dict(ws=ws.cpu()), dict(ws=ws[::2]), dict(ws=ws[:1].expand(ws.numel()))]:
        refused += [lambda k=kw: lib.offpolicy_loss_bwd(H, W, y, f, f, **k), lambda k=kw: lib.offpolicy_loss_bwd(H, W, y, f, f, **k, **phases)]
    for bad in (ws.cpu(), ws[::2]):
        refused += [lambda b=bad: lib.token_logprobs(H, W, y, ws=b), lambda b=bad: lib.token_logprobs_partial(H, W, y, 0, V, ws=b),
                    lambda b=bad: lib.offpolicy_loss_fwd(f, f, f, None, 1, N, ws=b)]
    refused += [lambda: lib.token_logprobs_partial(H, W, y, 0, V, m[:-1]), lambda: lib.token_logprobs_partial(H, W, y[:-1], 0, V),
                lambda: lib.offpolicy_loss_fwd(f, f, f, m, 1, N, targets=y[:-1], V=V)]
    out = f[:1].clone(), f.clone(), torch.zeros(5, device="cuda")
    refused += [lambda: lib.offpolicy_loss_fwd_static(f, f, f, m[:-1], 1, N, *out),
                lambda: lib.offpolicy_loss_fwd_static(f, f, f, m, 1, N, *out, targets=y[:-1], V=V)]
    for i, call in enumerate(refused):
        with pytest.raises(lib.LlamarlError) as e:
            call()
        assert e.value.status == lib.ERR_INVALID_ARG, i
    # larger ones are taken
    long = torch.zeros(N + 9, device="cuda")
    lib.offpolicy_loss_bwd(H, W, torch.cat([y, y[:9]]), long, long, dW=torch.empty(V + 3, d, dtype=W.dtype, device="cuda"),
                           dH=torch.empty(N + 1, d, dtype=H.dtype, device="cuda"), ws=ws.view(-1, 4).t())
    torch.cuda.synchronize()

"""The autograd wrapper: `loss.backward()` through `aipo_loss` must give the gradients the fp64 oracle gives for the
same upstream factor, for both storage types."""
import pytest
import torch

import synth
from parity_util import check_grad, f64, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,d,V,B,T", [("llama3_8b", 384, 2100, 3, 333), ("tiny_fp32", 256, 1024, 4, 64)])
def test_backward_through_the_wrapper_matches_the_oracle(lib, name, d, V, B, T):
    from paper_2505_24034_amd.autograd import aipo_loss
    base = synth.WORKLOADS[name]
    w = synth.scaled(base, d=d, V=V, B=B, T=T, len_lo=T // 4, len_hi=T, seed=77)
    x = synth.make_inputs(w, "cuda")
    H = x["H"].clone().requires_grad_(True)
    W = x["W"].clone().requires_grad_(True)
    loss, stats, logp = aipo_loss(H, W, x["targets"], x["mu_logp"], x["adv"], x["mask"], rho=1.1)
    assert loss.dim() == 0 and loss.requires_grad and not stats.requires_grad and not logp.requires_grad
    (3.0 * loss).backward()
    ref = run_oracle(x, rho=1.1, grad_loss=3.0)
    tol = 1e-4 if base.dtype == "f32" else 1e-2 * abs(ref["loss"]) + 1e-3
    assert abs(float(loss.detach()) - ref["loss"]) <= tol
    check_grad("H.grad", f64(H.grad), ref["dH"], base.dtype)
    check_grad("W.grad", f64(W.grad), ref["dW"], base.dtype)
    assert H.grad.dtype == H.dtype and W.grad.dtype == W.dtype


@pytest.mark.parametrize("name", ["llama3_8b", "tiny_fp32"])
@pytest.mark.parametrize("scale", [1.0, -2.5, 0.0, 1e-3])
def test_upstream_scalar_on_the_device(lib, name, scale):
    """the scale read on the device gives the bits of the scale passed from the host, through autograd as well; a
    non-finite one is refused and leaves no gradient"""
    from paper_2505_24034_amd.autograd import aipo_loss
    w = synth.scaled(synth.WORKLOADS[name], d=128, V=700, B=2, T=90, len_lo=20, len_hi=90, seed=78)
    x = synth.make_inputs(w, "cuda")
    H, W = x["H"].clone().requires_grad_(True), x["W"].clone().requires_grad_(True)

    def loss():
        return aipo_loss(H, W, x["targets"], x["mu_logp"], x["adv"], x["mask"], rho=1.1)[0]

    logp, lse = lib.token_logprobs(x["H"], x["W"], x["targets"], x["mask"].reshape(-1))
    _, coef, _ = lib.offpolicy_loss_fwd(logp, x["mu_logp"], x["adv"], x["mask"], 2, 90, rho=1.1, targets=x["targets"], V=700)
    dH, dW = lib.offpolicy_loss_bwd(x["H"], x["W"], x["targets"], lse, coef, grad_loss=scale)
    s = torch.tensor(scale, device="cuda")
    dH2, dW2 = lib.offpolicy_loss_bwd_device_scale(x["H"], x["W"], x["targets"], lse, coef, s)
    assert torch.equal(dH, dH2) and torch.equal(dW, dW2)
    loss().backward(gradient=s)
    assert torch.equal(H.grad, dH) and torch.equal(W.grad, dW)
    H.grad = W.grad = None
    for bad in (float("nan"), float("inf")):
        with pytest.raises(lib.LlamarlError):
            loss().backward(gradient=torch.tensor(bad, device="cuda"))
        assert H.grad is None and W.grad is None

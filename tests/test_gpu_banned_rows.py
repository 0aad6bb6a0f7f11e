"""A vocabulary row whose bias is -inf (a banned token) in the backward: its logits are -inf, its softmax and its gradient
are exactly zero, and the other rows and columns are what they are without it.  Positions past the active tokens are staged as
zero rows, against which such a row's logit is 0 * -inf: they must not reach the gradient."""
import pytest
import torch

from tile_util import loops
from test_gpu_f32_tiles import _inputs, _rel, _worst

pytestmark = pytest.mark.gpu


# active counts that leave 1 .. 63 positions of the last 64 empty
@pytest.mark.parametrize("dtype,N,V,d,loop", [
    ("bf16", 1, 300, 64, "64"), ("bf16", 100, 3000, 64, "64"), ("bf16", 383, 8065, 64, "128"), ("bf16", 500, 5003, 520, "128"),
    ("bf16", 31, 49200, 64, "256x128"), ("bf16", 150, 49200, 72, "256x160"), ("bf16", 300, 49200, 520, "256x160"),
    ("bf16", 1001, 49200, 136, "256x256"), ("bf16", 1275, 49200, 264, "256x256"),
    ("f32", 130, 300, 40, "64"), ("f32", 1, 700, 64, "64"), ("f32", 400, 9000, 40, "128"), ("f32", 1217, 8200, 260, "128"),
])
@pytest.mark.parametrize("masked", [False, True])
def test_banned_row_has_no_gradient(lib, dtype, N, V, d, loop, masked):
    assert loops(N, V, d, bf16=dtype == "bf16")[1] == loop
    H, W, t, coef = _inputs(N, V, d, N + d)
    if dtype == "bf16":
        H, W = H.bfloat16(), W.bfloat16()
    H[:, 0] = 1.0
    banned = torch.tensor([3, V // 2, V - 1], device="cuda")
    t = torch.where((t[:, None] == banned).any(1), torch.zeros_like(t), t)
    if masked:
        coef[2::3] = 0
    z = H.double() @ W.double().T
    z[:, banned] = -float("inf")
    W[banned, 0] = -float("inf")
    rlse = torch.logsumexp(z, dim=1)
    dz = -torch.exp(z - rlse[:, None])
    dz[torch.arange(N, device="cuda"), t.long()] += 1.0
    dz *= coef.double()[:, None]
    _, lse = lib.token_logprobs(H, W, t)
    assert float((lse.double() - rlse).abs().max()) <= 2e-5
    dH, dW = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    assert dW[banned].float().abs().nan_to_num(float("inf")).max().item() == 0.0
    # as test_tile_edges of either type
    rdW, rdH = dz.T @ H.double(), dz @ W.double()[:, 1:]         # column 0 of dH holds 0 * -inf
    tol = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -24 * (max(V, N, d) ** 0.5 + 16)
    assert _rel(dW, rdW) <= tol and _rel(dH[:, 1:], rdH) <= tol
    worst = 2 * tol if dtype == "bf16" else tol
    assert _worst(dW, rdW) <= worst and _worst(dH[:, 1:], rdH) <= worst

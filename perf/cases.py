"""Measured cases: what a trainer has this library do, through the entry points of the binding and the autograd op.

A case is a dict of plain values; `kind` says which call it makes:

  step      aipo_loss(...) and .backward(): token log-probs, off-policy loss and both gradients
  logprobs  token_logprobs alone: the reference policy's pass, scoring of finished generations
  backward  offpolicy_loss_bwd alone, optionally with an fp32 dW and in row passes with a bounded workspace
  shard     one rank's share of a vocabulary-parallel head: partial log-probs, merge with the other ranks' results,
            backward of the slice
  loss      offpolicy_loss_fwd alone on log-probs that are already there (several loss epochs over one batch)
  rewards   KL-shaped rewards and group advantages of a batch of generations

Sizes are those of the benchmark workloads (tiny fp32, Llama-3-8B / 70B heads, long reasoning), of the parity tests
and generic ones; B generations of T token slots, valid lengths uniform in [len_lo, T].
"""
import math

import torch

from paper_2505_24034_amd import binding as L
from paper_2505_24034_amd.autograd import aipo_loss

DEV = "cuda"
FULL_V = 128256
RHO = 2.0


def listed():
    return [
        # the smallest whole step: unit-test sized fp32 model, launch latency counts
        dict(name="step_fp32_tiny", kind="step", dtype="f32", d=256, V=1024, B=4, T=64, len_lo=16),
        # a small bf16 model with no size a multiple of a tile (debugging and CI runs of a trainer)
        dict(name="step_bf16_small_odd", kind="step", dtype="bf16", d=520, V=5003, B=3, T=347, len_lo=40),
        # fp32 run of a small model: numerics checks of a recipe before it goes to bf16
        dict(name="step_fp32_mid", kind="step", dtype="f32", d=516, V=20011, B=4, T=1200, len_lo=600),
        # a ~1B-class head, one micro-batch
        dict(name="step_bf16_mid", kind="step", dtype="bf16", d=1032, V=33001, B=5, T=1900, len_lo=950),
        # one short generation scored under an 8B head: few tokens against the whole vocabulary
        dict(name="logprobs_8b_one_short", kind="logprobs", dtype="bf16", d=4096, V=FULL_V, B=1, T=300, len_lo=300),
        # the reference policy's pass over a trainer batch at the 8B shape
        dict(name="logprobs_8b", kind="logprobs", dtype="bf16", d=4096, V=FULL_V, B=8, T=2048, len_lo=256),
        # the backward of the same batch
        dict(name="backward_8b", kind="backward", dtype="bf16", d=4096, V=FULL_V, B=8, T=2048, len_lo=256,
             dw_f32=False, max_rows=0),
        # long reasoning rollouts, fp32 head gradient, workspace bounded to 12288 active rows (two passes with work)
        dict(name="backward_long_bounded", kind="backward", dtype="bf16", d=4096, V=FULL_V, B=2, T=16384, len_lo=6000,
             dw_f32=True, max_rows=12288),
        # one of eight ranks of a vocabulary-parallel 70B head, one micro-batch
        dict(name="shard_70b_of_8", kind="shard", dtype="bf16", d=8192, V=FULL_V, shards=8, B=2, T=1500, len_lo=512),
        # the loss alone at the 8B batch size
        dict(name="loss_8b", kind="loss", B=8, T=2048, len_lo=256, per_token=False, norm=0, clip=0),
        # the loss over a whole rollout buffer, per-token advantages, sequence means, PPO clip
        dict(name="loss_buffer_4m", kind="loss", B=2048, T=2048, len_lo=256, per_token=True, norm=1, clip=1),
        # reward shaping of 16 prompts x 8 generations of up to 16 k tokens
        dict(name="rewards_long", kind="rewards", P=16, n=8, T=16384, len_lo=512, std=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "logprobs", "logprobs", "backward", "shard", "loss", "rewards"])
    if kind == "loss":
        T = _log_int(rng, 16, 16384)
        B = _log_int(rng, 1, max(2, min(2048, (1 << 22) // T)))
        return dict(kind=kind, B=B, T=T, len_lo=max(1, T // 8), per_token=rng.random() < 0.3,
                    norm=rng.randrange(3), clip=rng.randrange(2))
    if kind == "rewards":
        n = rng.choice([4, 8, 16])
        T = _log_int(rng, 64, 16384)
        P = _log_int(rng, 1, max(2, min(256, (1 << 22) // (n * T))))
        return dict(kind=kind, P=P, n=n, T=T, len_lo=max(1, T // 32), std=rng.random() < 0.5)
    dtype = "f32" if rng.random() < (0.3 if kind in ("step", "logprobs") else 0.0) else "bf16"
    while True:
        if dtype == "f32":
            d, V = 4 * _log_int(rng, 16, 512), _log_int(rng, 300, 40000)
            N = _log_int(rng, 32, 8192)
            limit = 6.0e11
        else:
            d = 8 * _log_int(rng, 16, 1024)
            V = FULL_V if rng.random() < 0.4 else _log_int(rng, 1000, FULL_V)
            N = _log_int(rng, 32, 24576)
            limit = 4.0e13
        if kind == "shard" and V < 8000:
            continue
        passes = {"step": 8, "logprobs": 2, "backward": 6, "shard": 2}[kind]
        if passes * N * V * d <= limit:
            break
    B = min(N, rng.choice([1, 2, 3, 4, 6, 8, 16]))
    T = N // B
    case = dict(kind=kind, dtype=dtype, d=d, V=V, B=B, T=T, len_lo=max(1, T // rng.choice([1, 2, 8])))
    if kind == "shard":
        case["shards"] = rng.choice([2, 4, 8])
    if kind == "backward":
        case["dw_f32"] = rng.random() < 0.4
        case["max_rows"] = 256 * max(1, N // 512) if rng.random() < 0.3 else 0
    return case


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 7)
    return g


def _rand(g, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype)


def _mask(g, B, T, len_lo):
    lo = min(len_lo, T)
    lens = lo + torch.floor(torch.rand(B, generator=g, device=DEV) * (T - lo + 1)).long().clamp_(max=T - lo)
    return (torch.arange(T, device=DEV)[None, :] < lens[:, None]).to(torch.uint8).contiguous()


def _advantages(g, B):
    a = _rand(g, B)
    return a if B == 1 else ((a - a.mean()) / (a.std(unbiased=False) + 1e-6)).contiguous()


def _drift(g, n):
    """log-ratio between the learner and the lagging generator: mostly small, a few tokens far off (those get clipped)"""
    return 0.08 * _rand(g, n) * torch.where(torch.rand(n, generator=g, device=DEV) < 0.03, 8.0, 1.0)


def _head(case, g):
    """H ~ N(0,1) (post-RMSNorm), W ~ N(0,1/d), tokens sampled from softmax(H W^T), the generator's log-probs a drift
    away from the learner's; lse and the shards' partials of the valid rows by plain fp32 products."""
    B, T, d, V = case["B"], case["T"], case["d"], case["V"]
    store = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    N = B * T
    H = _rand(g, N, d).to(store)
    W = (_rand(g, V, d) * d ** -0.5).to(store)
    mask = _mask(g, B, T, case["len_lo"])
    valid = mask.reshape(-1).nonzero()[:, 0]
    targets = torch.randint(0, V, (N,), generator=g, device=DEV)
    logp = torch.zeros(N, device=DEV)
    lse = torch.zeros(N, device=DEV)
    p = case.get("shards", 1)
    edges = [round(i * V / p) for i in range(p + 1)]
    m, s, zt = (torch.zeros(p, N, device=DEV) for _ in range(3))
    m.fill_(-math.inf)
    Wt = W.float().T
    for i in range(0, valid.numel(), 1024):
        r = valid[i:i + 1024]
        z = H[r].float() @ Wt
        u = torch.empty_like(z).exponential_(generator=g)
        y = torch.argmax(z - u.log_(), dim=1)                     # Gumbel-max: y ~ softmax(z)
        targets[r] = y
        zy = z.gather(1, y[:, None])[:, 0]
        lse[r] = torch.logsumexp(z, dim=1)
        logp[r] = zy - lse[r]
        if p > 1:
            for q in range(p):
                zq = z[:, edges[q]:edges[q + 1]]
                mq = zq.max(dim=1).values
                m[q, r] = mq
                s[q, r] = (zq - mq[:, None]).exp_().sum(dim=1)
                zt[q, r] = torch.where((y >= edges[q]) & (y < edges[q + 1]), zy, torch.zeros_like(zy))
        del z, u
    del Wt
    adv = _advantages(g, B)
    mu_logp = logp + _drift(g, N)
    coef = mask.reshape(-1).float() * -torch.exp(logp - mu_logp).clamp(max=RHO) * adv.repeat_interleave(T) / valid.numel()
    return dict(H=H, W=W, targets=targets.to(torch.int32), mask=mask, adv=adv, mu_logp=mu_logp, lse=lse, coef=coef,
                edges=edges, m=m, s=s, zt=zt)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    st = dict(case=case)
    if kind == "loss":
        B, T = case["B"], case["T"]
        logp = -2.0 * torch.empty(B * T, device=DEV).exponential_(generator=g)
        st.update(mask=_mask(g, B, T, case["len_lo"]), logp=logp, mu_logp=logp + _drift(g, B * T),
                  adv=_rand(g, B * T) if case["per_token"] else _advantages(g, B))
        return st
    if kind == "rewards":
        B, T = case["P"] * case["n"], case["T"]
        logp = -2.0 * torch.empty(B, T, device=DEV).exponential_(generator=g)
        st.update(mask=_mask(g, B, T, case["len_lo"]), logp=logp, base_logp=logp + 0.1 * _rand(g, B, T) - 0.005,
                  rewards=torch.where(torch.rand(B, generator=g, device=DEV) < 0.5, -1.0, 1.0).contiguous())
        return st
    x = _head(case, g)
    if kind == "step":
        x["H"].requires_grad_(True)
        x["W"].requires_grad_(True)
        keep = ("H", "W", "targets", "mu_logp", "adv", "mask")
    elif kind == "logprobs":
        keep = ("H", "W", "targets", "mask")
    elif kind == "backward":
        keep = ("H", "W", "targets", "lse", "coef")
    else:
        q = case["shards"] // 2                                    # a rank in the middle of the vocabulary
        v0, v1 = x["edges"][q], x["edges"][q + 1]
        others = [i for i in range(case["shards"]) if i != q]
        x["W_slice"] = x["W"][v0:v1].clone()
        x["v0"] = v0
        x["others"] = tuple(x[k][others].contiguous() for k in ("m", "s", "zt"))
        keep = ("H", "W_slice", "v0", "others", "targets", "mask", "coef")
    st.update({k: x[k] for k in keep})
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        st["H"].grad = None
        st["W"].grad = None
        loss, stats, logp = aipo_loss(st["H"], st["W"], st["targets"], st["mu_logp"], st["adv"], st["mask"], rho=RHO)
        loss.backward()
        return dict(loss=loss.detach(), stats=stats, logp=logp, dH=st["H"].grad, dW=st["W"].grad)
    if kind == "logprobs":
        logp, lse = L.token_logprobs(st["H"], st["W"], st["targets"], st["mask"].reshape(-1))
        return dict(logp=logp, lse=lse)
    if kind == "backward":
        dH, dW = L.offpolicy_loss_bwd(st["H"], st["W"], st["targets"], st["lse"], st["coef"],
                                      dW_dtype=torch.float32 if case["dw_f32"] else None,
                                      max_rows_per_pass=case["max_rows"] or None)
        return dict(dH=dH, dW=dW)
    if kind == "shard":
        m, s, zt = L.token_logprobs_partial(st["H"], st["W_slice"], st["targets"], st["v0"], case["V"],
                                            st["mask"].reshape(-1))
        every = [torch.cat([o, own[None]]) for o, own in zip(st["others"], (m, s, zt))]   # what an all-gather leaves
        logp, lse = L.merge_partials(*every)
        dH, dW = L.offpolicy_loss_bwd_slice(st["H"], st["W_slice"], st["targets"], st["v0"], lse, st["coef"])
        return dict(logp=logp, lse=lse, dH=dH, dW=dW)
    if kind == "loss":
        loss, coef, stats = L.offpolicy_loss_fwd(st["logp"], st["mu_logp"], st["adv"], st["mask"], case["B"], case["T"],
                                                 rho=RHO, norm_mode=case["norm"], clip_mode=case["clip"])
        return dict(loss=loss, coef=coef, stats=stats)
    shaped, kl = L.kl_shaped_rewards(st["rewards"], st["logp"], st["base_logp"], st["mask"], 0.05)
    adv = L.group_advantages(shaped, case["n"], normalise_std=case["std"])
    return dict(shaped=shaped, kl=kl, adv=adv)


def _mean_valid(case):
    return case["B"] * (min(case["len_lo"], case["T"]) + case["T"]) / 2.0


def work(case):
    """Mean number of valid tokens n; a contraction is 2 n V d.  Bytes: operands read once, results written once."""
    kind = case["kind"]
    if kind == "loss":
        n = case["B"] * case["T"]
        return dict(bytes=n * (4 + 4 + 1 + 4 + (4 if case["per_token"] else 0)) + 4 * case["B"] + 24, flops=20 * n)
    if kind == "rewards":
        n = case["P"] * case["n"] * case["T"]
        return dict(bytes=9 * n + 16 * case["P"] * case["n"], flops=2 * n)
    es = 4 if case["dtype"] == "f32" else 2
    N, d = case["B"] * case["T"], case["d"]
    V = case["V"] // case.get("shards", 1)
    n = _mean_valid(case)
    fwd_bytes = (V * d + n * d) * es + N * (4 + 1) + 8 * N
    bwd_bytes = (V * d + n * d + N * d) * es + V * d * (4 if case.get("dw_f32") else es) + 12 * N
    if kind == "logprobs":
        return dict(bytes=fwd_bytes, flops=2 * n * V * d)
    if kind == "backward":
        return dict(bytes=bwd_bytes, flops=6 * n * V * d)     # the logits have to be recomputed
    return dict(bytes=fwd_bytes + bwd_bytes + 12 * N, flops=8 * n * V * d)


def tolerance(case):
    # fp32 outputs of fp32 sums (bf16 products are exact in fp32): 1e-5.  Gradients in bf16 carry the rounding of the
    # staged dz and of the result, measured 2.3 - 2.5e-3 relative against 64 bits: four times that.
    if case["kind"] in ("loss", "rewards", "logprobs") or case["dtype"] == "f32":
        return dict(rel=1e-5)
    return dict(rel=1e-2)


def _exact_loss(case, logp, mu_logp, adv, mask, per_token, norm, clip):
    """logp, mu_logp float64 [N]; adv float64; returns loss [1], coef [N], stats [5]"""
    B, T = case["B"], case["T"]
    m = mask.reshape(-1).bool()
    A = adv if per_token else adv.repeat_interleave(T)
    lens = mask.reshape(B, T).sum(dim=1).double()
    nv = lens.sum().clamp(min=1.0)
    if norm == 0:
        Z = nv.expand(B * T)
    elif norm == 1:
        Z = ((lens > 0).sum().clamp(min=1) * lens.clamp(min=1.0)).repeat_interleave(T)
    else:
        Z = torch.full((B * T,), float(B), dtype=torch.float64, device=logp.device)
    delta = torch.where(m, logp - mu_logp, torch.zeros_like(logp))
    r = delta.exp()
    if clip == 0:
        coef = -r.clamp(max=RHO) * A / Z
        term = coef * logp
        clipped = r > RHO
    else:
        lo, hi = 1.0 - 0.2, 1.0 + 0.2
        u, k = r * A, r.clamp(lo, hi) * A
        coef = torch.where(u <= k, -A * r / Z, torch.zeros_like(r))
        term = -torch.minimum(u, k) / Z
        clipped = u > k
    zero = torch.zeros_like(logp)
    coef = torch.where(m, coef, zero)
    loss = torch.where(m, term, zero).sum()
    stats = torch.stack([lens.sum(), torch.where(m, r, zero).sum() / nv, (clipped & m).sum().double() / nv,
                         delta.sum() / nv, torch.zeros((), dtype=torch.float64, device=logp.device)])
    return loss.reshape(1), coef, stats


def _exact_forward(H, W, targets, valid):
    N = H.shape[0]
    logp = torch.zeros(N, dtype=torch.float64, device=DEV)
    lse = torch.zeros(N, dtype=torch.float64, device=DEV)
    W64 = W.double()
    for i in range(0, valid.numel(), 2048):
        r = valid[i:i + 2048]
        z = H[r].double() @ W64.T
        lse[r] = torch.logsumexp(z, dim=1)
        logp[r] = z.gather(1, targets[r].long()[:, None])[:, 0] - lse[r]
    return logp, lse


def _exact_backward(H, W, targets, v0, lse, coef, valid):
    """dH, dW of the rows [v0, v0 + V) of the head"""
    W64 = W.double()
    V = W64.shape[0]
    dH = torch.zeros(H.shape, dtype=torch.float64, device=DEV)
    dW = torch.zeros(W.shape, dtype=torch.float64, device=DEV)
    for i in range(0, valid.numel(), 2048):
        r = valid[i:i + 2048]
        Hr = H[r].double()
        dz = torch.exp(Hr @ W64.T - lse[r][:, None]).neg_()
        y = targets[r].long() - v0
        own = (y >= 0) & (y < V)
        dz[own.nonzero()[:, 0], y[own]] += 1.0
        dz *= coef[r][:, None]
        dH[r] = dz @ W64
        dW += dz.T @ Hr
    return dH, dW


def exact(case, seed):
    with torch.no_grad():
        st = prepare(case, seed)
        kind = case["kind"]
        if kind == "loss":
            loss, coef, stats = _exact_loss(case, st["logp"].double(), st["mu_logp"].double(), st["adv"].double(),
                                            st["mask"], case["per_token"], case["norm"], case["clip"])
            return dict(loss=loss, coef=coef, stats=stats)
        if kind == "rewards":
            m = st["mask"].bool()
            diff = st["logp"].double() - st["base_logp"].double()
            kl = torch.where(m, diff, torch.zeros_like(diff)).sum(dim=1)
            shaped = st["rewards"].double() - 0.05 * kl
            grp = shaped.reshape(case["P"], case["n"])
            adv = grp - grp.mean(dim=1, keepdim=True)
            if case["std"]:
                adv = adv / (grp.std(dim=1, unbiased=False, keepdim=True) + 1e-6)
            return dict(shaped=shaped, kl=kl, adv=adv.reshape(-1))
        if kind == "backward":
            valid = (st["coef"] != 0).nonzero()[:, 0]
            dH, dW = _exact_backward(st["H"], st["W"], st["targets"], 0, st["lse"].double(), st["coef"].double(), valid)
            return dict(dH=dH, dW=dW)
        valid = st["mask"].reshape(-1).nonzero()[:, 0]
        if kind == "logprobs":
            logp, lse = _exact_forward(st["H"], st["W"], st["targets"], valid)
            return dict(logp=logp, lse=lse)
        if kind == "shard":
            N = st["H"].shape[0]
            W64 = st["W_slice"].double()
            m, s, zt = (torch.cat([o.double(), torch.zeros(1, N, dtype=torch.float64, device=DEV)]) for o in st["others"])
            m[-1] = -math.inf
            for i in range(0, valid.numel(), 2048):
                r = valid[i:i + 2048]
                z = st["H"][r].double() @ W64.T
                m[-1, r] = z.max(dim=1).values
                s[-1, r] = torch.exp(z - m[-1, r][:, None]).sum(dim=1)
                y = st["targets"][r].long() - st["v0"]
                own = (y >= 0) & (y < W64.shape[0])
                zt[-1, r[own]] = z[own.nonzero()[:, 0], y[own]]
            lse = torch.zeros(N, dtype=torch.float64, device=DEV)
            logp = torch.zeros(N, dtype=torch.float64, device=DEV)
            lse[valid] = torch.logsumexp(m[:, valid] + s[:, valid].log(), dim=0)
            logp[valid] = zt[:, valid].sum(dim=0) - lse[valid]
            dH, dW = _exact_backward(st["H"], st["W_slice"], st["targets"], st["v0"], lse, st["coef"].double(), valid)
            return dict(logp=logp, lse=lse, dH=dH, dW=dW)
        H, W = st["H"].detach(), st["W"].detach()
        logp, lse = _exact_forward(H, W, st["targets"], valid)
        loss, coef, stats = _exact_loss(case, logp, st["mu_logp"].double(), st["adv"].double(), st["mask"], False, 0, 0)
        dH, dW = _exact_backward(H, W, st["targets"], 0, lse, coef, valid)
        return dict(loss=loss.reshape(()), stats=stats, logp=logp, dH=dH, dW=dW)

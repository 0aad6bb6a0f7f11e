"""bf16 contractions on every tile size and width: sizes at the edges of the tiles, of a K slab (64) and of the rules that pick
them, the loops at one slab and a few, against float64.  Each test asks the rules whether its sizes still reach what it names."""
import pytest
import torch

from tile_util import loops
from test_gpu_f32_tiles import _inputs, _reference, _rel, _worst

pytestmark = pytest.mark.gpu


# logits: bf16 products are exact in fp32, see the fp32 bound; gradients: dz and the results are rounded to bf16 once
# each, 2^-9 relative at most and independent per entry: 2 x 2^-9 bounds either result's relative error; twice that for a
# single row or column, whose sum can cancel to a fraction of its terms
@pytest.mark.parametrize("N,V,d,expected", [      # forward, dz, dH, dW
    (1, 64, 8, "64 64 64 64"),
    (64, 63, 64, "64 64 64 64"),
    (65, 129, 72, "64 64 64 64"),
    (127, 1025, 136, "64 64 64 64"),
    (129, 257, 200, "64 64 64 64"),
    (383, 5300, 136, "64 64 64 64"),
    (256, 8065, 64, "128 128 64 64"),
    (500, 24000, 72, "128 128 64 128"),
    (500, 5003, 520, "128 128 64 128"),
    (1041, 5003, 520, "128 128 128 128"),
    (300, 12000, 1032, "128 128 128 128"),
    (300, 24577, 64, "256x160 256x160 64 128"),      # 1 and 2 slabs
    (257, 33001, 128, "256x128 256x128 64 128"),
    (400, 32700, 136, "256x256 256x256 64 128"),      # 3 slabs
    (40, 33000, 1032, "128 128 64 256"),      # dW on 256-tiles, K of 1 and 2 slabs
    (70, 33000, 1032, "128 128 64 256"),
    (130, 33000, 520, "256x160 128 64 256"),      # ... of 3
    (200, 32768, 1024, "128 128 128 256"),      # full dW tiles, K of 4 slabs
    (330, 33000, 1024, "256x128 256x128 256 256"),      # ... of 6
    (260, 16384, 520, "128 128 64 128"),      # dH split along K
    (520, 16400, 2056, "256x256 256x256 256 256"),
])
@pytest.mark.parametrize("masked", [False, True])
def test_tile_edges(lib, N, V, d, expected, masked):
    assert " ".join(loops(N, V, d)) == expected
    H, W, t, coef = _inputs(N, V, d, 3 * N + V + d)
    H, W = H.bfloat16(), W.bfloat16()
    if masked:
        coef[1::3] = 0
    logp, lse = lib.token_logprobs(H, W, t)
    rlogp, rlse, rdH, rdW = _reference(H, W, t, coef)
    bound = 2.0 ** -24 * d ** 0.5
    assert float((lse.double() - rlse).abs().max()) <= 8 * bound + 2e-6
    assert float((logp.double() - rlogp).abs().max()) <= 16 * bound + 2e-6
    dH, dW = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    assert _rel(dH, rdH) <= 2.0 ** -8 and _rel(dW, rdW) <= 2.0 ** -8
    assert _worst(dH, rdH) <= 2.0 ** -7 and _worst(dW, rdW) <= 2.0 ** -7
    _, dW32 = lib.offpolicy_loss_bwd(H, W, t, lse, coef, dW_dtype=torch.float32)
    assert _rel(dW32, rdW) <= 2.0 ** -8 and _worst(dW32, rdW) <= 2.0 ** -7
    total = dW32.clone()
    lib.offpolicy_loss_bwd(H, W, t, lse, coef, dW=total, accumulate_dW=True)
    assert torch.equal(total, 2 * dW32)


@pytest.mark.parametrize("N", [1, 64, 127, 128, 129, 255, 256, 257, 320, 384, 385, 640])
@pytest.mark.parametrize("d", [64, 136, 264])                   # 1, 3 and 5 slabs
def test_narrow_last_token_column(lib, N, d):
    # 192 or more tiles of 256 x 256 at every N, on the widths that cost least: mostly 128 and 160
    assert all(x.startswith("256x") for x in loops(N, 49200, d)[:2])
    _check_head(lib, N, 49200, d)


# 256 columns: the last one holds 1 .. 256 tokens, half of the wavefronts idle up to 128; one tile a workgroup and two
@pytest.mark.parametrize("N", [1281, 1344, 1407, 1408, 1409, 1535, 1536, 3073, 3136, 3201])
@pytest.mark.parametrize("d", [40, 72, 136, 264])               # 1, 2, 3 and 5 slabs
def test_wide_last_token_column(lib, N, d):
    assert loops(N, 8200, d)[:2] == ("256x256", "256x256")
    _check_head(lib, N, 8200, d)


# 128 or 160 columns of tokens (dz of the last two sizes at short K: 128 x 128 tiles): one column, two, several, the last one
# full, of one token, of more than the left half; 1, 2, 3, 4 and 9 slabs of the three that are resident
@pytest.mark.parametrize("N,V", [(31, 49200), (128, 49200), (129, 49200), (159, 49200), (160, 49200), (300, 70000), (319, 70000),
                                 (320, 70000), (600, 33000), (900, 10487), (1700, 5412)])
@pytest.mark.parametrize("d", [8, 128, 192, 256, 520])
def test_narrow_token_tiles(lib, N, V, d):
    assert loops(N, V, d)[0] in ("256x128", "256x160")
    assert loops(N, V, d)[1] in ("256x128", "256x160") or (V < 20000 and d <= 128)
    _check_head(lib, N, V, d)


# 320 columns of tokens: one column, several, the last one of one token, of half of its wavefronts, full; 10, 11 and 17 slabs, the
# last one up to its half and past it; slabs taken from another one than the first on
@pytest.mark.parametrize("N,V", [(257, 49200), (320, 49200), (1041, 16380), (1280, 16380), (2241, 8190), (1601, 32700)])
@pytest.mark.parametrize("d", [584, 640, 648, 704, 1032])
def test_wide_token_tiles(lib, N, V, d):
    assert loops(N, V, d)[0] == "256x320"
    _check_head(lib, N, V, d)


# ... at 1, 2, 3, 5 and 9 slabs, the last one up to its half, past it and full
@pytest.mark.parametrize("N,V", [(257, 49200), (300, 49200), (320, 49200), (1041, 16380), (2241, 8190), (2300, 16032)])
@pytest.mark.parametrize("d", [8, 40, 72, 104, 168, 192, 264, 520, 576])
def test_wide_token_tiles_of_few_slabs(lib, N, V, d):
    assert loops(N, V, d)[0] == "256x320"
    _check_head(lib, N, V, d)


# 256 columns, slabs taken from another one than the first on up to 1024 tokens, in order beyond: one column of tiles, two, the last
# of each loop and the first of the other; whole slabs and a rest
@pytest.mark.parametrize("N,d", [(200, 264), (256, 576), (500, 576), (500, 520), (1024, 264), (1024, 520), (1025, 264), (1025, 520)])
def test_turned_slabs(lib, N, d):
    assert loops(N, 49200, d)[:2] == ("256x256", "256x256")
    _check_head(lib, N, 49200, d)


# the last slab up to its half, just past it and full, alone and after others: 128 x 128 tiles, 160 columns, 128 and 256
@pytest.mark.parametrize("d", [32, 40, 64, 96, 104, 160, 168])
@pytest.mark.parametrize("N,V", [(40, 33000), (400, 33000), (1000, 49200)])
def test_last_slab(lib, N, V, d):
    assert loops(N, V, d)[0] == {40: "128", 400: "256x160", 1000: "256x256" if d > 104 else "256x128"}[N]
    _check_head(lib, N, V, d)


# ... 256 columns throughout
@pytest.mark.parametrize("d", [32, 40, 96, 104, 128, 160, 168])
def test_last_slab_of_wide_tiles(lib, d):
    assert loops(1409, 8200, d)[:2] == ("256x256", "256x256")
    _check_head(lib, 1409, 8200, d)


# dH on tiles of 160, 192, 224 and 256 columns, its rows past the last whole tile in one half and in both
@pytest.mark.parametrize("N,V,d", [(6700, 8200, 264), (4000, 8200, 520), (2100, 8200, 1032), (2200, 8200, 1288),
                                   (2305, 8200, 1160), (4100, 8200, 1024)])
def test_narrow_gradient_tiles(lib, N, V, d):
    assert loops(N, V, d)[2] == "256"
    _check_head(lib, N, V, d)


# dz^T is written as far as dW reads it, the next 32 active rows: with NaN in what nothing writes, the gradients are the same
@pytest.mark.parametrize("N,V,d,expected", [(129, 49200, 72, "256x160 64 128"), (160, 49200, 520, "256x160 64 256"),
                                            (450, 33000, 1032, "256x160 256 256"), (97, 49200, 264, "256x128 64 256"),
                                            (65, 900, 64, "64 64 64"), (400, 8065, 64, "128 64 64")])
def test_dz_past_what_is_written(lib, N, V, d, expected):
    assert " ".join(loops(N, V, d)[1:]) == expected
    H, W, t, coef = _inputs(N, V, d, N + d)
    H, W = H.bfloat16(), W.bfloat16()
    _, lse = lib.token_logprobs(H, W, t)
    plain = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    ws = torch.full((lib.workspace_bytes(N, d, V, lib.BF16, lib.PASS_LOSS_BWD),), 255, dtype=torch.uint8, device="cuda")
    poisoned = lib.offpolicy_loss_bwd(H, W, t, lse, coef, ws=ws)
    assert all(torch.equal(a, b) for a, b in zip(plain, poisoned))


# dH in up to 32 parts a tile: 64-, 128- and 256-tiles, a last round that fills every XCD and one that does not
@pytest.mark.parametrize("N,V,d,edge", [(1, 70000, 64, "64"), (64, 40000, 512, "64"), (129, 33000, 520, "64"), (300, 70000, 264, "64"),
                                        (300, 70000, 1032, "256"), (520, 60000, 776, "256"), (140, 20000, 2048, "128")])
def test_many_parts(lib, N, V, d, edge):
    assert loops(N, V, d)[2] == edge
    _check_head(lib, N, V, d)


def _check_head(lib, N, V, d):
    H, W, t, coef = _inputs(N, V, d, N + d)
    H, W = H.bfloat16(), W.bfloat16()
    t[0] = V - 1
    logp, lse = lib.token_logprobs(H, W, t)
    rlogp, rlse, rdH, rdW = _reference(H, W, t, coef)
    bound = 2.0 ** -24 * d ** 0.5
    assert float((lse.double() - rlse).abs().max()) <= 8 * bound + 2e-6
    assert float((logp.double() - rlogp).abs().max()) <= 16 * bound + 2e-6
    dH, dW = lib.offpolicy_loss_bwd(H, W, t, lse, coef)
    assert _rel(dH, rdH) <= 2.0 ** -8 and _rel(dW, rdW) <= 2.0 ** -8
    assert _worst(dH, rdH) <= 2.0 ** -7 and _worst(dW, rdW) <= 2.0 ** -7

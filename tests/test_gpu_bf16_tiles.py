"""bf16 contractions on the three tile sizes: sizes at the edges of the tiles, of a K slab (64) and of the rule that
picks the tile, and the 256 x 256 loops at one, two and three slabs, against float64."""
import pytest
import torch

from test_gpu_f32_tiles import _inputs, _reference, _rel, _worst

pytestmark = pytest.mark.gpu


# logits: bf16 products are exact in fp32, see the fp32 bound; gradients: dz and the results are rounded to bf16 once
# each, 2^-9 relative at most and independent per entry: 2 x 2^-9 bounds either result's relative error; twice that for a
# single row or column, whose sum can cancel to a fraction of its terms
@pytest.mark.parametrize("N,V,d", [
    (1, 64, 8), (64, 63, 64), (65, 129, 72), (127, 1025, 136), (129, 257, 200),       # 64-tiles
    (256, 8065, 64), (383, 5300, 136), (500, 24000, 72),                               # 128-tiles
    (300, 24577, 64), (257, 33001, 128), (400, 32700, 136),                            # 256-tiles, K of 1, 2, 3 slabs
    (40, 33000, 1032), (70, 33000, 1032), (130, 33000, 520),                           # dW on 256-tiles, K of 1, 2, 3 slabs
    (200, 32768, 1024), (330, 33000, 1024),                                            # full dW tiles, K of 4 and 6 slabs
    (260, 16384, 520), (520, 16400, 2056),                                             # dH on 128- and 256-tiles, split along K
])
@pytest.mark.parametrize("masked", [False, True])
def test_tile_edges(lib, N, V, d, masked):
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
    # 192 or more tiles of 256 x 256 at every N: the last column holds 1 .. 256 tokens, half of the wavefronts idle up to 128
    _check_head(lib, N, 49200, d)


# 128 or 160 columns of tokens: one column, two, several, the last one full, of one token, of more than the left half;
# 1, 2, 3, 4 and 9 slabs of the three that are resident
@pytest.mark.parametrize("N,V", [(31, 49200), (128, 49200), (129, 49200), (159, 49200), (160, 49200), (300, 49200), (319, 49200),
                                 (320, 49200), (600, 33000), (900, 10487), (1700, 5412)])
@pytest.mark.parametrize("d", [8, 128, 192, 256, 520])
def test_narrow_token_tiles(lib, N, V, d):
    _check_head(lib, N, V, d)


# the last slab up to its half, just past it and full, alone and after another: narrow tiles, 256 and 64 columns
@pytest.mark.parametrize("d", [32, 40, 64, 96, 104, 160, 168])
@pytest.mark.parametrize("N,V", [(40, 33000), (400, 33000), (1000, 49200)])
def test_last_slab(lib, N, V, d):
    _check_head(lib, N, V, d)


# dH on tiles of 160, 192, 224 and 256 columns, its rows past the last whole tile in one half and in both
@pytest.mark.parametrize("N,V,d", [(6700, 8200, 264), (4000, 8200, 520), (2100, 8200, 1032), (2200, 8200, 1288),
                                   (2305, 8200, 1160), (4100, 8200, 1024)])
def test_narrow_gradient_tiles(lib, N, V, d):
    _check_head(lib, N, V, d)


# dH in up to 32 parts a tile: 64-, 128- and 256-tiles, a last round that fills every XCD and one that does not
@pytest.mark.parametrize("N,V,d", [(1, 70000, 64), (64, 40000, 512), (129, 33000, 520), (300, 70000, 264), (300, 70000, 1032),
                                   (520, 60000, 776), (140, 20000, 2048)])
def test_many_parts(lib, N, V, d):
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

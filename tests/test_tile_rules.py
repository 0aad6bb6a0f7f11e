"""The rules by which the library cuts its contractions into tiles and deals them out, asked for on the CPU."""
import pytest

from paper_2505_24034_amd import binding


@pytest.fixture(scope="module")
def rules():
    return binding._load_native()


# 256 workgroups are an MI355X's; others a part with fewer CUs, or a small problem's
@pytest.mark.parametrize("workgroups", [1, 3, 7, 8, 12, 60, 64, 100, 120, 228, 248, 252, 256, 304, 512])
def test_every_tile_is_taken_once(rules, workgroups):
    for tiles_m in (1, 2, 3, 4, 5, 21, 63, 64, 130, 501):
        for tiles_n in (1, 2, 3, 4, 5, 7, 8, 15, 32):
            walks = rules.tile_walk(tiles_m, tiles_n, workgroups)
            assert sorted(t for w in walks for t in w) == list(range(tiles_m * tiles_n)), (tiles_m, tiles_n)
            rounds = -(-tiles_m * tiles_n // workgroups)
            if workgroups >= 8 and workgroups % 8 == 0:
                assert max(map(len, walks)) == rounds


def test_the_columns_that_hold_tokens_write_all_of_dz(rules):
    # a column of tiles past them would walk all of W for zeros, at a cost the width rule does not count
    for bf16, widths in ((1, (64, 128, 160, 256)), (0, (64, 128))):
        for n in range(1, 3000):
            read = rules.dz_columns(n, bf16)
            assert n <= read < n + 64
            assert all(-(-read // w) == -(-n // w) for w in widths), (n, bf16)

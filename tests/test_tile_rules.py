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


# forward call and dz at (N, V, d) on an MI355X, microseconds on tiles of 256 vocabulary rows and on 128 x 128 ones
MEASURED = [
    ((1024, 8192, 1024), (27.2, 28.3), (24.6, 24.0)), ((1041, 5003, 520), (19.8, 20.4), (19.3, 17.6)),
    ((882, 10487, 7808), (126.7, 203.7), (128.8, 225.8)), ((1700, 5412, 1888), (42.7, 66.9), (40.2, 63.7)),
    ((256, 33000, 1024), (38.5, 35.3), (37.6, 31.5)), ((300, 16400, 512), (19.5, 19.1), (17.3, 15.6)),
    ((512, 12000, 512), (19.1, 18.9), (17.3, 15.7)), ((512, 12000, 2048), (35.6, 38.0), (32.3, 34.0)),
    ((512, 24000, 1024), (36.8, 43.2), (33.8, 38.6)), ((700, 8192, 1024), (24.5, 24.6), (22.4, 21.4)),
    ((2000, 5003, 1024), (35.9, 42.0), (34.2, 38.2)), ((2000, 5003, 4096), (101.3, 121.7), (98.7, 117.9)),
    ((3000, 3000, 1024), (29.7, 39.4), (26.4, 36.6)), ((4096, 2048, 512), (20.1, 19.9), (18.6, 16.2)),
    ((4000, 2048, 2048), (39.4, 42.3), (36.5, 37.6)), ((1024, 8192, 512), (19.0, 19.0), (18.2, 16.2)),
    ((1024, 8192, 256), (16.3, 15.6), (15.4, 13.0)), ((1024, 8192, 4096), (62.7, 70.1), (60.7, 66.5)),
    ((1500, 6000, 520), (22.3, 29.8), (21.2, 28.8)), ((1500, 6000, 1032), (31.2, 48.1), (28.9, 45.1)),
    ((640, 10000, 264), (17.3, 16.9), (17.1, 14.8)), ((640, 16032, 1024), (29.5, 42.0), (26.2, 37.7)),
    ((1000, 10000, 1024), (36.1, 41.2), (33.8, 37.8)), ((2048, 4096, 264), (18.0, 17.6), (17.1, 14.6)),
    ((8000, 1024, 512), (20.7, 20.2), (18.4, 16.1)), ((10000, 1024, 2048), (45.1, 69.4), (41.9, 64.7)),
    ((400, 24000, 4096), (94.0, 119.6), (117.9, 133.6)), ((600, 7000, 512), (18.6, 18.0), (18.0, 15.5)),
]


@pytest.mark.parametrize("shape,forward,dz", MEASURED)
def test_the_tile_rule_takes_what_measured_faster(rules, shape, forward, dz):
    for backward, (wide, small) in enumerate((forward, dz)):
        taken = wide if rules.logits_tile(*shape, 1, backward) == 256 else small
        assert taken <= 1.04 * min(wide, small), ("forward", "dz")[backward]

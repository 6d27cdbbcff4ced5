"""Host-side checks of what the LM-head pass runs on: no GPU needed."""
import pytest

from plan import plan

CUS = 256


@pytest.mark.parametrize("V", [20000, 126464, 152064])
@pytest.mark.parametrize("rows", [32769, 40000, 49153, 65535, 65536, 65537, 131072, 1 << 20])
def test_many_rows_take_the_fewest_rounds(rows, V):
    """Where a row tile's share is the whole vocabulary, the tile with the
    fewest rounds of workgroups."""
    tile, wgs, _ = plan(rows, 8, V, 8)
    assert wgs == -(-rows // tile)
    assert -(-wgs // CUS) == -(-rows // (256 * CUS))


@pytest.mark.parametrize("rows,d,V,want", [
    (4, 768, 20000, 0), (32, 2048, 50000, 0), (64, 1024, 126464, 0), (256, 4096, 32000, 0), (32, 4096, 32768, 0),
    (32, 4096, 32769, 1), (256, 4096, 50000, 1), (1, 4096, 126464, 1), (64, 3584, 152064, 1),
    (512, 4096, 126464, 0), (32, 4104, 126464, 0),
])
def test_only_an_lm_head_beyond_the_last_level_cache_is_streamed(rows, d, V, want):
    """Non-temporal copies: one row tile, rows of whole lines, over 256 MiB."""
    assert plan(rows, d, V, 8)[2] == want


@pytest.mark.parametrize("rows", [33, 64, 65, 128])
def test_shares_hold_a_whole_tile(rows):
    """At 33 to 128 rows thresholds are seeded from a whole 256-token tile:
    below 256 shares of one tile (cut at multiples of 16) every share but the
    last is a run of whole tiles."""
    for V in (20000, 32768, 33000, 50000, 65536, 69631):
        assert plan(rows, 2048, V, 8)[1] <= -(-V // 256), V
    assert plan(rows, 2048, 69632, 8)[1] == CUS

"""Host-side checks of what the LM-head pass runs on: no GPU needed."""
import ctypes

import pytest

import paper_2609_33390_amd as brisk

CUS = 256


def _plan(rows, V, K):
    fn = getattr(brisk.lib(), "_ZN5brisk17propose_plan_infoEiiiPi")   # internal, not part of the C ABI
    out = (ctypes.c_int * 2)()
    fn(rows, V, K, out)
    return list(out)


@pytest.mark.parametrize("V", [20000, 126464, 152064])
@pytest.mark.parametrize("rows", [32769, 40000, 49153, 65535, 65536, 65537, 131072, 1 << 20])
def test_many_rows_take_the_fewest_rounds(rows, V):
    """Where a row tile's share is the whole vocabulary, the tile with the
    fewest rounds of workgroups."""
    tile, wgs = _plan(rows, V, 8)
    assert wgs == -(-rows // tile)
    assert -(-wgs // CUS) == -(-rows // (256 * CUS))

"""What the LM-head pass runs on, from the library's host code."""
import ctypes

import paper_2609_33390_amd as brisk


def plan(rows, d, V, K):
    """Rows of a row tile, workgroups, non-temporal lm_head copies."""
    fn = getattr(brisk.lib(), "_ZN5brisk17propose_plan_infoEiiiiPi")   # internal, not part of the C ABI
    out = (ctypes.c_int * 3)()
    fn(rows, d, V, K, out)
    return list(out)

"""Default tile limits per segment (CPU, plans interpreted in numpy)."""
import pytest

import workloads as W
from tests.test_planner import check_plan


@pytest.mark.parametrize("n", [10, 13, 14, 15, 17])
@pytest.mark.parametrize("kind", ["tfim", "qpe", "qft_mixed"])
def test_default_tiles_per_segment(n, kind):
    """13 bits with QFT stages, the smallest tile with the same number of groups
    otherwise; what the plan does is unchanged."""
    if kind == "tfim":
        stream = W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 2)
    elif kind == "qpe":
        stream = W.qpe_ladder_stream(n - 1, 0.4)
    else:
        stream = (W.qft_stream(n) + W.random_stream(n, 40, n) + W.random_perm_block(n, 20, n)
                  + W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 1))
    d = check_plan(n, stream, window_k=-1)
    sizes = [L["L"] + L["h"] for L in d["layers"] if L["kind"] == "tile"]
    if kind == "tfim":
        assert max(sizes) == {10: 10, 13: 13, 14: 10, 15: 10, 17: 11}[n]
    else:
        assert max(sizes) <= 13
    # a limit given by the caller holds as before
    d = check_plan(n, stream, window_k=-1, max_tile_bits=13)
    assert max(L["L"] + L["h"] for L in d["layers"] if L["kind"] == "tile") == min(n, 13)

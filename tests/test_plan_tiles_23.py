"""Default tile limits at 23 qubits (CPU): 13 bits leave two high groups of five
bits there, which segments without diagonal layers keep."""
import numpy as np
import pytest

import workloads as W


def _tiles(n, gates, **opts):
    import paper_2609_19147_amd as qs
    d = qs.Plan(n, gates, window_k=-1, **opts).describe()
    return [(L["L"], L["h"]) for L in d["layers"] if L["kind"] == "tile"]


@pytest.mark.parametrize("n,bits", [(22, 13), (23, 13), (24, 12), (25, 12)])
@pytest.mark.parametrize("kind", ["wht", "product", "permuted"])
def test_product_segments(kind, n, bits):
    rng = np.random.default_rng(n)
    u = [W.G("U", q, mat=W.random_unitary(2, rng)) for q in range(n)]
    gates = {"wht": W.wht_stream(n), "product": u, "permuted": u + W.random_perm_block(n, 30, 1) + u}[kind]
    tiles = _tiles(n, gates)
    assert {L + h for L, h in tiles} == {bits}
    assert len(tiles) == len(_tiles(n, gates, max_tile_bits=13))  # no pass more


@pytest.mark.parametrize("n,bits", [(22, 13), (23, 12), (24, 12)])
def test_segments_with_diagonals(n, bits):
    tiles = _tiles(n, W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 1))
    assert max(L + h for L, h in tiles) == bits

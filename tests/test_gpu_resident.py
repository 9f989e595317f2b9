"""Layers on both sides of the sizes where states stay in the last-level cache
(32, 128 and 256 MiB): phase layers against closed form, tile passes and dense
blocks against the per-gate path."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _state(qs, n, dtype, seed):
    st = qs.State(n, dtype, init=None)
    W.gaussian_state_torch(n, seed, dtype, out=st.tensor())
    return st


@pytest.mark.parametrize("n,dtype", [(21, "c64"), (22, "c64"), (25, "c64"), (26, "c64"), (20, "c128"), (21, "c128"),
                                     (24, "c128"), (25, "c128")])
def test_phase_layer_closed_form(n, dtype):
    import torch
    import paper_2609_19147_amd as qs
    st = _state(qs, n, dtype, n)
    ref = st.tensor().to(torch.complex128)
    th = 0.37
    i = torch.arange(1 << n, device="cuda")
    x = (i ^ (i >> 1)) & ((1 << (n - 1)) - 1)
    cnt = torch.zeros_like(i)
    for b in range(n - 1):
        cnt += (x >> b) & 1
    ref *= torch.polar(torch.ones(1 << n, dtype=torch.float64, device="cuda"), th * cnt.double() - 0.5 * th * (n - 1))
    plan = qs.Plan(n, [W.G("RZZ", q, q + 1, theta=th) for q in range(n - 1)])
    assert [L["kind"] for L in plan.describe()["layers"]] == ["diag"]
    qs.apply(st, plan)
    err = torch.linalg.vector_norm(st.tensor().to(torch.complex128) - ref).item()
    # one rounded phase and one complex product per amplitude of a unit vector
    assert err <= (4e-7 if dtype == "c64" else 1e-15 * 4)


@pytest.mark.parametrize("n,dtype", [(23, "c64"), (24, "c64"), (25, "c64"), (26, "c64"), (24, "c128")])
def test_tile_and_dense_layers_against_plain(n, dtype):
    import torch
    import paper_2609_19147_amd as qs
    stream = (W.dense_block_stream(n, 1, 4, n) + W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 1)
              + W.dense_block_stream(n, 1, 5, n + 1) + W.wht_stream(n) + W.dense_block_stream(n, 1, 6, n + 2))
    a, b = _state(qs, n, dtype, n), _state(qs, n, dtype, n)
    fused, plain = qs.Plan(n, stream), qs.Plan(n, stream, mode="plain")
    nrm = qs.apply_norm2(a, fused)
    qs.apply(b, plain)
    assert abs(nrm - 1.0) <= (1e-5 if dtype == "c64" else 1e-12)
    err = torch.linalg.vector_norm((a.tensor() - b.tensor()).to(torch.complex128)).item()
    assert err <= (1e-5 if dtype == "c64" else 1e-12)  # the relative L2 parity bars

"""Rounds over the same register bits that run as one (QFT stages, forward and
inverse, with Hadamards and single-qubit windows between them) against the
per-gate path."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _streams(n):
    qft, wht = W.qft_stream(n), W.wht_stream(n)
    rx = [W.G("RY", q, theta=0.3 + 0.1 * q) for q in range(n)]
    return {"qft": qft, "qft_wht": qft + wht, "qft_windows": qft + rx + qft, "phase_estimation": W.qpe_ladder_stream(n - 1, 0.7)}


@pytest.mark.parametrize("name", ["qft", "qft_wht", "qft_windows", "phase_estimation"])
@pytest.mark.parametrize("n,bits,dtype", [(11, 0, "c64"), (15, 10, "c64"), (17, 0, "c128"), (18, 11, "c64"),
                                          (18, 12, "c128"), (19, 13, "c128"), (20, 0, "c64"), (21, 14, "c64"),
                                          (21, 13, "c128")])
def test_against_plain(n, bits, dtype, name):
    import torch
    import paper_2609_19147_amd as qs
    stream = _streams(n)[name]
    a, b = qs.State(n, dtype, init=None), qs.State(n, dtype, init=None)
    W.gaussian_state_torch(n, n, dtype, out=a.tensor())
    b.tensor().copy_(a.tensor())
    psi0 = a.tensor().clone()
    fused = qs.Plan(n, stream, max_tile_bits=bits) if bits else qs.Plan(n, stream)
    qs.apply(a, fused)
    qs.apply(b, qs.Plan(n, stream, mode="plain"))
    bar = 1e-5 if dtype == "c64" else 1e-12  # the relative L2 parity bars
    assert torch.linalg.vector_norm((a.tensor() - b.tensor()).to(torch.complex128)).item() <= bar
    qs.apply(a, fused.inverse())
    assert torch.linalg.vector_norm((a.tensor() - psi0).to(torch.complex128)).item() <= bar

"""Gradients of plans whose tiles are too large for the two-state passes."""
import numpy as np
import pytest

import workloads as W
from oracle import gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [13, 14])
def test_complex128_13_bit_tiles(n):
    """2^13 complex128 amplitudes of two states do not fit in LDS: every
    parameter's sums come from the per-bit reductions."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    stream = W.hea_stream(n, 1)
    params = W.hea_params(n, 1, n)
    terms = W.xxz_terms(n)
    plan = qs.Plan(n, stream, n_params=len(params), params=params, max_tile_bits=13)
    e, g = qs.adjoint_grad(qs.State(n, "c128"), plan, terms)
    ref = gradients.parameter_shift(n, stream, params, terms)
    assert np.max(np.abs(g - ref)) <= 1e-11  # the complex128 gradient bar

"""States of one tile: layer sequences run as one launch (apply) and one
backward launch (adjoint), at the sizes where the launch shape changes, against
the oracle; partial layer ranges and plans that cannot run as a sequence."""
import numpy as np
import pytest

import workloads as W
from oracle import gradients, statevec as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [4, 5, 7, 10, 12, 13, 14])
def test_sequences_and_ranges(n, dtype):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    stream = (W.tfim_strang_stream(n, 1.0, 0.8, 0.3, 6) + W.random_perm_block(n, 30, n) + W.random_stream(n, 60, n)
              + W.random_perm_block(n, 30, n + 1) + W.qft_stream(n))
    plan = qs.Plan(n, stream, window_k=-1)
    psi = W.gaussian_state(n, n).astype(np.complex64 if dtype == "c64" else np.complex128)
    ref = sv.run(psi.astype(np.complex128), n, stream)
    bar = 1e-5 if dtype == "c64" else 1e-12
    st = qs.State(n, dtype, init=None).upload(psi)
    qs.apply(st, plan)
    assert np.linalg.norm(st.download() - ref) <= bar
    # any split of the layers, the recorded graph, the fused norm and the way back
    L = plan.num_layers()
    st.upload(psi)
    cut = [0, 1, L // 2, L]
    for a, b in zip(cut, cut[1:]):
        qs.apply(st, plan, a, b - a)
    assert np.linalg.norm(st.download() - ref) <= bar
    for _ in range(3):
        st.upload(psi)
        qs.apply_graph(st, plan)
        assert np.linalg.norm(st.download() - ref) <= bar
    st.upload(psi)
    assert abs(qs.apply_norm2(st, plan) - np.linalg.norm(psi.astype(np.complex128)) ** 2) <= bar
    qs.apply(st, plan.inverse())
    assert np.linalg.norm(st.download() - psi) <= 2 * bar


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [4, 6, 9, 11, 12, 13])
def test_backward_sequence(n, dtype):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    layers = 2
    stream = W.hea_stream(n, layers)
    params = W.hea_params(n, layers, n)
    terms = W.xxz_terms(n) + W.x_terms(n)
    plan = qs.Plan(n, stream, n_params=len(params))
    st = qs.State(n, dtype, init=None)
    for shift in (0.0, 0.4):  # tables updated in between
        plan.set_params(params + shift)
        e, g = qs.adjoint_grad(st.set_basis(0), plan, terms)
        zero = sv.basis(n, 0)
        psi = sv.run(zero, n, stream, params + shift)
        assert abs(e - sv.expect(psi, n, terms)) <= (1e-5 if dtype == "c64" else 1e-11) * n
        pick = np.random.default_rng(n).choice(len(params), size=6, replace=False)
        for k in pick:
            p1, p2 = (params + shift).copy(), (params + shift).copy()
            p1[k] += np.pi / 2
            p2[k] -= np.pi / 2
            ref = 0.5 * (sv.expect(sv.run(zero, n, stream, p1), n, terms) - sv.expect(sv.run(zero, n, stream, p2), n, terms))
            assert abs(g[k] - ref) <= (1e-5 if dtype == "c64" else 1e-11) * n
        assert np.linalg.norm(st.download() - psi) <= (1e-5 if dtype == "c64" else 1e-12)

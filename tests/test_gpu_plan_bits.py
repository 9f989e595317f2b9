"""Plans of the same gates give the same bits."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [14, 16, 20])
def test_plans_of_the_same_gates_agree_in_every_bit(n, dtype):
    """Whatever the host's memory held where their tables are built (the choice of a QFT round's form
    depended on it)."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    layers = W.qft_stream(n) + W.wht_stream(n)
    psi = W.gaussian_state(n, n)
    st = qs.State(n, dtype, init=None)
    first, others = None, []
    for k in range(24):
        other = qs.Plan(n, layers + W.random_perm_block(n, 5 * k + 1, k))
        qs.apply(st, other)
        others.append(other)
        if k % 3 == 0:
            others.append(qs.Plan(n, W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 1 + k)))
        if k % 4 == 0:
            others = others[::2]
        st.upload(psi)
        qs.apply(st, qs.Plan(n, layers))
        got = st.download()
        first = got if first is None else first
        assert np.array_equal(got, first), k

"""Marginals over selections below, above and across the row boundary (9 state
bits), and block masses of partial sub-blocks and blocks, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import readout

pytestmark = pytest.mark.gpu


def _pick(n, which, rng):
    bits = {"low": range(0, min(n, 9)), "high": range(9, n), "mixed": range(n), "edge": [b for b in (0, 8, 9) if b < n],
            "none_low": range(max(0, n - 5), n), "sixteen": rng.permutation(n)[:16]}[which]
    bits = list(bits)[:16] if which != "mixed" else [int(b) for b in rng.choice(n, size=min(n, 7), replace=False)]
    return sorted(n - 1 - int(b) for b in bits)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("which", ["low", "high", "mixed", "edge", "none_low", "sixteen"])
@pytest.mark.parametrize("n", [2, 8, 9, 10, 13, 18])
def test_marginal_rows(n, which, dtype):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(n)
    sel = _pick(n, which, rng)
    if not sel:
        pytest.skip("no such bits at this size")
    psi = W.gaussian_state(n, 40 + n).astype(np.complex64 if dtype == "c64" else np.complex128)
    st = qs.State(n, dtype, init=None).upload(psi)
    ref = readout.marginal(psi.astype(np.complex128), n, sel)
    # FP64 sums of non-negative terms in another order
    assert np.allclose(qs.marginal(st, sel), ref, rtol=1e-12, atol=0)


@pytest.mark.parametrize("n", [4, 6, 8, 14, 16])
def test_scaled_and_massless_states(n):
    """Draws follow |psi|^2 / ||psi||^2 whatever the norm; no mass is an error."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    psi = W.gaussian_state(n, n)
    u = np.random.default_rng(n).random(200)
    st = qs.State(n, "c128", init=None)
    one = qs.sample(st.upload(psi), u)
    assert np.array_equal(qs.sample(st.upload(4.0 * psi), u), one)
    for bad in (0.0 * psi, np.where(np.arange(1 << n) == 1, np.nan, psi)):
        st.upload(bad)
        with pytest.raises(qs.QsError):
            qs.sample(st, u)
        with pytest.raises(qs.QsError):
            qs.sample_noalloc(st, u)
    assert np.array_equal(qs.sample(st.upload(psi), u), one)

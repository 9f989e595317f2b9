"""Which Pauli sums of a few terms take a reduction and which the tile sets, and
their values against torch in FP64."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,few_z,few_x", [("c64", 22, 0, 0), ("c64", 23, 2, 1), ("c128", 21, 0, 0),
                                                 ("c128", 22, 8, 4)])
def test_few_terms_of_one_mask(dtype, n, few_z, few_x):
    """From 64 MiB on, up to few_z Z-type terms (few_x of one X mask) alone are one
    reduction; one more, or a second mask, goes to the tile sets."""
    import torch
    import paper_2609_19147_amd as qs
    st = qs.State(n, dtype, init=None)
    W.gaussian_state_torch(n, 7, dtype, out=st.tensor())
    psi = st.tensor().to(torch.complex128)
    idx = torch.arange(1 << n, device="cuda")

    def mask(m):  # qubit q is index bit n - 1 - q
        return sum(1 << (n - 1 - q) for q in range(n) if m >> q & 1)

    def exact(term):
        c, xm, zm = term
        par = idx & mask(zm)
        for sh in (16, 8, 4, 2, 1):
            par = par ^ (par >> sh)
        sign = 1.0 - 2.0 * (par & 1).to(torch.float64)
        # Z first, then X: X Z = -i Y on a shared qubit
        phase = 1j ** bin(xm & zm).count("1")
        return c * (phase * (psi[idx ^ mask(xm)].conj() * sign * psi).sum()).real.item()

    def check(terms, tiled):
        with qs.profile() as prof:
            got = qs.expect(st, terms, per_term=True)[1]
        names = {r["kernel"] for r in prof.report}
        assert ("expect_tiles" in names) == tiled, names
        assert np.abs(got - [exact(t) for t in terms]).max() <= 64 * np.finfo(np.float64).eps

    z = [W.pauli(1.0, {q: "Z", (q + 5) % n: "Z"}) for q in range(9)]
    x = [W.pauli(1.0, {0: "XY"[q % 2], n - 1: "X", q + 2: "Z"}) for q in range(9)]
    for one, few in ((z, few_z), ([x[k] for k in (0, 2, 4, 6, 8)], few_x)):
        for count in {1, few or 1, few + 1}:
            check(one[:count], count > few)
    check(x[:2], few_x < 2)  # an even and an odd number of Y factors
    check([z[0], x[0]], True)

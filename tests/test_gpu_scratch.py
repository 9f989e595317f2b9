"""Device memory that a state holds on to after its read-out calls."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_expectation_keeps_no_more_scratch_than_stated():
    """8192 Z-type terms on 22 qubits: 32 sets of partial sums, 4 MiB each."""
    import torch
    import paper_2609_19147_amd as qs
    n = 22
    st = qs.State(n, "c64", init=None)
    W.gaussian_state_torch(n, 1, "c64", out=st.tensor())
    rng = np.random.default_rng(0)
    terms = [(1.0, 0, int(z)) for z in rng.choice(np.arange(1, 1 << n), size=8192, replace=False)]
    qs.expect(st, terms[:8])
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    got = qs.expect(st, terms, per_term=True)[1]
    kept = before - torch.cuda.mem_get_info()[0]
    assert kept <= (64 << 20) + (4 << 20), kept  # allocations are whole pages of up to 2 MiB
    # and the sums of the sets are those of the same terms one set at a time
    some = np.concatenate([qs.expect(st, terms[k:k + 128], per_term=True)[1] for k in (0, 4096, 8064)])
    assert np.abs(some - np.concatenate([got[k:k + 128] for k in (0, 4096, 8064)])).max() <= 64 * 2.0 ** -52

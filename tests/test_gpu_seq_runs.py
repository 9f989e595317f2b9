"""Which layer runs of a state of one tile are one launch, and their results."""
import numpy as np
import pytest

import workloads as W
from oracle import statevec as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13])
@pytest.mark.parametrize("kind", ["pass_gather", "gather_pass", "three", "two_passes"])
def test_runs_of_layers(kind, n, dtype):
    """A pass and a gather alone run apart from 10 qubits on, in complex64 up to 11."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(n)
    u = [W.G("U", q, mat=W.random_unitary(2, rng)) for q in range(n)]
    v = [W.G("U", q, mat=W.random_unitary(2, rng)) for q in range(n)]
    perm = W.random_perm_block(n, 40, 1)
    gates = {"pass_gather": u + perm, "gather_pass": perm + u, "three": u + perm + v,
             "two_passes": W.tfim_strang_stream(n, 1.0, 0.8, 0.05, 6)}[kind]
    plan = qs.Plan(n, gates, window_k=-1)
    kinds = [L["kind"] for L in plan.describe()["layers"]]
    assert kinds == {"pass_gather": ["tile", "gf2"], "gather_pass": ["gf2", "tile"], "three": ["tile", "gf2", "tile"],
                     "two_passes": ["tile", "tile"]}[kind]
    psi = W.gaussian_state(n, n).astype(np.complex64)
    st = qs.State(n, dtype, init=None).upload(psi)
    with qs.profile() as prof:
        qs.apply(st, plan)
    names = {r["kernel"] for r in prof.report}
    apart = n >= 10 and (dtype == "c128" or n <= 11) and len(kinds) == 2 and "gf2" in kinds
    assert ("seq_passes" in names) == (not apart), names
    ref = sv.run(psi.astype(np.complex128), n, gates)
    # a float (double) rounding or two per gate, all of the size of the state
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    assert np.linalg.norm(st.download() - ref) <= 4 * np.sqrt(len(gates)) * 4 * eps


@pytest.mark.parametrize("kind", ["pass_gather", "gather_pass"])
def test_a_state_of_one_buffer_stays_in_it(kind):
    """Nothing is allocated for a pair that a sequence runs in place (a capture or a memory cap may forbid it)."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    n = 10
    rng = np.random.default_rng(n)
    u = [W.G("U", q, mat=W.random_unitary(2, rng)) for q in range(n)]
    perm = W.random_perm_block(n, 40, 1)
    gates = u + perm if kind == "pass_gather" else perm + u
    psi = W.gaussian_state(n, n)
    st = qs.State(n, "c128", init=None, lazy_scratch=True).upload(psi)
    plan = qs.Plan(n, gates, window_k=-1)
    held = qs.memory_info()[0]
    for _ in range(2):
        qs.apply(st, plan)
    torch.cuda.synchronize()
    assert qs.memory_info()[0] == held
    ref = sv.run(sv.run(psi, n, gates), n, gates)
    assert np.linalg.norm(st.download() - ref) <= 4 * np.sqrt(2 * len(gates)) * 4 * 2.0 ** -53


@pytest.mark.parametrize("kind", ["pass_gather", "gather_pass"])
def test_a_captured_pair_goes_on_from_replay_to_replay(kind):
    """Recorded by the caller's own capture, a pair that a sequence runs in place reads its last result."""
    import torch
    import paper_2609_19147_amd as qs
    n = 10
    rng = np.random.default_rng(n)
    u = [W.G("U", q, mat=W.random_unitary(2, rng)) for q in range(n)]
    perm = W.random_perm_block(n, 40, 1)
    gates = u + perm if kind == "pass_gather" else perm + u
    psi = W.gaussian_state(n, n)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = qs.State(n, "c128", init=None).upload(psi)
        plan = qs.Plan(n, gates, window_k=-1)
        qs.apply(st, plan)
    torch.cuda.synchronize()
    ref = sv.run(psi, n, gates)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        qs.apply(st, plan)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        ref = sv.run(ref, n, gates)
        assert np.linalg.norm(st.download() - ref) <= 4 * np.sqrt((k + 2) * len(gates)) * 4 * 2.0 ** -53, k

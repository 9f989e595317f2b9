"""Norm, overlap and infidelity on both sides of the size from which a state is
streamed past the last-level cache (256 MiB, two states together where two are
read), against torch in FP64."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n", [("c64", 5), ("c64", 21), ("c64", 24), ("c64", 25), ("c64", 26),
                                     ("c128", 20), ("c128", 23), ("c128", 24), ("c128", 25)])
def test_reductions_around_the_cache_size(dtype, n):
    import torch
    import paper_2609_19147_amd as qs
    a, b = qs.State(n, dtype, init=None), qs.State(n, dtype, init=None)
    W.gaussian_state_torch(n, 1, dtype, out=a.tensor())
    W.gaussian_state_torch(n, 2, dtype, out=b.tensor())
    b.tensor().add_(a.tensor())
    b.tensor()[3] += 0.25
    x, y = a.tensor().to(torch.complex128), b.tensor().to(torch.complex128)
    nx, ny = [torch.view_as_real(v).pow(2).sum().item() for v in (x, y)]
    ov = torch.vdot(x, y).item()
    # 2^27 products at most, summed pairwise or in blocks on both sides: a few
    # dozen roundings of the sum of their sizes
    tol = 64 * 2.0 ** -52
    assert abs(qs.norm2(a) - nx) <= tol * nx and abs(qs.norm2(b) - ny) <= tol * ny
    assert abs(qs.overlap(a, b) - ov) <= tol * (nx * ny) ** 0.5 * 2
    assert abs(qs.infidelity(a, b) - (1 - abs(ov) ** 2 / (nx * ny))) <= 8 * tol

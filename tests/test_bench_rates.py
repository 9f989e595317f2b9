"""The benchmark's rates of the dense blocks are those of the instructions that run."""
import pytest


@pytest.mark.parametrize("dt,k,products,peak", [("c64", 4, 1, 157.3), ("c64", 5, 7, 2516.6), ("c64", 6, 7, 2516.6),
                                                ("c128", 4, 1, 78.6), ("c128", 6, 1, 78.6)])
def test_dense_matrix_work(dt, k, products, peak):
    import bench
    assert bench.dense_matrix_work(dt, k) == (products, peak)

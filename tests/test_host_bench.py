"""Host tests of the benchmark's choice of byte model: the kernel that a census
of a size, a scheme and a graph runs."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


@pytest.mark.parametrize("k,scheme,n,m,sizes,want", [
    (3, 0, 10, 20, 1, "copies<3>"), (4, 1, 5120, 5120, 1, "kr_kernel<4>"), (4, 1, 5120, 5121, 1, "copies<4>"),
    (4, 1, 5121, 100, 1, "copies<4>"), (4, 1, 100, 500, 2, "copies<4>"), (4, 2, 100, 500, 1, "k4_kernel"),
    (5, 1, 65536, 1 << 20, 1, "copies<5>"), (5, 1, 65537, 100, 1, "kr_kernel<5>"),
    (5, 1, 65536, (1 << 20) + 1, 3, "kr_kernel<5>"), (5, 1, 100, 3300, 1, "copies<5>"),
    (5, 1, 100, 3301, 1, "kr_kernel<5>"), (5, 2, 100, 300, 1, "k5_kernel")])
def test_kernel_name(k, scheme, n, m, sizes, want):
    import bench
    assert bench.kernel_name(k, scheme, n, m, sizes) == want

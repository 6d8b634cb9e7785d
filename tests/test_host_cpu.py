"""Host parts of the library that need no device."""

import ctypes as C

import numpy as np
import pytest


@pytest.mark.parametrize("n0,n1,span", [(0, 5, 10), (1, 1, 1), (1, 1, 2), (7, 9, 12), (1000, 700, 1500),
                                        (5000, 4096, 9216), (300, 300, 300)])
def test_common_nodes_counts_the_intersection(n0, n1, span):
    from paper_1802_05421_amd.api import _lib
    rng = np.random.default_rng(n0 + n1)
    a, b = (np.sort(rng.choice(span, n, replace=False)).astype(np.int32) for n in (n0, n1))
    keep = [np.append(x, np.int32(0)) for x in (a, b)]
    pa, pb = (x.ctypes.data for x in keep)
    count = C.c_int64(-1)
    assert _lib().cdl_common_nodes(n0, pa, n1, pb, C.byref(count)) == 0
    assert count.value == np.intersect1d(a, b).size
    assert _lib().cdl_common_nodes(-1, pa, n1, pb, C.byref(count)) == 1
    assert _lib().cdl_common_nodes(n0, None, n1, pb, C.byref(count)) == 1

"""Tile shapes and launch rules at their edges: sizes where a product takes
another tile shape, a last tile is nearly empty or a split is short, against
the CPU FP64 oracle."""

import numpy as np
import pytest
import torch

import gen
import oracle

pytestmark = pytest.mark.gpu

SEED = gen.grid.PROJ_SEED


@pytest.fixture(scope="module")
def cdl():
    import paper_1802_05421_amd as cdl
    return cdl


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# The FP64 product with W takes a tile shape by the number of 16-column groups
# (1 group: 32-row tiles; 5: 80; 7: 112; 9 and 10: two or three tiles; whole
# panels of 128 and 256 columns: the large tiles), by n and by the split.  Both
# solves end at a relative residual of 1e-12; kappa of these graphs is below
# 10, so Z is within 1e-11 of L^+ Y and 1e-10 allows for the oracle's rounding.
@pytest.mark.parametrize("n,k", [(2, 1), (257, 16), (300, 33), (513, 70), (300, 112), (640, 128),
                                 (300, 130), (511, 150), (1030, 200), (700, 256), (300, 300)])
def test_products_of_every_column_count(cdl, n, k):
    X = np.random.default_rng(n + k).standard_normal((n, 24))
    o = oracle.build_graph(X, sigma=6.0)
    want = oracle.solve_embedding(o["W"], oracle.rhs(o["W"], k, SEED))
    print("product case n=%d k=%d" % (n, k), flush=True)
    g = cdl.build_graph(dev(X), sigma=6.0)
    ch = cdl.build_chain(g, prec="fp32", depth_max=8, lazy=n == 2)
    Z, info = cdl.solve_embedding(g, ch, k, SEED, tol=1e-12, max_iter=60)
    assert info.converged and rel(host(Z), want) <= 1e-10
    if n > 2:
        # panels of 256 rows: the recomputed weights in the same products
        _, Zs, info = cdl.stream_embedding(dev(X), k, SEED, sigma=6.0, tol=1e-12, max_iter=60,
                                           panel_rows=256)
        assert info.converged and rel(host(Zs), want) <= 1e-10

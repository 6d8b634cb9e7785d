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


def score_inputs(cdl, n, k, weighted, rng):
    """Embeddings and graphs of two snapshots straight from random numbers."""
    Z = [rng.standard_normal((n, k)) for _ in range(2)]
    Z[1] = 0.9 * Z[0] + 0.3 * Z[1]
    vol = [float(n * n) / 3, float(n * n) / 4]
    gs, W = [], []
    for t in range(2):
        A = np.zeros((cdl.ld(n), cdl.ld(n)))
        if weighted:
            B = rng.uniform(0.1, 1.0, (n, n))
            A[:n, :n] = np.triu(B, 1) + np.triu(B, 1).T
        W.append(A[:n, :n])
        gs.append(cdl.Graph(W=dev(A), deg=dev(np.ones(n)), stats=dev(np.array([vol[t], 1.0, 1.0, 1.0])), n=n))
    return Z, vol, W, gs


def edge_matrix(Z, vol, W, weighted, m0, m1):
    E = np.zeros((len(m0), len(m0)))
    for z, v, m, s in ((Z[0], vol[0], m0, 1.0), (Z[1], vol[1], m1, -1.0)):
        z = z[m] * np.sqrt(v)
        sq = (z * z).sum(1)
        E += s * (sq[:, None] + sq[None, :] - 2.0 * z @ z.T)
    np.fill_diagonal(E, 0.0)
    E = np.abs(E)
    return E * np.abs(W[1][np.ix_(m1, m1)] - W[0][np.ix_(m0, m0)]) if weighted else E


# The score Gram takes 64 x 64, 128 x 128 or 256 x 128 tiles by m; its k range
# is two halves padded to 16 columns.  Each dc is a sum of 2k products rounded
# in FP64 (numpy's the same, in another order): relative error of F below
# (2k + 3) 2^-53 times the cancellation in sq_a + sq_b - 2 G, here under 1e3.
@pytest.mark.parametrize("n,m,k,weighted", [(2, 2, 1, False), (65, 64, 16, True), (300, 257, 17, False),
                                            (700, 641, 40, True), (2600, 2305, 33, True),
                                            (3100, 3100, 130, False), (4700, 4353, 8, False)])
def test_scores_of_every_tile_shape(cdl, n, m, k, weighted):
    rng = np.random.default_rng(n + m)
    print("score case n=%d m=%d k=%d" % (n, m, k), flush=True)
    Z, vol, W, gs = score_inputs(cdl, n, k, weighted, rng)
    maps = [np.arange(n) if m == n else np.sort(rng.choice(n, m, replace=False)) for _ in range(2)]
    E = edge_matrix(Z, vol, W, weighted, *maps)
    want = E.sum(1)
    kw = {} if m == n else dict(map0=dev(maps[0].astype(np.int32)), map1=dev(maps[1].astype(np.int32)))
    mode, K = ("delta_a" if weighted else "unweighted"), min(50, m)
    Zd = [dev(z) for z in Z]
    F, top = cdl.anomaly_scores(Zd[0], gs[0], Zd[1], gs[1], mode=mode, top_k=K, **kw)
    tol = (2 * k + 3) * 2.0 ** -53 * 1e3
    assert np.abs(host(F) - want).max() <= tol * np.abs(want).max()
    Fh = host(F)
    np.testing.assert_array_equal(host(top), np.lexsort((np.arange(m), -Fh))[:K])
    if m > 2:
        F2, a, b, v = cdl.anomaly_edges(Zd[0], gs[0], Zd[1], gs[1], top_k=K, mode=mode, **kw)
        np.testing.assert_array_equal(host(F2), Fh)
        iu = np.triu_indices(m, 1)
        order = np.argsort(-E[iu], kind="stable")[:K]
        assert np.abs(host(v) - E[iu][order]).max() <= tol * E.max()
        got = E[host(a), host(b)]
        assert np.all(host(a) < host(b)) and np.abs(got - host(v)).max() <= tol * E.max()


# Top-K over one chunk of 512, several, and enough for two further rounds, with
# exact ties (ordered by index).
@pytest.mark.parametrize("m,K", [(2, 1), (511, 50), (513, 256), (5000, 256), (70000, 50)])
def test_topk_rounds_and_ties(cdl, m, K):
    K = min(K, m)
    rng = np.random.default_rng(m)
    # scores through the public call: one column, two clusters at distance 0 or
    # d_c, so that many nodes tie exactly; the order must be (-F, index)
    lev = rng.integers(0, 3, m).astype(np.float64)
    Z0, Z1 = lev[:, None], np.zeros((m, 1))
    st = dev(np.array([1.0, 1.0, 1.0, 1.0]))
    g = cdl.Graph(W=None, deg=dev(np.ones(m)), stats=st, n=m)
    F, top = cdl.anomaly_scores(dev(Z0), g, dev(Z1), g, top_k=K)
    Fh = host(F)
    np.testing.assert_array_equal(host(top), np.lexsort((np.arange(m), -Fh))[:K])


# The median selection: one workgroup up to 512 nodes, passes over the bracket
# buffer above, the matrix when the bracket is switched off; many ties (integer
# series: digits below the tied value are empty), one value only, and the tile
# shapes of the Gram at their edges.  Integer series have exact distances, so
# sigma is the oracle's to the bit; the others round in the Gram's order.
@pytest.mark.parametrize("n,T,kind", [(2, 1, "normal"), (3, 400, "integer"), (64, 16, "normal"),
                                      (257, 33, "integer"), (512, 20, "normal"), (513, 20, "integer"),
                                      (1100, 120, "normal"), (1500, 3, "integer"), (700, 5, "constant"),
                                      (2300, 7, "normal")])
def test_median_and_graph_of_every_size(cdl, n, T, kind):
    rng = np.random.default_rng(n + T)
    X = {"normal": lambda: rng.standard_normal((n, T)),
         "integer": lambda: rng.integers(-3, 4, (n, T)).astype(float),
         "constant": lambda: np.tile(np.eye(n)[:, :1], (1, T)) * 2.0}[kind]()
    if kind == "constant":   # one node off by a vector, all others equal
        X = X + 1.0
        want = None
    else:
        want = oracle.bandwidth(oracle.sq_distances(X))
    print("median case n=%d T=%d %s" % (n, T, kind), flush=True)
    sig = []
    for mode in (0, 1):
        cdl.set_select(mode)
        try:
            g = cdl.build_graph(dev(X), check=False)
        finally:
            cdl.set_select(0)
        sig.append(g.host_stats()["sigma"])
    assert sig[0] == sig[1] or (np.isnan(sig[0]) and np.isnan(sig[1]))
    if kind == "integer":
        assert sig[0] == want
    elif kind == "normal":
        assert sig[0] == pytest.approx(want, rel=1e-13)
        o = oracle.build_graph(X)
        W = host(g.W)
        np.testing.assert_allclose(W[:n, :n], o["W"], rtol=0, atol=2e-13)
        np.testing.assert_array_equal(W, W.T)
        np.testing.assert_allclose(host(g.deg), o["deg"], rtol=1e-12)
        s = g.host_stats()
        assert s["deg_min"] == host(g.deg).min() and s["deg_max"] == host(g.deg).max()
    else:
        assert sig[0] == 0.0


# A non-finite series must reach the caller whatever the selection does with it.
@pytest.mark.parametrize("n", [40, 700])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_series_is_reported(cdl, n, bad):
    X = np.random.default_rng(n).standard_normal((n, 12))
    X[n // 3, 5] = bad
    with pytest.raises(cdl.CdlError):
        cdl.build_graph(dev(X))


# FP32 and FP64 levels are squared in tiles of 128, 64 or (FP64, one tile row)
# 32 by their count, and applied in tiles by the live 32-column groups, the
# column padding and n.  A level is the product of its predecessor with itself:
# a sum of nonnegative products rounded at most ld + 2 times.  A depth of 8
# leaves rho^256 < 1e-11 on these graphs (kappa < 10) and a sum's rounding, at
# most 8 ld 2^-24 < 1e-3 in FP32, of an application, so four corrections reach
# 1e-12; a missing or misplaced tile would leave its nodes uncorrected.
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,k", [(2, 1), (200, 32), (256, 33), (300, 70), (520, 112), (1000, 160),
                                 (1300, 96), (1800, 260), (700, 512)])
def test_levels_and_applications_of_every_tile_shape(cdl, prec, n, k):
    X = np.random.default_rng(n + k).standard_normal((n, 24))
    o = oracle.build_graph(X, sigma=6.0)
    want = oracle.solve_embedding(o["W"], oracle.rhs(o["W"], k, SEED))
    print("level case n=%d k=%d %s" % (n, k, prec), flush=True)
    g = cdl.build_graph(dev(X), sigma=6.0)
    ch = cdl.build_chain(g, prec=prec, depth=8, depth_max=8, lazy=n == 2)
    eps = 2.0 ** (-24 if prec == "fp32" else -53)
    for l in (0, 3):
        A, B = (host(cdl.level(ch, q)).astype(np.float64) for q in (l, l + 1))
        ref = A @ A
        assert np.abs(B - ref).max() <= (cdl.ld(n) + 2) * eps * np.abs(ref).max()
        np.testing.assert_array_equal(B, B.T)
    cdl.set_solve_depth(8)   # all eight, also where fewer would do
    try:
        Z, info = cdl.solve_embedding(g, ch, k, SEED, tol=1e-12, max_iter=4)
    finally:
        cdl.set_solve_depth(0)
    assert info.converged and rel(host(Z), want) <= 1e-10


# 16-bit levels go through 256 x 256 tiles whose rows and mirrored rows leave
# through one transposed copy.  An element is a sum of products (exact in FP32)
# rounded at most ld times in FP32 and once to its type; the dense product adds
# the two factors first, and its lower triangle is the upper one's copy (rounded
# factors do not quite commute).
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("n", [2, 255, 257, 900])
def test_16bit_levels_and_dense_product(cdl, prec, n):
    print("16-bit level case n=%d %s" % (n, prec), flush=True)
    X = np.random.default_rng(n).standard_normal((n, 24))
    g = cdl.build_graph(dev(X), sigma=4.0)
    ch = cdl.build_chain(g, prec=prec, depth=2, depth_max=3, lazy=n == 2)
    sc = cdl.level_scale(ch)
    A, B = (host(cdl.level(ch, q).double()) / sc for q in (0, 1))
    ulp, least = (2.0 ** -8, 0.0) if prec == "bf16" else (2.0 ** -11, 2.0 ** -25 / sc)
    acc = (cdl.ld(n) + 3) * 2.0 ** -24
    ref, mag = A @ A, np.abs(A) @ np.abs(A)
    assert np.all(np.abs(B - ref) <= ulp * np.abs(ref) + 2 * acc * mag + least)
    np.testing.assert_array_equal(B, B.T)
    cdl.chain_densify(ch)
    Q = host(cdl.level(ch, 0).double()) / sc
    ref, mag = A + B + A @ B, np.abs(A) + np.abs(B) + np.abs(A) @ np.abs(B)
    ref, mag = (np.triu(m) + np.triu(m, 1).T for m in (ref, mag))
    assert np.all(np.abs(Q - ref) <= ulp * np.abs(ref) + 2 * acc * mag + least)
    np.testing.assert_array_equal(Q, Q.T)


# A whole row panel computes the upper tiles of its own square once and stores
# them mirrored: with one panel, panels whose square ends in the padding, and
# either tile shape (a few tiles or many), the sweeps must see the stored path's
# weights: degrees agree to the rounding of their sums, (n + 2) 2^-53, and Z, each
# solved to a relative residual of 1e-12 with kappa below 10, to 2e-11.
@pytest.mark.parametrize("n,panel", [(256, 256), (700, 256), (700, 512), (1300, 1536), (3000, 1024),
                                     (5000, 5120)])
def test_panels_mirror_their_own_square(cdl, n, panel):
    print("panel case n=%d panel=%d" % (n, panel), flush=True)
    X = np.random.default_rng(n).standard_normal((n, 24))
    ref = cdl.build_graph(dev(X), sigma=6.0)
    g, Z, info = cdl.stream_embedding(dev(X), 3, SEED, sigma=6.0, tol=1e-12, max_iter=60, panel_rows=panel)
    assert info.converged
    d0, d1 = host(ref.deg), host(g.deg)
    assert np.abs(d1 - d0).max() <= (n + 2) * 2.0 ** -53 * d0.max()
    ch = cdl.build_chain(ref, prec="fp32", depth_max=8)
    Z0, info = cdl.solve_embedding(ref, ch, 3, SEED, tol=1e-12, max_iter=60)
    assert info.converged and rel(host(Z), host(Z0)) <= 2e-11


# The panel products' tiles differ with the panel's size, the order of their sums
# does not: the same bits for every panel size, at column counts of every tile
# and at whole 128-column panels.
@pytest.mark.parametrize("n,k", [(300, 5), (700, 48), (1100, 70), (1300, 112), (900, 128), (600, 200)])
def test_panel_size_leaves_every_bit(cdl, n, k):
    print("panel bits n=%d k=%d" % (n, k), flush=True)
    X = dev(np.random.default_rng(n + k).standard_normal((n, 24)))
    Z = [host(cdl.stream_embedding(X, k, SEED, sigma=6.0, tol=1e-12, max_iter=60, panel_rows=p)[1])
         for p in (256, 768, 0)]
    np.testing.assert_array_equal(Z[0], Z[1])
    np.testing.assert_array_equal(Z[0], Z[2])

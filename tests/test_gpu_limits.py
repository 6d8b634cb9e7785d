"""Calls at the ends of their ranges: groups that mix very small and large
snapshots, edge scores that are no numbers, sizes past 32-bit offsets and launch
limits."""

import numpy as np
import pytest
import torch

import gen

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


def mixed_snapshots(sizes, T, seed):
    """Random series on random subsets of one range of ids that share its ids 0..9."""
    rng = np.random.default_rng(seed)
    top = max(sizes) + 10
    Xs, gids = [], []
    for n in sizes:
        ids = np.sort(np.append(np.arange(10), 10 + rng.choice(top - 10, n - 10, replace=False)))
        Xs.append(dev(rng.standard_normal((n, T))))
        gids.append(torch.from_numpy(ids.astype(np.int32)).cuda())
    return Xs, gids


def batched_equals_per_snapshot(cdl, Xs, gids, **kw):
    """The one-pass sequence with its choices pinned: the per-snapshot path's bits."""
    base = dict(k=16, seed=SEED, depth=2, tol=0.0, max_iter=3, top_k=5, **kw)
    cdl.force_choice("apply", 0)
    cdl.force_choice("residual", 0)
    try:
        wF, wT, _ = cdl.score_sequence(Xs, gids, cdl.SeqParams(**base))
        Fb, Tb, _ = cdl.score_sequence(Xs, gids, cdl.SeqParams(**base, asynchronous=True, batched=True))
    finally:
        cdl.force_choice("apply", -1)
        cdl.force_choice("residual", -1)
    for t in range(len(wF)):
        np.testing.assert_array_equal(host(Fb[t]), host(wF[t]), err_msg="pair %d" % t)
        np.testing.assert_array_equal(host(Tb[t]), host(wT[t]), err_msg="pair %d" % t)


# Beside a snapshot of more than 512 nodes the small ones' medians take the passes
# of the whole chip.  Up to about 148 nodes a bracket holds at most 512 keys, which
# the first pass already collects, while the snapshot's other workgroups may still
# be reading the counts that say so.  The scores depend on every snapshot's
# bandwidth, so equal bits mean equal bandwidths.
@pytest.mark.parametrize("sizes", [[70, 3000, 100, 140], [600, 64, 148, 149, 70, 128] + [96, 127, 65, 141] * 5])
def test_small_snapshots_beside_large_ones(cdl, sizes):
    print("mixed group", sizes, flush=True)
    Xs, gids = mixed_snapshots(sizes, 20, len(sizes))
    batched_equals_per_snapshot(cdl, Xs, gids, prec="fp32")


# Edge scores that are no numbers: the finite ones come first, in order, and
# -infinity fills the rest.  With k = 1, vol = 1 and Z1 = 0 the score of (a, b) is
# (z_a - z_b)^2, exact for small integers.
@pytest.mark.parametrize("m,finite,K", [(300, 0, 20), (2, 0, 1), (300, 2, 20), (300, 5, 256), (700, 40, 50)])
def test_edges_without_enough_numbers(cdl, m, finite, K):
    print("edges m=%d with %d finite nodes, K=%d" % (m, finite, K), flush=True)
    rng = np.random.default_rng(m + finite)
    z = np.full(m, np.nan)
    at = np.sort(rng.choice(m, finite, replace=False))
    z[at] = rng.permutation(finite).astype(float)
    st = dev(np.ones(4))
    g = cdl.Graph(W=None, deg=dev(np.ones(m)), stats=st, n=m)
    F, a, b, v = cdl.anomaly_edges(dev(z[:, None]), g, dev(np.zeros((m, 1))), g, top_k=K)
    a, b, v = host(a), host(b), host(v)
    i, j = np.triu_indices(finite, 1)
    score = (z[at[i]] - z[at[j]]) ** 2
    order = np.argsort(-score, kind="stable")[:K]   # ascending (a, b) among equals
    c = len(order)
    np.testing.assert_array_equal(v[:c], score[order])
    np.testing.assert_array_equal(a[:c], at[i[order]])
    np.testing.assert_array_equal(b[:c], at[j[order]])
    assert np.all(v[c:] == -np.inf)
    assert np.isnan(host(F)).all()


# With k = 1, vol = 1 and Z1 = 0 the score of (a, b) is (z_a - z_b)^2: F_a = m z_a^2 -
# 2 z_a S1 + S2, every sum an integer below 2^53 and so exact.
def one_column(cdl, z):
    m = len(z)
    g = cdl.Graph(W=None, deg=dev(np.ones(m)), stats=dev(np.ones(4)), n=m)
    return dev(z[:, None]), g, dev(np.zeros((m, 1))), g


def one_column_scores(z):
    z = z.astype(np.int64)
    return (len(z) * z * z - 2 * z * z.sum() + (z * z).sum()).astype(np.float64)


# The tiles of the score Gram of 525000 common nodes have 2^32 work-items and more.
def test_scores_past_a_launch_of_32_bits(cdl):
    m = 525000
    print("scores m=%d" % m, flush=True)
    z = np.random.default_rng(m).integers(0, 4096, m).astype(float)
    F, top = cdl.anomaly_scores(*one_column(cdl, z), top_k=50)
    want = one_column_scores(z)
    np.testing.assert_array_equal(host(F), want)
    np.testing.assert_array_equal(host(top), np.lexsort((np.arange(m), -want))[:50])


# So have the eight parts of every 256 x 128 tile of 371000 nodes, of which the
# collection keeps those that reach the threshold.  The largest score is that of a
# 0 and a 4095, which many pairs share: the first fifty in order of (a, b).
def test_edges_past_a_launch_of_32_bits(cdl):
    m, K = 371000, 50
    print("edges m=%d" % m, flush=True)
    z = np.random.default_rng(m).integers(0, 4096, m).astype(float)
    F, a, b, v = cdl.anomaly_edges(*one_column(cdl, z), top_k=K)
    np.testing.assert_array_equal(host(F), one_column_scores(z))
    ends = np.flatnonzero((z == 0) | (z == 4095))
    pairs = [(i, j) for i in ends for j in ends if i < j and z[i] != z[j]][:K]
    assert len(pairs) == K and np.all(host(v) == 4095.0 ** 2)
    assert list(zip(host(a).tolist(), host(b).tolist())) == pairs


# Series so long that a tile's rows lie 2^32 bytes apart (64 rows of 2^23 values).
# Small integers: every distance is exact, whatever the order of its sum.
@pytest.mark.parametrize("n,T", [(70, (1 << 23) + 5), (3, (1 << 22) + 7)])
def test_series_past_32_bit_offsets(cdl, n, T):
    print("long series n=%d T=%d" % (n, T), flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randint(-2, 3, (n, T), generator=g, device="cuda").double()
    G = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    for c in range(0, T, 1 << 21):
        G += X[:, c:c + (1 << 21)] @ X[:, c:c + (1 << 21)].T.contiguous()
    D2 = host(G.diag()[:, None] + G.diag()[None, :] - 2.0 * G)
    d = np.sort(D2[np.triu_indices(n, 1)])
    sigma = np.sqrt(d[(len(d) - 1) // 2])
    W = np.exp(-D2 / sigma ** 2)
    np.fill_diagonal(W, 0.0)
    for mode in (0, 1):
        cdl.set_select(mode)
        try:
            got = cdl.build_graph(X)
        finally:
            cdl.set_select(0)
        assert got.host_stats()["sigma"] == sigma
        np.testing.assert_allclose(host(got.W)[:n, :n], W, rtol=1e-14)
        del got
    st, Z, info = cdl.stream_embedding(X, 2, SEED, tol=1e-9, max_iter=60)
    assert info.converged and st.host_stats()["sigma"] == sigma
    np.testing.assert_allclose(host(st.deg), W.sum(1), rtol=1e-13)
    del st, Z
    if n > 4:
        gid = torch.arange(n, dtype=torch.int32, device="cuda")
        batched_equals_per_snapshot(cdl, [X, X], [gid, gid], prec="fp32")


# Embeddings of so many columns that a score tile's rows lie 2^32 bytes apart; small
# integers, so that every score is exact.
@pytest.mark.parametrize("mode", ["unweighted", "delta_a"])
def test_scores_past_32_bit_offsets(cdl, mode):
    n, k, K = 70, (1 << 22) + 3, 20
    print("scores of %d columns, %s" % (k, mode), flush=True)
    gen_ = torch.Generator(device="cuda").manual_seed(k)
    Z, C, W, gs = [], [], [], []
    for t in range(2):
        z = torch.randint(-1, 2, (n, k), generator=gen_, device="cuda").double()
        G = z @ z.T.contiguous()
        C.append(host(G.diag()[:, None] + G.diag()[None, :] - 2.0 * G))
        A = np.zeros((cdl.ld(n), cdl.ld(n)))
        B = np.triu(np.random.default_rng(t).integers(1, 9, (n, n)), 1).astype(float)
        A[:n, :n] = B + B.T
        Z.append(z)
        W.append(A[:n, :n])
        gs.append(cdl.Graph(W=dev(A), deg=dev(np.ones(n)), stats=dev(np.ones(4)), n=n))
    E = np.abs(C[0] - C[1])
    if mode == "delta_a":
        E = E * np.abs(W[1] - W[0])
    F, top = cdl.anomaly_scores(Z[0], gs[0], Z[1], gs[1], mode=mode, top_k=K)
    np.testing.assert_array_equal(host(F), E.sum(1))
    F, a, b, v = cdl.anomaly_edges(Z[0], gs[0], Z[1], gs[1], mode=mode, top_k=K)
    np.testing.assert_array_equal(host(F), E.sum(1))
    i, j = np.triu_indices(n, 1)
    order = np.argsort(-E[i, j], kind="stable")[:K]
    np.testing.assert_array_equal(host(v), E[i, j][order])
    np.testing.assert_array_equal(host(a), i[order])
    np.testing.assert_array_equal(host(b), j[order])


# The score tiles' shape goes by the whole group, and the order in which a node's
# partial sums are added by the shape: with the choices pinned each pair takes the
# shape that it takes alone (3000 nodes: 64 x 64, five such pairs 128 x 128).
@pytest.mark.parametrize("mode,sizes", [("unweighted", [3000, 2900, 3100, 2950, 3050, 500]),
                                        ("delta_a", [700, 5200, 5100, 5000, 300])])
def test_pinned_groups_score_as_their_pairs_alone(cdl, mode, sizes):
    print("pinned group", mode, sizes, flush=True)
    Xs, gids = mixed_snapshots(sizes, 20, len(sizes))
    batched_equals_per_snapshot(cdl, Xs, gids, prec="fp32", mode=mode)


# Distances that crowd without being equal: 200 patterns at the corners of a rotated
# simplex are 2 apart but for rounding, and every node repeats one of them.  More
# keys than the bracket's buffer holds lie within a few units in the last place of
# the median; beside them some spread ones, or none.  The selection is exact: its
# result is one of the matrix's own distances, with the median's rank among them.
# The Gram's distances are not kept, but W = exp(-D2 / sigma^2) falls with them: the
# rank of sigma is bracketed by the weights above and below 1/e.
@pytest.mark.parametrize("n", [300, 513, 2100, 5000])
@pytest.mark.parametrize("spread", [0.0, 0.3])
def test_median_of_crowded_distances(cdl, n, spread):
    print("crowded n=%d spread=%.1f" % (n, spread), flush=True)
    rng = np.random.default_rng(n)
    C = 200
    Q = np.linalg.qr(rng.standard_normal((C, C)))[0]
    X = Q[rng.integers(0, C, n)]
    far = rng.random(n) < spread
    X[far] += 0.3 * rng.standard_normal((far.sum(), C)) / np.sqrt(C)
    sig, Ws = [], []
    for mode in (0, 1):
        cdl.set_select(mode)
        try:
            g = cdl.build_graph(dev(X))
        finally:
            cdl.set_select(0)
        sig.append(g.host_stats()["sigma"])
        Ws.append(host(g.W)[:n, :n])
    assert sig[0] == sig[1]
    np.testing.assert_array_equal(Ws[0], Ws[1])
    st, _, _ = cdl.stream_embedding(dev(X), 2, SEED, tol=1e-6, max_iter=64, panel_rows=512)
    assert st.host_stats()["sigma"] == sig[0]
    D2 = (X * X).sum(1)[:, None] + (X * X).sum(1)[None, :] - 2.0 * X @ X.T
    d = np.sort(D2[np.triu_indices(n, 1)])
    assert sig[0] ** 2 == pytest.approx(d[(len(d) - 1) // 2], rel=1e-13)
    w = Ws[0][np.triu_indices(n, 1)]
    rank, e1 = (len(d) - 1) // 2, np.exp(-1.0)
    assert (w > e1 * (1 + 1e-15)).sum() <= rank < (w >= e1 * (1 - 1e-15)).sum()


# Sequences whose smaller snapshots need larger workspaces than the largest one.
@pytest.mark.parametrize("prec,k,sizes", [("fp32", 128, [2560, 2304, 2500, 2250]), ("bf16", 16, [7100, 6900, 7000])])
def test_sequences_of_uneven_needs(cdl, prec, k, sizes):
    print("uneven needs", prec, k, sizes, flush=True)
    Xs, gids = mixed_snapshots(sizes, 20, len(sizes))
    base = dict(k=k, seed=SEED, prec=prec, depth=2, tol=0.0, max_iter=3, top_k=5)
    wF, wT, _ = cdl.score_sequence(Xs, gids, cdl.SeqParams(**base))
    F, T, _ = cdl.score_sequence(Xs, gids, cdl.SeqParams(**base, asynchronous=True))
    for t in range(len(wF)):
        np.testing.assert_array_equal(host(F[t]), host(wF[t]))
        np.testing.assert_array_equal(host(T[t]), host(wT[t]))


# Rounding of a node's sum over the tiles alone: with one column of integers below
# 2^23 and weights that differ by 1 every edge score and every sum over 64 of them is
# exact, and F's error is that of adding its 80 partial sums.  A rounding is
# uniform over half a unit in the last place, at most 0.58 2^-53 of the sum (rms).  In
# four chains the i-th of 20 sums is i / 80 of F: 4 sum (i / 80)^2 = 1.8, and the last
# additions are 2 / 4 and 1: rms at most 0.58 sqrt(1.8 + 0.5 + 1) 2^-53 = 1.06 2^-53.
# (One chain of 80: at least 0.29 sqrt(27) 2^-53 = 1.5 2^-53.)
def test_node_sums_round_little(cdl):
    m = 5003
    print("node sums m=%d" % m, flush=True)
    z = np.random.default_rng(m).integers(0, 1 << 23, m)
    A = np.zeros((cdl.ld(m), cdl.ld(m)))
    B = A.copy()
    B[:m, :m] = 1.0 - np.eye(m)
    g = [cdl.Graph(W=dev(w), deg=dev(np.ones(m)), stats=dev(np.ones(4)), n=m) for w in (A, B)]
    F, _ = cdl.anomaly_scores(dev(z[:, None].astype(float)), g[0], dev(np.zeros((m, 1))), g[1], mode="delta_a", top_k=0)
    want = m * z * z - 2 * z * z.sum() + (z * z).sum()
    err = (host(F).astype(np.int64) - want) / want.astype(float)
    assert np.sqrt((err * err).mean()) <= 1.1 * 2.0 ** -53


# Scores that are no numbers come first, in order of their index; none gives its
# place to the padding of a chunk.
@pytest.mark.parametrize("m,K", [(300, 256), (1300, 50)])
def test_top_nodes_of_nan_scores(cdl, m, K):
    z = np.arange(m, dtype=float)
    z[m // 2] = -np.nan
    F, top = cdl.anomaly_scores(*one_column(cdl, z), top_k=K)
    assert np.isnan(host(F)).all()
    np.testing.assert_array_equal(host(top), np.arange(K))


# Right-hand sides of 2^20 columns: 4096 groups of four 64-column blocks for every
# row are 2^32 work-items and more from 1024 rows on.  The first and the last
# block's columns against the definition.
def test_right_hand_sides_past_a_launch_of_32_bits(cdl):
    n, k = 1040, 1 << 20
    print("right-hand sides n=%d k=%d" % (n, k), flush=True)
    B = np.triu(np.random.default_rng(n).uniform(0.1, 1.0, (n, n)), 1)
    W = np.zeros((cdl.ld(n), cdl.ld(n)))
    W[:n, :n] = B + B.T
    Y = cdl.rhs(cdl.Graph(W=dev(W), deg=dev(np.ones(n)), stats=dev(np.ones(4)), n=n), k, SEED)

    def mix(z):
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
        return z ^ (z >> np.uint64(31))

    i, j = (np.triu(v, 1).astype(np.uint64) for v in np.indices((n, n)))
    root = np.sqrt(B)
    for beta in (0, k // 64 - 1):
        with np.errstate(over="ignore"):
            word = mix(mix(np.uint64(SEED)) ^ (np.uint64(beta << 40) | i << np.uint64(20) | j))
        for r in (0, 63):
            q = np.where((word >> np.uint64(r)) & np.uint64(1), -1.0, 1.0) * root   # (i < j: head i, tail j)
            want = (q.sum(1) - q.sum(0)) / np.sqrt(k)
            got = host(Y[:, beta * 64 + r].contiguous())
            assert np.abs(got - want).max() <= n * 2.0 ** -52 * np.abs(want).max()


# The same crowd in grouped launches, beside a snapshot of spread distances.
def test_median_of_crowded_distances_in_a_group(cdl):
    rng = np.random.default_rng(9)
    C = 64
    Q = np.linalg.qr(rng.standard_normal((C, C)))[0]
    sizes = [900, 150, 2000, 700]
    Xs, gids = mixed_snapshots(sizes, C, 9)
    for t in (0, 1, 2):
        Xs[t] = dev(Q[rng.integers(0, C, sizes[t])])
    print("crowded group", sizes, flush=True)
    batched_equals_per_snapshot(cdl, Xs, gids, prec="fp32")


# Two scales at once: most nodes are silent (distance 0 between them), the others
# repeat patterns of norm 1, so that the median's crowd lies at 1 but for rounding and
# the bracket may reach down to 0: half the pairs are silent.  Nested: some patterns
# have norms that differ from 1 at the scale of every 12 bits, so that no pass finds
# the crowd alone and four digits leave it unresolved.
@pytest.mark.parametrize("n", [400, 900, 2500, 4096])
@pytest.mark.parametrize("nested", [False, True])
def test_median_of_a_crowd_beside_zeros(cdl, n, nested):
    print("silent nodes n=%d nested=%d" % (n, nested), flush=True)
    rng = np.random.default_rng(n)
    C = 200
    Q = np.linalg.qr(rng.standard_normal((C, C)))[0]
    X = Q[rng.integers(0, C, n)]
    if nested:
        X *= np.sqrt(1.0 + rng.choice([0.0, 2.0 ** -13, 2.0 ** -25, 2.0 ** -37], (n, 1), p=[0.85, 0.05, 0.05, 0.05]))
    live = rng.permutation(n) < int(0.295 * n)
    X[~live] = 0.0
    sig = []
    for mode in (0, 1):
        cdl.set_select(mode)
        try:
            sig.append(cdl.build_graph(dev(X)).host_stats()["sigma"])
        finally:
            cdl.set_select(0)
    assert sig[0] == sig[1]
    st, _, _ = cdl.stream_embedding(dev(X), 2, SEED, tol=1e-6, max_iter=64, panel_rows=512)
    assert st.host_stats()["sigma"] == sig[0]
    zeros = (n - live.sum()) * (n - live.sum() - 1) // 2
    if (n * (n - 1) // 2 - 1) // 2 >= zeros:
        assert sig[0] ** 2 == pytest.approx(1.0, rel=1e-13)
    else:
        assert sig[0] == 0.0

"""GPU library against the CPU oracle: every share plane bit for bit, plus the
round and wire-byte counters.  All calls go through the C ABI."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1


def u64(vals):
    return np.array([int(v) & M64 for v in vals], dtype=np.uint64)


@pytest.fixture(scope="module")
def mods():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from oracle import Oracle
    from paper_2305_00645_amd import gtree
    gtree.load()
    return Oracle, gtree


def pair(mods, seed, tau=16, K=2):
    Oracle, gtree = mods
    return Oracle(seed, tau=tau, K=K), gtree.GTree(seed, tau=tau, K=K)


def same(gs, oc, what=""):
    """gs: gtree.Shares, oc: oracle components (3, n)."""
    comp = gs.components()
    assert comp.shape == oc.shape, (what, comp.shape, oc.shape)
    if not np.array_equal(comp, oc):
        bad = np.argwhere(comp != oc)
        raise AssertionError("%s: %d of %d words differ, first at %s" % (what, len(bad), comp.size, bad[0]))


def same_stats(o, g):
    ro, wo = o.stats()
    rg, wg, _ = g.stats()
    assert ro == rg and np.array_equal(wo, wg), (ro, rg, wo.tolist(), wg.tolist())
    assert o.op_counter() == g.op_counter()
    # what the kernels counted at their message stores (payload bits per directed pair)
    # against what the oracle's protocol steps sent
    bo, bg = o.wire_bits(), g.wire_bits_dev()
    assert np.array_equal(bo, bg), (bo.tolist(), bg.tolist())


@pytest.mark.parametrize("n", [1, 7, 8, 63, 64, 65, 1000, 4099])
def test_share_reconstruct(mods, seed, n):
    o, g = pair(mods, seed)
    rng = np.random.default_rng(n)
    x = rng.integers(0, M64, size=n, dtype=np.uint64)
    so, sg = o.share(x), g.share_a(x)
    same(sg, so, "share")
    assert np.array_equal(g.rec(sg), x)


@pytest.mark.parametrize("n", [511, 512, 513, 2047, 2049, 5 * 512 + 67])
def test_share_and_mult_at_tile_edges(mods, seed, n):
    """Tiles of 512 words whose PRF words change lanes: the last tile full, one short, one over."""
    o, g = pair(mods, seed)
    rng = np.random.default_rng(500 + n)
    x, y = (rng.integers(0, M64, size=n, dtype=np.uint64) for _ in range(2))
    xo, yo, xg, yg = o.share(x), o.share(y), g.share_a(x), g.share_a(y)
    same(xg, xo, "share")
    zg = g.mult(xg, yg)
    same(zg, o.mult(xo, yo), "mult")
    assert np.array_equal(g.rec(zg), x * y)
    same_stats(o, g)


def test_empty_vectors(mods, seed):
    o, g = pair(mods, seed)
    sg = g.share_a(np.zeros(0, dtype=np.uint64))
    o.share(np.zeros(0, dtype=np.uint64))
    assert g.mult(sg, sg).n == 0
    o.mult(np.zeros((3, 0), dtype=np.uint64), np.zeros((3, 0), dtype=np.uint64))
    assert o.op_counter() == g.op_counter()


@pytest.mark.parametrize("n", [1, 9, 512, 1531])
def test_mult(mods, seed, n):
    o, g = pair(mods, seed)
    rng = np.random.default_rng(10 + n)
    x = rng.integers(0, M64, size=n, dtype=np.uint64)
    y = rng.integers(0, M64, size=n, dtype=np.uint64)
    xo, yo = o.share(x), o.share(y)
    xg, yg = g.share_a(x), g.share_a(y)
    zo, zg = o.mult(xo, yo), g.mult(xg, yg)
    same(zg, zo, "mult")
    assert np.array_equal(g.rec(zg), x * y)
    same_stats(o, g)


@pytest.mark.parametrize("n,onto_y", [(255, False), (512 * 5 + 37, False), (512 * 5 + 37, True)])
def test_mult_in_place(mods, seed, n, onto_y):
    """The product over one of its factors: a party's next component is read from the plane of the party whose own it is, which that
    party overwrites."""
    _, gtree = mods
    o, g = pair(mods, seed)
    rng = np.random.default_rng(n)
    x, y = (rng.integers(0, M64, size=n, dtype=np.uint64) for _ in range(2))
    xo, yo, xg, yg = o.share(x), o.share(y), g.share_a(x), g.share_a(y)
    z = yg if onto_y else xg
    assert g.L.gt_mult(g.ctx, gtree._ref(xg), gtree._ref(yg), n, gtree._ref(z)) == 0
    same(z, o.mult(xo, yo), "mult in place")


def test_eq_public_and_shared(mods, seed):
    o, g = pair(mods, seed)
    rng = np.random.default_rng(3)
    xs, ys = [], []
    for b in range(64):
        v = int(rng.integers(0, M64, dtype=np.uint64))
        xs.append(v); ys.append(v ^ (1 << b))
    for v in [0, 1, M64, 1 << 63, (1 << 63) - 1]:
        xs += [v, v, v]; ys += [v, v + 1, v - 1]
    for _ in range(150):
        v = int(rng.integers(0, M64, dtype=np.uint64))
        xs.append(v); ys.append(v if rng.random() < 0.5 else int(rng.integers(0, M64, dtype=np.uint64)))
    x, y = u64(xs), u64(ys)
    xo, xg = o.share(x), g.share_a(x)
    eo, eg = o.eq_a(xo, y), g.eq_a(xg, y)
    same(eg, eo, "eq_a public")
    assert np.array_equal(g.rec(eg), (x == y).astype(np.uint64))
    yo, yg = o.share(y), g.share_a(y)
    do = xo - yo
    dg = g.new(x.size); dg.t.copy_(xg.t - yg.t)
    eo, eg = o.eq_a(do, None), g.eq_a(dg, None)
    same(eg, eo, "eq_a shared")
    same_stats(o, g)


def test_ge(mods, seed):
    o, g = pair(mods, seed)
    rng = np.random.default_rng(4)
    xs, ys = [], []
    smalls = [0, 1, 2, 5, 1 << 16, (1 << 40) - 1, 1 << 40, 1 << 62, (1 << 63) - 1]
    for a in smalls:
        for b in smalls:
            xs.append(a); ys.append(b)
    for b in range(63):
        v = int(rng.integers(0, 1 << 62))
        xs.append(v | (1 << b)); ys.append(v & ~(1 << b))
        xs.append(v & ~(1 << b)); ys.append(v | (1 << b))
    for _ in range(300):
        xs.append(int(rng.integers(0, 1 << 62))); ys.append(int(rng.integers(0, 1 << 62)))
    for a, b in [(-5, 3), (3, -5), (-1, -1), (-7, -8)]:
        xs.append(a); ys.append(b)
    x, y = u64(xs), u64(ys)
    zo = o.ge_a(o.share(x), o.share(y))
    zg = g.ge_a(g.share_a(x), g.share_a(y))
    same(zg, zo, "ge_a")
    want = u64([1 if a >= b else 0 for a, b in zip(xs, ys)])
    assert np.array_equal(g.rec(zg), want)
    same_stats(o, g)


@pytest.mark.parametrize("w,n", [(1, 5), (2, 64), (5, 100), (16, 513), (64, 1025), (37, 777)])
def test_oaa(mods, seed, w, n):
    o, g = pair(mods, seed)
    rng = np.random.default_rng(w * 1000 + n)
    Wp = rng.integers(0, M64, size=w, dtype=np.uint64)
    u = rng.integers(0, w + 2, size=n).astype(np.uint64)
    zo = o.oaa(o.share(Wp), o.share(u))
    zg = g.oaa(g.share_a(Wp), g.share_a(u))
    same(zg, zo, "oaa")
    want = np.array([Wp[int(i)] if int(i) < w else 0 for i in u], dtype=np.uint64)
    assert np.array_equal(g.rec(zg), want)
    same_stats(o, g)


@pytest.mark.parametrize("tau", [5, 16])
def test_div(mods, seed, tau):
    o, g = pair(mods, seed, tau=tau)
    rng = np.random.default_rng(6)
    Q = [1, 2, 3, 7, 1000, (1 << 40) - 1] + [int(rng.integers(1, 1 << 40)) for _ in range(200)]
    S = [int(rng.integers(0, q + 1)) for q in Q]
    S[0], S[1], S[2] = 1, 0, 3
    qo = o.div(o.share(u64(S)), o.share(u64(Q)))
    qg = g.div(g.share_a(u64(S)), g.share_a(u64(Q)))
    same(qg, qo, "div")
    assert np.array_equal(g.rec(qg), u64([(s << tau) // q for s, q in zip(S, Q)]))
    same_stats(o, g)


@pytest.mark.parametrize("w,n", [(1, 167), (3, 168), (7, 169), (300, 8), (41, 168 * 13 + 1)])
def test_oaa_at_tile_edges(mods, seed, w, n):
    """Tiles of 21 groups of 8 rows: one row short, full, one over; one group and many columns
    (every column range a wavefront of its own); many tiles with split columns."""
    o, g = pair(mods, seed)
    rng = np.random.default_rng(w + n)
    Wp = rng.integers(0, M64, size=w, dtype=np.uint64)
    u = rng.integers(0, w + 2, size=n).astype(np.uint64)
    same(g.oaa(g.share_a(Wp), g.share_a(u)), o.oaa(o.share(Wp), o.share(u)), "oaa")
    same_stats(o, g)


@pytest.mark.parametrize("n", [1, 19, 20, 21, 41, 20480, 20501])
def test_element_kernels_at_tile_edges(mods, seed, n):
    """Tiles of 20 elements whose mask words come from three blocks: short, full and over; for the
    division also the line between four wavefronts per tile and one."""
    o, g = pair(mods, seed, tau=4)
    rng = np.random.default_rng(n)
    x = rng.integers(0, 1 << 39, size=n).astype(np.uint64)
    y = np.where(rng.random(n) < 0.4, x, rng.integers(0, 1 << 39, size=n).astype(np.uint64))
    S, Q = np.minimum(x, y), np.maximum(x, y) + np.uint64(1)
    xo, yo, xg, yg = o.share(x), o.share(y), g.share_a(x), g.share_a(y)
    same(g.eq_a(xg, y), o.eq_a(xo, y), "eq")
    same(g.ge_a(xg, yg), o.ge_a(xo, yo), "ge")
    same(g.div(g.share_a(S), g.share_a(Q)), o.div(o.share(S), o.share(Q)), "div")
    same_stats(o, g)


# ------------------------------------------------------------------ training
def run_train_pair(mods, seed, w, tau=16, H=None, every_level=True):
    from oracle import X_T, X_F, X_M, X_C, X_GAMMA, X_SD, X_L, X_SCORE, X_C_PAPER
    H = w["H"] if H is None else H
    N, d, K = w["N"], w["d"], w["K"]
    o, g = pair(mods, seed, tau=tau, K=K)
    xo, yo = o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1))
    xg, yg = g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1))
    o.train_create(xo, yo, N, d, H)
    g.train_create(xg, yg, N, d, H)
    names = dict(M=X_M, L=X_L, C=X_C, SCORE=X_SCORE, SD=X_SD, GAMMA=X_GAMMA, F=X_F, T=X_T, CP=X_C_PAPER)
    for h in range(H):
        o.train_level(h)
        g.train_level(h)
        if every_level or h == H - 1:
            for nm, what in names.items():
                same(g.train_export(what), o.train_export(what), "level %d %s" % (h, nm))
        same_stats(o, g)
    fo, lo = o.train_finish()
    tree = g.train_finish()
    fg, lg = tree.export()
    same(fg, fo, "tree features")
    same(lg, lo, "tree labels")
    for nm in ("M", "L", "C", "F", "T"):
        same(g.train_export(names[nm]), o.train_export(names[nm]), "finish %s" % nm)
    same_stats(o, g)
    return o, g, tree, (fo, lo)


def test_train_c1(mods, seed):
    import plain_cart
    from paper_2305_00645_amd import workloads as wl
    w = wl.c1_train()
    o, g, tree, (fo, lo) = run_train_pair(mods, seed, w)
    ref = plain_cart.train(w["X"], w["y"], w["K"], w["H"], 16)
    fg, lg = tree.export()
    assert np.array_equal(g.rec(fg).astype(np.int64), ref["T"][:7])
    assert np.array_equal(g.rec(lg).astype(np.int64), ref["T"][7:])
    # inference with the trained tree, binary mode, against plaintext prediction
    rng = np.random.default_rng(5)
    I = (rng.random((333, w["d"])) < 0.5).astype(np.uint64)
    Ro = o.infer(fo, None, lo, w["H"], o.share(I.reshape(-1)), 333, w["d"])
    Rg = g.infer_batch(tree, g.share_a(I.reshape(-1)), 333, w["d"])
    same(Rg, Ro, "inference on trained tree")
    assert np.array_equal(g.rec(Rg).astype(np.int64), plain_cart.predict(ref["T"], w["H"], I))
    same_stats(o, g)


@pytest.mark.parametrize("keyseed", [1, 2])
def test_other_protocol_keys(mods, keyseed):
    """Fresh keys for all five roles: training, then inference with the trained tree."""
    from paper_2305_00645_amd import workloads as wl
    keys = np.random.default_rng(1000 + keyseed).integers(0, 1 << 63, size=(5, 4), dtype=np.uint64) * np.uint64(2) + np.uint64(keyseed & 1)
    w = wl.c1_train(N=300, d=10, depth=3)
    o, g, tree, (fo, lo) = run_train_pair(mods, keys, w, every_level=False)
    I = (np.random.default_rng(keyseed).random((129, w["d"])) < 0.5).astype(np.uint64)
    Ro = o.infer(fo, None, lo, w["H"], o.share(I.reshape(-1)), 129, w["d"])
    Rg = g.infer_batch(tree, g.share_a(I.reshape(-1)), 129, w["d"])
    same(Rg, Ro, "inference with other keys")
    same_stats(o, g)


def test_train_c2_depth7(mods, seed):
    from paper_2305_00645_amd import workloads as wl
    run_train_pair(mods, seed, wl.c2_train(), H=7, every_level=False)


def test_train_multiclass_ragged(mods, seed):
    rng = np.random.default_rng(77)
    N, d, K = 203, 9, 4
    X = (rng.random((N, d)) < 0.4).astype(np.uint64)
    y = (X[:, 0].astype(np.int64) * 2 + X[:, 3].astype(np.int64) + (rng.random(N) < 0.1)) % K
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=3), tau=10)


def test_train_c3_shape_reduced(mods, seed):
    from paper_2305_00645_amd import workloads as wl
    w = wl.c3_train(N=3000, H=4, n_thr=8)
    run_train_pair(mods, seed, w, every_level=False)


def test_train_degenerate(mods, seed):
    X = np.array([[0, 1], [1, 1], [1, 0], [0, 0], [1, 1]], dtype=np.uint64)
    y = np.ones(5, dtype=np.int64)
    Y = np.zeros((5, 2), dtype=np.uint64); Y[:, 1] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=5, d=2, K=2, H=2))
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=5, d=2, K=2, H=0))
    X1 = np.array([[0], [1], [1], [0]], dtype=np.uint64)
    y1 = np.array([0, 1, 1, 0])
    Y1 = np.zeros((4, 2), dtype=np.uint64); Y1[np.arange(4), y1] = 1
    run_train_pair(mods, seed, dict(X=X1, Y=Y1, y=y1, N=4, d=1, K=2, H=2))


def test_train_limits_of_classes_and_precision(mods, seed):
    """Largest class count and largest number of fractional bits the library accepts."""
    rng = np.random.default_rng(99)
    N, d, K = 130, 5, 16
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = (X[:, 0].astype(np.int64) * 8 + X[:, 2].astype(np.int64) * 4 + rng.integers(0, 4, N)) % K
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=3), tau=20)


@pytest.mark.parametrize("N,d,K,H", [(600, 4, 16, 3), (300, 3, 12, 2), (700, 5, 2, 3), (900, 21, 3, 3), (500, 40, 2, 4)])
def test_train_column_group_remainders(mods, seed, N, d, K, H):
    """The statistics contraction splits its d*K+K columns into groups of 64 and a remainder that
    takes its own path: 16 columns beside a full group (two passes of the packed 16-wide tile), 12
    class columns alone at the label level, 12 columns with no full group at all, 2 beside a full
    group, and a remainder of 18 (a launch of its own)."""
    rng = np.random.default_rng(1000 * d + K)
    X = (rng.random((N, d)) < 0.45).astype(np.uint64)
    y = (X[:, 0].astype(np.int64) * 3 + X[:, d - 1].astype(np.int64) + rng.integers(0, 2, N)) % K
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=H), tau=12)


SPLIT_LATE = [(20, 5000, 16, 3)]


@pytest.mark.parametrize("N,d,K,H", SPLIT_LATE)
def test_train_split_of_many_words(mods, seed, N, d, K, H):
    """The last level's node split loads its words after the block function, those before it ahead of it."""
    test_train_column_group_remainders(mods, seed, N, d, K, H)


# (test_shapes.py checks which tiles they take)
COUNT_FEW_NARROW = [(70, 7, 2, 5), (33, 16, 3, 4), (4100, 9, 5, 5), (2100, 37, 2, 4), (2100, 72, 4, 4)]
COUNT_FEW_WIDE = [(257, 63, 2, 4)]


@pytest.mark.parametrize("N,d,K,H", COUNT_FEW_NARROW + COUNT_FEW_WIDE)
def test_train_count_few_nodes(mods, seed, N, d, K, H):
    """Levels of up to eight nodes on the narrow tiles and of 16 on the wide ones: column counts of one tile of 16 with a
    remainder, of three and four tiles, of five (a second workgroup per chunk) and of 19 with a remainder; one sample block, an odd number of
    them and more than one chunk.  Last: few samples and more than 64 columns, on the wide tiles at every level."""
    rng = np.random.default_rng(N + d)
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = rng.integers(0, K, N)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=H), tau=3)


def test_train_count_few_nodes_of_few_columns(mods, seed):
    """Many samples and one column tile: the chunks' sums of a level meet at few lines.  Levels of 1 to 8 nodes on the narrow tiles take
    less than 1.4 times as long as 16 nodes on the wide ones.  Measured 0.95; with a lane's sums in four columns 1.9."""
    _, gtree = mods
    rng = np.random.default_rng(34)
    N, d, K, H = 50000, 16, 2, 5
    X, y = (rng.random((N, d)) < 0.5).astype(np.uint64), rng.integers(0, K, N)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    g = gtree.GTree(seed, tau=2, K=K, profile=True)
    Xs, Ys = g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1))
    g.train_create(Xs, Ys, N, d, H)
    ms = [1e9] * H
    for _ in range(6):
        g.train_reset(Xs, Ys)
        for h in range(H):
            g.stats_reset()
            g.train_level(h)
            ms[h] = min(ms[h], g.prof()["count"][0])
    g.close()
    assert max(ms[:4]) < 1.4 * ms[4], ms


@pytest.mark.parametrize("H", [7, 8])
@pytest.mark.parametrize("literal", [False, True])
def test_train_operand_layouts(mods, seed, H, literal):
    """Columns once per component with the sums on the leaf one-hot, or the sums on the columns:
    20 columns, and the leaf one-hot's 64 (H = 7) or 128 (H = 8) rows of sums on either side of the
    line between the two; both also read back by the learning protocol as printed."""
    from oracle import X_M, X_C, X_SD
    rng = np.random.default_rng(70 + H)
    N, d, K = 75, 9, 2
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = (X[:, 2] ^ X[:, 5]).astype(np.int64)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    if not literal:
        run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=H))
        return
    o, g = pair(mods, seed, K=K)
    o.train_create(o.share(X.reshape(-1)), o.share(Y.reshape(-1)), N, d, H)
    g.train_create(g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1)), N, d, H)
    o.train_set_literal(True); g.train_set_literal(True)
    for h in range(2):
        o.train_level(h); g.train_level(h)
        for what in (X_M, X_C, X_SD):
            same(g.train_export(what), o.train_export(what), "level %d" % h)
    same_stats(o, g)


@pytest.mark.parametrize("N,d,K,H", [(30, 1, 2, 2), (25, 2, 3, 2), (21, 512, 2, 1), (21, 513, 2, 2), (20, 1300, 2, 4)])
def test_train_argmax_widths(mods, seed, N, d, K, H):
    """The tournament of a node: one candidate (no round), one pair, the widest that stays in LDS, the
    narrowest that does not, and levels whose scores are on either side of the line between four
    wavefronts per tile and one."""
    rng = np.random.default_rng(d)
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = (X[:, 0].astype(np.int64) + X[:, d // 2].astype(np.int64)) % K
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=H), tau=6)


# 8, 4 and 2 nodes per wavefront (4, 8 and 16 candidates after padding), fewer nodes than one wavefront
# holds, a wavefront per node at its widest, two, four and eight, and a level whose first round runs in a
# launch of its own because its 4096 x 32 pairs fill the chip
@pytest.mark.parametrize("N,d,K,h", [(20, 3, 2, 5), (20, 5, 2, 1), (24, 12, 3, 4), (20, 32, 2, 2), (20, 33, 2, 3), (20, 128, 2, 2),
                                     (20, 129, 2, 2), (30, 33, 2, 12)])
def test_train_argmax_nodes_per_wavefront(mods, seed, N, d, K, h):
    from oracle import X_C, X_SD, X_SCORE, X_F, X_T
    from paper_2305_00645_amd import workloads as wl
    w = wl.c5_level(N=N, d=d, K=K, h=h)
    o, g = pair(mods, seed, tau=3, K=K)
    o.train_create(o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1)), N, d, h + 1)
    g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), N, d, h + 1)
    # random statistics: every node has scores of its own
    rng = np.random.default_rng(h * 1000 + d)
    n1 = rng.integers(0, 9, size=(1 << h, d, K))
    C = np.concatenate([n1.reshape(1 << h, d * K), n1.max(axis=1)], axis=1).astype(np.uint64)
    st = [w["M"], w["Tprev"], w["F"], C.reshape(-1), w["gamma"].reshape(-1)]
    o.train_import(h, *[o.share(a) for a in st])
    g.train_import(h, *[g.share_a(a) for a in st])
    o.train_level(h); g.train_level(h)
    for what in (X_C, X_SCORE, X_SD, X_F, X_T):
        same(g.train_export(what), o.train_export(what), "export %d" % what)
    same_stats(o, g)
    g.close()


@pytest.mark.parametrize("N,d,K,h", [(20, 1, 2, 5), (20, 1, 2, 6), (24, 2, 2, 6)])
def test_train_argmax_many_nodes_of_one_column(mods, seed, N, d, K, h):
    """32 and 64 nodes per wavefront and one or two columns: more nodes than a party has lanes in a wavefront."""
    test_train_argmax_nodes_per_wavefront(mods, seed, N, d, K, h)


def test_train_argmax_time_follows_the_candidates(mods, seed):
    """65,536 candidates cost about the same as one node's, as 128 nodes' or as 8192 nodes': the per-node
    protocols of a level (score to update) may differ by a factor of 2.2 between the three.  Measured 1.4; with a
    workgroup of eight wavefronts per node, whatever its number of candidates, 14 (one node) and 2.6 (8192)."""
    _, gtree = mods
    best = {}
    for h, d in ((0, 65536), (7, 512), (13, 8)):
        g = gtree.GTree(seed, tau=1, K=2, profile=True)
        N, nh = 8, 1 << h
        rng = np.random.default_rng(d)
        X, y = (rng.random((N, d)) < 0.5).astype(np.uint64), np.arange(N) % 2
        Y = np.zeros((N, 2), dtype=np.uint64); Y[np.arange(N), y] = 1
        Xs, Ys = g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1))
        g.train_create(Xs, Ys, N, d, h + 1)
        st = [g.share_a(np.full(n, v, dtype=np.uint64)) for n, v in
              ((N, nh // 2 - 1 if h else 0), (max(nh // 2, 1), 0), (nh, 1), (nh * 2 * (d + 1), 0), (nh * d, 1))]
        ms = []
        for _ in range(6):
            g.train_import(h, *st)
            g.stats_reset()
            g.train_level(h)
            ms.append(g.prof()["small"][0])
        best[(h, d)] = min(ms)
        g.close()
    assert max(best.values()) < 2.2 * min(best.values()), best


def test_train_deep_tree_few_samples(mods, seed):
    """Far more nodes than samples: 2^11 leaves for 40 samples, most nodes empty."""
    rng = np.random.default_rng(98)
    N, d, K, H = 40, 12, 2, 11
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = (X[:, 1] ^ X[:, 4] ^ X[:, 7]).astype(np.int64)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=H), every_level=False)


def test_train_reset_starts_an_equal_job(mods, seed):
    """gt_train_reset reuses every buffer of the object (limb tiles, partial sums, tree):
    a second job on different data must equal an oracle run started at the same operation
    counter, share by share, and give the plaintext tree."""
    import plain_cart
    from oracle import X_T, X_F, X_M, X_C, X_SD, X_GAMMA
    from paper_2305_00645_amd import workloads as wl
    N, d, H = 300, 11, 3
    wa, wb = wl.c1_train(N=N, d=d, depth=H, seed=31), wl.c1_train(N=N, d=d, depth=H, seed=32)
    o, g = pair(mods, seed)
    xa, ya = g.share_a(wa["X"].reshape(-1)), g.share_a(wa["Y"].reshape(-1))
    oxa, oya = o.share(wa["X"].reshape(-1)), o.share(wa["Y"].reshape(-1))
    g.train_create(xa, ya, N, d, H)
    o.train_create(oxa, oya, N, d, H)
    for h in range(H):
        g.train_level(h); o.train_level(h)
    t1 = g.train_finish(); o.train_finish()
    same(g.train_export(X_T), o.train_export(X_T), "first job T")
    t1.close()
    xb, yb = g.share_a(wb["X"].reshape(-1)), g.share_a(wb["Y"].reshape(-1))
    oxb, oyb = o.share(wb["X"].reshape(-1)), o.share(wb["Y"].reshape(-1))
    g.train_reset(xb, yb)
    o.train_create(oxb, oyb, N, d, H)          # the oracle has no reset: a new object, same operation counter
    assert o.op_counter() == g.op_counter()
    for h in range(H):
        g.train_level(h); o.train_level(h)
        for nm, what in (("M", X_M), ("C", X_C), ("SD", X_SD), ("GAMMA", X_GAMMA), ("F", X_F)):
            same(g.train_export(what), o.train_export(what), "second job level %d %s" % (h, nm))
    t2 = g.train_finish()
    fo, lo = o.train_finish()
    fg, lg = t2.export()
    same(fg, fo, "second job features"); same(lg, lo, "second job labels")
    ref = plain_cart.train(wb["X"], wb["y"], 2, H, 16)
    assert np.array_equal(g.rec(g.train_export(X_T)).astype(np.int64), ref["T"])
    same_stats(o, g)
    # a tree that is still alive when the object finishes again gets buffers of its own
    g.train_reset(xa, ya)
    for h in range(H):
        g.train_level(h)
    t3 = g.train_finish()
    assert np.array_equal(g.rec(t2.export()[0]).astype(np.int64), ref["T"][:(1 << H) - 1])
    ref_a = plain_cart.train(wa["X"], wa["y"], 2, H, 16)
    assert np.array_equal(g.rec(t3.export()[0]).astype(np.int64), ref_a["T"][:(1 << H) - 1])
    t2.close(); t3.close()


def test_levels_and_finish_allocate_nothing(mods, seed):
    """The partial sums of a level's partition (6 x 100,000 words) are there when the first level begins."""
    import torch
    _, gtree = mods
    N, d, H = 100000, 8, 3
    rng = np.random.default_rng(31)
    X, y = (rng.random((N, d)) < 0.5).astype(np.uint64), rng.integers(0, 2, N)
    Y = np.zeros((N, 2), dtype=np.uint64); Y[np.arange(N), y] = 1
    for job in range(2):                                  # the first one loads the kernels
        g = gtree.GTree(seed, K=2)
        Xs, Ys = g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1))
        g.train_create(Xs, Ys, N, d, H)
        torch.cuda.synchronize()
        free = [torch.cuda.mem_get_info()[0]]
        for h in range(H):
            g.train_level(h)
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])
        tree = g.train_finish()
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
        tree.close(); g.close()
    assert len(set(free)) == 1, free


def test_export_after_import_needs_a_level(mods, seed):
    Oracle, gtree = mods
    from oracle import X_C, X_M
    from paper_2305_00645_amd import workloads as wl
    w = wl.c5_level(N=100, d=5, K=2, h=2)
    g = gtree.GTree(seed, K=2)
    g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), 100, 5, 3)
    st = [w["M"], w["Tprev"], w["F"], np.zeros(4 * 12, dtype=np.uint64), w["gamma"].reshape(-1)]
    g.train_import(2, *[g.share_a(a) for a in st])
    assert np.array_equal(g.rec(g.train_export(X_M)), w["M"])
    with pytest.raises(gtree.GtError) as e:
        g.train_export(X_C)
    assert e.value.code == gtree.GT_ESTATE
    g.train_level(2)
    assert g.train_export(X_C).n == 4 * 12


@pytest.mark.parametrize("case", ["c1", "c2", "multi", "degenerate"])
def test_heuristic_by_reconstruction(mods, seed, case):
    """Reconstruct-and-score heuristic (host analogue of the TEE-based protocol): share by
    share against the oracle in the same mode, and the reconstructed tree against the
    plaintext CART (hence equal to the MPC heuristic's)."""
    import plain_cart
    from oracle import X_T, X_F, X_M, X_C, X_GAMMA, X_SD, X_SCORE
    from paper_2305_00645_amd import workloads as wl
    tau = 16
    if case == "c1":
        w = wl.c1_train()
    elif case == "c2":
        w = wl.c2_train(H=5)
    elif case == "multi":
        rng = np.random.default_rng(77)
        N, d, K = 203, 9, 4
        X = (rng.random((N, d)) < 0.4).astype(np.uint64)
        y = (X[:, 0].astype(np.int64) * 2 + X[:, 3].astype(np.int64) + (rng.random(N) < 0.1)) % K
        Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
        w, tau = dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=3), 10
    else:
        X = np.array([[0, 1], [1, 1], [1, 0], [0, 0], [1, 1]], dtype=np.uint64)
        y = np.ones(5, dtype=np.int64)
        Y = np.zeros((5, 2), dtype=np.uint64); Y[:, 1] = 1
        w = dict(X=X, Y=Y, y=y, N=5, d=2, K=2, H=2)
    N, d, K, H = w["N"], w["d"], w["K"], w["H"]
    o, g = pair(mods, seed, tau=tau, K=K)
    o.train_create(o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1)), N, d, H)
    g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), N, d, H)
    o.train_set_heuristic(True); g.train_set_heuristic(True)
    for h in range(H):
        o.train_level(h); g.train_level(h)
        for nm, what in (("M", X_M), ("C", X_C), ("SCORE", X_SCORE), ("SD", X_SD), ("GAMMA", X_GAMMA), ("F", X_F), ("T", X_T)):
            same(g.train_export(what), o.train_export(what), "level %d %s" % (h, nm))
    fo, lo = o.train_finish()
    tree = g.train_finish()
    fg, lg = tree.export()
    same(fg, fo, "features"); same(lg, lo, "labels")
    ref = plain_cart.train(w["X"], w["y"], K, H, tau)
    assert np.array_equal(g.rec(g.train_export(X_T)).astype(np.int64), ref["T"])
    assert np.array_equal(g.rec(g.train_export(X_F)).astype(np.int64), ref["F"])
    same_stats(o, g)
    assert o.scorer_bytes() == g.scorer_bytes()
    tree.close(); g.close()


@pytest.mark.parametrize("w,n", [(1, 5), (16, 513), (37, 100)])
def test_oaa_as_printed(mods, seed, w, n):
    """Array access element by element as the paper prints it: oracle's shares, W[u], and
    exactly N(4l-1) bits per party counted by the kernels."""
    o, g = pair(mods, seed)
    rng = np.random.default_rng(w * 1000 + n)
    Wp = rng.integers(0, M64, size=w, dtype=np.uint64)
    u = rng.integers(0, w + 2, size=n).astype(np.uint64)
    so, sg = (o.share(Wp), o.share(u)), (g.share_a(Wp), g.share_a(u))
    o.stats_reset(); g.stats_reset()
    zo, zg = o.oaa_literal(*so), g.oaa_literal(*sg)
    same(zg, zo, "oaa as printed")
    assert np.array_equal(g.rec(zg), np.array([Wp[int(i)] if int(i) < w else 0 for i in u], dtype=np.uint64))
    same_stats(o, g)
    assert int(g.wire_bits_dev()[0].sum()) == w * n * (4 * 64 - 1) and g.stats()[0] == 9
    same(g.oaa(*sg), o.oaa(*so), "fused access after the literal one (shared scratch left clean)")


@pytest.mark.parametrize("case", ["c1", "c2"])
def test_learning_as_printed(mods, seed, case):
    """Training with the learning protocol as printed (whole-tree scans, per-element
    SelectShare, local accumulation): share by share against the oracle in the same mode, the
    tree against the plaintext CART, the message volume against the fused mode."""
    import plain_cart
    from oracle import X_T, X_F, X_M, X_C, X_GAMMA, X_SD, X_SCORE
    from paper_2305_00645_amd import workloads as wl
    w = wl.c1_train(N=200, d=8, depth=3) if case == "c1" else wl.c2_train(H=4)
    N, d, K, H = w["N"], w["d"], w["K"], w["H"]
    o, g = pair(mods, seed, K=K)
    o.train_create(o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1)), N, d, H)
    g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), N, d, H)
    o.train_set_literal(True); g.train_set_literal(True)
    for h in range(H):
        o.train_level(h); g.train_level(h)
        for nm, what in (("M", X_M), ("C", X_C), ("SCORE", X_SCORE), ("SD", X_SD), ("GAMMA", X_GAMMA), ("F", X_F)):
            same(g.train_export(what), o.train_export(what), "level %d %s" % (h, nm))
    fo, lo = o.train_finish()
    tree = g.train_finish()
    fg, lg = tree.export()
    same(fg, fo, "features"); same(lg, lo, "labels")
    ref = plain_cart.train(w["X"], w["y"], K, H, 16)
    assert np.array_equal(g.rec(g.train_export(X_T)).astype(np.int64), ref["T"])
    same_stats(o, g)
    g2 = mods[1].GTree(seed, K=K)
    g2.train_create(g2.share_a(w["X"].reshape(-1)), g2.share_a(w["Y"].reshape(-1)), N, d, H)
    for h in range(H):
        g2.train_level(h)
    g2.train_finish().close()
    assert int(g.stats()[1][0].sum()) > 5 * int(g2.stats()[1][0].sum())      # what the fusion into inner products saves
    tree.close(); g.close(); g2.close()


@pytest.mark.parametrize("case", ["c1", "c2", "multi", "c3small"])
def test_partition_by_products(mods, seed, case):
    """Data partition by products with the previous level's leaf one-hot: share by share
    against the oracle in the same mode at every level, the tree against the plaintext CART."""
    import plain_cart
    from oracle import X_T, X_F, X_M, X_C, X_GAMMA, X_SD, X_SCORE, X_L
    from paper_2305_00645_amd import workloads as wl
    tau = 16
    if case == "c1":
        w = wl.c1_train()
    elif case == "c2":
        w = wl.c2_train(H=6)
    elif case == "c3small":
        w = wl.c3_train(N=3000, H=4, n_thr=8)
    else:
        rng = np.random.default_rng(77)
        N, d, K = 203, 9, 4
        X = (rng.random((N, d)) < 0.4).astype(np.uint64)
        y = (X[:, 0].astype(np.int64) * 2 + X[:, 3].astype(np.int64) + (rng.random(N) < 0.1)) % K
        Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
        w, tau = dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=3), 10
    N, d, K, H = w["N"], w["d"], w["K"], w["H"]
    o, g = pair(mods, seed, tau=tau, K=K)
    o.train_create(o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1)), N, d, H)
    g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), N, d, H)
    o.train_set_partition(True); g.train_set_partition(True)
    for h in range(H):
        o.train_level(h); g.train_level(h)
        for nm, what in (("M", X_M), ("L", X_L), ("C", X_C), ("SCORE", X_SCORE), ("SD", X_SD), ("GAMMA", X_GAMMA), ("F", X_F)):
            same(g.train_export(what), o.train_export(what), "level %d %s" % (h, nm))
    fo, lo = o.train_finish()
    tree = g.train_finish()
    fg, lg = tree.export()
    same(fg, fo, "features"); same(lg, lo, "labels")
    same(g.train_export(X_M), o.train_export(X_M), "M at the label level")
    ref = plain_cart.train(w["X"], w["y"], K, H, tau)
    assert np.array_equal(g.rec(g.train_export(X_T)).astype(np.int64), ref["T"])
    same_stats(o, g)
    tree.close(); g.close()


@pytest.mark.parametrize("N,d,H", [(75, 67, 7), (41, 130, 8), (33, 3, 9)])
def test_partition_by_products_deep(mods, seed, N, d, H):
    """More than one chunk of 32 nodes in the level before (64, 128 and 256 of them), columns just above one
    and two groups of 64 or far below, a ragged last block of samples: both products' chunks and the passes of
    zero-sharing words that are spread over them."""
    from oracle import X_M, X_L, X_C, X_SD
    rng = np.random.default_rng(10 * N + H)
    K = 2
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = rng.integers(0, K, N)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    o, g = pair(mods, seed, tau=4, K=K)
    o.train_create(o.share(X.reshape(-1)), o.share(Y.reshape(-1)), N, d, H)
    g.train_create(g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1)), N, d, H)
    o.train_set_partition(True); g.train_set_partition(True)
    for h in range(H):
        o.train_level(h); g.train_level(h)
        for what in (X_M, X_L, X_C, X_SD):
            same(g.train_export(what), o.train_export(what), "level %d, export %d" % (h, what))
    o.train_finish()
    g.train_finish().close()
    same(g.train_export(X_M), o.train_export(X_M), "M at the label level")
    same_stats(o, g)
    g.close()


@pytest.mark.parametrize("N,d,H", [(15, 31, 2), (17, 32, 3), (31, 33, 6), (32, 64, 2), (2049, 65, 3)])
def test_partition_by_products_few_nodes(mods, seed, N, d, H):
    """At most 32 nodes in the level before (16 samples x 32 columns per step): a last tile with one sample, without
    its second half and full, column counts around a step and around the limbs' padding to 64."""
    test_partition_by_products_deep(mods, seed, N, d, H)


PRODUCTS_WORDS = [(21, 67, 9), (19, 4097, 2)]


@pytest.mark.parametrize("N,d,H", PRODUCTS_WORDS)
def test_partition_by_products_words(mods, seed, N, d, H):
    """The one-hot of the last levels as words that a second launch turns into limbs, after levels that write bytes; of all levels, where the features are many."""
    test_partition_by_products_deep(mods, seed, N, d, H)


def test_train_errors(mods, seed):
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    w = wl.c1_train(N=32, d=4, depth=2)
    g = gtree.GTree(seed)
    xg, yg = g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1))
    g.train_create(xg, yg, 32, 4, 2)
    with pytest.raises(gtree.GtError) as e:
        g.train_level(1)                       # out of order
    assert e.value.code == gtree.GT_ESTATE
    with pytest.raises(gtree.GtError) as e:
        g.train_create(xg, yg, 33, 4, 2)       # buffers too small
    assert e.value.code == gtree.GT_EINVAL
    with pytest.raises(gtree.GtError):
        g.train_create(xg, yg, 32, 4, 99)      # depth over the limit


# ------------------------------------------------------------------ inference
@pytest.mark.parametrize("binary,NI,H", [(False, 1000, 7), (True, 1000, 7), (False, 77, 3), (True, 1, 2), (True, 5, 16), (False, 9, 13)])
def test_infer(mods, seed, binary, NI, H):
    import plain_cart
    from paper_2305_00645_amd import workloads as wl
    w = wl.c4_infer(NI=NI, H=H, binary=binary)
    o, g = pair(mods, seed)
    fo, lo = o.share(w["feat"]), o.share(w["leaf"])
    fg, lg = g.share_a(w["feat"]), g.share_a(w["leaf"])
    to = tg = None
    if not binary:
        to, tg = o.share(w["thr"]), g.share_a(w["thr"])
    Io, Ig = o.share(w["I"].reshape(-1)), g.share_a(w["I"].reshape(-1))
    tree = g.tree_import(fg, tg, lg, H)
    Ro = o.infer(fo, to, lo, H, Io, NI, w["d"])
    Rg = g.infer_batch(tree, Ig, NI, w["d"])
    same(Rg, Ro, "inference")
    T = np.concatenate([w["feat"], w["leaf"]]).astype(np.int64)
    thr = None if binary else np.concatenate([w["thr"], np.zeros(1 << H, dtype=np.uint64)])
    assert np.array_equal(g.rec(Rg).astype(np.int64), plain_cart.predict(T, H, w["I"], thr))
    same_stats(o, g)


@pytest.mark.parametrize("how", ["levelwise", 16, 32, 64])
@pytest.mark.parametrize("binary,NI,H,d", [(False, 333, 5, 16), (True, 1000, 7, 16), (True, 70, 9, 3), (False, 129, 3, 37), (True, 17, 0, 5)])
def test_infer_paths_agree(mods, seed, how, binary, NI, H, d):
    """The level-by-level path and the one-launch path with each of its three tile shapes (16, 32, 64
    instances per workgroup; column counts that are not a multiple of a step's columns and instance counts that
    leave a ragged tile) all give the oracle's shares, rounds, bytes and bits."""
    import plain_cart
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    w = wl.c4_infer(NI=NI, H=H, d=d, binary=binary, seed=4000 + H)
    flags = gtree.GT_FLAG_LEVELWISE_INFER if how == "levelwise" else gtree.GT_FLAG_INFER_TILE[how]
    o, g = Oracle(seed), gtree.GTree(seed, flags=flags)
    fo, lo = o.share(w["feat"]), o.share(w["leaf"])
    fg, lg = g.share_a(w["feat"]), g.share_a(w["leaf"])
    to = tg = None
    if not binary:
        to, tg = o.share(w["thr"]), g.share_a(w["thr"])
    Io, Ig = o.share(w["I"].reshape(-1)), g.share_a(w["I"].reshape(-1))
    tree = g.tree_import(fg, tg, lg, H)
    Ro = o.infer(fo, to, lo, H, Io, NI, d)
    Rg = g.infer_batch(tree, Ig, NI, d)
    same(Rg, Ro, "inference (%s)" % how)
    T = np.concatenate([w["feat"], w["leaf"]]).astype(np.int64)
    thr = None if binary else np.concatenate([w["thr"], np.zeros(1 << H, dtype=np.uint64)])
    assert np.array_equal(g.rec(Rg).astype(np.int64), plain_cart.predict(T, H, w["I"], thr))
    same_stats(o, g)
    tree.close(); g.close()


@pytest.mark.parametrize("binary,NI,H,d", [(False, 1, 2, 90), (False, 3, 7, 84), (True, 8, 3, 85), (False, 2501, 2, 19), (True, 70001, 1, 3), (False, 40009, 2, 6)])
def test_infer_tile_choice_extremes(mods, seed, binary, NI, H, d):
    """The split of the lanes chosen from the batch: one group of 8 instances with 42 or 84 columns a step (as many columns,
    one more, a few more), and single wavefronts with three groups and a ragged last tile."""
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    w = wl.c4_infer(NI=NI, H=H, d=d, binary=binary, seed=5000 + NI)
    o, g = Oracle(seed), gtree.GTree(seed)
    fo, lo, fg, lg = o.share(w["feat"]), o.share(w["leaf"]), g.share_a(w["feat"]), g.share_a(w["leaf"])
    to = tg = None
    if not binary:
        to, tg = o.share(w["thr"]), g.share_a(w["thr"])
    Io, Ig = o.share(w["I"].reshape(-1)), g.share_a(w["I"].reshape(-1))
    tree = g.tree_import(fg, tg, lg, H)
    same(g.infer_batch(tree, Ig, NI, d), o.infer(fo, to, lo, H, Io, NI, d), "inference")
    same_stats(o, g)
    tree.close(); g.close()


# (test_shapes.py checks which kernel and how many groups the cases of the following lists take)
SINGLE_WAVEFRONT_TILES = [(True, 33003, 2, 22), (False, 52005, 1, 12), (False, 30001, 1, 150), (True, 30001, 1, 294)]


@pytest.mark.parametrize("binary,NI,H,d", SINGLE_WAVEFRONT_TILES)
def test_infer_single_wavefront_tiles(mods, seed, binary, NI, H, d):
    """Batches of more tiles than k_infer_ahead takes: workgroups of one wavefront with two to four groups of 8 instances
    (10, 7, 5 columns a step, the last lanes idle where these do not divide 21), with a ragged last tile."""
    test_infer_tile_choice_extremes(mods, seed, binary, NI, H, d)


AHEAD_TILES = [(False, 1, 1, 1), (True, 4, 1, 64), (False, 5, 4, 22), (True, 2044, 8, 13), (False, 4101, 3, 43), (True, 8190, 4, 30),
               (False, 10004, 2, 200), (False, 13001, 4, 9), (True, 20011, 1, 70), (False, 16391, 2, 33), (True, 8, 9, 200), (False, 5, 5, 150), (True, 2699, 0, 5),
               (False, 133, 0, 3)]


@pytest.mark.parametrize("binary,NI,H,d", AHEAD_TILES)
def test_infer_ahead_tiles(mods, seed, binary, NI, H, d):
    """Batches whose tiles are all on the chip at once: one column and more than a step has, one step and several (an odd and
    an even number, so that either buffer of the material comes first), only the first half of a group's instances
    and one of the second, 84, 42 and 21 lanes per party, several workgroups on a compute unit."""
    test_infer_tile_choice_extremes(mods, seed, binary, NI, H, d)


@pytest.mark.parametrize("binary,ntrees,NI,H,d", [(True, 7, 150, 3, 9), (False, 3, 77, 4, 16), (True, 40, 1000, 2, 5)])
def test_forest_in_one_launch(mods, seed, binary, ntrees, NI, H, d):
    """Many shallow trees on one batch in one launch: shares, operation ids, rounds, bytes
    and bits are those of the oracle's single-tree inference called tree after tree."""
    import plain_cart
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    o, g = pair(mods, seed)
    rng = np.random.default_rng(500 + ntrees)
    I = rng.integers(0, 1 << 16, size=(NI, d)).astype(np.uint64)
    if binary:
        I &= np.uint64(1)
    Io, Ig = o.share(I.reshape(-1)), g.share_a(I.reshape(-1))
    plain = [wl.random_tree(H, d, rng, thresholds=not binary) for _ in range(ntrees)]
    so = [(o.share(f), None if t is None else o.share(t), o.share(l)) for f, t, l in plain]
    trees = []
    for f, t, l in plain:
        trees.append(g.tree_import(g.share_a(f), None if t is None else g.share_a(t), g.share_a(l), H))
    assert o.op_counter() == g.op_counter()
    forest = g.forest_create(trees)
    for tr in trees:
        tr.close()                               # the forest holds copies
    Rg = g.infer_forest(forest, Ig, NI, d).components()
    for t, (f, th, l) in enumerate(plain):
        Ro = o.infer(so[t][0], so[t][1], so[t][2], H, Io, NI, d)
        assert np.array_equal(Rg[:, t * NI:(t + 1) * NI], Ro), t
        T = np.concatenate([f, l]).astype(np.int64)
        thr = None if binary else np.concatenate([th, np.zeros(1 << H, dtype=np.uint64)])
        got = (Rg[0, t * NI:(t + 1) * NI] + Rg[1, t * NI:(t + 1) * NI] + Rg[2, t * NI:(t + 1) * NI]).astype(np.int64)
        assert np.array_equal(got, plain_cart.predict(T, H, I, thr))
    same_stats(o, g)
    forest.close(); g.close()


# k_infer_ahead with 21 lanes per party: 1 group of 8 instances with 21 columns a step (more and fewer features), ragged
# tiles of 2, 3 and 4 groups
FOREST_FEW = [(False, 300, 1, 3, 16), (False, 700, 5, 2, 9), (True, 600, 9, 2, 23), (True, 300, 30, 2, 16), (False, 500, 20, 3, 5), (True, 900, 30, 1, 3)]


@pytest.mark.parametrize("binary,ntrees,NI,H,d", FOREST_FEW)
def test_forest_on_few_instances(mods, seed, binary, ntrees, NI, H, d):
    test_forest_in_one_launch(mods, seed, binary, ntrees, NI, H, d)


# tiles asked for that are on the chip at once (k_infer_ahead, 21 and 42 lanes per party), and narrow rows on one and two wavefronts
SMALL_FORCED_TILES = [(16, True, 9001, 2, 5), (32, False, 20003, 2, 5), (32, True, 8300, 1, 100), (64, False, 17000, 1, 60), (64, True, 17003, 1, 40),
                      (64, True, 40007, 2, 5), (64, False, 33003, 1, 13), (32, True, 33003, 1, 13)]


@pytest.mark.parametrize("how,binary,NI,H,d", SMALL_FORCED_TILES)
def test_infer_small_forced_tiles(mods, seed, how, binary, NI, H, d):
    test_infer_paths_agree(mods, seed, how, binary, NI, H, d)


WIDE_FORCED_TILES = [(32, True, 33003, 1, 60), (32, False, 33010, 1, 50), (32, False, 20003, 1, 100), (64, True, 36001, 1, 50), (64, False, 33003, 1, 60),
                     (64, False, 20003, 1, 100)]


@pytest.mark.parametrize("how,binary,NI,H,d", WIDE_FORCED_TILES)
def test_infer_forced_tiles_of_wide_rows(mods, seed, how, binary, NI, H, d):
    """Tiles asked for, more of them than k_infer_ahead takes and rows that do not stay in the L2s: two and four wavefronts per tile."""
    test_infer_paths_agree(mods, seed, how, binary, NI, H, d)


# one or two groups per wavefront (the sums of one without thresholds meet through LDS): fewer tree slots and features than the
# columns of a step (21, 10), as many, more; a last tile with one group of two, a last group with one instance
ONE_OR_TWO_GROUPS_FORESTS = [(False, 1100, 7, 2, 23), (True, 1100, 7, 2, 23), (False, 1100, 3, 5, 5), (True, 1100, 3, 5, 22), (False, 1100, 13, 4, 12),
                       (True, 1100, 9, 4, 12), (False, 1100, 9, 2, 9), (True, 1100, 12, 1, 11)]
ONE_OR_TWO_GROUPS_TILES = [(16, False, 16401, 3, 12), (16, True, 16405, 2, 30), (16, False, 17001, 4, 9)]


@pytest.mark.parametrize("binary,ntrees,NI,H,d", ONE_OR_TWO_GROUPS_FORESTS)
def test_forest_one_or_two_groups(mods, seed, binary, ntrees, NI, H, d):
    test_forest_in_one_launch(mods, seed, binary, ntrees, NI, H, d)


@pytest.mark.parametrize("how,binary,NI,H,d", ONE_OR_TWO_GROUPS_TILES)
def test_infer_one_or_two_groups(mods, seed, how, binary, NI, H, d):
    test_infer_paths_agree(mods, seed, how, binary, NI, H, d)


OWN_ROWS_ALONE = (6495, 252)


def test_own_rows_wait_for_no_load(mods, seed):
    """A wavefront per SIMD: the grid over the rows' own values, fetched a step ahead, takes as long as the one against a
    shared array (within 2 %).  Measured 0.98 to 0.99; where a step waits for its fetch 1.05 to 1.06.  (Launches after a call's first, whose
    rows come from memory.)"""
    _, gtree = mods
    rng = np.random.default_rng(5)
    n, d = OWN_ROWS_ALONE
    g = gtree.GTree(seed, flags=gtree.GT_FLAG_LEVELWISE_INFER, profile=True)
    trees = {H: g.tree_import(g.share_a(rng.integers(0, d, (1 << H) - 1).astype(np.uint64)), None, g.share_a(u64([0, 1] * (1 << H - 1))), H) for H in (1, 9)}
    I = g.share_a((rng.random(n * d) < 0.5).astype(np.uint64))
    W, u = g.share_a(rng.integers(0, 9, d).astype(np.uint64)), g.share_a(rng.integers(0, d, n).astype(np.uint64))
    rows, common = {1: 1e9, 9: 1e9}, 1e9
    for _ in range(40):
        for H in rows:
            g.stats_reset(); g.infer_batch(trees[H], I, n, d); rows[H] = min(rows[H], g.prof()["eqgrid_rows"][0])
        g.stats_reset(); g.oaa(W, u); common = min(common, g.prof()["eqgrid"][0])
    g.close()
    assert (rows[9] - rows[1]) / 8 < 1.02 * common, (rows, common)


LEVELWISE_LARGE = (False, 30001, 6, 3)


def test_infer_levelwise_large(mods, seed):
    """Level by level with thresholds and two wavefronts per SIMD: the grid with two sums under issue priorities."""
    test_infer_paths_agree(mods, seed, "levelwise", *LEVELWISE_LARGE)


def test_forest_time_on_one_instance(mods, seed):
    """1,000 trees on one instance fit the wavefront slots at once: less than twice the time of 40 trees, which
    leave most of the chip idle.  Measured 1.2; with four wavefronts per tree 3.3, from two fillings of the slots."""
    _, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    rng, H, d, ms = np.random.default_rng(9), 3, 16, {}
    for ntrees in (40, 1000):
        g = gtree.GTree(seed, profile=True)
        trees = []
        for _ in range(ntrees):
            f, t, l = wl.random_tree(H, d, rng, thresholds=True)
            trees.append(g.tree_import(g.share_a(f), g.share_a(t), g.share_a(l), H))
        forest = g.forest_create(trees)
        for tr in trees:
            tr.close()
        I = g.share_a(rng.integers(0, 1 << 16, size=d).astype(np.uint64))
        times = []
        for _ in range(6):
            g.stats_reset()
            g.infer_forest(forest, I, 1, d)
            times.append(g.prof()["infer"][0])
        ms[ntrees] = min(times)
        forest.close(); g.close()
    assert ms[1000] < 2 * ms[40], ms


def test_infer_depth0(mods, seed):
    o, g = pair(mods, seed)
    lo, lg = o.share(u64([3])), g.share_a(u64([3]))
    Io, Ig = o.share(u64([1, 0, 1, 1])), g.share_a(u64([1, 0, 1, 1]))
    tree = g.tree_import(g.new(0), None, lg, 0)
    Ro = o.infer(np.zeros((3, 0), dtype=np.uint64), None, lo, 0, Io, 2, 2)
    Rg = g.infer_batch(tree, Ig, 2, 2)
    same(Rg, Ro, "depth 0")
    assert g.rec(Rg).tolist() == [3, 3]


# the shapes reach the variants of the statistics contraction: few nodes; 128 nodes with a
# remainder of 4 columns beside a full group of 64; 256 nodes with a remainder of 18 columns;
# exactly 64 columns; 64 nodes (two row tiles per workgroup) with a remainder above 32
# columns; 32 nodes (one row tile per workgroup) with exactly 64 columns.  The fourth shape (exactly
# 64 columns, 128 nodes) and the third keep the sums on the columns, the others on the leaf one-hot.
@pytest.mark.parametrize("N,d,K,h", [(5000, 12, 4, 3), (1500, 16, 4, 7), (700, 40, 2, 8),
                                     (900, 15, 4, 7), (900, 24, 4, 6), (600, 31, 2, 5)])
def test_single_level_from_imported_state(mods, seed, N, d, K, h):
    """One split-scoring level started from a synthetic state (reduced C5 recipe)."""
    from oracle import X_M, X_C, X_SD, X_SCORE, X_F
    from paper_2305_00645_amd import workloads as wl
    w = wl.c5_level(N=N, d=d, K=K, h=h)
    N, d, K, h = w["N"], w["d"], w["K"], w["h"]
    o, g = pair(mods, seed, K=K)
    xo, yo = o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1))
    xg, yg = g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1))
    o.train_create(xo, yo, N, d, h + 1)
    g.train_create(xg, yg, N, d, h + 1)
    CW = d * K + K
    st = [w["M"], w["Tprev"], w["F"], np.zeros((1 << h) * CW, dtype=np.uint64), w["gamma"].reshape(-1)]
    so = [o.share(a) for a in st]
    sg = [g.share_a(a) for a in st]
    o.train_import(h, *so)
    g.train_import(h, *sg)
    o.train_level(h)
    g.train_level(h)
    for what in (X_M, X_C, X_SCORE, X_SD, X_F):
        same(g.train_export(what), o.train_export(what), "import level, export %d" % what)
    # counts equal the plaintext histogram of the routed samples
    X, y = w["X"].astype(np.int64), w["y"]
    M = 2 * w["M"].astype(np.int64) + 1 + X[np.arange(N), w["Tprev"].astype(np.int64)[w["M"].astype(np.int64) - ((1 << (h - 1)) - 1)]]
    assert np.array_equal(g.rec(g.train_export(X_M)).astype(np.int64), M)
    C = g.rec(g.train_export(X_C)).astype(np.int64).reshape(1 << h, CW)
    for r in range(1 << h):
        sel = M == (1 << h) - 1 + r
        for c in range(K):
            assert C[r, d * K + c] == (sel & (y == c)).sum()
            assert np.array_equal(C[r, :d * K].reshape(d, K)[:, c], X[sel & (y == c)].sum(axis=0))
    same_stats(o, g)


# columns stored once per component: two groups of 128 nodes with a remainder of 10 columns (narrow tiles) and of
# 30 (a launch of its own); four row tiles with remainders of 18 and 38.  Sums on the columns: a remainder of 8
# columns beside a full group, with two groups of 128 nodes
@pytest.mark.parametrize("N,d,K,h", [(700, 100, 2, 8), (500, 110, 2, 8), (600, 40, 2, 7), (600, 50, 2, 7), (500, 17, 4, 8)])
def test_single_level_operand_layouts(mods, seed, N, d, K, h):
    test_single_level_from_imported_state(mods, seed, N, d, K, h)


def test_train_sums_on_columns_with_narrow_remainder(mods, seed):
    """72 columns and depth 9: the leaf one-hot has more rows than the columns, so the columns carry the sums at
    every level, and their remainder of 8 beside a full group meets one, two and four row tiles per workgroup."""
    rng = np.random.default_rng(179)
    N, d, K = 60, 17, 4
    X = (rng.random((N, d)) < 0.5).astype(np.uint64)
    y = (X[:, 0].astype(np.int64) * 2 + X[:, 16].astype(np.int64) + rng.integers(0, 2, N)) % K
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    run_train_pair(mods, seed, dict(X=X, Y=Y, y=y, N=N, d=d, K=K, H=9), tau=3, every_level=False)


def test_launch_and_message_pattern_is_data_independent(mods, seed):
    """Only sizes and depth may show (Sec. I, goals): two data sets of the same shape give
    the same operation count, rounds, wire bytes and kernel launches per class."""
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    seen = []
    for s in (21, 22):
        w = wl.c1_train(N=300, d=7, depth=3, seed=s)
        g = gtree.GTree(seed, K=2, profile=True)
        g.train_create(g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1)), 300, 7, 3)
        for h in range(3):
            g.train_level(h)
        tree = g.train_finish()
        g.infer_batch(tree, g.share_a(w["X"].reshape(-1)), 300, 7)
        rounds, wire, _ = g.stats()
        seen.append((g.op_counter(), rounds, wire.tolist(), {k: v[1] for k, v in g.prof().items()}))
        tree.close(); g.close()
    assert seen[0] == seen[1]
    assert seen[0][3]["eqgrid"] > 0 and seen[0][3]["count"] > 0


def test_calls_return_before_the_stream_drains(mods, seed):
    """Calls only enqueue: with a long kernel ahead of it on the context's stream a whole
    training level returns to the host while that kernel is still running, and the results
    still equal the oracle's."""
    import torch
    from oracle import X_C, X_SD, X_M
    Oracle, gtree = mods
    from paper_2305_00645_amd import workloads as wl
    w = wl.c1_train(N=500, d=9, depth=2)
    N, d, H = w["N"], w["d"], w["H"]
    o = Oracle(seed)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        g = gtree.GTree(seed, stream=st)
        xg, yg = g.share_a(w["X"].reshape(-1)), g.share_a(w["Y"].reshape(-1))
        g.train_create(xg, yg, N, d, H)
        g.train_level(0)
        st.synchronize()
        torch.cuda._sleep(int(2.0e9))            # about a second of GPU time on this stream
        g.train_level(1)
        tree = g.train_finish()
        pending = not st.query()                 # the sleep kernel (and everything behind it) has not finished
        st.synchronize()
        assert pending, "gt_train_level/gt_train_finish waited for the stream"
        o.train_create(o.share(w["X"].reshape(-1)), o.share(w["Y"].reshape(-1)), N, d, H)
        o.train_level(0); o.train_level(1)
        fo, lo = o.train_finish()
        fg, lg = tree.export()
        same(fg, fo, "features"); same(lg, lo, "labels")
        same(g.train_export(X_M), o.train_export(X_M), "M")
        same_stats(o, g)
        tree.close(); g.close()


def test_context_on_a_side_stream(mods, seed):
    """The library enqueues on the stream it is given (default priority)."""
    import torch
    Oracle, gtree = mods
    o = Oracle(seed)
    st = torch.cuda.Stream()
    rng = np.random.default_rng(9)
    x = rng.integers(0, M64, size=3000, dtype=np.uint64)
    y = rng.integers(0, M64, size=3000, dtype=np.uint64)
    with torch.cuda.stream(st):
        g = gtree.GTree(seed, stream=st)
        xg, yg = g.share_a(x), g.share_a(y)
        zg = g.mult(xg, yg)
        ug = g.oaa(g.share_a(x[:37]), g.share_a(np.arange(500, dtype=np.uint64) % 40))
        st.synchronize()
        zo = o.mult(o.share(x), o.share(y))
        uo = o.oaa(o.share(x[:37]), o.share(np.arange(500, dtype=np.uint64) % 40))
        same(zg, zo, "mult on side stream")
        same(ug, uo, "oaa on side stream")
        g.close()


OAA_THREE_WAVEFRONTS = [(64, 100003), (5, 364001), (500, 20003)]


@pytest.mark.parametrize("w,n", OAA_THREE_WAVEFRONTS)
def test_oaa_three_wavefronts(mods, seed, w, n):
    """Three wavefronts per SIMD, the rows' opened values in LDS: several ranges, one range of few columns, few rows."""
    test_oaa_at_tile_edges(mods, seed, w, n)


# one sample, one block and one over; few blocks, whose features go in parts of one to seven; classes of both variants; more blocks than workgroups; the
# columns kept per party (many nodes for the columns) and per component
SETUP_SHAPES = [(1, 1, 2, 1), (31, 33, 5, 1), (32, 32, 4, 2), (33, 65, 16, 1), (64, 31, 3, 2), (24601, 3, 4, 1), (65, 2, 5, 7), (40, 3, 2, 8)]


@pytest.mark.parametrize("N,d,K,H", SETUP_SHAPES)
def test_train_setup_shapes(mods, seed, N, d, K, H):
    """The launch that makes the transposed data, the products and the class columns, through whole trainings."""
    test_train_column_group_remainders(mods, seed, N, d, K, H)


# one part of 32 features, two of 17 and 16, two of 32, three; the same with the columns kept per party; two items of a workgroup, in two parts
# (test_shapes.py checks it)
SETUP_SPLITS = [(4129, 32, 2, 2), (4129, 33, 4, 2), (4129, 64, 5, 2), (4129, 65, 1, 9), (4129, 32, 5, 9), (13001, 64, 2, 2), (12500, 64, 5, 10)]


@pytest.mark.parametrize("N,d,K,H", SETUP_SPLITS)
def test_train_setup_splits(mods, seed, N, d, K, H):
    """The same launch where samples are many: the sums of all its columns at the root, and the samples' nodes and the sums at the level after it."""
    from oracle import X_M, X_C
    rng = np.random.default_rng(N + d)
    X = (rng.random((N, d)) < 0.45).astype(np.uint64)
    y = rng.integers(0, K, N)
    Y = np.zeros((N, K), dtype=np.uint64); Y[np.arange(N), y] = 1
    o, g = pair(mods, seed, tau=4, K=K)
    o.train_create(o.share(X.reshape(-1)), o.share(Y.reshape(-1)), N, d, H)
    g.train_create(g.share_a(X.reshape(-1)), g.share_a(Y.reshape(-1)), N, d, H)
    for h in range(2):
        o.train_level(h); g.train_level(h)
        for what in (X_M, X_C):
            same(g.train_export(what), o.train_export(what), "level %d, export %d" % (h, what))
        if h == 0:
            C = g.rec(g.train_export(X_C)).astype(np.int64)
            assert np.array_equal(C[:d * K].reshape(d, K), X.T.astype(np.int64) @ Y.astype(np.int64))
    same_stats(o, g)
    g.close()


# (test_shapes.py checks which kernel they take)
EQUALITY_PAIRS = [40959, 40960, 40961, 40979, 40981, 40999, 65536 * 40 + 3]


@pytest.mark.parametrize("n", EQUALITY_PAIRS)
def test_equality_two_elements_per_lane(mods, seed, n):
    """Tiles of 40 elements, two per lane, from 40 x 1,024 on: below, full, one element in the last tile, its lanes' second elements missing, one of
    them, one short; more tiles than workgroups."""
    o, g = pair(mods, seed)
    rng = np.random.default_rng(n)
    x = rng.integers(0, 1 << 39, size=n).astype(np.uint64)
    y = np.where(rng.random(n) < 0.4, x, rng.integers(0, 1 << 39, size=n).astype(np.uint64))
    xo, xg = o.share(x), g.share_a(x)
    z = g.eq_a(xg, y)
    same(z, o.eq_a(xo, y), "eq")
    assert np.array_equal(g.rec(z), (x == y).astype(np.uint64))
    same_stats(o, g)

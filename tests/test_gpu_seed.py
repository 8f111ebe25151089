"""GPU parity of the K-means++ seeding (D^2 sampling in feature space) with the oracle.

Floating point decides integers here (which index a uniform draws), and the
engine forms the distances in fp32 from its own kernel entries while the
oracle forms them in fp64 from the definitions, so the draws are compared
conditionally: for each center t the oracle recomputes D from the engine's
centers 0..t-1 and checks that the engine's pick i holds the target u_t * S
inside its prefix interval [P(i-1), P(i)] up to a band of BAND * S, with
D(i) > 0 (equal picks are the common case and are counted).  The initial
ids must be a nearest center of the oracle's distances up to the near-tie
band of the step tests.  Repeated calls and the three K storage modes must
agree bitwise (the seeding reads the staged points, not K).
"""
import numpy as np
import pytest

from gpu_helpers import TIE, Engine
from paper_2601_17136_amd import datagen

pytestmark = pytest.mark.gpu

BAND = 1e-5
MODES = ["resident", "packed", "onthefly"]


def _uniforms(seed, k):
    return np.random.default_rng(20_000 + seed).random(k)


def validate_seed(oracle, kern, X, k, u, centers, V):
    """Checks the engine's centers and ids against the oracle, conditionally on
    the engine's earlier picks; returns how many of the k - 1 draws picked the
    oracle's own index."""
    X = np.ascontiguousarray(X, dtype=np.float32)
    n = X.shape[0]
    centers = np.asarray(centers, dtype=np.int64)
    assert centers.shape == (k,) and np.all((centers >= 0) & (centers < n)), centers
    assert centers[0] == min(int(np.floor(u[0] * n)), n - 1)
    diagK = kern.diag(X)
    dist = [oracle.feature_sq_dist(kern, X, int(centers[0]), diagK)]
    D = dist[0].copy()
    same = 0
    for t in range(1, k):
        g = int(centers[t])
        ref = oracle.draw_index(D, u[t], centers[:t])
        if g == ref:
            same += 1
        else:
            P = np.cumsum(D)
            S = P[-1]
            assert S > 0, f"t={t}: S=0 draws the lowest unused index {ref}, engine drew {g}"
            target = u[t] * S
            lo = P[g - 1] if g > 0 else 0.0
            assert lo <= target + BAND * S and P[g] >= target - BAND * S and D[g] > BAND * S / n, \
                (t, g, ref, lo / S, P[g] / S, u[t])
        dist.append(oracle.feature_sq_dist(kern, X, g, diagK))
        D = np.minimum(D, dist[-1])
    Dall = np.stack(dist, axis=1)
    V = np.asarray(V)
    assert np.all((V >= 0) & (V < k))
    best = Dall.min(axis=1)
    scale = np.maximum(np.abs(Dall).max(axis=1), 1e-30)
    bad = Dall[np.arange(n), V] - best > TIE * scale
    assert not bad.any(), f"{bad.sum()} ids are not a nearest center: {np.nonzero(bad)[0][:5]}"
    return same


CASES = [  # (name, n, d, kind, gamma, coef0, degree, k)
    ("linear-300", 300, 5, "linear", 1.0, 0.0, 1, 7),
    ("poly-1000", 1000, 16, "poly", 0.1, 1.0, 2, 12),
    ("gauss-2049", 2049, 24, "gauss", 0.05, 0.0, 1, 20),
    ("gauss-k33", 777, 8, "gauss", 0.2, 0.0, 1, 33),
    ("poly3-513", 513, 3, "poly", 0.5, 1.0, 3, 9),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_seed_parity(oracle, case):
    name, n, d, kind, gamma, coef0, degree, k = case
    X = np.random.default_rng(n + d).normal(size=(n, d)).astype(np.float32)
    kern = oracle.Kernel(kind, gamma, coef0, degree)
    print(f"[gpu] seed parity {name}", flush=True)
    results = []
    for s in range(3):
        u = _uniforms(s, k)
        with Engine(X, kind, gamma, coef0, degree, mode="resident") as eng:
            centers, V = eng.seed(k, u)
            again = eng.seed(k, u)
        np.testing.assert_array_equal(again[0], centers)
        np.testing.assert_array_equal(again[1], V)
        results.append(validate_seed(oracle, kern, X, k, u, centers, V))
    print(f"[gpu] {name}: picks equal to the oracle's {results} of {k - 1} draws x3", flush=True)


@pytest.mark.parametrize("kind,gamma,coef0,degree", [("gauss", 0.1, 0.0, 1), ("poly", 0.2, 1.0, 2)])
def test_seed_modes_agree(kind, gamma, coef0, degree):
    X = np.random.default_rng(7).normal(size=(1500, 10)).astype(np.float32)
    u = _uniforms(9, 16)
    got = []
    for mode in MODES:
        with Engine(X, kind, gamma, coef0, degree, mode=mode) as eng:
            got.append(eng.seed(16, u))
    for c, V in got[1:]:
        np.testing.assert_array_equal(c, got[0][0])
        np.testing.assert_array_equal(V, got[0][1])


def test_seed_single_center():
    X = np.random.default_rng(1).normal(size=(100, 4)).astype(np.float32)
    with Engine(X, "gauss", 0.5) as eng:
        centers, V = eng.seed(1, [0.999999])
    assert list(centers) == [99] and np.all(V == 0)


def test_seed_every_point_a_center(oracle):
    X = np.random.default_rng(2).normal(size=(9, 3)).astype(np.float32)
    u = _uniforms(3, 9)
    with Engine(X, "poly", 1.0, 1.0, 2) as eng:
        centers, V = eng.seed(9, u)
    assert sorted(centers) == list(range(9))
    np.testing.assert_array_equal(centers[V], np.arange(9))
    validate_seed(oracle, oracle.Kernel("poly", 1.0, 1.0, 2), X, 9, u, centers, V)


def test_seed_identical_points():
    """Every distance is exactly 0 after the first center: lowest unused indices."""
    X = np.full((10, 3), 0.25, dtype=np.float32)
    for kind in ("linear", "poly", "gauss"):
        with Engine(X, kind, 0.5, 1.0, 2) as eng:
            centers, V = eng.seed(3, [0.5, 0.2, 0.9])
        assert list(centers) == [5, 0, 1], (kind, centers)
        assert np.all(V == 0)


def test_seed_never_repeats_a_point(oracle):
    """Duplicated points have distance exactly 0 to a center that equals them,
    so while other points remain no center is a copy of an earlier one."""
    rng = np.random.default_rng(4)
    base = rng.normal(size=(40, 6)).astype(np.float32)
    X = np.concatenate([base, base[:25], base[:10]])[rng.permutation(75)]
    for kind, g in (("linear", 1.0), ("gauss", 0.1)):
        u = _uniforms(5, 40)
        with Engine(X, kind, g, 1.0, 2) as eng:
            centers, V = eng.seed(40, u)
        pts = {tuple(X[c]) for c in centers}
        assert len(pts) == 40, kind
        validate_seed(oracle, oracle.Kernel(kind, g, 1.0, 2), X, 40, u, centers, V)


def test_seed_extreme_uniforms(oracle):
    X = np.random.default_rng(6).normal(size=(600, 5)).astype(np.float32)
    kern = oracle.Kernel("gauss", 0.3)
    for u in ([0.0] * 8, [0.999999] * 8, [0.5, 0.0, 0.999999, 0.0, 0.999999, 0.25, 0.75, 0.0]):
        with Engine(X, "gauss", 0.3) as eng:
            centers, V = eng.seed(8, u)
        validate_seed(oracle, kern, X, 8, np.array(u), centers, V)


def test_seed_argument_errors():
    from paper_2601_17136_amd import kkm
    X = np.random.default_rng(8).normal(size=(50, 4)).astype(np.float32)
    with Engine(X, "linear") as eng:
        for k, u in ((0, []), (51, [0.1] * 51), (3, [0.1, 1.0, 0.2]), (3, [0.1, -0.1, 0.2]),
                     (2, [0.1, float("nan")])):
            with pytest.raises(kkm.KKMError) as e:
                eng.seed(k, u)
            assert e.value.code == kkm.KKM_ERR_ARG, (k, u)
    import torch
    ctx = kkm.kkm_create(kkm.current_stream_handle())
    try:
        with pytest.raises(kkm.KKMError) as e:
            kkm.kkm_init_kmeanspp(ctx, 2, [0.1, 0.2], torch.zeros(50, dtype=torch.int32, device="cuda"))
        assert e.value.code == kkm.KKM_ERR_STATE
    finally:
        kkm.kkm_destroy(ctx)


@pytest.mark.parametrize("cfg", [2, 5])
def test_seed_full_size(oracle, cfg):
    w, X, _ = datagen.workload(cfg)
    kern = oracle.Kernel(w.kind, w.gamma, w.coef0, w.degree)
    u = _uniforms(100 + cfg, w.k)
    print(f"[gpu] full-size seeding: {w.describe()}", flush=True)
    with Engine(X, w.kind, w.gamma, w.coef0, w.degree, mode="packed") as eng:
        centers, V = eng.seed(w.k, u)
        cl, it, hist = eng.iterate(V, w.k, 3)
    same = validate_seed(oracle, kern, X, w.k, u, centers, V)
    assert it == 3 and np.all(np.diff(hist) <= 1e-5 * np.abs(hist[:-1]))
    print(f"[gpu] cfg {cfg}: centers {list(centers)} ({same} of {w.k - 1} draws equal), J {hist}", flush=True)


@pytest.mark.parametrize("n", [102400, 102401, 150000])
def test_draws_where_the_draw_gets_its_own_launch(n):
    """Points of small integers: every distance and sum is exact, so the drawn
    indices are those of the rule, on both sides of 1600 blocks of 64 points."""
    k, d = 9, 4
    rng = np.random.default_rng(n)
    X = rng.integers(0, 6, (n, d)).astype(np.float32)
    u = rng.random(k)
    with Engine(X, "linear", mode="onthefly") as eng:
        centers, V = eng.seed(k, u)
    Z = X.astype(np.float64)
    want, D = [int(u[0] * n)], None
    ids = np.zeros(n, np.int32)
    for t in range(k):
        if t:
            P = np.cumsum(D)
            want.append(int(np.searchsorted(P, u[t] * P[-1], side="right")))
        d2 = ((Z - Z[want[-1]]) ** 2).sum(1)
        if t:
            ids[d2 < D] = t
        D = d2 if D is None else np.minimum(D, d2)
    np.testing.assert_array_equal(centers, want)
    np.testing.assert_array_equal(V, ids)


@pytest.mark.parametrize("n,k", [(1500, 1000), (257, 257), (120000, 40)])
def test_points_all_alike_take_the_lowest_indices(n, k):
    """No distance is left after the first center: the lowest index not yet taken follows, k times."""
    X = np.ones((n, 8), np.float32)
    u = np.full(k, 0.01)
    with Engine(X, "poly", 1.0, 1.0, 2, mode="onthefly") as eng:
        centers, V = eng.seed(k, u)
    first = int(0.01 * n)
    rest = [i for i in range(k) if i != first][: k - 1]
    np.testing.assert_array_equal(centers, [first] + rest)
    assert not V.any()

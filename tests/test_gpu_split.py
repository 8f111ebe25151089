"""The K build on the binary16 matrix cores (each coordinate as two binary16 values).

Sizes sit at the edges of its tiles: ragged last rows and columns, coordinate
counts below, at and above its chunks of 16 (from 25 coordinates up, where
split_wanted's size rule takes it), and one row tile more or less than the bands of eight its tiles are dealt in.
"""
import numpy as np
import pytest

from gpu_helpers import TOL, Engine, assignment_mismatches, rel_err, rowscaled_err

pytestmark = pytest.mark.gpu


def _torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _points(n, d, seed, spread=True):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d)).astype(np.float32)
    if spread:  # row scales over 8 binary orders, a zero row, coordinates over 8 more within a row
        # (much wider ranges keep the fp32 products: the tests of wide rows below)
        X *= np.exp2(rng.integers(-4, 5, size=(n, 1))).astype(np.float32)
        X *= np.exp2(rng.integers(-8, 1, size=(n, d))).astype(np.float32)
        X[n // 2] = 0.0
    return X


def _bound(X, d):
    """|K - x.y| for the linear kernel: a coordinate is held to 2^-24 of itself
    or 2^-39 of its row's largest, lo lo (2^-22 of a product) is left out, and
    the fp32 sum is rounded three times per 16 coordinates and once when the
    scales come off; all relative to |x_i||x_j| (Cauchy-Schwarz)."""
    nrm = np.sqrt((X.astype(np.float64) ** 2).sum(1))
    return (2.0 ** -22 + 2.0 ** -23 + (3 * (d // 16 + 1) + 1) * 2.0 ** -24) * np.outer(nrm, nrm)


CASES = [(1, 145), (127, 136), (128, 144), (129, 152), (2177, 32), (257, 164), (2100, 25), (385, 129), (1024, 161),
         (2049, 49), (1025, 137), (2305, 33), (2051, 100)]


@pytest.mark.parametrize("mode", ["packed", "resident"])
@pytest.mark.parametrize("n,d", CASES)
def test_linear_within_the_split_bound(n, d, mode):
    _torch_cuda()
    X = _points(n, d, 100 + n)
    with Engine(X, "linear", mode=mode) as eng:
        K, diag = eng.K_rows(), eng.diag()
    ref = X.astype(np.float64) @ X.astype(np.float64).T
    assert np.all(np.abs(K - ref) <= _bound(X, d)), float(np.max(np.abs(K - ref) / np.maximum(_bound(X, d), 1e-300)))
    assert np.array_equal(K, K.T) and np.array_equal(diag, np.diag(K))


@pytest.mark.parametrize("mode,storage,n", [("packed", "f32", 8200), ("resident", "f32", 8200), ("packed", "f32", 8193),
                                            ("packed", "f16", 8321), ("resident", "f16", 8321)])
def test_many_tiles_match_fp64(mode, storage, n):
    torch = _torch_cuda()
    d, g = 67, 0.01
    X = _points(n, d, 7, spread=False)
    with Engine(X, "gauss", g, mode=mode, storage=storage) as eng:
        out = torch.empty((n, n), device="cuda")
        eng.kkm.kkm_copy_kernel_rows(eng.ctx, 0, n, out)
        X64 = eng.X.double()
        sq = (X64 * X64).sum(1)
        ref = torch.exp(-g * (sq[:, None] + sq[None, :] - 2.0 * (X64 @ X64.T)).clamp(min=0.0))
        err = (out.double() - ref).abs()
        # entries are at most 1: the exponent's error is 2 gamma times the
        # product's plus a few roundings of its terms (below 16 here), and
        # exp2 is good to a few units in the last place
        nrm = float(sq.max())
        tol = 2 * g * (2.0 ** -22 + 2.0 ** -23 + 19 * 2.0 ** -24) * nrm + 64 * 2.0 ** -24
        tol += 2.0 ** -12 if storage == "f16" else 0.0
        assert float(err.max()) <= tol, (float(err.max()), tol)
        assert torch.equal(out, out.T)


@pytest.mark.parametrize("kind", ["linear", "gauss"])
@pytest.mark.parametrize("value", [np.inf, 3e19])
def test_a_norm_past_fp32_takes_the_fp32_build(kind, value):
    """One point with an infinite coordinate, or a finite one whose square is
    past fp32's range: the entries among the other points are as without it,
    and those with it are what fp32 products give."""
    _torch_cuda()
    X = np.abs(_points(200, 270, 3, spread=False)) + np.float32(0.5)
    Y = X.copy()
    Y[17, 4] = value
    with Engine(Y, kind, 0.01, mode="packed") as eng:
        K = eng.K_rows()
    keep = np.arange(200) != 17
    K64 = X.astype(np.float64) @ X.astype(np.float64).T
    if kind == "gauss":
        sq = np.diag(K64)
        K64 = np.exp(-0.01 * (sq[:, None] + sq[None, :] - 2 * K64))
    np.testing.assert_allclose(K[np.ix_(keep, keep)], K64[np.ix_(keep, keep)], rtol=2e-5)
    if kind == "linear":
        row = Y[17].astype(np.float64) @ Y[keep].astype(np.float64).T
        np.testing.assert_allclose(K[17, keep], row, rtol=1e-5)
        assert np.isinf(K[17, 17])


@pytest.mark.parametrize("mode", ["packed", "resident"])
def test_without_room_for_the_split_points(mode):
    """A budget of exactly what kkm_plan asks for has no room for the split
    points: the build runs on the fp32 matrix cores, and iterating works."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    X = _points(700, 150, 5)
    _, need = kkm.kkm_plan(700, 150, 9, kkm.KKM_LINEAR, 1 << 40, kkm.MODES[mode])
    ref = X.astype(np.float64) @ X.astype(np.float64).T
    nrm = np.sqrt(np.diag(ref))
    with Engine(X, "linear", mode=mode, mem_budget=need + 4096, k_hint=9) as eng:
        K = eng.K_rows()
        _, it, _ = eng.iterate(np.arange(700, dtype=np.int32) % 9, 9, 3)
        assert eng.info()["bytes_total"] <= need + 4096 and it == 3
    assert np.all(np.abs(K - ref) <= 150 * 2.0 ** -24 * np.outer(nrm, nrm))


def test_the_split_points_give_way_to_scratch():
    """The split points fit beside the build but not beside the scratch of a
    larger k: the scratch takes their room, and a rebuild gives the same K."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    n, d = 1500, 784
    X = _points(n, d, 6, spread=False)
    _, need1 = kkm.kkm_plan(n, d, 1, kkm.KKM_LINEAR, 1 << 40, kkm.KKM_MODE_PACKED)
    _, need = kkm.kkm_plan(n, d, 60, kkm.KKM_LINEAR, 1 << 40, kkm.KKM_MODE_PACKED)
    split = (n + 36) * (d * 4 + 4)  # n = 1536 padded, d = 784
    budget = max(need, need1 + split) + (1 << 16)
    assert budget < need + split
    with Engine(X, "linear", mode="packed", mem_budget=budget) as eng:
        K = eng.K_rows()
        cl = (np.arange(n) % 60).astype(np.int32)
        held = eng.info()["bytes_total"]
        _, it, _ = eng.iterate(cl, 60, 2)
        assert it == 2 and eng.info()["bytes_total"] <= budget and held <= budget
        P = kkm.make_params(mode=kkm.KKM_MODE_PACKED)
        kkm.kkm_build_kernel(eng.ctx, eng.X, n, d, kkm.KKM_LINEAR, P)
        np.testing.assert_allclose(eng.K_rows(), K, rtol=0, atol=float(_bound(X, d).max()) * 2)


def _check_step(X, kind, g, c, p, cl, k, eng, oracle):
    ref = oracle.step_full(oracle.Kernel(kind, g, c, p).matrix(X), cl, k)
    out = eng.step(cl, k)
    np.testing.assert_array_equal(out["counts"], ref["counts"])
    assert rowscaled_err(out["E"], ref["E"]) <= 1e-5 and rowscaled_err(out["D"], ref["D"]) <= TOL
    assert rel_err(out["z"], ref["z"]) <= 1e-5
    assignment_mismatches(out["cl"], ref["cl"], ref["D"])
    return out


@pytest.mark.parametrize("kind", ["gauss", "poly", "linear"])
@pytest.mark.parametrize("n,d,k", [(1, 32, 1), (1, 70, 1), (1025, 25, 3), (1152, 33, 2), (1153, 48, 9), (1300, 56, 40),
                                   (1664, 64, 5), (127, 66, 3), (257, 65, 3), (700, 100, 30), (385, 130, 7)])
def test_on_the_fly_step(oracle, n, d, k, kind):
    """Sweeps of two to four chunks held in LDS and of chunks staged per tile;
    blocks of one cluster and of several, ragged last tiles."""
    _torch_cuda()
    X = _points(n, d, 40 + n, spread=False) + np.float32(0.25)
    cl = np.random.default_rng(n).integers(0, k, n).astype(np.int32)
    g, c, p = {"gauss": (1.0 / d, 0.0, 1), "poly": (1.0 / d, 1.0, 2 if d % 2 else 3), "linear": (1.0, 0.0, 1)}[kind]
    with Engine(X, kind, g, c, p, mode="onthefly") as eng:
        out = _check_step(X, kind, g, c, p, cl, k, eng, oracle)
        again = eng.step(cl, k)
        assert np.array_equal(out["E"], again["E"]) and out["J"] == again["J"]


@pytest.mark.parametrize("d", [40, 90])
def test_on_the_fly_fixups_and_small_budgets(oracle, d):
    """Points far from the origin, so that Gaussian entries are recomputed from
    the differences inside the sweep; once with the split points and once in
    exactly the budget kkm_plan asks for, which has no room for them."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    n, k = (1100 if d == 40 else 500), 6
    X = 0.3 * _points(n, d, 9, spread=False) + np.float32(20.0)
    cl = np.random.default_rng(1).integers(0, k, n).astype(np.int32)
    with Engine(X, "gauss", 0.05, mode="onthefly") as eng:
        _check_step(X, "gauss", 0.05, 0.0, 1, cl, k, eng, oracle)
    _, need = kkm.kkm_plan(n, d, k, kkm.KKM_GAUSS, 1 << 40, kkm.KKM_MODE_ONTHEFLY)
    with Engine(X, "gauss", 0.05, mode="onthefly", mem_budget=need + 4096, k_hint=k) as eng:
        _check_step(X, "gauss", 0.05, 0.0, 1, cl, k, eng, oracle)
        assert eng.info()["bytes_total"] <= need + 4096


@pytest.mark.parametrize("d", [40, 90])
def test_on_the_fly_past_fp32_norms(d):
    """A point whose squared norm is past fp32's range: the other clusters'
    sums over the other points are finite and as without it."""
    _torch_cuda()
    n = 1100 if d == 40 else 300
    X = np.abs(_points(n, d, 3, spread=False)) + np.float32(0.5)
    X[17, 4] = 3e19
    cl = (np.arange(n) % 3).astype(np.int32)
    cl[17] = 2
    with Engine(X, "linear", mode="onthefly") as eng:
        E = eng.step(cl, 3)["E"]
    X64 = X.astype(np.float64)
    keep = np.arange(n) != 17
    for j in (0, 1):
        ref = X64[keep] @ X64[cl == j].sum(0)
        np.testing.assert_allclose(E[keep, j], ref, rtol=1e-5)
    assert np.isinf(E[17, 2])


@pytest.mark.parametrize("mode,d", [("packed", 25), ("packed", 54), ("packed", 301), ("resident", 784)])
def test_diagonal_has_no_bias(mode, d):
    """tr K, and with it the objective, sees the mean error of the diagonal.  Rounded norms of random sign leave
    2^-25 / sqrt(n) = 2^-30.5 of it at n = 2100; the bound is 2^-28 (a square without its lo lo is low by about 2^-25)."""
    _torch_cuda()
    X = np.random.default_rng(d).random((2100, d), dtype=np.float32)
    with Engine(X, "linear", mode=mode) as eng:
        K, diag = eng.K_rows(), eng.diag().astype(np.float64)
    ref = (X.astype(np.float64) ** 2).sum(1)
    assert np.array_equal(np.diag(K), diag)
    assert abs(np.mean((diag - ref) / ref)) <= 2.0 ** -28


def _wide(case, n, d, size, seed):
    """Points whose rows hold coordinates of very different size, such that
    some pairs of points share only small ones."""
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d)).astype(np.float32)
    big = np.arange(n) < n // 10
    X[:, :2] = 0.0
    if case == "one column":  # a tenth of the points have a large coordinate the others lack
        X[big, 0] = size * (1 + rng.random(big.sum()))
    elif case == "two columns":  # every point has a large one, in one column or the other
        X[big, 0] = size * (1 + rng.random(big.sum()))
        X[~big, 1] = size * (1 + rng.random((~big).sum()))
    elif case == "sparse":  # two nonzero coordinates, or the small one of them alone
        X[:] = 0.0
        X[:, 3] = 1 + rng.random(n)
        X[big, 0] = size * (1 + rng.random(big.sum()))
    else:  # "few": one small coordinate in ordinary rows, large points in that column alone
        X[:, 3] = (1 + rng.random(n)) * (100.0 / size)
        X[big] = 0.0
        X[big, 3] = size * (1 + rng.random(big.sum()))
    return X, big


WIDE = [("one column", 1e6), ("one column", 1e8), ("one column", 1e12), ("two columns", 1e9), ("sparse", 1e10), ("few", 1e10)]


@pytest.mark.parametrize("case,size", WIDE)
@pytest.mark.parametrize("n,d", [(2100, 32), (300, 130)])
def test_rows_of_wide_range_keep_fp32_products(n, d, case, size):
    """Every entry within what fp32 products give, relative to the sum of its
    own terms' sizes (and not to the points' norms); K is the one that a budget
    without room for the split points builds."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    X, big = _wide(case, n, d, size, n + d)
    X64 = X.astype(np.float64)
    B, S = X64 @ X64.T, np.abs(X64) @ np.abs(X64).T
    off = ~np.eye(n, dtype=bool)
    for kind, mode in [("linear", "packed"), ("linear", "resident"), ("poly", "packed")]:
        args = (kind, 1.0, 1.0, 2) if kind == "poly" else (kind,)
        with Engine(X, *args, mode=mode) as eng:
            K = eng.K_rows()
        if kind == "linear":
            assert np.all((np.abs(K - B) <= (d + 2) * 2.0 ** -24 * S)[off])
        else:
            ref = (B + 1) ** 2
            ok = (np.abs(K - ref) <= 2 * (np.abs(B) + 1) * (d + 4) * 2.0 ** -24 * (S + 1)) | (ref > 1e38)
            assert np.all(ok[off])
        _, need = kkm.kkm_plan(n, d, 1, kkm.KINDS[kind], 1 << 40, kkm.MODES[mode])
        with Engine(X, *args, mode=mode, mem_budget=need + 4096, k_hint=1) as eng:
            assert np.array_equal(eng.K_rows(), K)


@pytest.mark.parametrize("case,size", WIDE)
@pytest.mark.parametrize("d", [32, 130])
def test_rows_of_wide_range_on_the_fly(d, case, size):
    """The sweep and a block of one GPU's share on the same points: sums of the
    large points' entries over the small points' cluster."""
    torch = _torch_cuda()
    from paper_2601_17136_amd import kkm
    n = 1100 if d == 32 else 256
    X, big = _wide(case, n, d, size, d)
    cl = np.where(big, 0, 1).astype(np.int32)
    X64 = X.astype(np.float64)
    V = np.eye(2)[cl]
    ref, S = X64 @ (X64.T @ V), np.abs(X64) @ (np.abs(X64).T @ V)
    bound = (d + 2 + n) * 2.0 ** -24 * S
    other = V == 0  # the entries between the groups
    with Engine(X, "linear", mode="onthefly") as eng:
        E = eng.step(cl, 2)["E"]
    assert np.all((np.abs(E - ref) <= bound)[other])
    ctx = kkm.kkm_create(kkm.current_stream_handle())
    try:
        kkm.kkm_build_block(ctx, torch.from_numpy(X).cuda(), n, d, kkm.KKM_LINEAR, kkm.make_params(), 0, n, 0, n)
        E = torch.empty((n, 2), device="cuda")
        kkm.kkm_block_spmm(ctx, torch.from_numpy(cl).cuda(), 2, E)
        assert np.all((np.abs(E.cpu().numpy() - ref) <= bound)[other])
    finally:
        kkm.kkm_destroy(ctx)


@pytest.mark.parametrize("kind,gamma,scale", [("gauss", 1e31, 1e12), ("gauss", 1e-36, 1e8), ("poly", 1e30, 1e15),
                                              ("poly", 1e-36, 1e-3), ("linear", 1.0, 1e-30)])
def test_factors_at_the_ends_of_fp32(kind, gamma, scale):
    """Scales and kernel widths whose product with a row's factor leaves fp32's
    range: K is the one that fp32 products give.  Half of the points share no
    coordinate with the other half."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    n, d = 200, 280
    X = np.random.default_rng(8).random((n, d)).astype(np.float32) + np.float32(0.5)
    X[: n // 2, 140:] = 0.0
    X[n // 2:, :140] = 0.0
    X *= np.float32(scale)
    args = (kind, gamma, 0.5, 1)
    with Engine(X, *args, mode="packed") as eng:
        K = eng.K_rows()
    _, need = kkm.kkm_plan(n, d, 1, kkm.KINDS[kind], 1 << 40, kkm.KKM_MODE_PACKED)
    with Engine(X, *args, mode="packed", mem_budget=need + 4096, k_hint=1) as eng:
        assert np.array_equal(eng.K_rows(), K, equal_nan=True)
    X64 = X.astype(np.float64)
    off = ~np.eye(n, dtype=bool)
    if kind == "gauss":
        sq = (X64 * X64).sum(1)
        ref = np.exp(-gamma * np.maximum(sq[:, None] + sq[None] - 2 * X64 @ X64.T, 0.0))
        assert np.all(np.abs(K - ref)[off] <= 1e-4)
    else:
        apart = np.zeros((n, n), bool)
        apart[: n // 2, n // 2:] = apart[n // 2:, : n // 2] = True
        assert np.all(K[apart] == (0.5 if kind == "poly" else 0.0))


def test_a_rebuild_is_not_charged_for_what_it_can_free():
    """The split points and the seeding scratch of one build make way for the
    next on the same context, as on a new one: more points in an explicit mode,
    more clusters announced under AUTO, the same build after seeding, and an
    update after seeding, in budgets that hold just what kkm_plan asks for."""
    torch = _torch_cuda()
    from paper_2601_17136_amd import kkm
    d, L = 400, kkm.KKM_LINEAR
    X = _points(1500, d, 6, spread=False)
    Xd = torch.from_numpy(X).cuda()
    plan = lambda n, k, mode: kkm.kkm_plan(n, d, k, L, 1 << 40, mode)[1]

    need = plan(1500, 1, kkm.KKM_MODE_PACKED) + 4096
    assert plan(600, 1, kkm.KKM_MODE_PACKED) + 640 * (d * 4 + 4) + 8192 < need
    with Engine(X[:600], "linear", mode="packed", mem_budget=need) as eng:
        held = eng.info()["bytes_total"]
        assert held > 640 * (d * 4 + 4) * 2  # the split points are held
        kkm.kkm_build_kernel(eng.ctx, Xd, 1500, d, L, kkm.make_params(mode=kkm.KKM_MODE_PACKED))
        assert eng.info()["n"] == 1500 and eng.info()["bytes_total"] <= need

    need = plan(1500, 60, kkm.KKM_MODE_PACKED) + 4096
    assert plan(1500, 1, kkm.KKM_MODE_PACKED) + 1536 * (d * 4 + 4) + 8192 < need
    with Engine(X, "linear", mode="auto", mem_budget=need, k_hint=1) as eng:
        assert eng.info()["mode"] == kkm.KKM_MODE_PACKED
        kkm.kkm_build_kernel(eng.ctx, eng.X, 1500, d, L, kkm.make_params(k_hint=60))
        assert eng.info()["mode"] == kkm.KKM_MODE_PACKED
        _, it, _ = eng.iterate((np.arange(1500) % 60).astype(np.int32), 60, 2)
        assert it == 2 and eng.info()["bytes_total"] <= need

    need = plan(1500, 9, kkm.KKM_MODE_PACKED) + 4096
    with Engine(X, "linear", mode="packed", mem_budget=need, k_hint=9) as eng:
        _, V = eng.seed(9, np.random.default_rng(0).random(9))
        kkm.kkm_build_kernel(eng.ctx, eng.X, 1500, d, L, kkm.make_params(mode=kkm.KKM_MODE_PACKED, k_hint=9))
        _, it, _ = eng.iterate(V, 9, 2)
        assert it == 2 and eng.info()["bytes_total"] <= need


@pytest.mark.parametrize("spare", [0, 4096, 20000, 60000, 400000])
def test_on_the_fly_bits_do_not_depend_on_seeding(spare):
    """With little or no room beside the split points, the same update gives the
    same bits before and after seeding; a request that fails takes nothing away."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    n, d, k = 2000, 90, 7
    X = _points(n, d, 5, spread=False)
    cl = (np.arange(n) % k).astype(np.int32)
    _, need = kkm.kkm_plan(n, d, k, kkm.KKM_LINEAR, 1 << 40, kkm.KKM_MODE_ONTHEFLY)
    split = 2048 * (6 * 64 + 8)
    with Engine(X, "linear", mode="onthefly", mem_budget=need + split + spare, k_hint=k) as eng:
        first = eng.step(cl, k)
        with pytest.raises(kkm.KKMError) as e:
            eng.step((np.arange(n) % 1000).astype(np.int32), 1000, want_E=False, want_D=False)
        assert e.value.code == kkm.KKM_ERR_OOM
        again = eng.step(cl, k)
        eng.seed(k, np.random.default_rng(1).random(k))
        after = eng.step(cl, k)
    for key in ("E", "D", "z", "cl"):
        assert np.array_equal(first[key], again[key]) and np.array_equal(first[key], after[key]), key


@pytest.mark.parametrize("d", [33, 54, 100, 128, 301])
def test_entries_have_no_bias(d):
    """Sums of K over a cluster, and the objective, see the mean error of its
    entries.  Roundings of random sign leave next to nothing of it over 4
    million entries (the rows' own, 2^-25 over sqrt(d) and over sqrt(2100) rows,
    2^-33 at most); a turn of the sum's sign at the wrong chunk leaves 2e-9."""
    _torch_cuda()
    X = np.random.default_rng(d).random((2100, d), dtype=np.float32)
    with Engine(X, "linear", mode="packed") as eng:
        K = eng.K_rows().astype(np.float64)
    ref = X.astype(np.float64) @ X.astype(np.float64).T
    off = ~np.eye(len(X), dtype=bool)
    assert abs((K - ref)[off].sum() / ref[off].sum()) <= 2.0 ** -30


@pytest.mark.parametrize("kind", ["linear", "poly", "gauss"])
@pytest.mark.parametrize("n,d", [(1000, 270), (4225, 33), (1000, 70), (897, 33), (2050, 40)])
def test_blocks_hold_the_bits_of_the_full_k(n, d, kind):
    """Entry (i, j) of any block is entry (i, j) of the full K, bit for bit, above,
    on and below the diagonal, ragged ends of rows and columns included; the
    Gaussian with many entries recomputed.  (Blocks of few narrow points, whose
    full K takes another kernel: of one block that holds everything.)"""
    torch = _torch_cuda()
    from paper_2601_17136_amd import kkm
    rng = np.random.default_rng(n)
    X = (rng.standard_normal((9, d))[rng.integers(0, 9, n)] + 0.05 * rng.standard_normal((n, d))).astype(np.float32)
    g, c, p = {"linear": (1.0, 0.0, 1), "poly": (0.5, 1.0, 3), "gauss": (20.0 / d, 0.0, 1)}[kind]
    Xd = torch.from_numpy(X).cuda()
    ctx = kkm.kkm_create(kkm.current_stream_handle())
    if d > 256 or n > 4096:
        with Engine(X, kind, g, c, p, mode="resident") as eng:
            K = eng.K_rows()
            assert kind != "gauss" or eng.info()["fixups"] > n
    else:
        kkm.kkm_build_block(ctx, Xd, n, d, kkm.KINDS[kind], kkm.make_params(g, c, p), 0, n, 0, n)
        out = torch.empty((n, n), device="cuda")
        kkm.kkm_copy_kernel_rows(ctx, 0, n, out)
        K = out.cpu().numpy()
    assert np.array_equal(K, K.T)
    try:
        for r0, r1, c0, c1 in [(0, n, 0, n), (n // 256 * 128, n, 0, n // 256 * 128), (128, n, 0, 700),
                               (0, 300, 256, n), (256, 700, 128, 650), (640, n, 640, n),
                               (384, 400, 384, 500), (384, 500, 384, 400), (128, 129, 128, 129)]:
            kkm.kkm_build_block(ctx, Xd, n, d, kkm.KINDS[kind], kkm.make_params(g, c, p), r0, r1, c0, c1)
            out = torch.empty((r1 - r0, c1 - c0), device="cuda")
            kkm.kkm_copy_kernel_rows(ctx, r0, r1, out)
            assert np.array_equal(out.cpu().numpy(), K[r0:r1, c0:c1]), (r0, r1, c0, c1)
            # the columns past the block's end are zero: sums over them too
            E = torch.empty((c1 - c0, 1), device="cuda")
            kkm.kkm_block_spmm(ctx, torch.zeros(r1 - r0, dtype=torch.int32, device="cuda"), 1, E)
            ref = K[r0:r1, c0:c1].astype(np.float64).sum(0)
            scale = np.abs(K[r0:r1, c0:c1]).astype(np.float64).sum(0)
            assert np.all(np.abs(E.cpu().numpy()[:, 0] - ref) <= 2.0 ** -24 * (r1 - r0 + 2) * scale)
    finally:
        kkm.kkm_destroy(ctx)


@pytest.mark.parametrize("kind", ["linear", "poly", "gauss"])
@pytest.mark.parametrize("layout,n,d", [("packed", 2048, 128), ("packed", 2049, 128), ("packed", 2049, 24),
                                        ("packed", 700, 129), ("packed", 4096, 64), ("packed", 4097, 64),
                                        ("packed", 2048, 200), ("packed", 2049, 200), ("packed", 300, 257),
                                        ("resident16", 700, 33), ("resident16", 4097, 33), ("onthefly", 1024, 64),
                                        ("onthefly", 1025, 64), ("block", 4096, 40), ("block", 4097, 40), ("block", 600, 65)])
def test_both_sides_of_the_size_rule(layout, n, d, kind):
    """The sizes at which the products change hands: E of a few clusters against 64 bits on either side."""
    torch = _torch_cuda()
    from paper_2601_17136_amd import kkm
    X = _points(n, d, n + d, spread=False)
    k, g = 5, 1.0 / d
    cl = (np.arange(n) % k).astype(np.int32)
    X64 = torch.from_numpy(X).cuda().double()
    B = X64 @ X64.T
    sq = B.diagonal()
    K = B if kind == "linear" else (g * B + 1) ** 2 if kind == "poly" else torch.exp(-g * (sq[:, None] + sq[None] - 2 * B))
    V = torch.nn.functional.one_hot(torch.from_numpy(cl).cuda().long(), k).double()
    prm = (kind, g, 1.0 if kind == "poly" else 0.0, 2 if kind == "poly" else 1)
    if layout == "block":
        ctx = kkm.kkm_create(kkm.current_stream_handle())
        E = torch.empty((n, k), device="cuda")
        kkm.kkm_build_block(ctx, torch.from_numpy(X).cuda(), n, d, kkm.KINDS[kind], kkm.make_params(*prm[1:]), 0, n, 0, n)
        kkm.kkm_block_spmm(ctx, torch.from_numpy(cl).cuda(), k, E)
        kkm.kkm_destroy(ctx)
        E = E.cpu().numpy()
    else:
        with Engine(X, *prm, mode=layout.replace("16", ""), storage="f16" if "16" in layout else "f32") as eng:
            E = eng.step(cl, k)["E"]
    ref = (K @ V).cpu().numpy()
    scale = (K.abs() @ V).cpu().numpy()
    # fp32 products and sums; binary16 entries carry 2^-11 and the row bound's share
    assert np.all(np.abs(E - ref) <= (2.0 ** -10 if "16" in layout else 4e-6) * scale + (
        2.0 ** -25 * n * np.abs(ref).max() if "16" in layout else 0.0))

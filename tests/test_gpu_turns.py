"""Contexts used in turn, and memory used again: a pass gives the same bits
whatever ran in between, in every layout of K.

Also the blocks whose Gaussian entries are too small to be recomputed and too
ill-conditioned for two products to agree: they keep the fp32 products."""
import numpy as np
import pytest

from gpu_helpers import Engine

pytestmark = pytest.mark.gpu


def _torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _rings(n, d, k, seed):
    rng = np.random.default_rng(seed)
    lab = rng.permutation(n) % k
    theta = rng.random(n) * 2 * np.pi
    X = 0.1 * rng.standard_normal((n, d))
    r = lab + 1 + 0.05 * rng.standard_normal(n)
    X[:, 0], X[:, 1] = r * np.cos(theta), r * np.sin(theta)
    return X.astype(np.float32), lab.astype(np.int32)


def _K64(X, kind, g, rows, cols):
    X = X.astype(np.float64)
    B = X[rows] @ X[cols].T
    if kind == "gauss":
        sq = (X * X).sum(1)
        return np.exp(-g * np.maximum(sq[rows][:, None] + sq[cols][None] - 2 * B, 0))
    return (g * B + 1.0) ** 2 if kind == "poly" else B


class _Share:
    """A block of K on a context of its own."""

    def __init__(self, X, kind, g, rows, cols):
        import torch
        from paper_2601_17136_amd import kkm
        self.kkm, self.torch, self.kind, self.n, self.d = kkm, torch, kind, X.shape[0], X.shape[1]
        self.rows, self.cols, self.X = rows, cols, torch.from_numpy(X).cuda()
        self.prm = kkm.make_params(g, 1.0 if kind == "poly" else 0.0, 2 if kind == "poly" else 1)
        self.ctx = kkm.kkm_create(kkm.current_stream_handle())

    def build(self):
        (r0, r1), (c0, c1) = self.rows, self.cols
        self.kkm.kkm_build_block(self.ctx, self.X, self.n, self.d, self.kkm.KINDS[self.kind], self.prm, r0, r1, c0, c1)

    def K(self):
        out = self.torch.empty((self.rows[1] - self.rows[0], self.cols[1] - self.cols[0]), device="cuda")
        self.kkm.kkm_copy_kernel_rows(self.ctx, self.rows[0], self.rows[1], out)
        return out.cpu().numpy()

    def run(self, cl, k):
        torch, kkm = self.torch, self.kkm
        self.build()
        (r0, r1), (c0, c1) = self.rows, self.cols
        E = torch.empty((c1 - c0, k), device="cuda")
        kkm.kkm_block_spmm(self.ctx, torch.from_numpy(np.ascontiguousarray(cl[r0:r1])).cuda(), k, E)
        ids = torch.from_numpy(np.ascontiguousarray(cl[c0:c1])).cuda()
        zp, cnt = kkm.kkm_block_zpart(self.ctx, E, ids, c0, c1, k)
        new = torch.empty(c1 - c0, dtype=torch.int32, device="cuda")
        kkm.kkm_block_assign(self.ctx, E, c0, c1, k, zp / np.maximum(cnt, 1.0) ** 2, cnt, new)
        return {"E": E.cpu().numpy(), "z": np.array(zp), "cl": new.cpu().numpy()}

    def close(self):
        self.kkm.kkm_destroy(self.ctx)


class _Whole:
    """All of K (packed, resident or on the fly) on a context of its own."""

    def __init__(self, X, kind, g, mode):
        self.mode = mode
        self.args = (kind, g, 1.0 if kind == "poly" else 0.0, 2 if kind == "poly" else 1)
        self.eng = Engine(X, *self.args, mode=mode)

    def run(self, cl, k):
        e = self.eng
        e.kkm.kkm_build_kernel(e.ctx, e.X, e.n, e.d, e.kkm.KINDS[self.args[0]],
                               e.kkm.make_params(*self.args[1:], e.kkm.MODES[self.mode]))
        out = e.step(cl, k)
        return {key: out[key] for key in ("E", "z", "cl")}

    def close(self):
        self.eng.close()


def _of(layout, X, kind, g):
    n = X.shape[0]
    half = n // 256 * 128
    return _Share(X, kind, g, (half, n), (0, half)) if layout == "block" else _Whole(X, kind, g, layout)


@pytest.mark.parametrize("kind,d", [("gauss", 130), ("gauss", 54), ("poly", 100), ("linear", 20)])
@pytest.mark.parametrize("layout", ["block", "packed", "resident", "onthefly"])
def test_a_pass_does_not_depend_on_what_ran_before(layout, kind, d):
    """Own pass, another context's, own pass again: the same bits, those of a
    new context, and what 64 bits give."""
    _torch_cuda()
    n, k, g = 2900, 12, 0.5 if kind == "gauss" else 1.0
    X, cl = _rings(n, d, k, d)
    Y, cl2 = _rings(n, d, k, d + 1)
    a, b = _of(layout, X, kind, g), _of(layout, Y, kind, g)
    first = a.run(cl, k)
    b.run(cl2, k)
    third = a.run(cl, k)
    b.close()
    a.close()
    c = _of(layout, X, kind, g)
    fresh = c.run(cl, k)
    c.close()
    for key in first:
        assert np.array_equal(first[key], third[key]) and np.array_equal(first[key], fresh[key]), key
    half = n // 256 * 128
    rows, cols = (slice(half, n), slice(0, half)) if layout == "block" else (slice(0, n), slice(0, n))
    ref = _K64(X, kind, g, rows, cols).T @ np.eye(k)[cl[rows]]
    # fp32 sums of a cluster's entries; Gaussian entries are let stand 2e-6 off
    bound = 4e-6 * np.abs(ref).max(1, keepdims=True) + (2e-6 * n / k if kind == "gauss" else 0.0)
    assert np.all(np.abs(first["E"] - ref) <= bound)


@pytest.mark.parametrize("layout", ["block", "packed", "onthefly"])
def test_memory_of_a_large_k_is_used_again(layout):
    """A K of 5 GB is built, stepped and freed between two passes of a smaller
    problem whose buffers can then lie where that K was."""
    torch = _torch_cuda()
    X, cl = _rings(6000, 100, 9, 1)
    big, clb = _rings(50000, 16, 9, 2)
    outs = []
    for turn in range(2):
        s = _of(layout, X, "poly", 1.0)
        outs.append(s.run(cl, 9))
        s.close()
        if turn == 0:
            w = _Whole(big, "gauss", 0.5, "packed")
            w.run(clb, 9)
            w.close()
            torch.cuda.synchronize()
    for key in outs[0]:
        assert np.array_equal(outs[0][key], outs[1][key]), key


@pytest.mark.parametrize("d", [70, 392])
def test_far_gaussian_blocks_keep_the_fp32_products(d):
    """Rings of radius up to 61 under a kernel of width 1: an entry's exponent
    is good to 1e-3 only, and entries below that are not recomputed.  The block
    holds what the fp32 products give, bit for bit: the same entries of a full K
    whose budget has no room for the split points."""
    _torch_cuda()
    from paper_2601_17136_amd import kkm
    n, k = 1500, 61
    X, cl = _rings(n, d, k, d)
    _, need = kkm.kkm_plan(n, d, 1, kkm.KKM_GAUSS, 1 << 40, kkm.KKM_MODE_RESIDENT)
    with Engine(X, "gauss", 0.5, mode="resident", mem_budget=need + 4096, k_hint=1) as eng:
        K = eng.K_rows()
    for rows, cols in [((640, n), (0, 700)), ((0, n), (256, 1000)), ((128, 900), (768, n))]:
        s = _Share(X, "gauss", 0.5, rows, cols)
        s.build()
        got = s.K()
        s.close()
        assert np.array_equal(got, K[rows[0]:rows[1], cols[0]:cols[1]]), (rows, cols)

"""The work a user has this engine do, as cases for a timing harness.

A case is one call sequence through the public binding (``kkm``) at one size:

* ``fit``: a whole job, the K build and then the clustering loop;
* ``build``: the K build and one full step (E, z, new ids, sizes, objective);
* ``update``: the clustering loop on a K that is already built;
* ``onthefly``: one full step with K recomputed instead of stored;
* ``share``: one process's block of the 1.5D split, build and one update;
* ``seed``: K-means++ seeding on staged points.

Sizes, kernels and point distributions are those of the repository's
workloads (n = 2000 .. 200000, d = 16 .. 784, k = 7 .. 64) and of its tests
(ragged n, odd d, more than 64 clusters, binary16 K), kept small enough that
three built problems fit one GPU together.  Points are generated on the GPU
from the seed; the ids a clustering starts from are the generating labels with
a share of them redrawn (a warm start), so that a rounding difference does not
send the loop down another trajectory.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_17136_amd import kkm

# Share of the generating labels redrawn at random for the initial ids.
SCRAMBLE = 0.1


def listed():
    return [
        # The smallest job users run (and the first thing they try): launches
        # and synchronisations count, the arithmetic does not.
        _case("fit-small", "fit", "blobs", "poly", n=2000, d=16, k=8, iters=20),
        # An image-like data set of ordinary size, build and loop of like weight.
        _case("fit-medium", "fit", "protos", "gauss", n=20000, d=784, k=10, iters=30),
        # The paper's kernel on wide points: the K build is most of a job.
        _case("build-wide", "build", "protos", "poly", n=60000, d=780, k=10),
        # Low-dimensional tabular data at a large n: K's bytes outweigh its flops.
        _case("build-narrow", "build", "tabular", "gauss", n=120000, d=54, k=7),
        # Concentric rings: large norms next to small distances, so many entries
        # are recomputed from the differences; the most labels packed K takes.
        _case("build-rings", "build", "rings", "gauss", n=50000, d=128, k=64),
        # Binary16 storage at ragged sizes with the linear kernel.
        _case("build-half", "build", "protos", "linear", n=40001, d=301, k=20, storage="f16"),
        # The loop alone until it converges (tol = 0), on a handful of points:
        # a host round trip per update.
        _case("update-tiny", "update", "blobs", "linear", n=999, d=9, k=5, iters=50, tol=0.0),
        # The loop alone on a large packed K with many labels: HBM bound.
        _case("update-packed", "update", "rings", "gauss", n=100000, d=128, k=64, iters=5),
        # More clusters than packed storage takes: the full K is streamed.
        _case("update-full", "update", "blobs", "gauss", n=30000, d=40, k=300, iters=5),
        # K never stored: what runs when K does not fit.
        _case("onthefly-narrow", "onthefly", "tabular", "gauss", n=60000, d=54, k=7),
        # One process of a 2 x 2 grid.
        _case("share-block", "share", "tabular", "gauss", n=50000, d=100, k=16),
        # K-means++ on a large data set with many centers.
        _case("seed-large", "seed", "rings", "gauss", n=100000, d=128, k=64),
    ]


def draw(rng):
    """One more case of the listed ones' ranges; none costs more than the largest of them."""
    family = rng.choice(["fit", "fit", "build", "build", "build", "update", "update", "onthefly", "share", "seed"])
    points = rng.choice(["blobs", "protos", "tabular", "rings"])
    kernel = {"blobs": ["poly", "linear", "gauss"], "protos": ["poly", "gauss", "linear"],
              "tabular": ["gauss", "poly"], "rings": ["gauss"]}[points]
    kernel = rng.choice(kernel)
    top_n = {"fit": 20000, "build": 60000, "update": 60000, "onthefly": 40000, "share": 40000, "seed": 100000}[family]
    low_n = {"share": 3000}.get(family, 900)
    n = _log_between(rng, low_n, top_n)
    d = _log_between(rng, 6, 784)
    k = _log_between(rng, 3, 64)
    iters, tol, storage = 1, -1.0, "f32"
    if family == "fit":
        iters = rng.randint(5, 30)
    elif family == "update":
        iters = rng.randint(2, 10)
        if rng.random() < 0.3:
            k = _log_between(rng, 65, 300)
            n = max(n, 20 * k)
        elif rng.random() < 0.3:
            # far apart, so that the loop stops after a known number of updates
            tol, points, kernel, d, k = 0.0, "blobs", "linear", max(d, 16), min(k, 16)
    if family in ("fit", "build", "update") and rng.random() < 0.25:
        storage = "f16"
    if points == "rings":
        d = max(d, 8)
    return {key: v for key, v in _case("", family, points, kernel, n, d, k, iters, tol, storage).items()
            if key != "name"}


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _case(name, family, points, kernel, n, d, k, iters=1, tol=-1.0, storage="f32"):
    return {"name": name, "family": family, "points": points, "kernel": kernel, "n": n, "d": d, "k": k,
            "iters": iters, "tol": tol, "storage": storage}


# ------------------------------------------------------------------ inputs

def _labels(n, k, unequal, gen):
    """Generating labels in a random order: i mod k, or sizes in proportion to 1 .. k."""
    i = torch.arange(n, device="cuda")
    if unequal:
        edges = torch.cumsum(torch.arange(1, k + 1, device="cuda", dtype=torch.float64), 0)
        lab = torch.searchsorted(edges / edges[-1] * n, i.double() + 0.5)
        lab = lab.clamp_(max=k - 1)
    else:
        lab = i % k
    return lab[torch.randperm(n, device="cuda", generator=gen)]


def _inputs(case, seed):
    """Points (n x d fp32) and initial ids (int32) on the GPU, from the seed alone."""
    n, d, k = case["n"], case["d"], case["k"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)

    def uniform(*shape):
        return torch.rand(*shape, device="cuda", generator=gen)

    def normal(*shape):
        return torch.randn(*shape, device="cuda", generator=gen)

    lab = _labels(n, k, case["points"] == "tabular", gen)
    if case["points"] == "blobs":        # isotropic blobs, centres in [-10, 10]^d
        X = (uniform(k, d) * 20 - 10)[lab] + normal(n, d)
    elif case["points"] == "protos":     # image-like: prototypes in [0, 1]^d plus noise, clipped
        X = (uniform(k, d)[lab] + (uniform(n, d) * 0.6 - 0.3)).clamp_(0.0, 1.0)
    elif case["points"] == "rings":      # dims 0-1 on k rings, the others small
        theta = uniform(n) * (2 * math.pi)
        r = lab + 1 + 0.05 * normal(n)
        X = 0.1 * normal(n, d)
        X[:, 0] = r * torch.cos(theta)
        X[:, 1] = r * torch.sin(theta)
    else:                                # unequal Gaussian clusters, features standardised
        X = normal(k, d)[lab] + normal(n, d)
        X = (X - X.mean(0)) / X.std(0)
    redrawn = uniform(n) < SCRAMBLE
    cl = torch.where(redrawn, torch.randint(0, k, (n,), device="cuda", generator=gen), lab)
    return X.float().contiguous(), cl.to(torch.int32).contiguous()


def _kernel(case):
    """(gamma, coef0, degree): the polynomial is the paper's, the Gaussian's width follows the points."""
    if case["kernel"] == "poly":
        return 1.0, 1.0, 2
    if case["kernel"] == "gauss":
        return (0.5 if case["points"] == "rings" else 0.02 if case["points"] == "blobs" else 1.0 / case["d"]), 0.0, 1
    return 1.0, 0.0, 1


def _mode(case):
    return kkm.KKM_MODE_ONTHEFLY if case["family"] in ("onthefly", "seed") else kkm.KKM_MODE_AUTO


def _ranges(case):
    """The block of the (1, 0) process of a 2 x 2 grid, rows and columns, and its piece of the columns."""
    n = case["n"]
    half = (n // 2 + 127) // 128 * 128
    return half, n, 0, half, half // 2, half


# ------------------------------------------------------------------ one pass

class Problem:
    """A context with its inputs and outputs; the context's memory goes with it."""

    def __init__(self, case, seed):
        n, k = case["n"], case["k"]
        self.case, self.ctx = case, None
        self.X, self.cl0 = _inputs(case, seed)
        self.V = self.cl0.clone()
        self.params = kkm.make_params(*_kernel(case), _mode(case), kkm.STORAGES[case["storage"]], k)
        self.kind = kkm.KINDS[case["kernel"]]
        self.ctx = kkm.kkm_create(kkm.current_stream_handle())
        if case["family"] in ("build", "onthefly"):
            self.E = torch.empty((n, k), device="cuda")
            self.z = torch.empty(k, device="cuda")
            self.cl = torch.empty(n, dtype=torch.int32, device="cuda")
            self.counts = torch.empty(k, dtype=torch.int32, device="cuda")
        elif case["family"] == "share":
            r0, r1, c0, c1, a0, a1 = _ranges(case)
            self.rows, self.piece = self.cl0[r0:r1].clone(), self.cl0[a0:a1].clone()
            self.E = torch.empty((c1 - c0, k), device="cuda")
            self.cl = torch.empty(a1 - a0, dtype=torch.int32, device="cuda")
        elif case["family"] == "seed":
            u = np.random.default_rng(int(seed) + 5).random(k)
            self.u = np.minimum(u, 1 - 2.0 ** -30)
        if case["family"] in ("update", "seed"):
            self.build()

    def build(self):
        kkm.kkm_build_kernel(self.ctx, self.X, self.case["n"], self.case["d"], self.kind, self.params)

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            kkm.kkm_destroy(self.ctx)
            self.ctx = None


def prepare(case, seed):
    return Problem(case, seed)


def run(p):
    case, k = p.case, p.case["k"]
    family = case["family"]
    if family in ("fit", "update"):
        if family == "fit":
            p.build()
        p.V.copy_(p.cl0)
        done, hist = kkm.kkm_iterate(p.ctx, p.V, k, case["iters"], case["tol"])
        return {"ids": p.V, "objective": hist, "updates": done}
    if family in ("build", "onthefly"):
        p.build()
        J = kkm.kkm_step(p.ctx, p.cl0, k, E=p.E, z=p.z, cl_out=p.cl, counts_out=p.counts)
        return {"E": p.E, "z": p.z, "ids": p.cl, "sizes": p.counts, "objective": J}
    if family == "share":
        r0, r1, c0, c1, a0, a1 = _ranges(case)
        kkm.kkm_build_block(p.ctx, p.X, case["n"], case["d"], p.kind, p.params, r0, r1, c0, c1)
        kkm.kkm_block_spmm(p.ctx, p.rows, k, p.E)
        Ep = p.E[a0 - c0:a1 - c0]
        zpart, counts = kkm.kkm_block_zpart(p.ctx, Ep, p.piece, a0, a1, k)
        # the exchanges between processes are the caller's; here the block's own parts stand for the sums
        z = zpart / np.maximum(counts.astype(np.float64), 1.0) ** 2
        kkm.kkm_block_assign(p.ctx, Ep, a0, a1, k, z, counts, p.cl)  # (the sizes it returns are those of the ids)
        return {"E": p.E, "zpart": zpart, "sizes": counts, "ids": p.cl}
    centers = kkm.kkm_init_kmeanspp(p.ctx, k, p.u, p.V)
    return {"centers": centers, "ids": p.V}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    n, d, k, it = case["n"], case["d"], case["k"], case["iters"]
    entry = 2 if case["storage"] == "f16" else 4
    triangle = n * (n + 1) // 2                    # distinct entries of K
    points, ids = 4 * n * d, 8 * n                 # ids in and out
    if case["family"] == "fit":                    # K written once, read by each update
        return {"bytes": points + ids + (1 + it) * entry * triangle, "flops": 2 * triangle * d + 2 * it * triangle}
    if case["family"] == "build":
        return {"bytes": points + ids + 4 * n * k + 2 * entry * triangle, "flops": 2 * triangle * (d + 1)}
    if case["family"] == "update":                 # tol = 0 on these points stops after two updates
        it = min(it, 2) if case["tol"] >= 0 else it
        return {"bytes": ids + it * entry * triangle, "flops": 2 * it * triangle}
    if case["family"] == "onthefly":
        return {"bytes": points + ids + 4 * n * k, "flops": 2 * triangle * (d + 1)}
    if case["family"] == "share":
        r0, r1, c0, c1, a0, a1 = _ranges(case)
        block = (r1 - r0) * (c1 - c0)
        return {"bytes": 4 * (r1 - r0 + c1 - c0) * d + 8 * block + 4 * (c1 - c0) * k, "flops": 2 * block * (d + 1)}
    return {"bytes": k * points + 4 * n, "flops": 2 * k * n * d}   # every center is one pass over the points


def tolerance(case):
    """32-bit sums over a cluster's rows and over d, about four times the largest error
    against 64 bits measured on these ranges (2e-6 in fp32, where Gaussian entries are let
    stand up to 2e-6 off; binary16 entries carry 2^-12 each, averaged over a cluster's
    members).  The ids may differ where two distances tie: a point or two of the smallest
    problem."""
    rel = 1e-4 if case["storage"] == "f16" else 8e-6
    return {"rel": rel, "max": 40 * rel, "differ": 2e-3}


# ------------------------------------------------------------------ the same in 64 bits

def _k_rows(case, X, rows, cols=slice(None)):
    """Rows of K in fp64 by the kernel's definition (the Gaussian from fp64 norms and products)."""
    gamma, coef0, degree = _kernel(case)
    B = X[rows] @ X[cols].T
    if case["kernel"] == "linear":
        return B
    if case["kernel"] == "poly":
        return (gamma * B + coef0) ** degree
    sq = (X * X).sum(1)
    B.mul_(-2.0).add_(sq[rows][:, None]).add_(sq[cols][None, :]).clamp_(min=0.0)
    return B.mul_(-gamma).exp_()


def _sums(case, X, ids, k, rows, cols=slice(None)):
    """E of the points `rows`: their entries of K summed per id of the points `cols`."""
    V = torch.nn.functional.one_hot(ids.long(), k).double()
    lo, hi, _ = rows.indices(X.shape[0])
    step = max(1, int(4e8 // max(1, V.shape[0])))
    return torch.cat([_k_rows(case, X, slice(r, min(hi, r + step)), cols) @ V for r in range(lo, hi, step)])


def _diag(case, X):
    gamma, coef0, degree = _kernel(case)
    sq = (X * X).sum(1)
    return torch.ones_like(sq) if case["kernel"] == "gauss" else (gamma * sq + coef0) ** degree if case["kernel"] == "poly" else sq


def _update(case, X, diag, ids, k):
    """(E, z, new ids, sizes, objective) of one update from `ids`."""
    E = _sums(case, X, ids, k, slice(0, X.shape[0]))
    sizes = torch.bincount(ids.long(), minlength=k)
    own = E.gather(1, ids.long()[:, None])[:, 0]
    total = torch.zeros(k, dtype=torch.float64, device="cuda").index_add_(0, ids.long(), own)
    m = sizes.clamp(min=1).double()
    z = total / m ** 2
    D = diag[:, None] - 2.0 * E / m + z
    D[:, sizes == 0] = math.inf
    return E, z, D.argmin(1).to(torch.int32), sizes.to(torch.int32), float(diag.sum() - (total / m).sum())


def exact(case, seed):
    k, family = case["k"], case["family"]
    if family == "seed":
        return None  # indices only
    X32, ids = _inputs(case, seed)
    X, diag = X32.double(), _diag(case, X32.double())
    if family in ("fit", "update"):
        hist = []
        for _ in range(case["iters"]):
            _, _, new, _, J = _update(case, X, diag, ids, k)
            hist.append(J)
            same = bool((new == ids).all())
            ids = new
            if case["tol"] >= 0 and same:
                break
        return {"ids": ids, "objective": np.array(hist), "updates": len(hist)}
    if family in ("build", "onthefly"):
        E, z, new, sizes, J = _update(case, X, diag, ids, k)
        return {"E": E, "z": z, "ids": new, "sizes": sizes, "objective": J}
    r0, r1, c0, c1, a0, a1 = _ranges(case)
    E = _sums(case, X, ids[r0:r1], k, slice(c0, c1), slice(r0, r1))
    piece = ids[a0:a1].long()
    own = E[a0 - c0:a1 - c0].gather(1, piece[:, None])[:, 0]
    zpart = torch.zeros(k, dtype=torch.float64, device="cuda").index_add_(0, piece, own)
    return {"E": E, "zpart": zpart.cpu().numpy(), "sizes": None, "ids": None}

"""Timed cases of the framework: what its users run, through its public entry points.

A case is one call of a user's program on points (or a tree) that already lie on the GPU: clustering points, building their
minimum spanning tree, sweeping k on a tree, computing full-graph weights, or one training step with the points' gradients.
The sizes are those of the standard workloads in paper_1702_04739_amd/datagen.py and of the tests, with smaller and ragged ones
beside them; the points are drawn on the GPU by the same recipes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1702_04739_amd as iso

DEV = "cuda"
IMAGE_D = 28 * 28


# ------------------------------------------------------------------ cases

def listed():
    return [
        # a table of a few hundred rows: the call is all launches, copies and waits
        dict(name="cluster-150x5", kind="cluster", data="mixture", n=150, d=5, k=3, precision="fp32", recheck="fp32"),
        # the small standard workload: isotropic clusters with outliers, below the size where tile pairs are pruned
        dict(name="cluster-2000x16", kind="cluster", data="mixture", n=2000, d=16, k=5, precision="fp32", recheck="fp32"),
        # overlapping Gaussian data (nothing to prune), ordered by exact FP64 distances; ragged n
        dict(name="cluster-20011x40-fp64", kind="cluster", data="normal", n=20011, d=40, k=7, precision="fp32", recheck="fp64"),
        # the anisotropic mixture workload, default precision
        dict(name="cluster-50000x64", kind="cluster", data="aniso", n=50_000, d=64, k=20, precision="fp32", recheck="fp32"),
        # the headline workload: image-like rows with the BF16 screen
        dict(name="cluster-200000x784-bf16", kind="cluster", data="image", n=200_000, d=IMAGE_D, k=10, precision="bf16",
             recheck="fp32"),
        # a middle-sized set of 8-bit images with the exact integer screen; ragged n
        dict(name="cluster-59999x784-int8", kind="cluster", data="image", n=59_999, d=IMAGE_D, k=10, precision="int8",
             recheck="fp32"),
        # the high-dimensional sparse-communities workload: the tree alone, heavy-tailed norms
        dict(name="mst-100000x4096-bf16", kind="mst", data="sparse", n=100_000, d=4096, precision="bf16", recheck="fp32"),
        # clustering with the full-graph vertex weights and a potential (eqs. 2.2 and 2.3)
        dict(name="cluster-20000x128-full", kind="cluster", data="blobs", n=20_000, d=128, k=16, precision="fp32",
             recheck="fp32", omega="full", alpha=0.05),
        # learnable points: a forward and backward step on a small and on a full batch
        dict(name="train-777x5", kind="train", data="blobs", n=777, d=5, k=4, precision="fp32", recheck="fp32"),
        dict(name="train-20000x128", kind="train", data="blobs", n=20_000, d=128, k=16, precision="fp32", recheck="fp32"),
        # choosing k: every k up to 10 on one large tree that is already there
        dict(name="sweep-200000", kind="sweep", data="image", n=200_000, d=IMAGE_D, k=10, precision="bf16", recheck="fp32"),
        # the full-graph weights by themselves
        dict(name="weights-50000x64", kind="weights", data="aniso", n=50_000, d=64, alpha=0.05),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["cluster", "cluster", "image", "image", "mst", "full", "train", "sweep", "weights"])
    recheck = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "cluster":
        return dict(kind="cluster", data=rng.choice(["mixture", "normal", "aniso", "blobs"]), n=_log_int(rng, 150, 50_000),
                    d=_log_int(rng, 2, 128), k=rng.randint(2, 20), precision="fp32", recheck=recheck)
    if kind == "image":
        return dict(kind="cluster", data="image", n=_log_int(rng, 2000, 200_000), d=IMAGE_D, k=rng.randint(2, 20),
                    precision=rng.choice(["bf16", "int8"]), recheck=recheck)
    if kind == "mst":
        return dict(kind="mst", data="sparse", n=_log_int(rng, 5000, 60_000), d=_log_int(rng, 1024, 4096), precision="bf16",
                    recheck="fp32")
    if kind == "full":
        return dict(kind="cluster", data=rng.choice(["mixture", "aniso", "blobs"]), n=_log_int(rng, 500, 20_000),
                    d=_log_int(rng, 2, 128), k=rng.randint(2, 16), precision="fp32", recheck="fp32", omega="full",
                    alpha=rng.choice([0.0, 0.05]))
    if kind == "train":
        return dict(kind="train", data=rng.choice(["blobs", "normal"]), n=_log_int(rng, 300, 20_000), d=_log_int(rng, 2, 128),
                    k=rng.randint(2, 16), precision="fp32", recheck="fp32")
    if kind == "sweep":
        return dict(kind="sweep", data="image", n=_log_int(rng, 2000, 200_000), d=IMAGE_D, k=rng.randint(4, 16),
                    precision="bf16", recheck="fp32")
    return dict(kind="weights", data=rng.choice(["aniso", "blobs"]), n=_log_int(rng, 1000, 50_000), d=_log_int(rng, 2, 64),
                alpha=rng.choice([0.0, 0.05]))


# ------------------------------------------------------------------ inputs

def _points(case, seed):
    """The case's points, float32 (n, d) on the GPU, rows in random order (the recipes of datagen.py)."""
    n, d, data = case["n"], case["d"], case["data"]
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    r = np.random.default_rng(int(seed))

    def rand(*shape):
        return torch.rand(shape, generator=g, device=DEV)

    def randn(*shape):
        return torch.randn(shape, generator=g, device=DEV)

    def randint(hi, *shape):
        return torch.randint(hi, shape, generator=g, device=DEV)

    if data == "mixture":  # 5 isotropic clusters and 2 % uniform outliers
        X = 20.0 * rand(5, d)[randint(5, n)] - 10.0 + randn(n, d)
        out = rand(n) < 0.02
        X = torch.where(out[:, None], 26.0 * rand(n, d) - 13.0, X)
    elif data == "normal":  # clusters that overlap
        X = 2.0 * rand(4, d)[randint(4, n)] - 1.0 + randn(n, d)
    elif data == "aniso":  # 20 anisotropic clusters of uneven sizes
        props = torch.from_numpy(r.dirichlet(np.ones(20)).cumsum().astype(np.float32)).to(DEV)
        lab = torch.searchsorted(props, rand(n)).clamp_(max=19)
        means, stds = 40.0 * rand(20, d) - 20.0, 0.5 + 1.5 * rand(20, d)
        X = means[lab] + stds[lab] * randn(n, d)
    elif data == "blobs":  # 16 isotropic clusters
        X = (30.0 * rand(16, d) - 15.0)[randint(16, n)] + randn(n, d)
    elif data == "image":  # 10 blurred patterns with multiplicative noise, 8-bit values q / 256
        yy, xx = np.mgrid[0:28, 0:28].astype(np.float64)
        centres = np.zeros((10, IMAGE_D), np.float32)
        for c in range(10):
            img = np.zeros((28, 28))
            for _ in range(int(r.integers(3, 7))):
                amp, width, (cy, cx) = r.uniform(0.5, 1.0), r.uniform(2.0, 4.0), r.uniform(0, 28, size=2)
                img += amp * np.exp(-((yy - cy) ** 2 + (xx - cx) ** 2) / (2 * width * width))
            img = np.clip(img, 0.0, 1.0)
            img[img < 0.1] = 0.0
            centres[c] = img.ravel()
        X = torch.from_numpy(centres).to(DEV)[randint(10, n)]
        X = torch.round(255.0 * (X * (1.0 + 0.1 * randn(n, IMAGE_D))).clamp_(0.0, 1.0)) / 256.0
    else:  # "sparse": 50 communities that share supports, 1 % lognormal nonzeros
        nnz = max(1, round(0.01 * d))
        supports = torch.from_numpy(np.stack([r.choice(d, size=nnz, replace=False) for _ in range(50)])).to(DEV)
        own = torch.gather(supports[randint(50, n)], 1, randint(nnz, n, nnz))
        cols = torch.where(rand(n, nnz) < 0.8, own, randint(d, n, nnz))
        X = torch.zeros(n, d, device=DEV).scatter_reduce_(1, cols, randn(n, nnz).exp_(), "amax")
    return X.contiguous()


def _sigma(case):
    """A scale near the edges' lengths, as a program that sets it by itself would."""
    return math.sqrt(case["d"])


def prepare(case, seed):
    X = _points(case, seed)
    if case["kind"] == "sweep":  # the tree is there from an earlier call; the points are no longer needed
        parent, length, _ = iso.mst(X, precision=case["precision"], recheck=case["recheck"])
        return dict(case=case, parent=parent, length=length)
    if case["kind"] == "train":
        return dict(case=case, points=X.requires_grad_(True),
                    sigma=torch.tensor(_sigma(case), dtype=torch.float64, device=DEV, requires_grad=True))
    return dict(case=case, points=X)


# ------------------------------------------------------------------ one pass

def run(state):
    c = state["case"]
    if c["kind"] == "cluster":
        labels, i_k, info = iso.cluster(state["points"], c["k"], precision=c["precision"], recheck=c["recheck"],
                                        omega=c.get("omega", "tree"), alpha=c.get("alpha", 0.0))
        return dict(labels=labels, i_k=i_k, parent=info["parent"], length=info["length"], weight=info["mst"]["mst_weight"])
    if c["kind"] == "mst":
        parent, length, info = iso.mst(state["points"], precision=c["precision"], recheck=c["recheck"])
        return dict(parent=parent, length=length, weight=info["mst_weight"])
    if c["kind"] == "sweep":
        i_k, labels, _ = iso.subpartition_all_k(state["parent"], state["length"], c["k"])
        return dict(labels=labels, i_k=i_k)
    if c["kind"] == "train":
        X, sigma = state["points"], state["sigma"]
        X.grad = sigma.grad = None
        W, i_k, labels = iso.MSTIsoCost.apply(X, sigma, c["k"], c["precision"], c["recheck"])
        (W + i_k).backward()
        return dict(labels=labels, i_k=i_k.detach(), weight=W.detach(), grad=X.grad, grad_sigma=sigma.grad)
    omega, p0 = iso.graph_weights(state["points"], _sigma(c), alpha=c["alpha"])
    return dict(omega=omega) if p0 is None else dict(omega=omega, p0=p0)


def work(case):
    """Every input read once and every output written once.  Operations: the distances within a cluster for a tree (pairs of
    far clusters need none), every pair's distance for the weights."""
    n, d, kind = case["n"], case["d"], case["kind"]
    clusters = {"mixture": 5, "aniso": 20, "blobs": 16, "image": 10}.get(case["data"], 1)
    tree = dict(bytes=4 * n * d + 12 * n, flops=d * n * n / clusters)
    weights = dict(bytes=4 * n * d + 16 * n, flops=1.5 * d * n * n)
    if kind == "mst":
        return tree
    if kind == "weights":
        return weights
    if kind == "sweep":
        return dict(bytes=12 * n + 4 * n * (case["k"] - 1), flops=0)
    if kind == "train":
        return dict(bytes=tree["bytes"] + 4 * n * d + 4 * n, flops=tree["flops"])
    full = case.get("omega") == "full" or case.get("alpha", 0.0) > 0.0
    return dict(bytes=tree["bytes"] + 4 * n, flops=tree["flops"] + (weights["flops"] if full else 0))


# ------------------------------------------------------------------ the same in 64 bits, in plain torch

def _tree64(X):
    """Prim's tree from vertex 0 with float64 distances: parents and lengths.  Edges are ordered by (squared length, smaller
    end, larger end), which settles the ties of 8-bit data (whose squared lengths are exact here)."""
    n = X.shape[0]
    X = X.double()
    s = X.square().sum(1)
    number = torch.arange(n, device=X.device)
    key = torch.full((n,), math.inf, dtype=torch.float64, device=X.device)
    parent = torch.full((n,), -1, dtype=torch.int64, device=X.device)
    v = torch.zeros(1, dtype=torch.int64, device=X.device)
    for _ in range(n - 1):
        key.index_fill_(0, v, -math.inf)
        d2 = torch.addmv(s + s[v], X, X.index_select(0, v)[0], alpha=-2.0)
        nearer = (d2 < key) | ((d2 == key) & (v < parent))
        key = torch.where(nearer, d2, key)
        parent = torch.where(nearer, v, parent)
        open_ = torch.where(key == -math.inf, math.inf, key)
        ends = torch.minimum(parent, number) * n + torch.maximum(parent, number)
        v = torch.where(open_ == open_.min(), ends, n * n).argmin(0, keepdim=True)
    length = (X - X[parent.clamp(min=0)]).square().sum(1).sqrt()
    length[0] = 0.0
    return parent, length


class _Sub64:
    """The optimal k-subpartitions of a tree rooted at vertex 0 (Algorithms 1, 2 and 4) with float64 weights, for several k at once.
    On the CPU, where sums are taken in one order: the bisection's last threshold has to give the same cuts again."""

    def __init__(self, parent, length, sigma=None, omega=None, p0=None):
        parent, length, omega, p0 = (x if x is None else x.cpu() for x in (parent, length, omega, p0))
        n = parent.shape[0]
        up, depth = parent.clamp(min=0), (parent >= 0).long()
        while int((up != 0).sum()):
            depth, up = depth + depth[up], up[up]
        order = torch.argsort(-depth, stable=True)  # deepest first, by vertex number within a depth
        place = torch.empty_like(order).scatter_(0, order, torch.arange(n))
        sizes = torch.bincount(depth.max() - depth).tolist()
        ends = np.cumsum(sizes).tolist()
        self.levels = [(e - s, e) for s, e in zip(sizes, ends)]
        self.n, self.order, self.length = n, order, length[order]
        self.up = place[parent.clamp(min=0)][order]  # of the root: itself
        self.sigma = float(torch.sort(length[1:]).values[(n - 2) // 2]) if sigma is None else sigma
        self.flow = torch.exp(-self.length / self.sigma)
        self.flow[n - 1] = 0.0
        self.omega = omega[order] if omega is not None else self.flow.clone().index_add_(0, self.up[:-1], self.flow[:-1])
        self.p0 = p0[order] if p0 is not None else torch.zeros_like(self.omega)

    def decide(self, N):
        """Cut and joined flags of every vertex, and the sets' weight and boundary, at each threshold of N."""
        w, p = (x[:, None].repeat(1, N.shape[0]) for x in (self.omega, self.p0))
        cut = torch.empty_like(w, dtype=torch.bool)
        join = torch.zeros_like(cut)
        for s, e in self.levels:
            f, room = self.flow[s:e, None], N * w[s:e]
            cut[s:e] = f + p[s:e] <= room
            if e < self.n:
                join[s:e] = ~cut[s:e] & (p[s:e] - f < room)
                zero = torch.zeros_like(room)
                w.index_add_(0, self.up[s:e], torch.where(join[s:e], w[s:e], zero))
                p.index_add_(0, self.up[s:e], torch.where(join[s:e], p[s:e], f.expand_as(room)))
        return cut, join, w, p

    def solve(self, ks):
        """For each k: the cost, the labels in tree order and the cluster that attains the cost."""
        k = torch.tensor(ks)
        edges = self.flow[:-1]
        lo = float((edges.min() + self.p0.min()) / self.omega.sum())
        hi = float((edges.sum() + self.p0.sum()) / self.omega.min())
        lo, hi = (2.0 ** (math.frexp(x)[1] + m) for x, m in ((lo, -1), (hi, 0)))
        lo, hi = (torch.full((len(ks),), x, dtype=torch.float64) for x in (lo, hi))
        while True:
            mid = lo + 0.5 * (hi - lo)
            open_ = (mid > lo) & (mid < hi)
            if not bool(open_.any()):
                break
            yes = self.decide(mid)[0].sum(0) >= k
            hi, lo = torch.where(open_ & yes, mid, hi), torch.where(open_ & ~yes, mid, lo)
        cut, join, w, p = self.decide(hi)
        rep = torch.arange(self.n)[:, None].repeat(1, len(ks))
        for s, e in reversed(self.levels):
            if e < self.n:
                rep[s:e] = torch.where(join[s:e], rep[self.up[s:e]], rep[s:e])
        found = []
        for j, kk in enumerate(ks):
            at = torch.nonzero(cut[:, j])[:kk, 0]
            cost = (self.flow[at] + p[at, j]) / w[at, j]
            which = torch.full((self.n,), -1, dtype=torch.int64)
            which[at] = torch.arange(len(at))
            found.append((float(cost.max()), which[rep[:, j]], int(cost.argmax())))
        return found


def _weights64(X, sigma, alpha):
    n = X.shape[0]
    X = X.double()
    X = X - X.mean(0)
    sq = X.square().sum(1)
    omega, p0 = (torch.empty(n, dtype=torch.float64, device=X.device) for _ in range(2))
    for s in range(0, n, 1024):
        rows = X[s:s + 1024]
        D = (sq[s:s + 1024, None] + sq - 2.0 * (rows @ X.t().contiguous())).clamp_(min=0.0).sqrt_()
        own = torch.arange(rows.shape[0], device=X.device)
        D[own, s + own] = 0.0
        phi = torch.exp(-D / sigma)
        phi[own, s + own] = 0.0
        omega[s:s + 1024], p0[s:s + 1024] = phi.sum(1), alpha * D.sum(1)
    return omega, p0


def exact(case, seed):
    n, d, kind = case["n"], case["d"], case["kind"]
    if kind == "sweep":
        s = prepare(case, seed)
        return dict(labels=None, i_k=np.array([c for c, _, _ in _Sub64(s["parent"].long(), s["length"]).solve(list(range(2, case["k"] + 1)))]))
    if kind == "weights":
        omega, p0 = _weights64(_points(case, seed), _sigma(case), case["alpha"])
        return dict(omega=omega, p0=p0) if case["alpha"] > 0 else dict(omega=omega)
    if n * max(1.5e-4, n * d * 8 / 2.5e12) > 15.0:
        return None  # Prim's n steps in torch would take too long
    X = _points(case, seed)
    parent, length = _tree64(X)
    weight = length.sum() if kind == "train" else float(length.sum())
    if kind == "mst":
        return dict(parent=None, length=length, weight=weight)
    if kind == "cluster":
        om = p0 = None
        if case.get("omega", "tree") == "full":
            om, p0 = _weights64(X, float(torch.sort(length[1:]).values[(n - 2) // 2]), case["alpha"])
        (i_k, _, _), = _Sub64(parent, length, omega=om, p0=p0).solve([case["k"]])
        return dict(labels=None, i_k=i_k, parent=None, length=length, weight=weight)
    # the step's gradients: autograd through the lengths of the same tree and the cost of the same cluster
    sub = _Sub64(parent, length, sigma=_sigma(case))
    (i_k, which, best), = sub.solve([case["k"]])
    Xd = X.double().requires_grad_(True)
    sigma = torch.tensor(_sigma(case), dtype=torch.float64, device=X.device, requires_grad=True)
    a = torch.arange(1, n, device=X.device)
    b = parent[1:]
    lens = (Xd[a] - Xd[b]).square().sum(1).sqrt()
    flow = torch.exp(-lens / sigma)
    label = torch.empty_like(which).scatter_(0, sub.order, which).to(X.device)
    ina, inb = label[a] == best, label[b] == best
    cost = flow[ina != inb].sum() / (flow * (ina.double() + inb.double())).sum()
    (lens.sum() + cost).backward()
    return dict(labels=None, i_k=cost.detach(), weight=weight, grad=Xd.grad, grad_sigma=sigma.grad)

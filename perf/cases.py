"""Performance cases: what a program that counts tree templates asks of the library.

Each case is one call (or one training step) through the public entry points
on a seeded synthetic graph: ``kind`` says which entry point, ``graph`` which
generator ("er", "rmat", "chunglu"), ``n`` and ``deg`` its vertices and mean
degree, ``template`` and ``k`` the tree and the colours, ``colorings`` how
many colourings one call counts, ``mode`` the arithmetic.

Every pass draws its colourings on the device, as a program that runs more
and more colourings does.  FP32S counts carry single precision, so they are
returned in that type, in units of 1024 per template vertex to the power of
its size (a power of two that keeps them inside the type's range).
"""
import math

import numpy as np
import torch

import paper_2009_11665_amd as sg

DEV = "cuda"


# ---------------------------------------------------------------------------
# templates

def tree(name):
    """Parent array of a named template: path8, star5 (four leaves), bintree15
    (complete binary tree numbering), caterpillar10 (a spine, one leg on each
    inner spine vertex)."""
    shape = name.rstrip("0123456789")
    t = int(name[len(shape):])
    if shape == "path":
        return [-1] + list(range(t - 1))
    if shape == "star":
        return [-1] + [0] * (t - 1)
    if shape == "bintree":
        return [-1] + [(i - 1) // 2 for i in range(1, t)]
    if shape == "caterpillar":
        spine = t // 2 + 1
        return [-1] + list(range(spine - 1)) + list(range(1, t - spine + 1))
    raise ValueError(name)


def trees_of(case):
    """The case's templates: names joined by '+', or every free tree of a size."""
    name = case["template"]
    if name.startswith("alltrees"):
        return sg.trees(int(name[8:]))
    return [tree(p) for p in name.split("+")]


# ---------------------------------------------------------------------------
# graphs, made on the GPU from the seed

def _endpoints(case, count, gen):
    """`count` random vertex pairs of the case's generator."""
    n = case["n"]
    if case["graph"] == "er":
        return (torch.randint(0, n, (count,), device=DEV, generator=gen),
                torch.randint(0, n, (count,), device=DEV, generator=gen))
    if case["graph"] == "rmat":
        u = torch.zeros(count, dtype=torch.int64, device=DEV)
        v = torch.zeros(count, dtype=torch.int64, device=DEV)
        for _ in range(int(n).bit_length() - 1):
            q = torch.rand(count, device=DEV, generator=gen)
            # quadrants a, b, c, d with 0.57, 0.19, 0.19, 0.05
            u.mul_(2).add_(q >= 0.76)
            v.mul_(2).add_(((q >= 0.57) & (q < 0.76)) | (q >= 0.95))
        return u, v
    # Chung-Lu, power-law weights of exponent 2.1 up to sqrt(n * mean degree)
    beta, total = 1.0 / 1.1, n * case["deg"]
    lo, hi = 1e-3, float(n)
    for _ in range(100):
        i0 = math.sqrt(lo * hi)
        mass = ((n + i0) ** (1 - beta) - i0 ** (1 - beta)) / (1 - beta) * i0 ** beta
        lo, hi = (i0, hi) if mass * math.sqrt(total) < total else (lo, i0)
    cum = torch.cumsum((torch.arange(n, device=DEV, dtype=torch.float64) + i0) ** -beta, 0)
    draw = lambda: torch.searchsorted(cum, torch.rand(count, device=DEV, dtype=torch.float64, generator=gen) * cum[-1]).clamp_(max=n - 1)  # noqa: E731
    return draw(), draw()


def make_graph(case, seed):
    """Symmetric CSR (int64 row pointers, int32 sorted columns, float32 weights
    or None) of round(n * deg / 2) distinct undirected edges, vertices shuffled."""
    n = case["n"]
    m = int(round(n * case["deg"] / 2))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1000003 * int(seed) + 17)
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while keys.numel() < m:
        # small first draws, then what is missing: RMAT and Chung-Lu repeat pairs
        u, v = _endpoints(case, int((m - keys.numel()) * 1.25) + 256, gen)
        lo, hi = torch.minimum(u, v), torch.maximum(u, v)
        del u, v
        fresh = (lo * n + hi)[lo != hi]
        del lo, hi
        keys = torch.unique(torch.cat([keys, fresh]))
    if keys.numel() > m:
        keys = keys[torch.randperm(keys.numel(), device=DEV, generator=gen)[:m]]
    perm = torch.randperm(n, device=DEV, generator=gen)
    u, v = perm[keys // n], perm[keys % n]
    del keys
    both = torch.cat([u * n + v, v * n + u])
    del u, v
    w = None
    if case.get("weighted"):
        w = torch.rand(m, device=DEV, generator=gen) + 0.5
        both, order = torch.sort(both)
        w = torch.cat([w, w])[order]
    else:
        both = torch.sort(both)[0]
    row_ptr = torch.searchsorted(both, torch.arange(n + 1, device=DEV) * n)
    return row_ptr, (both % n).to(torch.int32), w


# ---------------------------------------------------------------------------
# the cases

def listed():
    return [
        # one colouring of a small graph: a test, a notebook, a request to a service
        dict(name="small-path5-fp64", kind="count", graph="er", n=1000, deg=8, template="path5", k=5,
             colorings=1, mode="fp64"),
        # the estimator with an error bound on that graph: thousands of colourings
        dict(name="small-estimate", kind="estimate", graph="er", n=1000, deg=8, template="path5", k=5,
             eps=0.25, delta=0.1, mode="fp64"),
        # a social-network sized graph, a few colourings at once
        dict(name="rmat16-bintree7-fp32s", kind="count", graph="rmat", n=65536, deg=32, template="bintree7", k=7,
             colorings=8, mode="fp32s"),
        # exact counts, as a check of the floating ones asks for
        dict(name="rmat16-path8-u64", kind="count", graph="rmat", n=65536, deg=32, template="path8", k=8,
             colorings=4, mode="u64"),
        # more colours than vertices and a vertex count that is no multiple of anything
        dict(name="odd-path7-k9-fp32s", kind="count", graph="chunglu", n=100003, deg=13, template="path7", k=9,
             colorings=3, mode="fp32s"),
        # weighted counting and its derivative in double, the differentiation workload
        dict(name="weighted-caterpillar10-fp64", kind="count", graph="chunglu", n=262144, deg=16,
             template="caterpillar10", k=10, colorings=1, mode="fp64", weighted=True),
        dict(name="grad-caterpillar10-fp64", kind="grad", graph="chunglu", n=262144, deg=16,
             template="caterpillar10", k=10, colorings=1, mode="fp64", weighted=True),
        # a training step on edge weights: forward and backward through autograd
        dict(name="train-caterpillar10-fp32s", kind="train", graph="chunglu", n=262144, deg=16,
             template="caterpillar10", k=10, colorings=1, mode="fp32s", weighted=True),
        # several templates, many colourings: the batching workload
        dict(name="batch-3x16-fp32s", kind="batch", graph="chunglu", n=500000, deg=20,
             template="bintree7+path8+caterpillar10", k=0, colorings=16, mode="fp32s"),
        # a treelet distribution: all 47 trees of nine vertices in one call
        dict(name="treelets9-fp32s", kind="multi", graph="chunglu", n=500000, deg=20, template="alltrees9", k=9,
             colorings=8, mode="fp32s"),
        # the plain FP64 method on a dense power-law graph
        dict(name="rmat18-bintree15-fp64", kind="count", graph="rmat", n=262144, deg=190, template="bintree15",
             k=15, colorings=1, mode="fp64", relabel=True),
        # the benchmark's graph and template: 200M entries, the 15-vertex tree
        dict(name="rmat20-bintree15-fp32s", kind="count", graph="rmat", n=1048576, deg=200e6 / 1048576,
             template="bintree15", k=15, colorings=1, mode="fp32s", relabel=True),
    ]


NAMES = ("path5", "path7", "path8", "star5", "bintree7", "caterpillar8", "caterpillar10", "bintree15")


def draw(rng):
    kind = rng.choice(("count", "count", "count", "grad", "train", "batch", "multi", "estimate"))
    graph = rng.choice(("er", "rmat", "chunglu"))
    if kind == "estimate":
        n = int(round(2 ** rng.uniform(8, 12)))
        t = rng.choice(("path5", "star5", "path4", "star4"))
        return dict(kind=kind, graph="er", n=n, deg=round(rng.uniform(4, 12), 2), template=t, k=int(t[-1]),
                    eps=round(rng.uniform(0.2, 0.4), 3), delta=0.1, mode=rng.choice(("fp64", "fp32s")))
    if kind in ("grad", "train"):
        t = rng.choice(("path5", "path8", "bintree7", "caterpillar8", "caterpillar10"))
        return dict(kind=kind, graph=graph if graph != "rmat" else "chunglu", n=int(round(2 ** rng.uniform(10, 17.5))),
                    deg=round(2 ** rng.uniform(2, 4.5), 2), template=t,
                    k=len(tree(t)) + rng.choice((0, 0, 1)), colorings=rng.choice((1, 1, 2)),
                    mode=rng.choice(("fp64", "fp32s")), weighted=True)
    if kind == "batch":
        t = "+".join(rng.sample(("path5", "path7", "path8", "star5", "bintree7", "caterpillar8", "caterpillar10"), rng.choice((2, 3))))
        return dict(kind=kind, graph=graph if graph != "rmat" else "chunglu", n=int(round(2 ** rng.uniform(11, 18.5))),
                    deg=round(rng.uniform(6, 20), 2), template=t, k=0, colorings=rng.randint(2, 16),
                    mode=rng.choice(("fp32s", "fp32s", "fp64")))
    if kind == "multi":
        s = rng.choice((6, 7, 8))
        return dict(kind=kind, graph=graph if graph != "rmat" else "chunglu", n=int(round(2 ** rng.uniform(10, 18))),
                    deg=round(rng.uniform(6, 20), 2), template="alltrees%d" % s, k=s, colorings=rng.randint(1, 8),
                    mode=rng.choice(("fp32s", "fp32s", "fp64")))
    t = rng.choice(NAMES)
    size = len(tree(t))
    mode = rng.choice(("fp32s", "fp32s", "fp64", "u64"))
    if size == 15:  # the large template: dense RMAT graphs
        scale = rng.choice((14, 15, 16, 17))
        return dict(kind=kind, graph="rmat", n=1 << scale, deg=round(2 ** rng.uniform(5, 7.5), 2), template=t, k=15,
                    colorings=rng.choice((1, 2)), mode=rng.choice(("fp32s", "fp64")), relabel=rng.random() < 0.7)
    n = 1 << rng.randint(10, 18) if graph == "rmat" else int(round(2 ** rng.uniform(10, 19)))
    return dict(kind=kind, graph=graph, n=n, deg=round(2 ** rng.uniform(2, 5), 2), template=t,
                k=size + rng.choice((0, 0, 1, 2)), colorings=rng.randint(1, 16), mode=mode,
                weighted=mode != "u64" and rng.random() < 0.3, relabel=rng.random() < 0.25)


# ---------------------------------------------------------------------------
# one pass

class State:
    pass


def prepare(case, seed):
    """The registered graph, the plan and the weights, as a program keeps them."""
    s = State()
    s.case, s.seed = case, int(seed)
    s.row_ptr, s.col_idx, s.w = make_graph(case, seed)
    ts = trees_of(case)
    if case["kind"] == "batch":
        s.plans = [sg.Plan(sg.reroot(t)[0]) for t in ts]
    elif case["kind"] == "multi":
        s.plan = sg.Plan.multi(ts, case["k"])
    else:
        s.plan = sg.Plan(ts[0], case["k"])
    s.unit = float(2.0 ** (-10 * max(len(t) for t in ts)))
    if case["kind"] == "train":
        s.w.requires_grad_(True)  # the graph is registered with the step's weights
    else:
        s.graph = sg.Graph(case["n"], s.row_ptr, s.col_idx, s.w, relabel=bool(case.get("relabel")))
    s.gc = np.linspace(1.0, 2.0, case.get("colorings", 1))
    return s


def _counts(s, x):
    """Counts in the precision of their mode."""
    if s.case["mode"] == "fp32s":
        return (np.asarray(x, np.float64) * s.unit).astype(np.float32)
    return np.asarray(x, np.float64)


def run(s):
    case = s.case
    kind, mode = case["kind"], case["mode"]
    if kind == "count":
        col = sg.Colorings(s.graph, case["k"], s.seed, case["colorings"])
        r = sg.count(s.plan, s.graph, col, mode)
        if mode == "u64":
            return {"colorful": r["colorful_u64"].view(np.int64), "overflow": r["overflow"]}
        return {"colorful": _counts(s, r["colorful"]), "estimate": _counts(s, r["estimate"])}
    if kind == "estimate":
        e, trace = sg.estimate(s.plan, s.graph, s.seed, case["eps"], case["delta"], mode)
        return {"mean": _counts(s, e.mean), "median": _counts(s, e.median_of_means),
                "trace": _counts(s, trace), "colorings": int(e.n_colorings)}
    if kind == "batch":
        cf, est = sg.count_batch(s.plans, s.graph, s.seed, case["colorings"], mode)
        return {"colorful": _counts(s, cf), "estimate": _counts(s, est)}
    if kind == "multi":
        col = sg.Colorings(s.graph, case["k"], s.seed, case["colorings"])
        r = sg.count_multi(s.plan, s.graph, col, mode)
        freq = r["frequency"].astype(np.float32) if mode == "fp32s" else r["frequency"]
        return {"colorful": _counts(s, r["colorful"]), "frequency": freq}
    if kind == "grad":
        col = sg.Colorings(s.graph, case["k"], s.seed, case["colorings"])
        g = sg.count_grad(s.plan, s.graph, col, s.gc, mode)
        return {"grad": g if mode == "fp64" else (g * s.unit).to(torch.float32)}
    # train: forward and backward of the colourful counts in the edge weights
    s.w.grad = None
    f = sg.SubgraphCount.apply(s.w, s.plan, s.row_ptr, s.col_idx, s.seed, case["colorings"], mode)
    (f * s.unit).sum().backward()
    return {"colorful": f.detach() if mode == "fp64" else (f.detach() * s.unit).to(torch.float32),
            "grad": s.w.grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _shapes(case):
    """Per template: (sizes of the distinct passive children, (size, active size) of the distinct splits)."""
    out = []
    for t in trees_of(case):
        ch = [[] for _ in t]
        for v, p in enumerate(t):
            if p >= 0:
                ch[p].append(v)
        seen, passives, splits = {}, {}, {}

        def walk(v, kept):
            if kept == 0:
                return (1, "o")
            a = walk(v, kept - 1)
            c = ch[v][kept - 1]
            p = walk(c, len(ch[c]))
            key = a[1] + "(" + p[1] + ")"
            passives[p[1]] = p[0]
            splits[key] = (a[0] + p[0], a[0])
            seen[key] = a[0] + p[0]
            return (a[0] + p[0], key)

        walk(t.index(-1), len(ch[t.index(-1)]))
        out.append((passives, splits, len(t)))
    return out


def work(case):
    """Bytes: the colours, the adjacency once per colouring (and once more for
    gradients), and the count tables once written and once read at their
    narrowest, the aggregated ones; flops: one addition per entry and aggregated
    column plus a multiply-add per split pair and vertex (three times as much
    with gradients)."""
    n, es = case["n"], 4 if case["mode"] == "fp32s" else 8
    nnz = 2 * int(round(n * case["deg"] / 2))
    passes = case.get("colorings", 1)
    if case["kind"] == "estimate":
        t = len(tree(case["template"]))
        p = math.factorial(case["k"]) / math.factorial(case["k"] - t) / case["k"] ** t
        passes = math.ceil(8 * math.log(1 / case["delta"])) * math.ceil(4 * (1 / p - 1) / case["eps"] ** 2)
    by, fl = 0.0, 0.0
    shared_p, shared_s = set(), set()
    for passives, splits, t in _shapes(case):
        k = case["k"] or t
        for key, m in passives.items():
            if (key, k) in shared_p:
                continue
            shared_p.add((key, k))
            cols = math.comb(k, m)
            by += 2.0 * n * cols * es
            fl += nnz * cols
        for key, (m, a) in splits.items():
            if (key, k) in shared_s:
                continue
            shared_s.add((key, k))
            fl += 2.0 * n * math.comb(k, m) * math.comb(m, a)
    by += n + nnz * (8.0 if case.get("weighted") else 4.0) / passes
    if case["kind"] in ("grad", "train"):
        by, fl = 3 * by + 8.0 * nnz, 3 * fl
    return {"bytes": by * passes, "flops": fl * passes}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch

def _colours(n, k, seed, j):
    """Colour of every vertex in colouring j (SplitMix64's finaliser, multiply-shift)."""
    def fin(z):
        with np.errstate(over="ignore"):
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))
    v = np.arange(n, dtype=np.uint64) | (np.uint64(j) << np.uint64(40))
    h = fin(np.uint64(seed) ^ fin(v))
    return ((h >> np.uint64(32)) * np.uint64(k) >> np.uint64(32)).astype(np.int64)


class _Spmm(torch.autograd.Function):
    """A(w) M with derivatives in both."""

    @staticmethod
    def forward(ctx, w, m, row_ptr, col_idx):
        n = row_ptr.numel() - 1
        a = torch.sparse_csr_tensor(row_ptr, col_idx.long(), w, (n, n))
        ctx.save_for_backward(w, m, row_ptr, col_idx)
        return torch.sparse.mm(a, m)

    @staticmethod
    def backward(ctx, gb):
        w, m, row_ptr, col_idx = ctx.saved_tensors
        n = row_ptr.numel() - 1
        rows = torch.repeat_interleave(torch.arange(n, device=w.device), row_ptr.diff())
        gw = torch.empty_like(w)
        for a in range(0, w.numel(), 1 << 19):
            b = min(w.numel(), a + (1 << 19))
            gw[a:b] = (gb[rows[a:b]] * m[col_idx[a:b].long()]).sum(1)
        adj = torch.sparse_csr_tensor(row_ptr, col_idx.long(), w, (n, n))  # symmetric
        return gw, torch.sparse.mm(adj, gb.contiguous()), None, None


def _sets(k, m):
    return sorted(x for x in range(1 << k) if bin(x).count("1") == m)


def _dp(t, k, colour, w, row_ptr, col_idx, memo, bs):
    """Colourful maps of tree t, by recursion over its rooted sub-trees; memo
    and bs keep the tables and their aggregations by rooted shape."""
    n = row_ptr.numel() - 1
    ch = [[] for _ in t]
    for v, p in enumerate(t):
        if p >= 0:
            ch[p].append(v)

    def shape(v, kept):
        return "(" + "".join(sorted(shape(c, len(ch[c])) for c in ch[v][:kept])) + ")"

    def agg(v):
        key = shape(v, len(ch[v]))
        if key not in bs:
            m = table(v, len(ch[v]))
            bs[key] = _Spmm.apply(w, m, row_ptr, col_idx)
        return bs[key]

    def size(v, kept):
        return 1 + sum(size(c, len(ch[c])) for c in ch[v][:kept])

    def table(v, kept):
        key = shape(v, kept)
        if key not in memo:
            if kept == 0:
                x = torch.zeros(n, k, dtype=torch.float64, device=DEV)
                x[torch.arange(n, device=DEV), colour] = 1.0
                memo[key] = x
            else:
                a, b = table(v, kept - 1), agg(ch[v][kept - 1])
                ma, mb = size(v, kept - 1), size(ch[v][kept - 1], len(ch[ch[v][kept - 1]]))
                ia = {s: i for i, s in enumerate(_sets(k, ma))}
                ib = {s: i for i, s in enumerate(_sets(k, mb))}
                pick = []
                for s in _sets(k, ma + mb):
                    q, x = [], s
                    while x:
                        if bin(x).count("1") == ma:
                            q.append((ia[x], ib[s ^ x]))
                        x = (x - 1) & s
                    pick.append(q)
                idx = torch.tensor(pick, device=DEV).permute(1, 2, 0).contiguous()
                if idx.shape[2] == 1:
                    out = sum((a[:, i[0]] * b[:, i[1]]).sum(1, keepdim=True) for i in idx[:, :, 0].T.split(512, 1))
                else:
                    out = 0
                    for q in range(idx.shape[0]):
                        out = out + a[:, idx[q, 0]] * b[:, idx[q, 1]]
                memo[key] = out
        return memo[key]

    return table(t.index(-1), len(ch[t.index(-1)])).sum()


def _scale(t, k):
    """Counts of colourful maps to copies: 1 / (colourful probability * automorphisms)."""
    ch = [[] for _ in t]
    nb = [[] for _ in t]
    for v, p in enumerate(t):
        if p >= 0:
            nb[v].append(p)
            nb[p].append(v)

    def canon(v, p):
        kids = sorted(canon(c, v) for c in nb[v] if c != p)
        aut = 1
        for c in kids:
            aut *= c[1]
        for s in set(c[0] for c in kids):
            aut *= math.factorial(sum(c[0] == s for c in kids))
        return ("(" + "".join(c[0] for c in kids) + ")", aut)

    del ch
    rooted = [canon(v, -1) for v in range(len(t))]
    alpha = rooted[0][1] * sum(r[0] == rooted[0][0] for r in rooted)
    p = math.factorial(k) / math.factorial(k - len(t)) / k ** len(t)
    return 1.0 / (p * alpha)


def exact(case, seed):
    kind, mode, n = case["kind"], case["mode"], case["n"]
    ts = trees_of(case)
    w64 = work(case)
    if mode == "u64" or kind == "estimate" or w64["flops"] > 6e11:
        return None  # whole numbers; thousands of colourings; too long in 64 bits
    row_ptr, col_idx, w = make_graph(case, seed)
    w = torch.ones(col_idx.numel(), dtype=torch.float64, device=DEV) if w is None else w.double()
    grads = kind in ("grad", "train")
    w.requires_grad_(grads)
    unit = 2.0 ** (-10 * max(len(t) for t in ts)) if mode == "fp32s" else 1.0
    f = torch.zeros(len(ts), case["colorings"], dtype=torch.float64)
    gc = np.linspace(1.0, 2.0, case["colorings"]) if kind == "grad" else np.full(case["colorings"], 2.0 ** (-10 * len(ts[0])))
    grad = torch.zeros_like(w) if grads else None
    for j in range(case["colorings"]):
        by_k = {}
        for r, t in enumerate(ts):
            k = case["k"] or len(t)
            if k not in by_k:
                by_k[k] = (torch.as_tensor(_colours(n, k, seed, j), device=DEV), {}, {})
            with torch.set_grad_enabled(grads):
                x = _dp(t, k, by_k[k][0], w, row_ptr, col_idx, by_k[k][1], by_k[k][2])
            f[r, j] = float(x)
            if grads:
                grad += torch.autograd.grad(x, w)[0] * gc[j]
    est = torch.stack([f[r] * _scale(t, case["k"] or len(t)) for r, t in enumerate(ts)])
    if kind == "batch":
        return {"colorful": f * unit, "estimate": est * unit}
    if kind == "multi":
        return {"colorful": f * unit, "frequency": est.mean(1) / est.mean(1).sum()}
    if kind == "grad":
        return {"grad": grad * unit}
    if kind == "train":
        return {"colorful": f[0] * unit, "grad": grad}
    return {"colorful": f[0] * unit, "estimate": est[0] * unit}

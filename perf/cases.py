"""The work this library is timed on, through its public Python entry points.

Every case is one call a program makes on graphs it already holds: a
minimum spanning forest (``Context.solve``) of one graph on the device or in
host memory, of a batch of graphs (``Context.solve_batched``), a burst of
requests to the server (``Server``), the multilinear kernel and connected
components on a kept graph (``Graph``).  The families and sizes are those of
the repository's benchmark and tests: Erdos-Renyi, R-MAT (0.57, 0.19, 0.19,
0.05) and 3D grids with 5% of the edges dropped; weights uint32 over the whole
range, float32 k * 2^-24 in (0, 1), or small integers 1..255 with many ties
(the usual weights of unweighted graphs).

Inputs are made on the GPU from the seed alone.  ``exact`` computes the same
answers with plain torch in 64 bits (Boruvka's rounds by scatter minima).
"""
import math

import numpy as np
import torch

import paper_2110_04865_amd as msf

DEV = "cuda:0"
BIG = (1 << 63) - 1


# ------------------------------------------------------------------ cases --

def listed():
    return [
        # the smallest calls: a graph of a few hundred edges, where the launch
        # and the host round trip are all there is
        dict(name="solve_tiny_er", kind="solve", family="er", n=100, m=400, w="u32", mem="dev"),
        # the small benchmark graph: one solve of 32K edges
        dict(name="solve_er_4096", kind="solve", family="er", n=4096, m=32768, w="u32",
             mem="dev"),
        # a medium skewed graph (social-network-like), resident on the device
        dict(name="solve_rmat_16", kind="solve", family="rmat", scale=16, ef=16, w="f32",
             mem="dev"),
        # a medium sparse graph of high diameter (road-network-like)
        dict(name="solve_grid_101", kind="solve", family="grid", side=101, w="u32", mem="dev"),
        # a program that holds its graph in host memory, small integer weights
        dict(name="solve_host_rmat_18", kind="solve", family="rmat", scale=18, ef=16, w="i255",
             mem="host"),
        # the headline graph: R-MAT scale 22, edge factor 16, float32
        dict(name="solve_rmat_22", kind="solve", family="rmat", scale=22, ef=16, w="f32",
             mem="dev"),
        # the large sparse graph of high diameter: 256^3 grid, uint32
        dict(name="solve_grid_256", kind="solve", family="grid", side=256, w="u32", mem="dev"),
        # the large batch: 10^4 graphs of 64 to 65536 vertices, 4 edges each
        dict(name="batch_10000", kind="batch", graphs=10000, lo=64, hi=65536, deg=4, w="u32",
             mem="dev"),
        # a batch of small float graphs
        dict(name="batch_small_f32", kind="batch", graphs=1500, lo=16, hi=3000, deg=4, w="f32",
             mem="dev"),
        # the multilinear kernel alone, parents as after the first round
        dict(name="multilinear_rmat_22", kind="multilinear", family="rmat", scale=22, ef=16,
             w="f32"),
        # connected components of a kept graph
        dict(name="components_rmat_20", kind="components", family="rmat", scale=20, ef=16,
             w="u32"),
        # a burst of mixed requests to the server, host arrays in and out
        dict(name="serve_pool_32", kind="serve", graphs=32, lo=10, hi=18, w="f32"),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _family(rng, top):
    """A graph of a random family and size, at most about `top` edges."""
    f = rng.choice(["er", "rmat", "grid"])
    if f == "er":
        n = _log(rng, 50, top // 8)
        return dict(family="er", n=n, m=int(n * rng.uniform(1.0, 8.0)) + 1)
    if f == "rmat":
        ef = rng.choice([8, 16])
        hi = int(math.log2(top / ef))
        return dict(family="rmat", scale=rng.randint(8, hi), ef=ef)
    return dict(family="grid", side=_log(rng, 5, int((top / 2.85) ** (1 / 3))))


def draw(rng):
    w = rng.choice(["u32", "f32", "i255"])
    kind = rng.choices(["solve", "host", "batch", "multilinear", "components", "serve"],
                       [8, 2, 4, 1, 1, 1])[0]
    if kind == "solve":
        return dict(kind="solve", w=w, mem="dev", **_family(rng, 1 << 26))
    if kind == "host":
        return dict(kind="solve", w=w, mem="host", **_family(rng, 1 << 22))
    if kind == "batch":
        hi = _log(rng, 100, 65536)
        graphs = _log(rng, 16, min(20000, (1 << 27) // hi))
        return dict(kind="batch", graphs=graphs, lo=rng.randint(2, 64), hi=hi,
                    deg=rng.randint(2, 8), w=w, mem=rng.choice(["dev", "dev", "host"])
                    if graphs * hi < (1 << 22) else "dev")
    if kind == "serve":
        return dict(kind="serve", graphs=rng.randint(4, 48), lo=rng.randint(8, 11),
                    hi=rng.randint(14, 17), w=w)
    return dict(kind=kind, w=w, **_family(rng, 1 << 25))


# ----------------------------------------------------------------- inputs --

_CTX = None


def _ctx():
    """The program's one context (it caches workspace between calls)."""
    global _CTX
    if _CTX is None:
        torch.cuda.set_device(0)
        _CTX = msf.Context(0)
    return _CTX


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weights(g, m, w):
    """(weights as a 32-bit device tensor, library weight type)"""
    if w == "f32":
        k = torch.randint(1, 1 << 24, (m,), generator=g, device=DEV, dtype=torch.int32)
        return k.to(torch.float32) * 2.0 ** -24, msf.W_F32
    if w == "i255":
        return torch.randint(1, 256, (m,), generator=g, device=DEV, dtype=torch.int32), msf.W_U32
    return torch.randint(-(1 << 31), 1 << 31, (m,), generator=g, device=DEV,
                         dtype=torch.int64).to(torch.int32), msf.W_U32


def _er(g, n, m):
    u = torch.randint(0, n, (m,), generator=g, device=DEV, dtype=torch.int32)
    v = torch.randint(0, n - 1, (m,), generator=g, device=DEV, dtype=torch.int32)
    v += (v >= u).to(torch.int32)
    return torch.stack([torch.minimum(u, v), torch.maximum(u, v)], 1)


def _rmat(g, scale, ef):
    """(min, max) pairs, sorted and unique, vertex ids relabelled at random."""
    n, draws = 1 << scale, ef << scale
    u = torch.zeros(draws, dtype=torch.int32, device=DEV)
    v = torch.zeros(draws, dtype=torch.int32, device=DEV)
    for _ in range(scale):
        x = torch.rand(draws, generator=g, device=DEV)
        u = 2 * u + (x >= 0.76).to(torch.int32)
        v = 2 * v + (((x >= 0.57) & (x < 0.76)) | (x >= 0.95)).to(torch.int32)
    perm = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
    u, v = perm[u.long()], perm[v.long()]
    key = torch.minimum(u, v).long() * n + torch.maximum(u, v)
    key = torch.unique(key[u != v])
    return torch.stack([(key >> scale).to(torch.int32), (key & (n - 1)).to(torch.int32)], 1)


def _grid(g, side):
    """Edges per vertex in id order (+x, +y, +z), 5% dropped."""
    v = torch.arange(side ** 3, device=DEV, dtype=torch.int32)
    x, y, z = v % side, v // side % side, v // (side * side)
    step = torch.tensor([1, side, side * side], device=DEV, dtype=torch.int32)
    e = torch.stack([v[:, None].expand(-1, 3), v[:, None] + step], 2)
    ok = torch.stack([x, y, z], 1) < side - 1
    ok &= torch.rand(ok.shape, generator=g, device=DEV) >= 0.05
    return e[ok]


def _graph(case, seed):
    """(n, edges [m, 2] int32, weights, library weight type) on the device"""
    g = _gen(seed)
    if case["family"] == "er":
        n, e = case["n"], _er(g, case["n"], case["m"])
    elif case["family"] == "rmat":
        n, e = 1 << case["scale"], _rmat(g, case["scale"], case["ef"])
    else:
        n, e = case["side"] ** 3, _grid(g, case["side"])
    w, wt = _weights(g, len(e), case["w"])
    return n, e.contiguous(), w, wt


def _batch_sizes(case):
    """Vertices per graph, log-uniform, and the offsets (the same for every seed)."""
    rng = np.random.RandomState(case["graphs"])
    n = np.floor(case["lo"] * (case["hi"] / case["lo"]) ** rng.rand(case["graphs"]))
    n = n.astype(np.int64)
    vo = np.concatenate([[0], np.cumsum(n)])
    return n, vo, vo * case["deg"]


def _batch(case, seed):
    """(vertex and edge offsets, local edges, weights, library weight type)"""
    n, vo, eo = _batch_sizes(case)
    g = _gen(seed)
    M = int(eo[-1])
    e = torch.empty((M, 2), dtype=torch.int32, device=DEV)
    ng = torch.from_numpy(n).to(DEV)
    of = torch.repeat_interleave(torch.arange(len(n), device=DEV, dtype=torch.int32),
                                 ng * case["deg"])
    nf = ng.to(torch.float64)
    step = 1 << 25
    for a in range(0, M, step):  # in pieces, to keep the temporaries small
        b = min(M, a + step)
        k = nf[of[a:b].long()]
        u = (torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64) * k).long()
        v = (torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64) * (k - 1)).long()
        v += v >= u
        e[a:b, 0] = torch.minimum(u, v)
        e[a:b, 1] = torch.maximum(u, v)
    w, wt = _weights(g, M, case["w"])
    return vo, eo, e, w, wt


def _pool(case, seed):
    """The requests of a serve case: R-MAT and grid graphs in turn, host arrays."""
    rng = np.random.RandomState(case["graphs"])  # sizes: the same for every seed
    out = []
    for k in range(case["graphs"]):
        lg = case["lo"] + (case["hi"] - case["lo"]) * rng.rand()
        if k % 2 == 0:
            c = dict(family="rmat", scale=int(round(lg)), ef=16, w=case["w"])
        else:
            c = dict(family="grid", side=max(2, int(round(2 ** (lg / 3)))), w=case["w"])
        n, e, w, wt = _graph(c, seed * 64 + k)
        out.append((n, e.cpu().numpy(), _host_w(w, wt), wt))
    return out


def _host_w(w, wt):
    a = w.cpu().numpy()
    return a.view(np.uint32) if wt == msf.W_U32 else a


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        pool = _pool(case, seed)
        return dict(kind=kind, pool=pool, server=msf.Server(_ctx(), 32 << 30),
                    out=[np.full(r[0] - 1, -1, np.int32) for r in pool])
    if kind == "batch":
        vo, eo, e, w, wt = _batch(case, seed)
        if case["mem"] == "host":
            return dict(kind=kind, vo=vo, eo=eo, e=e.cpu().numpy(), w=_host_w(w, wt), wt=wt,
                        out=None)
        return dict(kind=kind, vo=vo, eo=eo, e=e, w=w, wt=wt,
                    out=torch.empty(int(vo[-1]), dtype=torch.int32, device=DEV))
    n, e, w, wt = _graph(case, seed)
    if kind == "solve":
        if case["mem"] == "host":
            return dict(kind=kind, n=n, e=e.cpu().numpy(), w=_host_w(w, wt), wt=wt,
                        out=np.full(n - 1, -1, np.int32))
        return dict(kind=kind, n=n, e=e, w=w, wt=wt,
                    out=torch.full((n - 1,), -1, dtype=torch.int32, device=DEV))
    graph = msf.Graph(_ctx(), n, e, w, wtype=wt)
    if kind == "multilinear":
        p = _round1_parents(n, e, _order_key(w, wt))
        return dict(kind=kind, g=graph, p=p.to(torch.int32),
                    r=torch.empty(n, dtype=torch.int64, device=DEV))
    return dict(kind=kind, g=graph, labels=torch.empty(n, dtype=torch.int32, device=DEV))


def _unused(ids, vo, counts):
    """-1 in the slots past each graph's forest (the call leaves them as they
    were), so that the whole array is defined."""
    free = vo[1:] - vo[:-1] - counts
    at = np.repeat(vo[:-1] + counts, free)
    at += np.arange(len(at)) - np.repeat(np.cumsum(free) - free, free)
    ids[torch.from_numpy(at).to(DEV) if torch.is_tensor(ids) else at] = -1
    return ids


# -------------------------------------------------------------------- run --

def run(state):
    c, kind = _ctx(), state["kind"]
    if kind == "solve":
        out = state["out"]
        if torch.is_tensor(out):
            _, count, total = c.solve(state["n"], state["e"], state["w"], wtype=state["wt"],
                                      out=out)
        else:
            ids, count, total = c.solve(state["n"], state["e"], state["w"], wtype=state["wt"])
            out[:count] = ids
        return dict(ids=out, count=count, u64=total[0], f64=total[1])
    if kind == "batch":
        ids, counts, totals = c.solve_batched(state["vo"], state["eo"], state["e"], state["w"],
                                              wtype=state["wt"], out=state["out"])
        return dict(ids=_unused(ids, state["vo"], counts), counts=counts,
                    f64=totals._a["f64"])
    if kind == "serve":
        s = state["server"]
        tickets = [s.submit(n, e, w, wtype=wt) for n, e, w, wt in state["pool"]]
        f64 = []
        for t, r, out in zip(tickets, state["pool"], state["out"]):
            ids, count, total = s.result(t, r[0])
            out[:count] = ids
            f64.append(total[1])
        return dict(ids=state["out"], f64=np.array(f64))
    if kind == "multilinear":
        c.multilinear(state["g"], state["p"], state["r"])
        return state["r"]
    c.components(state["g"], state["labels"])
    return state["labels"]


# ------------------------------------------------------------------- work --

def _size(case):
    """(vertices, edges) of a single graph, edges to within a few percent."""
    if case["family"] == "er":
        return case["n"], case["m"]
    if case["family"] == "rmat":  # loops and duplicates dropped
        return 1 << case["scale"], int(0.93 * (case["ef"] << case["scale"]))
    s = case["side"]
    return s ** 3, int(0.95 * 3 * s * s * (s - 1))


def work(case):
    """Bytes of the inputs read once and the outputs written once: 12 per edge
    (endpoints and weight) and 4 per forest edge; a kept graph's entries are
    its adjacency matrix's (column 4, key 8; both directions)."""
    kind = case["kind"]
    if kind == "batch":
        lo, hi = case["lo"], case["hi"]
        n = case["graphs"] * (hi - lo) / math.log(hi / lo)
        return dict(bytes=12 * case["deg"] * n + 4 * n, flops=0)
    if kind == "serve":
        b = 0
        for k in range(case["graphs"]):
            s = (case["lo"] + case["hi"]) / 2
            b += 2 ** s * (12 * (15 if k % 2 == 0 else 2.8) + 4)
        return dict(bytes=b, flops=0)
    n, m = _size(case)
    if kind == "multilinear":
        return dict(bytes=24 * m + 16 * n, flops=0)
    if kind == "components":
        return dict(bytes=8 * m + 8 * n, flops=0)
    return dict(bytes=12 * m + 4 * n, flops=0)


# ------------------------------------------------------------------ exact --

def _order_key(w, wt):
    """The weights as int64 whose order is the weights' order (w >= 0)."""
    x = w.view(torch.int32).long()
    return x if wt == msf.W_F32 else x & 0xFFFFFFFF


def _minima(n, a, b, key):
    r = torch.full((n,), BIG, dtype=torch.int64, device=DEV)
    r.scatter_reduce_(0, a, key, "amin")
    return r.scatter_reduce_(0, b, key, "amin")


def _hook(r, a0, b0, comp):
    """Parents after every root hooked along its minimum edge (the smaller
    root of a mutual pair stays), trees shortcut; and the edges used."""
    n = len(r)
    root = (r < BIG).nonzero()[:, 0]
    e = r[root] & 0x7FFFFFFF
    a, b = comp[a0[e].long()], comp[b0[e].long()]
    p = torch.arange(n, device=DEV)
    p[root] = torch.where(a == root, b, a)
    stay = (p[p[root]] == root) & (root < p[root])
    p[root[stay]] = root[stay]
    used = e[~stay]
    while True:
        q = p[p]
        if torch.equal(q, p):
            return p, used
        p = q


def _round1_parents(n, e, wkey):
    """Every vertex's root after the first round: hooks along the minimum
    incident edges, then complete shortcutting."""
    key = (wkey << 31) | torch.arange(len(e), device=DEV)
    comp = torch.arange(n, device=DEV)
    r = _minima(n, e[:, 0].long(), e[:, 1].long(), key)
    return _hook(r, e[:, 0], e[:, 1], comp)[0]


def _forest(n, e, w, wt):
    """Ascending ids of the minimum spanning forest under (weight, edge id)."""
    a0, b0 = e[:, 0], e[:, 1]
    key = (_order_key(w, wt) << 31) | torch.arange(len(e), device=DEV)
    a, b = a0.long(), b0.long()
    comp = torch.arange(n, device=DEV)
    ids = [key[:0]]
    while len(key):
        p, used = _hook(_minima(n, a, b, key), a0, b0, comp)
        ids.append(used)
        comp = p[comp]
        a, b = p[a], p[b]
        live = a != b
        a, b, key = a[live], b[live], key[live]
    return torch.sort(torch.cat(ids))[0]


def _total(w, wt, ids):
    x = w[ids]
    return int(_order_key(x, wt).sum()) if wt == msf.W_U32 else 0, \
        float(_order_key(x, wt).sum() if wt == msf.W_U32 else x.double().sum())


def _padded(n, ids):
    out = torch.full((n - 1,), -1, dtype=torch.int32, device=DEV)
    out[:len(ids)] = ids.to(torch.int32)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "components":
        return None  # which vertex of a component is its label is not defined
    if kind == "serve":
        pool, ids, tot = _pool(case, seed), [], []
        for n, e, w, wt in pool:
            e = torch.from_numpy(e).to(DEV)
            w = torch.from_numpy(w.view(np.int32) if wt == msf.W_U32 else w).to(DEV)
            i = _forest(n, e, w, wt)
            ids.append(_padded(n, i).cpu().numpy())
            tot.append(_total(w, wt, i)[1])
        return dict(ids=ids, f64=np.array(tot))
    if kind == "batch":
        if case["graphs"] * case["hi"] > 1 << 28:
            return None  # the disjoint union takes too long
        vo, eo, e, w, wt = _batch(case, seed)
        of = torch.repeat_interleave(torch.arange(len(vo) - 1, device=DEV),
                                     torch.from_numpy(eo[1:] - eo[:-1]).to(DEV))
        dv, de = torch.from_numpy(vo).to(DEV), torch.from_numpy(eo).to(DEV)
        ids = _forest(int(vo[-1]), e + dv[of][:, None].to(torch.int32), w, wt)
        g = of[ids]
        counts = torch.bincount(g, minlength=len(vo) - 1)
        first = torch.cumsum(counts, 0) - counts
        out = torch.full((int(vo[-1]),), -1, dtype=torch.int32, device=DEV)
        out[dv[g] + torch.arange(len(ids), device=DEV) - first[g]] = \
            (ids - de[g]).to(torch.int32)
        x = w[ids].double() if wt == msf.W_F32 else _order_key(w[ids], wt)
        f = torch.zeros(len(counts), dtype=x.dtype, device=DEV).index_add_(0, g, x).double()
        return dict(ids=out, counts=counts.cpu().numpy(), f64=f.cpu().numpy())
    n, e, w, wt = _graph(case, seed)
    if kind == "multilinear":
        key, p = _order_key(w, wt), _round1_parents(n, e, _order_key(w, wt))
        if wt == msf.W_F32:
            key |= 1 << 31  # the key of a non-negative float has the sign bit set
        key = ((key - (1 << 31)) << 32) | torch.arange(len(e), device=DEV)
        a, b = p[e[:, 0].long()], p[e[:, 1].long()]
        live = a != b
        r = _minima(n, a[live], b[live], key[live])
        return r ^ (-1 << 63)
    ids = _forest(n, e, w, wt)
    u, f = _total(w, wt, ids)
    return dict(ids=_padded(n, ids), count=len(ids), u64=u, f64=f)

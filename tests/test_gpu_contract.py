"""Rounds over a contracted edge list (msf_solve's default above one
workgroup's size) against the oracle: bit-exact ids, count and totals."""
import math
import os

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U32, F32 = oracle.W_U32, oracle.W_F32


@pytest.fixture(scope="module")
def pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_04865_amd as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def ctx(pkg):
    """Every solve through the contracted rounds, whatever its size."""
    old = {k: os.environ.get(k) for k in ("MSF_CONTRACT", "MSF_SMALL_M")}
    os.environ.update(MSF_CONTRACT="2", MSF_SMALL_M="0")
    try:
        c = pkg.Context(0)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    yield c
    c.close()


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(a.reshape(-1).copy()).to("cuda:0")


def check(c, n, e, w, wt, label, path=4):
    print("[gpu-case]", label, f"n={n} m={len(e)} wt={wt}", flush=True)
    want_ids, want_cnt, want_tot = oracle.msf(n, e, w, wt)
    ids, cnt, tot = c.solve(n, dev(e), dev(w), wtype=wt)
    torch.cuda.synchronize()
    assert cnt == want_cnt, label
    assert np.array_equal(ids.cpu().numpy().astype(np.int64), want_ids), label
    assert wt == F32 or tot[0] == want_tot[0], label
    assert tot[1] == want_tot[1] or (math.isnan(tot[1]) and math.isnan(want_tot[1])), label
    st = c.stats()
    assert st["path"] == path, (label, st["path"])
    assert sum(st["hooks"]) == cnt, label  # every kept hook is one forest edge
    return st


def path_graph(n, w):
    e = np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    return n, e, np.asarray(w, np.uint32)


def ruler(n):
    """Path whose trees only double every round: weight ctz(i + 1)."""
    i = np.arange(1, n)
    return path_graph(n, np.log2((i & -i).astype(np.float64)).astype(np.uint32))


# vertices around powers of two near the sizes where one workgroup finishes a
# round (2048) and minima move to LDS (7680); edges around a wave's tile (256)
# and a sweep of every wave over one tile
@pytest.mark.parametrize("n,m", [(2, 1), (3, 255), (60, 256), (300, 257), (2047, 9000),
                                 (2049, 6000), (4096, 4095), (4097, 40000), (8191, 30000),
                                 (8192, 30000), (8193, 30000), (16385, 20000),
                                 (70001, 200003), (33000, 900001)])
def test_random_multigraphs(ctx, n, m):
    rng = np.random.default_rng(n + m)
    e = rng.integers(0, n, size=(m, 2)).astype(np.int32)  # loops and parallel edges among them
    check(ctx, n, e, rng.integers(0, 1 << 32, size=m, dtype=np.uint64).astype(np.uint32), U32,
          "u32")
    check(ctx, n, e, rng.integers(0, 3, size=m).astype(np.uint32), U32, "three weights")
    w = rng.standard_normal(m).astype(np.float32)
    w[::7] = -0.0
    w[1::7] = 0.0
    if m > 1000:
        w[5] = np.inf
    check(ctx, n, e, w, F32, "f32")


def test_shapes(ctx):
    rng = np.random.default_rng(5)
    n = 30000
    star = np.stack([np.zeros(n - 1), np.arange(1, n)], 1).astype(np.int32)
    check(ctx, n, star, np.full(n - 1, 9, np.uint32), U32, "star, equal weights")
    check(ctx, *path_graph(n, np.arange(n - 1, 0, -1)), U32, "path, one long chain of hooks")
    check(ctx, *path_graph(n, np.full(n - 1, 4)), U32, "path, equal weights")
    e = np.zeros((5, 2), np.int32)
    check(ctx, 4, e, np.arange(5).astype(np.uint32), U32, "loops only")
    e = np.array([[0, 1], [2999999, 5]], np.int32)
    check(ctx, 3000000, e, np.array([2, 1], np.uint32), U32, "isolated vertices")
    # weights in the order of the edges, and equal ones: the light edges are
    # then a stretch of the input
    e, _ = gen.er(20000, 200000, seed=3)
    check(ctx, 20000, e, np.arange(200000).astype(np.uint32), U32, "sorted weights")
    check(ctx, 20000, e, np.arange(200000, 0, -1).astype(np.uint32), U32, "falling weights")
    check(ctx, 20000, e, np.ones(200000, np.uint32), U32, "equal weights")


def test_more_rounds_than_enqueued(ctx):
    """Trees that only double every round need more rounds than a round's
    usual shrinking suggests: the solve goes on from the first open round, in
    the first phase and (with parallel heavier edges) where two phases run."""
    n, e, w = ruler(1 << 17)
    st = check(ctx, n, e, w, U32, "ruler path")
    assert st["hook_rounds"] == 17 and st["hooks"][:2] == [1 << 16, 1 << 15], st
    e4 = np.concatenate([e, e, e, e])
    w4 = np.concatenate([w, w + 40, w + 50, w + 60]).astype(np.uint32)
    check(ctx, n, e4, w4, U32, "ruler path with parallel edges")
    # light edges that leave the ruler to the second phase
    loops = np.stack([np.arange(n), np.arange(n)], 1).astype(np.int32)
    e5 = np.concatenate([loops, loops, loops, e])
    w5 = np.concatenate([np.zeros(3 * n), w + 100]).astype(np.uint32)
    check(ctx, n, e5, w5, U32, "ruler path among light loops")


@pytest.mark.parametrize("label", ["rmat14", "rmat17", "grid24", "grid 12, 40% dropped",
                                   "many vertices"])
def test_families(ctx, label):
    if label.startswith("rmat"):
        n, e, w = gen.rmat(int(label[4:]), 16, seed=7)
        check(ctx, n, e, w, F32, label)
    elif label == "many vertices":  # lookups through the bits of the largest tree
        n = (1 << 20) + 77
        e, w = gen.er(n, 3 * n, seed=8)
        check(ctx, n, e, w, U32, label)
    else:
        s, drop = (24, 0.05) if label == "grid24" else (12, 0.4)
        n, e, w = gen.grid(s, s, s, drop, seed=9)
        check(ctx, n, e, w, U32, label)


def test_default_route_and_bad_input(pkg):
    """A default context takes this path above 2^17 edges; bad input ends
    with MSF_EINVAL, the output untouched and the context still solving."""
    c = pkg.Context(0)
    n, m = 40000, (1 << 17) + 1
    e, w = gen.er(n, m, seed=11)
    check(c, n, e, w, U32, "default route")
    wf = gen.weights(m, gen.W_F32, seed=12)
    out = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    for what in ("endpoint", "negative", "nan"):
        be, bw = e.copy(), wf.copy()
        if what == "endpoint":
            be[m - 1, 1] = n
        elif what == "negative":
            be[m // 2, 0] = -1
        else:
            bw[m // 3] = np.nan
        with pytest.raises(pkg.MSFError) as ex:
            c.solve(n, dev(be), dev(bw), wtype=F32, out=out)
        assert ex.value.status == 1, what
        torch.cuda.synchronize()
        assert bool((out == -7).all()), what
        check(c, n, e, wf, F32, "valid after " + what)
    c.close()


@pytest.mark.parametrize("n,m", [(9000, 1 << 19), (9000, (1 << 19) + 1), (200, (1 << 19) + 1),
                                 (240000, (1 << 19) + 1), (7680, 600000), (7681, 600000),
                                 (2048, 600000), (2049, 600000)])
def test_one_or_two_phases(ctx, n, m):
    """One phase up to 2^19 edges, light edges first above (with more than
    two edges a light one); vertices around the sizes where one workgroup
    finishes a round."""
    rng = np.random.default_rng(n + m)
    e = rng.integers(0, n, size=(m, 2)).astype(np.int32)
    check(ctx, n, e, rng.integers(0, 1 << 32, size=m, dtype=np.uint64).astype(np.uint32), U32,
          "phases, u32")
    check(ctx, n, e, rng.integers(0, 3, size=m).astype(np.uint32), U32, "phases, three weights")


def test_more_rounds_than_enqueued_two_phases(ctx):
    """The ruler path above the line: in the first phase, and left to the
    second one by lighter loops."""
    n, e, w = ruler(1 << 17)
    e6 = np.concatenate([e] * 6)
    w6 = np.concatenate([w] + [w + 40 + 10 * k for k in range(5)]).astype(np.uint32)
    check(ctx, n, e6, w6, U32, "ruler path with five parallel edges each")
    loops = np.stack([np.arange(n), np.arange(n)], 1).astype(np.int32)
    e7 = np.concatenate([loops] * 5 + [e])
    w7 = np.concatenate([np.zeros(5 * n), w + 100]).astype(np.uint32)
    check(ctx, n, e7, w7, U32, "ruler path among many light loops")


@pytest.mark.parametrize("n,m", [(2, 1), (40, 2048), (40, 2049), (3248, 2048), (3249, 2048),
                                 (500, 4096), (500, 4097), (6499, 4096), (6500, 4096),
                                 (900, 8193), (130, 20000), (129, 60000)])
def test_edges_in_registers(pkg, n, m):
    """One-workgroup solves and batches around the sizes whose edges and
    state fit the registers and LDS of 256, 512 and 1024 threads."""
    c = pkg.Context(0)
    rng = np.random.default_rng(n * 7 + m)
    e = rng.integers(0, n, size=(m, 2)).astype(np.int32)
    wu = rng.integers(0, 5, size=m).astype(np.uint32)
    wf = rng.standard_normal(m).astype(np.float32)
    wf[::9] = -0.0
    check(c, n, e, wu, U32, "registers, ties", path=1)
    check(c, n, e, wf, F32, "registers, f32", path=1)
    # the same graph between a smaller one and one without edges
    vo, eo = np.array([0, 2, 2 + n, 5 + n]), np.array([0, 1, 1 + m, 1 + m])
    eb = np.concatenate([np.array([[0, 1]], np.int32), e])
    for w, wt in ((wu, U32), (wf, F32)):
        want, cnt, tot = oracle.msf(n, e, w, wt)
        wb = np.concatenate([w[:1], w])
        ids, counts, totals = c.solve_batched(vo, eo, dev(eb), dev(wb), wtype=wt)
        torch.cuda.synchronize()
        assert list(counts) == [1, cnt, 0]
        assert np.array_equal(ids.cpu().numpy()[2:2 + cnt].astype(np.int64), want)
        assert totals[1][1] == tot[1]
    c.close()


@pytest.mark.parametrize("n,m,path", [(1000, 66000, 1), (1000, 66001, 4), (22000, 24000, 1),
                                      (22000, 24001, 4), (33999, 2, 1), (34000, 1, 4)])
def test_one_workgroup_line(pkg, n, m, path):
    """A default context solves up to 68000 = edges + 2 * vertices in one
    workgroup, and one more by the contracted rounds."""
    c = pkg.Context(0)
    rng = np.random.default_rng(n + m)
    e = rng.integers(0, n, size=(m, 2)).astype(np.int32)
    check(c, n, e, rng.integers(0, 50, size=m).astype(np.uint32), U32, "line, ties", path=path)
    check(c, n, e, rng.standard_normal(m).astype(np.float32), F32, "line, f32", path=path)
    c.close()


def test_refused_allocations(pkg):
    """Every workspace allocation of the path refused in turn: MSF_ENOMEM,
    the output untouched, and the next solve right."""
    n, e, w = gen.rmat(13, 16, seed=13)
    want_ids, want_cnt, _ = oracle.msf(n, e, w, F32)
    de, dw = dev(e), dev(w)
    for k in range(40):
        keys = dict(MSF_CONTRACT="2", MSF_SMALL_M="0", MSF_TEST_FAIL_ALLOC_AFTER=str(k))
        old = {q: os.environ.get(q) for q in keys}
        os.environ.update(keys)
        try:
            c = pkg.Context(0)
        finally:
            for q, v in old.items():
                if v is None:
                    os.environ.pop(q, None)
                else:
                    os.environ[q] = v
        out = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
        failed = False
        try:
            c.solve(n, de, dw, wtype=F32, out=out)
        except pkg.MSFError as ex:
            assert ex.status == 2
            failed = True
        torch.cuda.synchronize()
        if failed:
            assert bool((out == -7).all()), k
        ids, cnt, _ = c.solve(n, de, dw, wtype=F32)
        torch.cuda.synchronize()
        assert cnt == want_cnt and np.array_equal(ids.cpu().numpy().astype(np.int64), want_ids), k
        c.close()
        if not failed:
            break
    assert 5 <= k < 39


# vertices where the pair matrix starts (32, 64, 128), where a round's minima
# and map stop fitting 32 / 64 / 150 KB of LDS (bytes / 10), where minima take
# a second range (bytes / 8) and where vertex numbers outgrow 16 bits; edges
# around two per vertex and the size from which light edges go first
BATCH_SIZES = [(0, 0), (1, 0), (2, 1), (31, 90), (33, 200), (64, 300), (65, 300), (128, 900),
               (129, 900), (511, 2047), (512, 2048), (512, 2049), (1024, 2048), (1025, 2049),
               (3275, 4096), (3276, 4097), (3277, 20000), (4095, 16385), (4097, 9000),
               (6552, 30000), (6553, 30000), (8193, 40000), (15358, 70000), (15359, 31000),
               (19199, 60000), (19201, 60000), (38401, 90000), (65536, 180000),
               (65537, 180000), (76801, 80000), (76801, 190000)]


@pytest.mark.parametrize("config", [0, 2, 3, 6, 7])
def test_batched_sizes(pkg, config):
    rng = np.random.default_rng(17)
    graphs = [rng.integers(0, max(n, 1), size=(m, 2)).astype(np.int32) for n, m in BATCH_SIZES]
    vo = np.cumsum([0] + [n for n, _ in BATCH_SIZES]).astype(np.int64)
    eo = np.cumsum([0] + [m for _, m in BATCH_SIZES]).astype(np.int64)
    e = np.concatenate(graphs)
    wide = rng.integers(0, 1 << 32, size=len(e), dtype=np.uint64).astype(np.uint32)
    ties = rng.integers(0, 3, size=len(e)).astype(np.uint32)
    f = rng.standard_normal(len(e)).astype(np.float32)
    c = pkg.Context(0)
    old = os.environ.get("MSF_BATCH_CONFIG")
    os.environ["MSF_BATCH_CONFIG"] = str(config)
    try:
        for w, wt, label in ((wide, U32, "wide"), (ties, U32, "ties"), (f, F32, "float")):
            print("[gpu-case] batched sizes", config, label, flush=True)
            ids, counts, totals = c.solve_batched(vo, eo, dev(e), dev(w), wtype=wt)
            torch.cuda.synchronize()
            ids = ids.cpu().numpy()
            for g, (n, m) in enumerate(BATCH_SIZES):
                wi, wc, wtot = oracle.msf(n, e[eo[g]:eo[g + 1]], w[eo[g]:eo[g + 1]], wt)
                assert counts[g] == wc, (label, n, m)
                assert np.array_equal(ids[vo[g]:vo[g] + wc].astype(np.int64), wi), (label, n, m)
                assert totals[g][1] == wtot[1], (label, n, m)
    finally:
        if old is None:
            os.environ.pop("MSF_BATCH_CONFIG", None)
        else:
            os.environ["MSF_BATCH_CONFIG"] = old
        c.close()


@pytest.mark.parametrize("before", ["large total", "refused"])
def test_batch_of_large_graphs_only(pkg, before):
    """A batch in which every graph is above the one-workgroup limits writes
    the caller's ids whatever the call before it left in the workspace: a
    total above 2^32 where the error word of two graphs lies, or a refused
    batch of as many graphs."""
    c = pkg.Context(0)
    if before == "large total":
        c.solve_batched(np.array([0, 3]), np.array([0, 2]), dev(np.array([[0, 1], [1, 2]], np.int32)),
                        dev(np.full(2, 0xFFFFFFF0, np.uint32)), wtype=U32)
    else:
        with pytest.raises(pkg.MSFError):
            c.solve_batched(np.array([0, 2, 4]), np.array([0, 1, 2]),
                            dev(np.array([[0, 1], [0, 2]], np.int32)),
                            dev(np.ones(2, np.uint32)), wtype=U32)
    rng = np.random.default_rng(29)
    n, m = (1 << 20) + 1, 3000
    e = rng.integers(0, n, size=(2 * m, 2)).astype(np.int32)
    w = rng.integers(0, 1000, size=2 * m).astype(np.uint32)
    out = torch.full((2 * n,), -7, dtype=torch.int32, device="cuda:0")
    ids, counts, totals = c.solve_batched(np.array([0, n, 2 * n]), np.array([0, m, 2 * m]), dev(e),
                                          dev(w), wtype=U32, out=out)
    torch.cuda.synchronize()
    assert c.stats()["batch_large"] == 2
    got = out.cpu().numpy().astype(np.int64)
    for g in range(2):
        want, cnt, tot = oracle.msf(n, e[g * m:(g + 1) * m], w[g * m:(g + 1) * m], U32)
        assert counts[g] == cnt and totals[g][0] == tot[0], g
        assert np.array_equal(got[g * n:g * n + cnt], want), g
    c.close()


def test_refused_multilinear_leaves_nothing_behind(pkg):
    """A multilinear call refused for its parents returns with nothing left
    on the stream (the caller may free them), and the statistics stay those
    of the last accepted call."""
    c = pkg.Context(0)
    e, w = gen.er(1000, 4000, seed=31)
    small, big_n = c.graph(1000, dev(e), dev(w), wtype=U32), 1 << 26
    be = (e.astype(np.int64) * 67000).astype(np.int32)  # few edges, many vertices
    big = c.graph(big_n, dev(be), dev(w), wtype=U32)
    p = torch.arange(big_n, dtype=torch.int32, device="cuda:0")
    r = torch.zeros(big_n, dtype=torch.int64, device="cuda:0")
    c.multilinear(big, p, r)
    bad = torch.full((1000,), 1000, dtype=torch.int32, device="cuda:0")
    r2 = torch.zeros(1000, dtype=torch.int64, device="cuda:0")
    with pytest.raises(pkg.MSFError):
        c.multilinear(small, bad, r2)
    st = c.stats()
    # the gather of the big call: 12 bytes a vertex, not above memory's peak
    assert st["pass_bytes"][0] == 12.0 * big_n
    assert st["pass_bytes"][0] <= st["pass_ms"][0] * 1e-3 * 8e12, st["pass_ms"]
    torch.cuda.synchronize()
    p[7] = big_n
    before = r.clone()
    torch.cuda.synchronize()
    with pytest.raises(pkg.MSFError, match="parent") as ex:
        c.multilinear(big, p, r)
    idle = torch.cuda.current_stream().query()
    assert idle and ex.value.status == 1
    torch.cuda.synchronize()
    assert torch.equal(r, before) and int(r2.abs().sum()) == 0
    c.close()


# hooks that all point along the path make one chain of its length; the last
# size gives a thread of the chase more than 64 vertices
@pytest.mark.parametrize("n", [1 << 21, 40 * 10 ** 6])
@pytest.mark.parametrize("falling", [False, True])
def test_long_chains(pkg, n, falling):
    """Paths with rising or falling weights: every edge is in the forest, and
    a chain of n hooks takes neither n steps nor n / 1000."""
    import time
    c = pkg.Context(0)
    i = torch.arange(n, dtype=torch.int32, device="cuda:0")
    e = torch.stack([i[:-1], i[1:]], 1).reshape(-1).contiguous()
    w = (i[:-1].flip(0) if falling else i[:-1]).contiguous()
    ids, cnt, tot = c.solve(n, e, w, wtype=U32)
    t0 = time.perf_counter()
    ids, cnt, tot = c.solve(n, e, w, wtype=U32)
    ms = (time.perf_counter() - t0) * 1e3
    assert cnt == n - 1 and torch.equal(ids[:cnt], i[:-1]) and tot[0] == (n - 1) * (n - 2) // 2
    assert c.stats()["path"] == 4
    assert ms < 50.0, ms  # (0.3 and 3 ms; a step per vertex and thread: 1 s and more)
    c.close()


@pytest.mark.parametrize("n", [6000, 20000, 22667])
@pytest.mark.parametrize("falling", [False, True])
def test_long_chains_in_one_workgroup(pkg, n, falling):
    """The same in one workgroup, alone and in a batch whose targets lie in
    LDS as 16-bit numbers and in device memory."""
    import time
    c = pkg.Context(0)

    def path(n):
        i = torch.arange(n, dtype=torch.int32, device="cuda:0")
        return (torch.stack([i[:-1], i[1:]], 1).reshape(-1).contiguous(),
                (i[:-1].flip(0) if falling else i[:-1]).contiguous(), i)

    e, w, i = path(n)
    c.solve(n, e, w, wtype=U32)
    t0 = time.perf_counter()
    ids, cnt, tot = c.solve(n, e, w, wtype=U32)
    ms = (time.perf_counter() - t0) * 1e3
    assert cnt == n - 1 and torch.equal(ids[:cnt], i[:-1]) and c.stats()["path"] == 1
    sizes = [n, 40000, 70000, 2]
    parts = [path(k) for k in sizes]
    vo, eo = np.cumsum([0] + sizes), np.cumsum([0] + [k - 1 for k in sizes])
    be, bw = torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
    os.environ["MSF_BATCH_CONFIG"] = "7"
    try:
        ids, counts, totals = c.solve_batched(vo, eo, be, bw, wtype=U32)
        t0 = time.perf_counter()
        ids, counts, totals = c.solve_batched(vo, eo, be, bw, wtype=U32)
        batch_ms = (time.perf_counter() - t0) * 1e3
    finally:
        os.environ.pop("MSF_BATCH_CONFIG")
    for g, k in enumerate(sizes):
        assert counts[g] == k - 1 and totals[g][0] == (k - 1) * (k - 2) // 2, k
        assert torch.equal(ids[vo[g]:vo[g] + k - 1], parts[g][2][:-1]), k
    if n >= 20000:  # (0.1 and 1.4 ms; a step per vertex and thread: 13 ms and more)
        assert ms < 5.0 and batch_ms < 20.0, (ms, batch_ms)
    c.close()


@pytest.mark.parametrize("config", [0, 2, 7])
def test_batched_equal_weights(pkg, config):
    """Where the threshold of a batch's light edges falls among equal
    weights, the edge decides: the same forests, and a graph of one weight
    takes no longer than one of many."""
    c = pkg.Context(0)
    rng = np.random.default_rng(37)
    sizes = [(512, 2048), (512, 2049), (1000, 4100), (3000, 20000), (20000, 70000), (70000, 300000)]
    e = np.concatenate([rng.integers(0, n, size=(m, 2)) for n, m in sizes]).astype(np.int32)
    vo = np.cumsum([0] + [n for n, _ in sizes])
    eo = np.cumsum([0] + [m for _, m in sizes])
    wide = rng.integers(0, 1 << 32, size=len(e), dtype=np.uint64).astype(np.uint32)
    os.environ["MSF_BATCH_CONFIG"] = str(config)
    try:
        for w, wt, label in ((np.full(len(e), 0xFFFFFFFF, np.uint32), U32, "largest"),
                             (np.zeros(len(e), np.uint32), U32, "zero"),
                             (np.where(wide & 1, wide, np.uint32(1 << 20)), U32, "half equal"),
                             (np.arange(len(e), dtype=np.uint32) // 5000, U32, "rising blocks"),
                             (np.full(len(e), -0.0, np.float32), F32, "float")):
            print("[gpu-case] equal weights", config, label, flush=True)
            ids, counts, totals = c.solve_batched(vo, eo, dev(e), dev(w), wtype=wt)
            torch.cuda.synchronize()
            ids = ids.cpu().numpy()
            for g, (n, m) in enumerate(sizes):
                wi, wc, wtot = oracle.msf(n, e[eo[g]:eo[g + 1]], w[eo[g]:eo[g + 1]], wt)
                assert counts[g] == wc and totals[g][1] == wtot[1], (label, n)
                assert np.array_equal(ids[vo[g]:vo[g] + wc].astype(np.int64), wi), (label, n)
        if config == 7:
            n, m, G = 40000, 160000, 200
            de = dev(np.tile(rng.integers(0, n, size=(m, 2)).astype(np.int32), (G, 1)))
            vo, eo = np.arange(G + 1) * n, np.arange(G + 1) * m
            ms = []
            for w in (rng.integers(0, 1 << 32, size=G * m, dtype=np.uint64).astype(np.uint32),
                      np.ones(G * m, np.uint32)):
                dw = dev(w)
                for _ in range(3):
                    c.solve_batched(vo, eo, de, dw, wtype=U32)
                ms.append(c.stats()["batch_ms"])
            assert ms[1] < 1.4 * ms[0], ms  # (0.9; 1.9 with every edge light)
    finally:
        os.environ.pop("MSF_BATCH_CONFIG")
        c.close()


TUNED_BATCH = """
import numpy as np, torch
import paper_2110_04865_amd as pkg
rng = np.random.default_rng(41)
n, m, G = 40000, 160000, 20
e = torch.from_numpy(rng.integers(0, n, size=2 * G * m).astype(np.int32)).to("cuda:0")
w = torch.from_numpy(rng.integers(0, 1 << 30, size=G * m).astype(np.int32)).to("cuda:0")
c = pkg.Context(0)
c.solve_batched(np.arange(G + 1) * n, np.arange(G + 1) * m, e, w, wtype=pkg.W_U32)
print("config", c.stats()["batch_config"], flush=True)
"""


def test_saved_choice_of_an_older_kernel(pkg, tmp_path):
    """The tuner passes over choices saved for an older form of the kernel
    (or for none) and keeps to those of its own."""
    import subprocess
    import sys
    path = tmp_path / "tune.txt"
    env = {k: v for k, v in os.environ.items() if k != "MSF_BATCH_CONFIG"}
    env.update(MSF_TUNE_CACHE=str(path),
               PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

    def run():
        out = subprocess.run([sys.executable, "-c", TUNED_BATCH], env=env, capture_output=True,
                             text=True, timeout=100)
        assert out.returncode == 0, out.stderr[-2000:]
        return int(out.stdout.split("config")[1])

    shape = "15 3 0"  # log2 of 40000 vertices and of 8 entries each, uint32
    path.write_text(f"gfx950 {shape} 0\ngfx950/1 {shape} 0\n")
    first = run()
    assert first != 0  # (256 threads and 32 KB: several times the fastest)
    lines = path.read_text().split("\n")
    assert len(lines) == 4 and lines[2].split()[1:] == f"{shape} {first}".split(), lines
    mine = lines[2].split()[0]
    path.write_text(f"{mine} {shape} 3\n")
    assert run() == 3
    assert path.read_text() == f"{mine} {shape} 3\n"


@pytest.mark.parametrize("sweeps", [1, 2, 3])
def test_chains_given_up(pkg, sweeps):
    """Where the chase of a large round gives up, the solve goes on behind
    launches that follow the chains: in either phase, more than once a
    solve, and after it on the same context."""
    old = {k: os.environ.get(k) for k in ("MSF_CONTRACT", "MSF_SMALL_M", "MSF_CONTRACT_SWEEPS")}
    os.environ.update(MSF_CONTRACT="2", MSF_SMALL_M="0", MSF_CONTRACT_SWEEPS=str(sweeps))
    try:
        c = pkg.Context(0)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    rng = np.random.default_rng(47)
    n = 300000
    check(c, *path_graph(n, np.arange(n - 1, 0, -1)), U32, "falling path")
    check(c, *path_graph(n, np.arange(n - 1)), U32, "rising path")
    # chains of 100 vertices, joined by random heavier edges: long chains in
    # a first round, others in the next
    i = np.arange(n - 1)
    check(c, *path_graph(n, np.where(i % 100 == 99, (1 << 20) + i[::-1], i[::-1])), U32, "pieces")
    # phase 1: loops are the light edges
    loops = np.stack([np.arange(n)] * 2, 1).astype(np.int32)
    e = np.concatenate([loops] * 6 + [path_graph(n, i)[1]])
    w = np.concatenate([np.zeros(6 * n), 5 + i[::-1]]).astype(np.uint32)
    check(c, n, e, w, U32, "falling path among light loops")
    e, w = gen.er(n, 4 * n, seed=48)
    check(c, n, e, w, U32, "random")
    e = rng.permutation(n).astype(np.int32)[path_graph(n, i)[1]]
    check(c, n, e, i[::-1].astype(np.uint32), U32, "permuted falling path")
    be = path_graph(n, i)[1].copy()
    be[77, 1] = n
    with pytest.raises(pkg.MSFError):
        c.solve(n, dev(be), dev(i.astype(np.uint32)), wtype=U32)
    check(c, n, *gen.er(n, n, seed=49), U32, "after a refused one")
    c.close()


def test_hubs_cost_no_more_than_random_edges(pkg):
    """Edges that all lead to a few hubs (a star among them) lower their
    minima in LDS in every workgroup, whatever other vertices share the hubs'
    places in the table: about the time of as many random edges."""
    import time
    c = pkg.Context(0)
    rng = np.random.default_rng(53)
    n, m = 500000, 2000000

    def ms(e, w):
        de, dw = dev(e), dev(w)
        best = 1e9
        for _ in range(5):
            t0 = time.perf_counter()
            ids, cnt, tot = c.solve(n, de, dw, wtype=U32)
            best = min(best, (time.perf_counter() - t0) * 1e3)
        want_ids, want_cnt, want_tot = oracle.msf(n, e, w, U32)
        assert cnt == want_cnt and tot[0] == want_tot[0]
        assert np.array_equal(ids.cpu().numpy().astype(np.int64), want_ids)
        return best

    w = rng.integers(0, 1 << 32, size=m, dtype=np.uint64).astype(np.uint32)
    spread = ms(rng.integers(0, n, size=(m, 2)).astype(np.int32), w)
    for k in (1, 3, 40):
        e = np.stack([rng.integers(0, k, size=m) * (n // k), rng.integers(0, n, size=m)], 1)
        hubs = ms(e.astype(np.int32), w)
        print("[gpu-case]", k, "hubs", hubs, "ms, random edges", spread, flush=True)
        assert hubs < 1.5 * spread, (k, hubs, spread)
    c.close()

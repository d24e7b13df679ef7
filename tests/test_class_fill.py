"""The class fill (a digit met by one split-match edge and no lookup): its
identity against the dense minimum on the CPU, and every table entry against
the oracle on the GPU at the sizes where its shapes change."""
import os

import numpy as np
import pytest

from workloads import random_graph
from workloads.gen import _Builder


def form(x):
    """The fill a vertex's plan reports (pase_vertex_info)."""
    if x["splits"] == 0:
        return "none"
    if x["tile_cols"]:
        return "rows"
    if x["kernel"] == 0:
        return "generic"
    if x["parts"] == 2:
        return "joint" if x["column"] >= 0 else "exchange"
    return "class" if x["column"] >= 0 else "minimum"


def star(dims, elems=(48, 48, 7), sizes=16, r=1, twice=()):
    """v0 with dims[0] loop dims joined to neighbours with dims[1:] loop dims,
    all joined to each other (so v0, the lowest id, comes first and its table
    has one digit per neighbour); small extents, so that ties are dense.
    twice: neighbours joined to v0 by a second edge (no class digit)."""
    b = _Builder("star", 4, comm_weight=r)
    for k, d in enumerate(dims):
        b.vertex(f"v{k}", [sizes + k] * d, [f"x{i}" for i in range(d)], [d - 1] if d > 1 else [], 1)
    for k in range(1, len(dims)):
        rank = max(1, min(dims[0], dims[k]) - (k == 1))
        b.edge(0, k, list(range(rank)), list(range(rank))[::-1], elems=elems[(k - 1) % 3])
        if k in twice:
            b.edge(0, k, list(range(rank)), list(range(rank)), elems=elems[k % 3])
    for k in range(1, len(dims)):
        for m in range(k + 1, len(dims)):
            b.edge(k, m, [0], [0], elems=elems[(k + m) % 3])
    return b.done()


@pytest.mark.parametrize("all_integers,p", [(False, 8), (False, 32), (True, 6), (True, 12)])
@pytest.mark.parametrize("seed", range(6))
def test_identity(seed, all_integers, p):
    """min over c of X + t_x(c, z) equals the three-part minimum over classes,
    value and lowest argmin, for edges of random graphs (unmapped dims, several
    tensor dims on one loop dim) under both configuration sets; X with ties."""
    from oracle.oracle import Oracle
    g = random_graph(3000 + seed, n=4, p=p, max_dims=3, extra_edges=2, max_size=40)
    o = Oracle(g)
    o.configs(p, all_integers=all_integers)
    rng = np.random.default_rng(seed)
    for k, e in enumerate(g["edges"]):
        t = o.edge_costs(k).astype(np.int64)                       # K_src x K_dst
        su, sv = o.splits(e["src"]).astype(np.int64), o.splits(e["dst"]).astype(np.int64)
        sig = [np.stack([s[:, d] if d >= 0 else np.ones(len(s), np.int64) for d in dims], 1)
               for s, dims in ((su, e["src_dim"]), (sv, e["dst_dim"]))]
        f = [g["comm_weight"] * -(-e["elems"] // s.prod(1)) for s in (su, sv)]
        K, Kz = t.shape
        X = rng.integers(0, 4, K) * (int(t.max()) // 6 + 1) * K + np.arange(K)   # keys: cost * K + c
        same = (sig[0][:, None, :] == sig[1][None, :, :]).all(2)
        dense = (X[:, None] + t * K).min(0)
        best = np.minimum((X[:, None] + f[0][:, None] * K).min(0), X.min() + f[1] * K)
        best = np.minimum(best, np.where(same, X[:, None], np.iinfo(np.int64).max).min(0))
        assert (best == dense).all()


def test_plan_rule():
    """Where the plan takes the class fill (reported as a column digit with no
    tile columns): not with caller-given costs, the volume model, a tile knob
    or the generic kernel mode, and back again; the launch plan checks in
    every case."""
    from paper_2407_04001_amd import pase as P
    P.load()
    g = star((3, 3, 3, 2))

    def classes(pg):
        assert pg.plan_check() > 0
        return [v for v in range(pg.nv) if (x := pg.vertex_info(v))["kernel"] == 1 and x["column"] >= 0
                and x["tile_cols"] == 0]
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 0)
    pg.enumerate_configs(16)
    base = classes(pg)
    assert base
    for opt, on, off in ((P.OPT_TILE_ROWS, 1, 0), (P.OPT_C_SPLITS, 2, 0), (P.OPT_KERNEL, 1, 0),
                         (P.OPT_HOIST_ELEMS, 1, 1 << 20), (P.OPT_KEY_TYPE, 2, 0)):
        pg.set_option(opt, on)
        assert not classes(pg), opt
        pg.set_option(opt, off)
        assert classes(pg) == base, opt
    zeros = [np.zeros(k, np.uint64) for k in pg.K], [np.zeros((pg.K[e["src"]], pg.K[e["dst"]]), np.uint64)
                                                    for e in g["edges"]]
    pg.override_costs(*zeros)
    assert not classes(pg)
    pg.enumerate_configs(16)
    assert classes(pg) == base
    pg.set_option(P.OPT_TRANSFER, 1)
    pg.enumerate_configs(16)
    assert not classes(pg)


# (loop dims of v0 and its neighbours, p, every integer): one-row tables, few rows (no staging) with odd
# counts, rows past a workgroup's, 64 rows with X in LDS (K 84) and formed twice (K 252: 31 752 rows)
SHAPES = [((1, 1), 2, False), ((3, 2), 8, False), ((2, 3), 16, False), ((3, 3, 2), 16, False),
          ((2, 3, 3), 7, True), ((3, 3, 3, 2), 8, False), ((3, 4, 3, 2), 16, False), ((3, 3, 3), 24, True),
          ((3, 4, 4, 4), 16, False), ((2, 4, 4, 4, 2), 8, False), ((5, 4, 5, 5), 16, False),
          ((4, 5, 4, 5), 32, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("key", [0, 1])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_shapes_every_entry(shape, key):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    dims, p, every = SHAPES[shape]
    g = star(dims)
    print(f"class fill shape {dims} p={p} every={every} key={key}", flush=True)
    o = Oracle(g)
    o.configs(p, all_integers=every)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.enumerate_configs(p, all_integers=every)
    pg.set_option(P.OPT_KEY_TYPE, key)
    for keep in (1, 0):
        pg.set_option(P.OPT_KEEP_TABLES, keep)
        assert pg.find_best_strategy() == o.result()
        if keep:
            for i, v in enumerate(o.sequence()):
                assert pg.fingerprint(v) == o.fingerprint(i), (v, pg.vertex_info(v))


# a class digit of few configurations beside large rest digits: (loop dims, neighbours joined twice, p, every
# integer, whether v0 takes the class fill); K 84 to 731, Kz 6 to 56
SMALL_DIGITS = [((5, 5, 5, 1), (1, 2), 32, False, False), ((5, 5, 5, 3), (1, 2), 32, False, True),
                ((4, 5, 5, 3), (1, 2), 32, False, True), ((5, 4, 4, 1), (1, 2), 64, False, False),
                ((3, 4, 4, 2), (1, 2), 64, False, True), ((5, 3, 3, 1), (1, 2), 24, True, False)]


@pytest.mark.parametrize("case", range(len(SMALL_DIGITS)))
def test_small_digit_plan(case):
    """The class fill only where its digit saves more than its own cost per
    cell; otherwise the dense fill."""
    from paper_2407_04001_amd import pase as P
    P.load()
    dims, twice, p, every, classes = SMALL_DIGITS[case]
    pg = P.Graph(star(dims, twice=twice))
    pg.enumerate_configs(p, all_integers=every)
    x = pg.vertex_info(0)
    assert x["kernel"] == 1 and (x["tile_cols"] == 0) == classes, x
    assert classes is False or x["column"] == len(dims) - 1
    for sched in (0, 1, 4, 5):
        pg.set_option(P.OPT_SCHEDULE, sched)
        assert pg.plan_check() > 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(SMALL_DIGITS)))
def test_small_digit_every_entry(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    dims, twice, p, every, _ = SMALL_DIGITS[case]
    print(f"small class digit {SMALL_DIGITS[case]}", flush=True)
    g = star(dims, twice=twice)
    o = Oracle(g)
    o.configs(p, all_integers=every)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.enumerate_configs(p, all_integers=every)
    for keep in (1, 0):
        pg.set_option(P.OPT_KEEP_TABLES, keep)
        assert pg.find_best_strategy() == o.result()
        if keep:
            for i, v in enumerate(o.sequence()):
                assert pg.fingerprint(v) == o.fingerprint(i), (v, pg.vertex_info(v))


@pytest.mark.gpu
@pytest.mark.parametrize("key", [0, 1])
@pytest.mark.parametrize("shape", range(7))
def test_volume_minimum(shape, key):
    """The volume model at direct sizes: the plain minimum with every edge's
    matrix as a lookup (up to three edges and a lookup per vertex, either end of
    an edge), and with a smaller direct size, where some vertices take the dense
    fills."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    dims, p, every = SHAPES[shape]
    g = star(dims)
    print(f"volume minimum {dims} p={p} every={every} key={key}", flush=True)
    o = Oracle(g)
    o.configs(p, all_integers=every, volume=True)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.set_option(P.OPT_TRANSFER, 1)
    pg.enumerate_configs(p, all_integers=every)
    pg.set_option(P.OPT_KEY_TYPE, key)
    pg.set_option(P.OPT_KEEP_TABLES, 1)
    for cells in (1 << 30, 1000):
        pg.set_option(P.OPT_DIRECT_CELLS, cells)
        assert pg.find_best_strategy() == o.result(), cells
        for i, v in enumerate(o.sequence()):
            assert pg.fingerprint(v) == o.fingerprint(i), (v, cells, pg.vertex_info(v))


@pytest.mark.gpu
@pytest.mark.parametrize("p,every", [(16, False), (7, True)])
@pytest.mark.parametrize("key", [0, 1])
def test_lookups_alone(p, every, key):
    """A vertex without edges past the direct size (the decoder's context GEMM:
    no column digit fits, its lookups are small) on the plain minimum: every
    table against the oracle, and the strategy without kept tables."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    from workloads import transformer
    g = transformer(p=p, enc_layers=1, dec_layers=2)
    print(f"lookups alone p={p} every={every} key={key}", flush=True)
    o = Oracle(g)
    o.configs(p, all_integers=every)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.enumerate_configs(p, all_integers=every)
    pg.set_option(P.OPT_KEY_TYPE, key)
    info = [pg.vertex_info(v) for v in range(pg.nv)]
    assert any(x["kernel"] == 1 and x["column"] == -1 and x["tile_cols"] == 0 for x in info)
    for keep in (1, 0):
        pg.set_option(P.OPT_KEEP_TABLES, keep)
        assert pg.find_best_strategy() == o.result()
        if keep:
            for i, v in enumerate(o.sequence()):
                assert pg.fingerprint(v) == o.fingerprint(i), (v, pg.vertex_info(v))


# ------------------------------------------------------------------ joint fill
def triangle(di, dj, dy, has_e, looks, perm=False, r=1, upper=2):
    """v_j (1) joined to v_i (2), y (3) and an upper digit (4); v_i joined to y
    (has_e) and, twice, to a lower digit (5), so that no digit of v_i meets it
    in one edge alone; the digits joined to each other.  looks: a vertex (0)
    whose table over (v_j, the upper digit) v_j looks up, and the edge j-upper
    left out.  Without has_e there is no upper digit either (v_i would come
    first).  The order is (0,) v_j, v_i, ..."""
    b = _Builder("triangle", 4, comm_weight=r)
    dims = (2, dj, di, dy, upper, 1)
    for k, d in enumerate(dims):
        if k == 0 and not looks:
            b.vertex("pad", [3], ["x0"], [], 1)
            continue
        b.vertex(f"v{k}", [12 + k] * d, [f"x{i}" for i in range(d)], [d - 1] if d > 2 else [], 1)

    def edge(u, v, elems):
        d = list(range(max(1, min(dims[u] if u or looks else 1, dims[v]))))
        b.edge(u, v, d, d[::-1] if perm else d, elems=elems)
    edge(1, 2, 40)
    edge(1, 3, 24)
    if has_e:
        edge(2, 3, 33)
    edge(2, 5, 5)
    edge(2, 5, 9)
    if has_e and not looks:
        edge(1, 4, 17)
    for u, v in ((3, 4), (3, 5), (4, 5)):
        b.edge(u, v, [0], [0], elems=11)
    if looks:
        edge(0, 1, 21)
        if has_e:
            edge(0, 4, 6)
    else:
        b.edge(0, 5, [0], [0], elems=3)
    return b.done()


# (dims of v_i, v_j, y; edge from v_i to y; v_j looks a table up; permuted maps; p, every integer): K 35 to
# 252 on one configuration per thread, 738 on one of 768 threads, 796 on two; classes of one and of several
# configurations, of five on both sides of an entry in the last two (y of three dims, its neighbours of four)
TRIANGLES = [(4, 4, 4, True, False, False, 8, False), (4, 4, 4, True, True, True, 16, False),
             (5, 4, 4, True, False, True, 16, False), (4, 5, 4, True, True, False, 16, False),
             (4, 4, 3, False, False, True, 16, False), (4, 4, 3, False, True, False, 32, False),
             (3, 4, 4, True, False, False, 12, True), (4, 4, 3, False, True, True, 10, True),
             (5, 4, 5, True, True, True, 32, False), (3, 2, 2, False, False, True, 64, True),
             (3, 2, 2, True, False, False, 60, True), (4, 4, 3, True, False, True, 16, False),
             (4, 4, 3, True, True, True, 16, False)]


def maps(rng, nu, nv):
    """A tensor whose dims map at least all but one loop dim of either end:
    permuted, some dims unmapped at one end, some loop dims mapped twice."""
    for _ in range(1000):
        rank = int(rng.integers(max(1, max(nu, nv) - 1), max(nu, nv) + 3))
        if rank > 8:
            continue
        su, sv = rng.integers(-1, nu, rank), rng.integers(-1, nv, rank)
        if len(set(su) - {-1}) >= nu - 1 and len(set(sv) - {-1}) >= nv - 1:
            return [int(k) for k in su], [int(k) for k in sv]
    raise AssertionError("no map")


def random_triangle(seed):
    """triangle() with its three edges between v_i, v_j and y mapped at random."""
    rng = np.random.default_rng(seed)
    di, dj, dy = (int(k) for k in rng.integers(3, 5, 3))
    g = triangle(di, dj, dy, True, False)
    dims = {1: dj, 2: di, 3: dy}
    for e in g["edges"]:
        if {e["src"], e["dst"]} <= {1, 2, 3}:
            e["src_dim"], e["dst_dim"] = maps(rng, dims[e["src"]], dims[e["dst"]])
    return g


# (in the last three an entry's pair of combined classes has several configurations on both sides)
RANDOM_TRIANGLES = list(range(12)) + [30, 77, 106]


@pytest.mark.parametrize("every,p", [(False, 16), (True, 8)])
@pytest.mark.parametrize("case", range(len(RANDOM_TRIANGLES) + len(TRIANGLES)))
def test_joint_identity(case, every, p):
    """The minima over classes, with at most one pair of combined classes per
    entry, against the dense minimum over both configurations: value and the
    lowest v_i, at every y, for the edges of joint plans; costs with ties."""
    from oracle.oracle import Oracle
    from paper_2407_04001_amd import pase as P
    P.load()
    if case < len(RANDOM_TRIANGLES):
        g = random_triangle(RANDOM_TRIANGLES[case])
    else:
        di, dj, dy, has_e, looks, perm = TRIANGLES[case - len(RANDOM_TRIANGLES)][:6]
        g = triangle(di, dj, dy, has_e, looks, perm)
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.enumerate_configs(p, all_integers=every)
    if form(pg.vertex_info(2)) != "joint":
        pytest.skip("not a joint fill")
    o = Oracle(g)
    o.configs(p, all_integers=every)
    K = {v: len(o.splits(v)) for v in (1, 2, 3)}
    rng = np.random.default_rng(case)
    big = np.int64(1) << 60

    def edge(u, v):
        """t (K_u x K_v), f of either end, same class; None without an edge."""
        at = [k for k, e in enumerate(g["edges"]) if {e["src"], e["dst"]} == {u, v}]
        if not at:
            return None
        e, k = g["edges"][at[0]], at[0]
        t = o.edge_costs(k).astype(np.int64)
        sig = {}
        for x, dims in ((e["src"], e["src_dim"]), (e["dst"], e["dst_dim"])):
            sp = o.splits(x).astype(np.int64)
            sig[x] = np.stack([sp[:, d] if d >= 0 else np.ones(len(sp), np.int64) for d in dims], 1)
        f = [g["comm_weight"] * -(-e["elems"] // o.splits(x).astype(np.int64).prod(1)) for x in (u, v)]
        return t if e["src"] == u else t.T, f[0], f[1], (sig[u][:, None, :] == sig[v][None, :, :]).all(2)
    to, fio, fjo, so = edge(2, 1)
    tj, fjy, fyj, sj = edge(1, 3)
    has_e = edge(2, 3) is not None
    ti, fiy, fyi, si = edge(2, 3) or (np.zeros((K[2], K[3]), np.int64), None, None, None)
    hi = int(max(to.max(), tj.max(), ti.max())) // 4 + 1
    XI = rng.integers(0, 5, K[2]) * hi * K[2] + np.arange(K[2])    # keys of v_i
    XJ = rng.integers(0, 5, K[1]) * hi * K[2]
    to, tj, ti, fio, fjo, fjy, fyj = (x * K[2] for x in (to, tj, ti, fio, fjo, fjy, fyj))
    if has_e:
        fiy, fyi = fiy * K[2], fyi * K[2]
    pair = XI[:, None] + XJ[None, :] + to                           # c, c'
    J0, J1 = (XJ[None, :] + to).min(1), (XJ[None, :] + fjy[None, :] + to).min(1)
    I0 = (XI[:, None] + to).min(0)
    I1 = (XI[:, None] + fiy[:, None] + to).min(0) if has_e else None
    several = 0
    for y in range(K[3]):
        dense = (pair + ti[:, y][:, None] + tj[:, y][None, :]).min()
        best = (ti[:, y] + XI + np.minimum(J0 + fyj[y], J1)).min()
        cj = np.flatnonzero(sj[:, y])
        ci = np.flatnonzero(si[:, y]) if has_e else np.arange(0)
        if len(cj):
            both = np.minimum(I0[cj] + fyi[y], I1[cj]) if has_e else I0[cj]
            best = min(best, (XJ[cj] + both).min())
        if len(cj) and len(ci):
            # t(c', c) as one of the f, and as 0 in the one pair of combined classes
            best = min(best, XI[ci].min() + (XJ + fjo)[cj].min(), (XI + fio)[ci].min() + XJ[cj].min())
            at = so[np.ix_(ci, cj)]
            if at.any():
                a, b = np.flatnonzero(at.any(1)), np.flatnonzero(at.any(0))
                assert at[np.ix_(a, b)].all(), (y, "more than one pair of combined classes")
                best = min(best, XI[ci[a]].min() + XJ[cj[b]].min())
                several += len(a) > 1 and len(b) > 1
        assert best == dense < big, y
    if case < len(RANDOM_TRIANGLES) and RANDOM_TRIANGLES[case] >= 30:
        assert several


@pytest.mark.parametrize("case", range(len(TRIANGLES)))
def test_joint_plan(case):
    """Every triangle plans v_i as a joint fill (a class form column digit y,
    found in a lookup), under every schedule, tables kept and not; the launch
    plan checks; a smaller workspace without v_j's table."""
    from paper_2407_04001_amd import pase as P
    P.load()
    di, dj, dy, has_e, looks, perm, p, every = TRIANGLES[case]
    g = triangle(di, dj, dy, has_e, looks, perm, upper=1 if p > 48 else 2)
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.enumerate_configs(p, all_integers=every)
    x = pg.vertex_info(2)
    assert (x["kernel"], x["column"], x["tile_cols"]) == (1, 3, 0) and x["lookups"] >= 1, x
    assert form(x) == "joint" and form(pg.vertex_info(1)) == "none"
    assert 2 in pg.dependent_set(1) and 3 in pg.dependent_set(1) and 3 in pg.dependent_set(2)
    for sched in (0, 1, 4, 5):
        for hoist in (0, 1 << 20):
            pg.set_option(P.OPT_SCHEDULE, sched)
            pg.set_option(P.OPT_HOIST_ELEMS, hoist)
            pg.set_option(P.OPT_KEEP_TABLES, 1)
            assert pg.plan_check() > 0 and form(pg.vertex_info(1)) == "class" and form(pg.vertex_info(2)) == "joint"
            kept = pg.workspace_size()
            pg.set_option(P.OPT_KEEP_TABLES, 0)
            assert pg.plan_check() > 0 and pg.workspace_size() <= kept


@pytest.mark.gpu
@pytest.mark.parametrize("key", [0, 1])
@pytest.mark.parametrize("seed", RANDOM_TRIANGLES)
def test_random_maps_every_table(seed, key):
    """Unmapped and repeated tensor dims on the three edges of a joint fill (or
    of the fill the plan takes in its place): every table, then the strategy
    without v_j's."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    g = random_triangle(seed)
    print(f"random maps seed={seed} key={key}", flush=True)
    o = Oracle(g)
    o.configs(16)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.set_option(P.OPT_KEY_TYPE, key)
    pg.enumerate_configs(16)
    for keep in (1, 0):
        pg.set_option(P.OPT_KEEP_TABLES, keep)
        assert pg.find_best_strategy() == o.result()
        if keep:
            for i, v in enumerate(o.sequence()):
                assert pg.fingerprint(v) == o.fingerprint(i), (v, pg.vertex_info(v))


@pytest.mark.gpu
@pytest.mark.parametrize("key", [0, 1])
@pytest.mark.parametrize("case", range(len(TRIANGLES)))
def test_joint_every_table(case, key):
    """Joint fills against the oracle: every table with tables kept, and the
    strategy with v_j's table left out (its argmin evaluated afterwards), under
    each schedule, with the half fill in its own slot or just before the fill,
    and through the allocation-free entry point."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    di, dj, dy, has_e, looks, perm, p, every = TRIANGLES[case]
    g = triangle(di, dj, dy, has_e, looks, perm, upper=1 if p > 48 else 2)
    print(f"joint fill {TRIANGLES[case]} key={key}", flush=True)
    o = Oracle(g)
    o.configs(p, all_integers=every)
    o.solve(threads=os.cpu_count() or 1)
    pg = P.Graph(g)
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.enumerate_configs(p, all_integers=every)
    pg.set_option(P.OPT_KEY_TYPE, key)
    for sched, hoist in ((5, 1 << 20), (0, 1 << 20), (1, 1 << 20), (5, 0)):
        pg.set_option(P.OPT_SCHEDULE, sched)
        pg.set_option(P.OPT_HOIST_ELEMS, hoist)
        for keep in (1, 0):
            pg.set_option(P.OPT_KEEP_TABLES, keep)
            assert form(pg.vertex_info(2)) == "joint"
            assert pg.find_best_strategy() == o.result(), (sched, hoist, keep)
            if keep:
                for i, v in enumerate(o.sequence()):
                    assert pg.fingerprint(v) == o.fingerprint(i), (v, sched, hoist)
    if pg.workspace_size() <= P.NOALLOC_WORKSPACE_BYTES:
        assert P.pase_find_best_strategy_noalloc(pg.h, pg.nv) == o.result()


# --------------------------------------------------------------- exchange fill
def exchange(dj, di, dy, dz, perm=False, r=1, elems=(40, 24, 33, 17, 11, 9)):
    """v_j (3) with three lookups -- leaves joined to it and to v_i (4), y (5)
    and z (6) -- and no edges of its own; v_i joined to y and to z, y to z.  The
    order is the leaves, v_j, v_i, y, z."""
    b = _Builder("exchange", 4, comm_weight=r)
    dims = (2, 2, 2, dj, di, dy, dz)
    for k, d in enumerate(dims):
        b.vertex(f"v{k}", [12 + k] * d, [f"x{i}" for i in range(d)], [d - 1] if d > 2 else [], 1)

    def edge(u, v, el):
        d = list(range(min(dims[u], dims[v])))
        b.edge(u, v, d, d[::-1] if perm else d, elems=el)
    for leaf, other in ((0, 4), (1, 5), (2, 6)):
        edge(leaf, 3, elems[leaf])
        edge(leaf, other, elems[leaf] + 2)
    edge(4, 5, elems[3])
    edge(4, 6, elems[4])
    edge(5, 6, elems[5])
    return b.done()


# (dims of v_j, v_i, y, z; permuted maps; p, every integer): K_i 28 to 556, K_y and K_z odd, below and past a
# wave, K_j 3 (a wave of the fill without a c) to 43
EXCHANGES = [(2, 4, 4, 4, False, 8, False), (4, 4, 3, 4, True, 8, False), (1, 4, 4, 3, True, 8, False),
             (4, 3, 3, 2, False, 7, True), (2, 5, 4, 5, True, 16, False), (1, 4, 5, 4, False, 32, False),
             (2, 3, 4, 3, True, 7, True), (1, 4, 3, 3, True, 24, True), (1, 6, 5, 5, False, 4, False),
             (1, 5, 4, 4, True, 23, True)]


@pytest.mark.parametrize("seed", range(8))
def test_exchange_identity(seed):
    """The five cases per (c, y, z), with their minima over classes and pairs
    of classes, against the dense minimum over c and x, value and lowest
    argmin, at every entry; costs with ties."""
    from oracle.oracle import Oracle
    dj, di, dy, dz, perm, p, every = EXCHANGES[seed]
    p = min(p, 8)
    g = exchange(dj, di, dy, dz, perm)
    o = Oracle(g)
    o.configs(p, all_integers=every)
    K = [len(o.splits(v)) for v in range(7)]
    at = {(e["src"], e["dst"]): k for k, e in enumerate(g["edges"])}
    rng = np.random.default_rng(seed)
    hi = 40
    L, A, B, C = (rng.integers(0, hi, s) for s in ((K[3],), (K[3], K[4]), (K[3], K[5]), (K[3], K[6])))
    Li = rng.integers(0, hi, K[4])
    t, f, sig = [], [], []
    for w in (5, 6):
        k = at[(4, w)]
        e = g["edges"][k]
        t.append(o.edge_costs(k).astype(np.int64))
        s = [np.stack([o.splits(v).astype(np.int64)[:, d] if d >= 0 else np.ones(K[v], np.int64) for d in dims], 1)
             for v, dims in ((4, e["src_dim"]), (w, e["dst_dim"]))]
        sig.append((s[0][:, None, :] == s[1][None, :, :]).all(2))            # x, other end
        f.append([g["comm_weight"] * -(-e["elems"] // o.splits(v).astype(np.int64).prod(1)) for v in (4, w)])
    Ki, big = K[4], 1 << 40
    T = (L[:, None, None] + B[:, :, None] + C[:, None, :]) * Ki                # c, y, z
    dense = np.full((K[5], K[6]), big)
    best = np.full((K[5], K[6]), big)
    for c in range(K[3]):
        X = (A[c] + Li) * Ki + np.arange(Ki)
        dense = np.minimum(dense, T[c] + (X[:, None, None] + Ki * (t[0][:, :, None] + t[1][:, None, :])).min(0))
        over = lambda v, m: np.where(m, v[:, None], big).min(0)                # minima over the other end's class
        f1x, f1y, f2x, f2z = (q * Ki for q in (*f[0], *f[1]))
        a1 = np.minimum(np.minimum(X.min() + f1y, (X + f1x).min()), over(X, sig[0]))
        b1 = np.minimum(np.minimum((X + f2x).min() + f1y, (X + f1x + f2x).min()), over(X + f2x, sig[0]))
        q1, q2 = over(X, sig[1]), over(X + f1x, sig[1])
        both = np.where(sig[0][:, :, None] & sig[1][:, None, :], X[:, None, None], big).min(0)
        case = np.minimum(np.minimum(a1[:, None] + f2z[None], b1[:, None]), np.minimum(q1[None] + f1y[:, None], q2[None]))
        best = np.minimum(best, T[c] + np.minimum(case, both))
    assert (best == dense).all()


@pytest.mark.parametrize("case", range(len(EXCHANGES)))
def test_exchange_plan(case):
    """The pair is an exchange fill without v_j's table (with it, filled by
    itself, when tables are kept): the launch plan checks under every schedule;
    not with the option off."""
    from paper_2407_04001_amd import pase as P
    P.load()
    dj, di, dy, dz, perm, p, every = EXCHANGES[case]
    pg = P.Graph(exchange(dj, di, dy, dz, perm))
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.enumerate_configs(p, all_integers=every)
    for sched in (0, 1, 4, 5):
        pg.set_option(P.OPT_SCHEDULE, sched)
        for hoist in (0, 1 << 20):
            pg.set_option(P.OPT_HOIST_ELEMS, hoist)
            pg.set_option(P.OPT_KEEP_TABLES, 1)
            assert pg.plan_check() > 0
            assert form(pg.vertex_info(3)) in ("rows", "generic") and form(pg.vertex_info(4)) == "exchange"
            kept = pg.workspace_size()
            pg.set_option(P.OPT_KEEP_TABLES, 0)
            assert pg.plan_check() > 0 and pg.workspace_size() <= kept
            assert (form(pg.vertex_info(3)), form(pg.vertex_info(4))) == ("none", "exchange")
            assert (pg.vertex_info(3)["fused"], pg.vertex_info(4)["fused"]) == (1, 2)
    pg.set_option(P.OPT_FUSED_MIN, 0)
    assert not any(pg.vertex_info(v)["fused"] for v in range(7))
    assert "exchange" not in [form(pg.vertex_info(v)) for v in range(7)]


def test_exchange_lanes():
    """The lanes follow the fills that run: a pair whose dense fill would take
    past the bulk threshold (84 x 462 x 210 x 210 cells), whose exchange fill
    takes 12 us, is on the lane of the small vertices."""
    from paper_2407_04001_amd import pase as P
    P.load()
    pg = P.Graph(exchange(3, 5, 4, 4))
    pg.enumerate_configs(64)
    assert form(pg.vertex_info(4)) == "exchange"
    assert [pg.vertex_info(v)["lane"] for v in (3, 4, 5, 6)] == [0, 0, 0, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("key", [0, 1])
@pytest.mark.parametrize("case", range(len(EXCHANGES)))
def test_exchange_strategies(case, key):
    """Against the oracle under each schedule, with the half fill in v_j's slot
    or just before the fill, for several tensor sizes: every table with tables
    kept, and the strategy with v_j's left out (its argmin evaluated
    afterwards)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    dj, di, dy, dz, perm, p, every = EXCHANGES[case]
    sizes = ((40, 24, 33, 17, 11, 9), (5, 90, 700, 300, 2, 60), (900, 4, 4, 3000, 2000, 1), (1, 1, 1, 1, 1, 1))
    for elems in sizes[:1] if p == 23 else sizes:
        g = exchange(dj, di, dy, dz, perm, elems=elems)
        print(f"exchange fill {EXCHANGES[case]} key={key} elems={elems}", flush=True)
        o = Oracle(g)
        o.configs(p, all_integers=every)
        o.solve(threads=os.cpu_count() or 1)
        want = [o.fingerprint(i) for i in range(7)]
        pg = P.Graph(g)
        pg.set_option(P.OPT_DIRECT_CELLS, 1)
        pg.enumerate_configs(p, all_integers=every)
        pg.set_option(P.OPT_KEY_TYPE, key)
        for sched, hoist in ((5, 1 << 20), (0, 1 << 20), (1, 1 << 20), (5, 0)):
            pg.set_option(P.OPT_SCHEDULE, sched)
            pg.set_option(P.OPT_HOIST_ELEMS, hoist)
            for keep in (1, 0):
                pg.set_option(P.OPT_KEEP_TABLES, keep)
                assert form(pg.vertex_info(4)) == "exchange"
                assert pg.find_best_strategy() == o.result(), (elems, sched, hoist, keep)
                if keep:
                    for i, v in enumerate(o.sequence()):
                        assert pg.fingerprint(v) == want[i], (v, elems, sched, hoist)
        if pg.workspace_size() <= P.NOALLOC_WORKSPACE_BYTES:
            assert P.pase_find_best_strategy_noalloc(pg.h, pg.nv) == o.result()


@pytest.mark.gpu
def test_memory_limits():
    """A chain of small vertices in a lent workspace, a memory budget and the
    static workspace that only the dense fills fit: the same strategy."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from workloads import chain_graph
    pg = P.Graph(chain_graph(1, 600, p=64, max_dims=5))
    pg.enumerate_configs(64)
    want, need = pg.find_best_strategy(), pg.workspace_size()
    pg.set_option(P.OPT_C_SPLITS, 1)   # (a tile knob: the dense fills)
    dense = pg.workspace_size()
    assert dense < need and pg.find_best_strategy() == want
    pg.set_option(P.OPT_C_SPLITS, 0)
    ws = torch.empty(dense + 256, dtype=torch.uint8, device="cuda")
    at = -ws.data_ptr() % 256
    P.pase_set_workspace(pg.h, ws.data_ptr() + at, dense)
    assert P.pase_find_best_strategy(pg.h, pg.nv) == want and pg.workspace_size() == dense
    P.pase_set_workspace(pg.h, 0, 0)
    assert P.pase_find_best_strategy(pg.h, pg.nv) == want and pg.workspace_size() == need
    pg.set_option(P.OPT_MEMORY_BUDGET, dense)
    assert P.pase_find_best_strategy(pg.h, pg.nv) == want and pg.workspace_size() <= dense
    big = P.Graph(chain_graph(1, 6100, p=64, max_dims=5))
    big.enumerate_configs(64)
    assert big.workspace_size() > P.NOALLOC_WORKSPACE_BYTES
    assert P.pase_find_best_strategy_noalloc(big.h, big.nv) == P.pase_find_best_strategy(big.h, big.nv)


# -------------------------------------------------------------- key edges
def scaled(g, m):
    """The graph with every cost about m times as large (and no multiple of it:
    the splits round up)."""
    return dict(g, vertices=[dict(v, flops_per_point=v["flops_per_point"] * m) for v in g["vertices"]],
                edges=[dict(e, elems=e["elems"] * m + k % 3) for k, e in enumerate(g["edges"])])


# graph, p, every integer, the vertex whose fill is looked at and its form
EDGE_GRAPHS = [(lambda: star((3, 3, 3, 2)), 16, False, 0, "class"),
               (lambda: triangle(4, 4, 3, True, True, True), 16, False, 2, "joint"),
               (lambda: triangle(4, 4, 3, False, False, True), 16, False, 2, "joint"),
               (lambda: exchange(2, 5, 4, 5, True), 16, False, 4, "exchange"),
               (lambda: exchange(4, 3, 3, 2), 7, True, 4, "exchange")]


def edge_plan(P, graph, p, every, m):
    """A handle planned at m; None past 64-bit costs."""
    pg = P.Graph(scaled(graph, m))
    pg.set_option(P.OPT_DIRECT_CELLS, 1)
    pg.set_option(P.OPT_KEEP_TABLES, 1)
    try:
        pg.enumerate_configs(p, all_integers=every)
    except P.PaseError as e:
        assert e.status == P.OVERFLOW, e
        return None
    return pg


def edge_scales(P, case):
    """The largest m with fp64 keys, with the structured form in uint64 keys,
    and with 64-bit keys (bisection on the host), in that order."""
    build, p, every, v, kind = EDGE_GRAPHS[case]
    g = build()

    def largest(accept):
        lo, hi = 1, 1 << 56
        while hi - lo > 1:
            mid = (lo + hi) // 2
            pg = edge_plan(P, g, p, every, mid)
            if pg is not None and accept(pg.vertex_info(v)):
                lo = mid
            else:
                hi = mid
        return lo
    return g, [largest(lambda x: x["key_type"] == 0), largest(lambda x: x["key_type"] < 2 and form(x) == kind),
               largest(lambda x: x["key_type"] < 2)]


@pytest.mark.parametrize("case", range(len(EDGE_GRAPHS)))
def test_key_edge_plan(case):
    """The key types meet at 2^53 and 2^64; in uint64 keys the joint and the
    exchange fill stop where the sums they form could wrap (2^64, and 2^60 for
    the mark of an empty class), the class fill, whose sums are those of the
    dense fill, nowhere before."""
    from paper_2407_04001_amd import pase as P
    P.load()
    g, (a, b, c) = edge_scales(P, case)
    _, p, every, v, kind = EDGE_GRAPHS[case]

    def top(m):
        pg = edge_plan(P, g, p, every, m)
        return max((int(x["key_bound"]) + 1) << max(0, (int(k) - 1).bit_length())
                   for x, k in ((pg.vertex_info(u), pg.K[u]) for u in range(pg.nv)))
    assert top(a) <= 1 << 53 < top(a + 1) and top(c) <= 1 << 64
    assert a < b <= c
    below, past = edge_plan(P, g, p, every, b), edge_plan(P, g, p, every, b + 1)
    assert form(below.vertex_info(v)) == kind and below.plan_check() > 0
    if kind == "class":
        assert b == c
    else:
        assert past.vertex_info(v)["key_type"] == 1 and form(past.vertex_info(v)) != kind and past.plan_check() > 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(EDGE_GRAPHS)))
def test_key_edge_every_table(case):
    """Every table on both sides of each edge (fp64 and uint64 keys with the
    structured fill; uint64 keys with and without it; uint64 and 128-bit keys)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_04001_amd import pase as P
    from oracle.oracle import Oracle
    g, scales = edge_scales(P, case)
    _, p, every, v, kind = EDGE_GRAPHS[case]
    for m in sorted({x for s in scales for x in (s, s + 1)}):
        pg = edge_plan(P, g, p, every, m)
        if pg is None:
            continue
        x = pg.vertex_info(v)
        print(f"key edge {kind} m={m} key type {x['key_type']} {form(x)}", flush=True)
        o = Oracle(scaled(g, m))
        o.configs(p, all_integers=every)
        o.solve(threads=os.cpu_count() or 1)
        assert pg.find_best_strategy() == o.result(), m
        for i, u in enumerate(o.sequence()):
            assert pg.fingerprint(u) == o.fingerprint(i), (u, m, pg.vertex_info(u))
        pg.set_option(P.OPT_KEEP_TABLES, 0)
        assert pg.find_best_strategy() == o.result(), m

"""The class fill (a digit met by one split-match edge and no lookup): its
identity against the dense minimum on the CPU, and every table entry against
the oracle on the GPU at the sizes where its shapes change."""
import os

import numpy as np
import pytest

from workloads import random_graph
from workloads.gen import _Builder


def star(dims, elems=(48, 48, 7), sizes=16, r=1):
    """v0 with dims[0] loop dims joined to neighbours with dims[1:] loop dims,
    all joined to each other (so v0, the lowest id, comes first and its table
    has one digit per neighbour); small extents, so that ties are dense."""
    b = _Builder("star", 4, comm_weight=r)
    for k, d in enumerate(dims):
        b.vertex(f"v{k}", [sizes + k] * d, [f"x{i}" for i in range(d)], [d - 1] if d > 1 else [], 1)
    for k in range(1, len(dims)):
        rank = max(1, min(dims[0], dims[k]) - (k == 1))
        b.edge(0, k, list(range(rank)), list(range(rank))[::-1], elems=elems[(k - 1) % 3])
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

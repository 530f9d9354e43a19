"""The octree's nodes at the edges of the build: tiles of 1024 particles, leaf
sizes around the window limit of 1024, depth caps, coincident particles, both
curves, forests; node sets against the oracle, child links through the masses
that the multipole pass sums along them."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


def points(n, seed):
    """A third uniform, a third in a tight clump, the rest copies of a few points."""
    rng = np.random.default_rng(seed)
    p = rng.uniform(size=(n, 3))
    k = n // 3
    p[:k] = 0.3 + 1e-4 * rng.normal(size=(k, 3))
    if n > 10:
        p[k:2 * k] = p[rng.integers(2 * k, n, size=k) % max(1, n // 50) + 2 * k if n > 200 else np.full(k, n - 1)]
    return np.mod(p, 1.0)[rng.permutation(n)]


def export(g, ctx, tree):
    g.g4_compute_multipoles(ctx, tree, 3)
    return {k: v.cpu().numpy() for k, v in g.g4_tree_export(ctx, tree).items()}


def check_links(ex, n, nroot=1):
    """Mass of every node = its particle count (unit masses; sums up to 2^24 are exact in FP32):
    wrong child links would lose or repeat particles.  Levels contiguous and in curve order."""
    assert np.array_equal(ex["mass"], ex["count"].astype(np.float64))
    assert np.all(np.diff(ex["level"]) >= 0)
    for l in range(ex["level"].max() + 1):
        f, c = ex["first"][ex["level"] == l], ex["count"][ex["level"] == l]
        assert np.all(f[1:] >= f[:-1] + c[:-1])
    assert np.all(ex["level"][:nroot] == 0) and ex["count"][:nroot].sum() == n


@pytest.mark.parametrize("n,B,maxd,keys", [
    (1, 1, 21, 0), (2, 1, 21, 0), (8, 8, 21, 0), (9, 8, 21, 0), (1023, 8, 21, 0), (1024, 1, 21, 1), (1025, 32, 21, 0),
    (4099, 1, 21, 0), (4099, 16, 21, 1), (4099, 5, 1, 0), (4099, 5, 3, 1), (5000, 1023, 21, 0), (5000, 1024, 21, 0),
    (5000, 1025, 21, 0), (9001, 3000, 21, 1), (3000, 3000, 21, 0), (3001, 3000, 21, 0), (200003, 24, 21, 0),
    # the sort's small forms: up to 128 tiles of 1024 keys, then of 2048
    (511, 4, 21, 0), (513, 4, 21, 1), (65536, 8, 21, 0), (65537, 8, 21, 1), (131072, 24, 21, 0), (131073, 24, 21, 1),
    (262144, 32, 21, 1), (262145, 32, 21, 0)])
@pytest.mark.parametrize("periodic", [True, False])
def test_nodes_match_oracle(g, n, B, maxd, keys, periodic):
    ctx = g.Context()
    pos = points(n, n + B)
    tp = g.tree_params(periodic, 1.0, leaf_max=B, max_depth=maxd, key_kind=keys)
    x, y, z = g.g4_quantize(ctx, torch.from_numpy(pos).cuda(), tp)
    m = torch.ones(n, device="cuda")
    tree = g.g4_build_tree(ctx, g.particles(x, y, z, m), tp)
    ex = export(g, ctx, tree)
    X, Y, Z = (v.cpu().numpy().view(np.uint32) for v in (x, y, z))
    ot = oracle.Tree(X, Y, Z, np.ones(n), periodic, 1.0, B, max_depth=maxd)
    level, cell, count, leaf = ot.nodes()
    mine = np.column_stack([ex["level"], ex["cell"].view(np.uint32), ex["count"], ex["leaf"]]).astype(np.int64)
    ref = np.column_stack([level, cell, count, leaf]).astype(np.int64)
    assert mine.shape == ref.shape
    assert np.array_equal(mine[np.lexsort(mine.T)], ref[np.lexsort(ref.T)])
    check_links(ex, n)
    nn, starts = g.g4_tree_info(ctx, tree)
    assert nn == len(level) and starts[-1] == nn


@pytest.mark.parametrize("B", [1, 8, 1500])
def test_forest_nodes(g, B):
    """Boxes of 1, 2, B, B + 1, ... particles, some ending on the tile edge: the nodes of each box
    are those of its own tree."""
    ctx = g.Context()
    sizes = [1, 2, B, B + 1, 1024 - (2 * B + 4) % 1024, 1, 1024, 1025, 3000, 7, 5]
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    pos = np.concatenate([points(s, 100 + i) for i, s in enumerate(sizes)])
    tp = g.tree_params(True, 1.0, leaf_max=B)
    xyz = g.g4_quantize(ctx, torch.from_numpy(pos).cuda(), tp)
    m = torch.ones(n, device="cuda")
    ex = export(g, ctx, g.g4_build_forest(ctx, off, g.particles(*xyz, m), tp))
    check_links(ex, n, len(sizes))
    box = np.searchsorted(off, ex["first"], side="right") - 1
    for b in range(len(sizes)):
        lo, hi = int(off[b]), int(off[b + 1])
        sub = [v[lo:hi].contiguous() for v in xyz]
        one = export(g, ctx, g.g4_build_tree(ctx, g.particles(*sub, m[lo:hi].contiguous()), tp))
        sel = box == b
        assert np.array_equal(ex["first"][sel] - lo, one["first"])
        for k in ("level", "cell", "count", "leaf", "com", "q2", "q3"):
            assert np.array_equal(ex[k][sel], one[k]), k


# windows in memory, eight values a pass: leaf sizes at powers of eight, sets of one more than a leaf, odd ends
@pytest.mark.parametrize("n,B", [(1026, 1025), (4111, 1026), (4098, 4097), (20011, 4094), (20011, 4095), (20011, 4096),
                                 (70003, 32767), (70003, 32768), (70002, 70001), (70002, 70002), (70001, 100000)])
def test_nodes_of_large_leaves(g, n, B):
    ctx = g.Context()
    pos = points(n, n + B)
    tp = g.tree_params(True, 1.0, leaf_max=B)
    x, y, z = g.g4_quantize(ctx, torch.from_numpy(pos).cuda(), tp)
    tree = g.g4_build_tree(ctx, g.particles(x, y, z, torch.ones(n, device="cuda")), tp)
    ex = export(g, ctx, tree)
    X, Y, Z = (v.cpu().numpy().view(np.uint32) for v in (x, y, z))
    level, cell, count, leaf = oracle.Tree(X, Y, Z, np.ones(n), True, 1.0, B).nodes()
    mine = np.column_stack([ex["level"], ex["cell"].view(np.uint32), ex["count"], ex["leaf"]]).astype(np.int64)
    ref = np.column_stack([level, cell, count, leaf]).astype(np.int64)
    assert np.array_equal(mine[np.lexsort(mine.T)], ref[np.lexsort(ref.T)])
    check_links(ex, n)

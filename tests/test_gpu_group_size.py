"""The group size that a caller names is the one the walk uses: a forest equals
the separate trees of its boxes bit for bit at every size of the set, and
small groups make more tree entries than groups of 64."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


KW = dict(kernel=1, r_s=0.01, r_cut=0.07, eps0=0.0005, criterion=1, alpha=0.002, theta_seed=0.7)


def make_forest(g, ctx, sizes, leaf=16):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    pos = torch.from_numpy(np.concatenate([workloads.clustered_box(s, seed=s + k, nhalo=max(1, s // 400)).pos
                                           for k, s in enumerate(sizes)])).cuda()
    mass = torch.full((n,), 1.0 / n, device="cuda")
    tp = g.tree_params(True, 1.0, leaf_max=leaf)
    xyz = g.g4_quantize(ctx, pos, tp)
    f = g.g4_build_forest(ctx, off, g.particles(*xyz, mass), tp)
    g.g4_compute_multipoles(ctx, f, 3)
    return off, f, xyz, mass, tp


# below and above 2^18 particles in all; None: the binding's own default
@pytest.mark.parametrize("sizes,group", [([200003, 50021, 9001, 4001, 70], None), ([200003, 50021, 9001, 4001, 70], 20),
                                         ([131000, 131001, 700], 64), ([90001, 20002, 33], None)])
def test_forest_is_bitwise_its_boxes(g, sizes, group):
    ctx = g.Context()
    off, f, xyz, mass, tp = make_forest(g, ctx, sizes)
    wp = g.walk_params(**KW, **({} if group is None else dict(group_size=group)))
    out = g.g4_treepm_shortrange(ctx, f, wp, want_pot=True)
    for b in range(len(sizes)):
        lo, hi = int(off[b]), int(off[b + 1])
        t = g.g4_build_tree(ctx, g.particles(*[v[lo:hi].contiguous() for v in xyz], mass[lo:hi].contiguous()), tp)
        g.g4_compute_multipoles(ctx, t, 3)
        ref = g.g4_treepm_shortrange(ctx, t, wp, want_pot=True)
        for k in ("ax", "ay", "az", "pot"):
            assert torch.equal(out[k][lo:hi], ref[k]), (b, k)


def test_named_group_size_is_used(g):
    """One wavefront pops the entries of one group, so groups of 8 make more of them than
    groups of 64, of which there are an eighth."""
    ctx = g.Context()
    n = 8192
    ps = workloads.clustered_box(n, seed=4, nhalo=20)
    tp = g.tree_params(True, 1.0, leaf_max=8)
    xyz = g.g4_quantize(ctx, torch.from_numpy(ps.pos).cuda(), tp)
    t = g.g4_build_tree(ctx, g.particles(*xyz, torch.full((n,), 1.0 / n, device="cuda")), tp)
    g.g4_compute_multipoles(ctx, t, 3)
    kw = dict(kernel=1, criterion=0, theta=0.7, r_s=0.03, r_cut=0.2, eps0=0.003)
    e = {s: g.g4_treepm_shortrange(ctx, t, g.walk_params(group_size=s, **kw), want_stats=True)["stats"]["w_entry"]
         for s in (64, 32, 8)}
    assert e[8] > e[32] > e[64] and e[8] >= 2 * e[64], e


# boxes, particles of each, and the group that the rule gives
@pytest.mark.parametrize("nbox,size,group", [(320, 800, 31), (1000, 250, 64), (1100, 30, 64), (12, 2000, 9)])
def test_unset_group_of_a_forest_follows_its_total(g, nbox, size, group):
    """With the size left open a forest is cut by its total (31 a group for 2.56e5 particles)
    or, with many short boxes, into groups of 64; never box by box into groups of 8."""
    ctx = g.Context()
    off, f, xyz, mass, tp = make_forest(g, ctx, [size] * nbox)
    e = {s: g.g4_treepm_shortrange(ctx, f, g.walk_params(group_size=s, **{**KW, "criterion": 0}),
                                   want_stats=True)["stats"]["w_entry"] for s in (0, group)}
    assert e[0] == e[group], e


# 16 targets and eight siblings are the fewest that make 128 slots
@pytest.mark.parametrize("kind", ["box", "plummer"])
@pytest.mark.parametrize("criterion", [0, 1])
def test_group_decisions_by_group_size(g, kind, criterion, monkeypatch):
    """Decisions for whole groups start at 128 (node, target) slots: groups of 15 take none, groups of
    16 to 64 take some, and counts and forces equal those of a walk without any."""
    ctx = g.Context()
    n = 20011
    if kind == "box":
        pos, tp = workloads.clustered_box(n, seed=6, nhalo=40).pos, g.tree_params(True, 1.0, leaf_max=8)
        kw = dict(kernel=1, r_s=0.02, r_cut=0.14, eps0=0.002)
    else:
        pos, tp = workloads.plummer(n, seed=6).pos, g.tree_params(False, 44.0, origin=(-22.0,) * 3, leaf_max=8)
        kw = dict(kernel=0, eps0=0.01)
    xyz = g.g4_quantize(ctx, torch.from_numpy(np.ascontiguousarray(pos)).cuda(), tp)
    t = g.g4_build_tree(ctx, g.particles(*xyz, torch.full((n,), 1.0 / n, device="cuda")), tp)
    g.g4_compute_multipoles(ctx, t, 3)
    geo = g.g4_tree_force(ctx, t, g.walk_params(criterion=0, theta=0.7, **kw))
    seed = torch.sqrt(geo["ax"] ** 2 + geo["ay"] ** 2 + geo["az"] ** 2).float()
    crit = dict(criterion=1, alpha=0.002, a_seed=seed) if criterion else dict(criterion=0, theta=0.6)
    for group in (15, 16, 33, 63, 64):
        out = []
        for per_target in ("0", "1"):
            monkeypatch.setenv("G4_WALK_PER_TARGET", per_target)
            out.append(g.g4_tree_force(ctx, t, g.walk_params(group_size=group, **crit, **kw), want_counts=True,
                                       want_stats=True))
        a, b = out
        assert (a["stats"]["n_group_use"] > 0) == (group >= 16) and b["stats"]["n_group_use"] == 0, group
        assert torch.equal(a["counts"], b["counts"])
        for k in ("ax", "ay", "az"):
            # the same FP32 terms in FP64 sums of another order, some 10^3 of them
            assert (a[k] - b[k]).abs().max().item() <= 1e-12 * b[k].abs().max().item(), (group, k)

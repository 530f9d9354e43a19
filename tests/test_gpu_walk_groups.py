"""The walk cuts small sets into groups smaller than asked for: interaction
counts equal those of other group sizes, forces differ only by the order of
the FP64 sums."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


# 8 targets per wavefront up to 20735 particles, 9 from 20736 on, the full 64 from 2^20 on
@pytest.mark.parametrize("n,leaf", [(1, 8), (2, 8), (63, 8), (20735, 8), (20737, 16), (131007, 24), (1048583, 32)])
def test_group_size_of_small_sets(g, n, leaf):
    ctx = g.Context()
    ps = workloads.clustered_box(n, seed=21, nhalo=max(1, n // 1000)) if n > 100 else workloads.plummer(n, seed=3)
    pos = torch.from_numpy(np.ascontiguousarray(np.mod(ps.pos, 1.0))).cuda()
    mass = torch.full((n,), 1.0 / n, device="cuda")
    scale = (128 ** 3 / n) ** (1 / 3)
    kw = dict(kernel=1, r_s=1.25 / 256 * min(scale, 20.0), r_cut=7 * 1.25 / 256 * min(scale, 20.0),
              eps0=min(scale, 20.0) / (40 * 128))
    tp = g.tree_params(True, 1.0, leaf_max=leaf)
    tree = g.g4_build_tree(ctx, g.particles(*g.g4_quantize(ctx, pos, tp), mass), tp)
    g.g4_compute_multipoles(ctx, tree, 3)
    g.g4_treepm_shortrange(ctx, tree, g.walk_params(criterion=0, theta=0.7, **kw))
    outs = [g.g4_treepm_shortrange(ctx, tree, g.walk_params(criterion=1, alpha=0.002, seed_from_tree=1, group_size=s,
                                                            **kw), want_counts=True, want_pot=True)
            for s in (64, 0, 1, 7)]
    a = outs[0]
    for b in outs[1:]:
        assert torch.equal(a["counts"], b["counts"])
        for k in ("ax", "ay", "az", "pot"):
            # ~10^3 FP64 terms in another order: 10^3 x 2^-53 of the summed magnitudes
            assert (a[k] - b[k]).abs().max().item() <= 1e-12 * max(a[k].abs().max().item(), 1e-300)


def test_forest_groups(g):
    """A forest large enough to fill the chip (2^18 particles) is cut by its total, a smaller one box by
    box: counts as in separate trees, forces to the order of the FP64 sums."""
    ctx = g.Context()
    sizes = [200003, 50021, 9001, 4001]
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    pos = torch.from_numpy(np.concatenate([workloads.clustered_box(s, seed=s, nhalo=20).pos for s in sizes])).cuda()
    mass = torch.full((n,), 1.0 / n, device="cuda")
    kw = dict(kernel=1, r_s=0.01, r_cut=0.07, eps0=0.0005, criterion=1, alpha=0.002, theta_seed=0.7)
    tp = g.tree_params(True, 1.0, leaf_max=16)
    xyz = g.g4_quantize(ctx, pos, tp)
    f = g.g4_build_forest(ctx, off, g.particles(*xyz, mass), tp)
    g.g4_compute_multipoles(ctx, f, 3)
    out = g.g4_treepm_shortrange(ctx, f, g.walk_params(**kw), want_counts=True)
    for b in range(len(sizes)):
        lo, hi = int(off[b]), int(off[b + 1])
        t = g.g4_build_tree(ctx, g.particles(*[v[lo:hi].contiguous() for v in xyz], mass[lo:hi].contiguous()), tp)
        g.g4_compute_multipoles(ctx, t, 3)
        ref = g.g4_treepm_shortrange(ctx, t, g.walk_params(**kw), want_counts=True)
        assert torch.equal(out["counts"][lo:hi], ref["counts"])
        for k in ("ax", "ay", "az"):
            assert (out[k][lo:hi] - ref[k]).abs().max().item() <= 1e-12 * ref[k].abs().max().item()

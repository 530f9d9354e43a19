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


# 2 targets per wavefront up to 4355 particles, 3 from 4356 on, the full 64 from 1982464 on
@pytest.mark.parametrize("n,leaf", [(1, 8), (2, 8), (63, 8), (4355, 8), (4357, 16), (31007, 24), (1982471, 32)])
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

"""The leaf-node pass of the FMM where its packing changes (leaf sizes around
the 16 targets of a walk, one to many pairs per wavefront, coincident particles
in depth-capped leaves, both criteria): the same interactions as the
sorted-list mode, forces to FP32 round-off of the sums."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


@pytest.mark.parametrize("n,leaf,maxd,kernel,crit", [
    (40, 1, 21, 0, 0), (700, 1, 21, 1, 0), (3001, 4, 21, 0, 1), (5003, 15, 21, 1, 0), (5003, 16, 21, 1, 1),
    (5003, 17, 21, 0, 0), (8009, 40, 21, 1, 0), (8009, 100, 21, 0, 0), (6007, 8, 3, 1, 0), (6007, 8, 4, 0, 1)])
@pytest.mark.parametrize("pot", [False, True])
def test_leaf_node_pass(g, n, leaf, maxd, kernel, crit, pot):
    ctx = g.Context()
    pos = workloads.clustered_box(max(n, 100), seed=n, nhalo=max(1, n // 400)).pos[:n]
    if n > 1000:
        pos[:40] = pos[40]  # a pile deeper than any leaf
    scale = min((128 ** 3 / n) ** (1 / 3), 15.0)
    kw = dict(kernel=kernel, theta=0.5, eps0=scale / (40 * 128))
    if kernel == 1:
        kw.update(r_s=1.25 / 256 * scale, r_cut=4.5 * 1.25 / 256 * scale)
    tp = g.tree_params(True, 1.0, leaf_max=leaf, max_depth=maxd)
    xyz = g.g4_quantize(ctx, torch.from_numpy(np.ascontiguousarray(pos)).cuda(), tp)
    mass = torch.rand(n, generator=torch.Generator("cuda").manual_seed(n), device="cuda") + 0.5
    tree = g.g4_build_tree(ctx, g.particles(*xyz, mass), tp)
    g.g4_compute_multipoles(ctx, tree, 3)
    if crit:
        o = g.g4_fmm_force(ctx, tree, g.fmm_params(deterministic=1, **kw))
        kw.update(criterion=1, alpha=0.003,
                  a_seed=torch.sqrt(o["ax"] ** 2 + o["ay"] ** 2 + o["az"] ** 2).float().clamp_min(1e-3).contiguous())
    det = g.g4_fmm_force(ctx, tree, g.fmm_params(deterministic=1, **kw), want_pot=pot, want_stats=True)
    fast = g.g4_fmm_force(ctx, tree, g.fmm_params(deterministic=0, **kw), want_pot=pot, want_stats=True)
    for k in ("n_pp", "n_pn", "n_nn"):
        assert det["stats"][k] == fast["stats"][k], k
    a, b = (torch.stack([o["ax"], o["ay"], o["az"]], 1) for o in (fast, det))
    # up to ~10^3 FP32 terms per sum in another order: 10^3 x 6e-8 at worst against the rms force
    rms = b.square().sum(1).mean().sqrt()
    assert ((a - b).norm(dim=1) / torch.maximum(rms, b.norm(dim=1))).max().item() <= 6e-5
    if pot:
        assert ((fast["pot"] - det["pot"]).abs() / det["pot"].abs().max()).max().item() <= 6e-5

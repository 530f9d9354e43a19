"""The direct sum over all splits of its targets and sources (targets per
block, waves per block, near-pair lists or not), against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


# n: sources, nt: targets (0: all); reach (12 r_s) in box sides; truncate: r_cut in box sides (0: off)
@pytest.mark.parametrize("kernel,n,nt,reach,truncate", [
    (1, 1, 1, 0.1, 0.0), (1, 2, 0, 0.1, 0.0), (1, 63, 0, 0.3, 0.0), (1, 65, 0, 0.34, 0.0), (1, 3000, 1023, 0.1, 0.0),
    (1, 3001, 1024, 0.05, 0.0), (1, 5003, 2049, 0.2, 0.0), (1, 5003, 0, 0.1, 0.03), (1, 5003, 0, 0.5, 0.0),
    (1, 4099, 4097, 0.02, 0.0), (0, 4099, 0, 0.0, 0.2), (0, 2500, 2049, 0.0, 0.0), (0, 777, 5, 0.0, 0.0),
    (0, 2048, 1025, 0.0, 0.0)])
def test_direct_splits(g, kernel, n, nt, reach, truncate):
    ps = workloads.clustered_box(n, seed=5, nhalo=max(1, n // 300))
    ctx = g.Context()
    tp = g.tree_params(True, 1.0, leaf_max=8)
    mass = torch.from_numpy(ps.mass.astype(np.float32)).cuda()
    x, y, z = g.g4_quantize(ctx, torch.from_numpy(ps.pos).cuda(), tp)
    kw = dict(eps0=0.004, **(dict(r_s=reach / 12) if kernel else {}))
    wp = g.walk_params(kernel=kernel, r_cut=truncate or 1e30, **kw)
    tg = torch.from_numpy(workloads.sample_indices(n, nt, seed=4)).cuda() if nt else None
    parts = g.particles(x, y, z, mass)
    out = g.g4_direct_force(ctx, parts, tp, wp, targets=tg, truncate=bool(truncate))
    X, Y, Z = (v.cpu().numpy().view(np.uint32) for v in (x, y, z))
    okw = dict(kw, r_cut=truncate, truncate=True) if truncate else kw
    ref, pref = oracle.direct(X, Y, Z, mass.cpu().numpy().astype(np.float64), 2.0 ** -32, kernel=kernel,
                              targets=None if tg is None else tg.cpu().numpy(), nthreads=8, **okw)
    a = torch.stack([out["ax"], out["ay"], out["az"]], 1).cpu().numpy()
    # n FP64 terms in another order, libm and device erfc/exp within a few ulp of each other
    tol = 1e-12 * np.abs(ref).max() if n > 1 else 0.0
    np.testing.assert_allclose(a, ref, rtol=1e-11, atol=max(tol, 1e-300))
    np.testing.assert_allclose(out["pot"].cpu().numpy(), pref, rtol=1e-11, atol=1e-12 * np.abs(pref).max())
    # the order of the sums is fixed: a second call gives the same bits
    again = g.g4_direct_force(ctx, parts, tp, wp, targets=tg, truncate=bool(truncate))
    for k in ("ax", "ay", "az", "pot"):
        assert torch.equal(out[k], again[k])

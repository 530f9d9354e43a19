"""The direct sum's near-pair lists at reaches up to half the box, for targets
and sources on both sides of the box faces, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


# n sources around the edges of a step (4 x 64 per wavefront, 8 or 16 wavefronts), nt targets around
# the changes of targets per block; reach in box sides (12 r_s of the
# split force in a periodic box, r_cut of the truncated Newtonian sum in an open one), 0.4938 the largest with lists
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("n,nt,reach", [
    (255, 3, 0.4938), (256, 256, 0.4939), (257, 40, 0.25), (2049, 1025, 0.4), (4097, 2047, 0.45), (4095, 2049, 0.02),
    (1300, 8191, 0.3), (700, 8193, 0.4938), (9000, 300, 2e-5)])
def test_direct_reach(g, periodic, n, nt, reach):
    rng = np.random.default_rng(n + nt)
    pos = rng.random((n, 3))
    k = n // 3
    # a third within 1e-4 of the faces, a few exactly one reach from another one along an axis
    pos[:k] = np.where(rng.random((k, 3)) < 0.5, pos[:k] * 1e-4, 1.0 - pos[:k] * 1e-4)
    pos[k + 1] = pos[k] + [reach, 0.0, 0.0]
    pos[k + 2] = pos[k] - [0.0, reach, 0.0]
    pos -= np.floor(pos)
    pos[pos >= 1.0] = 0.0
    ctx = g.Context()
    tp = g.tree_params(periodic, 1.0, leaf_max=8)
    unit = 2.0 ** -32 if periodic else 2.0 ** -31
    x, y, z = g.g4_quantize(ctx, torch.from_numpy(pos).cuda(), tp)
    m = rng.random(n).astype(np.float32)
    # softened pairs lie within the reach
    kw = dict(eps0=min(0.002, reach / 20), **(dict(r_s=reach / 12) if periodic else dict(r_cut=reach)))
    tg = torch.from_numpy(rng.integers(0, n, nt)).cuda()
    out = g.g4_direct_force(ctx, g.particles(x, y, z, torch.from_numpy(m).cuda()), tp,
                            g.walk_params(kernel=int(periodic), **dict(dict(r_cut=1e30), **kw)), targets=tg,
                            truncate=not periodic)
    X, Y, Z = (v.cpu().numpy().view(np.uint32) for v in (x, y, z))
    ref, pref = oracle.direct(X, Y, Z, m.astype(np.float64), unit, kernel=int(periodic),
                              targets=tg.cpu().numpy(), truncate=not periodic, nthreads=8, **kw)
    a = torch.stack([out["ax"], out["ay"], out["az"]], 1).cpu().numpy()
    # n FP64 terms in another order, libm and device erfc/exp within a few ulp; a pair at the reach is 1e-16 of a near one
    np.testing.assert_allclose(a, ref, rtol=1e-11, atol=max(1e-12 * np.abs(ref).max(), 1e-300))
    np.testing.assert_allclose(out["pot"].cpu().numpy(), pref, rtol=1e-11, atol=max(1e-12 * np.abs(pref).max(), 1e-300))

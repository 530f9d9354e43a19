"""The PM force at every mesh size (line lengths 8 to 1024, each radix
sequence of the transforms) against the same steps in 64-bit torch."""
import math

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2010_03567_amd.g4hip as m
    return m


def reference(X, mass, ng, box, r_s, G):
    """CIC, real FFT, Green's function with the window deconvolved, 4th-order differences, CIC."""
    sh = 32 - int(math.log2(ng))
    cell, f = X >> sh, (X & ((1 << sh) - 1)).double() / 2.0 ** sh

    def at(o):
        i = [(cell[:, k] + o[k]) & (ng - 1) for k in range(3)]
        return (i[0] * ng + i[1]) * ng + i[2]

    def weight(o):
        return math.prod((f[:, k] if o[k] else 1 - f[:, k]) for k in range(3))

    corners = [(c >> 2, (c >> 1) & 1, c & 1) for c in range(8)]
    M = torch.zeros(ng ** 3, dtype=torch.float64, device="cuda")
    for o in corners:
        M.index_add_(0, at(o), mass * weight(o))
    F = torch.fft.rfftn(M.view(ng, ng, ng))
    n = torch.fft.fftfreq(ng, d=1.0 / ng, device="cuda", dtype=torch.float64)
    nz = n[:ng // 2 + 1].abs()
    sc, scz = torch.sinc(n / ng) ** 4, torch.sinc(nz / ng) ** 4
    kf = 2 * math.pi / box
    for i in range(ng):
        k2 = (n[i] ** 2 + n[:, None] ** 2 + nz[None, :] ** 2) * kf ** 2
        gr = -G * 4 * math.pi / box ** 3 * torch.exp(-k2 * r_s ** 2) / k2 / (sc[i] * sc[:, None] * scz[None, :]) * ng ** 3
        if i == 0:
            gr[0, 0] = 0
        F[i] *= gr
    phi = torch.fft.irfftn(F, s=(ng, ng, ng)).reshape(-1)
    acc, pot = [], sum(weight(o) * phi[at(o)] for o in corners)
    for k in range(3):
        a = torch.zeros_like(pot)
        for o in corners:
            for d, c in ((1, 2 / 3), (2, -1 / 12)):
                for sg in (1, -1):
                    oo = list(o)
                    oo[k] += sg * d
                    a -= weight(o) * (sg * c * ng / box) * phi[at(oo)]
        acc.append(a)
    return acc, pot


@pytest.mark.parametrize("ng,n,keys", [(8, 1, 0), (8, 300, 0), (16, 3001, 0), (32, 777, 1), (64, 3001, 0), (128, 3001, 0),
                                       (256, 20011, 0), (512, 20011, 1), (1024, 3001, 0), (32, 70001, 0), (64, 500009, 1),
                                       # tiles (from 5e5 particles, a third of that from 128^3 on, and 100 per
                                       # 16^3 cells): one cube, staged or not, several items a cube
                                       (16, 500000, 0), (32, 500003, 1), (128, 500003, 0), (256, 600011, 1),
                                       (128, 166665, 0), (128, 166666, 1), (128, 1300003, 0), (256, 409600, 0)])
def test_pm_sizes(g, ng, n, keys):
    ctx = g.Context()
    box, G = 2.5, 0.7
    ps = workloads.clustered_box(max(n, 100), seed=9, nhalo=max(1, n // 500))
    tp = g.tree_params(True, box, leaf_max=16, key_kind=keys)
    pos = torch.from_numpy(ps.pos[:n] * box).cuda().contiguous()
    m = torch.rand(n, generator=torch.Generator("cuda").manual_seed(n), device="cuda") + 0.5
    x, y, z = g.g4_quantize(ctx, pos, tp)
    tree = g.g4_build_tree(ctx, g.particles(x, y, z, m), tp)
    r_s = 1.25 * box / ng
    ws = torch.empty(g.g4_pm_workspace_bytes(ng) + 256, dtype=torch.uint8, device="cuda")
    out = g.g4_pm_longrange(ctx, tree, g.pm_params(ng, r_s, G), ws=ws, want_pot=True)
    X = torch.stack([v.long() & 0xffffffff for v in (x, y, z)], 1)
    acc, pot = reference(X, m.double(), ng, box, r_s, G)
    # FP32 mesh values with about 3 log2 ng roundings each way; the differences cancel all but
    # ~ 1 / 3 of a neighbour's potential: 3e-6 of the rms force, tails of the sampled noise 30 times that
    rms = torch.stack(acc).square().mean().sqrt().clamp_min(1e-300)
    if n == 1:  # only its own mesh force, zero up to rounding
        return
    for k, c in enumerate(("ax", "ay", "az")):
        d = (out[c] - acc[k]).abs() / torch.maximum(rms, acc[k].abs())
        assert d.square().mean().sqrt().item() <= 3e-6 and d.max().item() <= 1e-4, (c, d.max().item())
    assert ((out["pot"] - pot).abs() / pot.abs().max()).max().item() <= 3e-6
    # the accumulate mode adds the same values (the deposit's atomics round in another order)
    more = g.g4_pm_longrange(ctx, tree, g.pm_params(ng, r_s, G), ws=ws, accumulate=True,
                             out=tuple(torch.ones_like(out["ax"]) for _ in range(4)))
    for c in ("ax", "ay", "az", "pot"):
        assert (more[c] - 1 - out[c]).abs().max().item() <= 1e-4 * max(rms.item(), out[c].abs().max().item())


@pytest.mark.parametrize("ng", [16, 64])
def test_pm_of_one_particle(g, ng):
    """A single particle feels no force but its own mesh force, which vanishes up to rounding; its
    potential is that of the 64-bit reference; accumulating adds the same."""
    ctx = g.Context()
    box, G = 2.5, 0.7
    tp = g.tree_params(True, box, leaf_max=16)
    pos = torch.tensor([[0.3, 1.9, 2.4]], dtype=torch.float64, device="cuda")
    m = torch.tensor([1.5], device="cuda")
    x, y, z = g.g4_quantize(ctx, pos, tp)
    tree = g.g4_build_tree(ctx, g.particles(x, y, z, m), tp)
    r_s = 1.25 * box / ng
    out = g.g4_pm_longrange(ctx, tree, g.pm_params(ng, r_s, G), want_pot=True)
    X = torch.stack([v.long() & 0xffffffff for v in (x, y, z)], 1)
    acc, pot = reference(X, m.double(), ng, box, r_s, G)
    assert (out["pot"] - pot).abs().item() <= 3e-6 * pot.abs().item()
    # the antisymmetric differences cancel to the rounding of the potential over a cell
    for k, c in enumerate(("ax", "ay", "az")):
        assert (out[c] - acc[k]).abs().item() <= 1e-5 * pot.abs().item() * ng / box, c
    more = g.g4_pm_longrange(ctx, tree, g.pm_params(ng, r_s, G), accumulate=True,
                             out=tuple(torch.ones_like(out["ax"]) for _ in range(4)))
    for c in ("ax", "ay", "az", "pot"):
        assert (more[c] - 1 - out[c]).abs().item() <= 1e-5 * pot.abs().item() * ng / box, c


def test_pm_of_an_infinite_split_scale(g):
    """exp(-k^2 r_s^2) is zero for every wave but k = 0, which the force drops: all zero."""
    ctx = g.Context()
    tp = g.tree_params(True, 1.0, leaf_max=16)
    ps = workloads.clustered_box(1000, seed=3, nhalo=4)
    x, y, z = g.g4_quantize(ctx, torch.from_numpy(ps.pos).cuda(), tp)
    tree = g.g4_build_tree(ctx, g.particles(x, y, z, torch.ones(1000, device="cuda")), tp)
    out = g.g4_pm_longrange(ctx, tree, g.pm_params(32, math.inf), want_pot=True)
    for c in ("ax", "ay", "az", "pot"):
        assert torch.all(out[c] == 0), c

"""The direct sum for more targets than one launch's grid can hold."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# near-pair lists (8 targets a block of 512 threads) and sums without them (4 a block of 256): both
# reach 2^32 threads at 2^26 targets; one block past that, the last one not full
@pytest.mark.parametrize("reach", [0.3, 0.6])
def test_more_targets_than_a_grid_holds(reach):
    import paper_2010_03567_amd.g4hip as g
    ctx = g.Context()
    n, nt = 3, 2 ** 26 + 13
    pos = torch.tensor([[0.1, 0.2, 0.3], [0.15, 0.22, 0.31], [0.6, 0.7, 0.4]], dtype=torch.float64, device="cuda")
    tp = g.tree_params(True, 1.0)
    p = g.particles(*g.g4_quantize(ctx, pos, tp), torch.tensor([1.0, 2.0, 3.0], device="cuda"))
    wp = g.walk_params(kernel=1, r_s=reach / 12, eps0=0.001)
    few = g.g4_direct_force(ctx, p, tp, wp, targets=torch.arange(n, dtype=torch.int64, device="cuda"))
    targets = torch.arange(nt, dtype=torch.int64, device="cuda") % n
    many = g.g4_direct_force(ctx, p, tp, wp, targets=targets)
    for k in ("ax", "ay", "az", "pot"):
        # two terms a sum: their order does not matter
        assert torch.equal(many[k], few[k][targets]), k

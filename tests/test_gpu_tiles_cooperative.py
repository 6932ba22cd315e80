"""V-cycles whose small levels run in the fused steps (csrc/tile.hip) against the same cycle
as one cooperative launch (csrc/coarse.hip), as either may be chosen by timing: the same
sums in another order."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dims,levels", [((32, 16, 16), 4), ((24, 20, 28), 3)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_cooperative_cycle_equals_the_fused_steps(dims, levels, dtype):
    from paper_2201_12931_amd import hexmg

    print(f"case tiles cooperative {dims} levels={levels} {dtype}", flush=True)
    g = W.Grid(*dims)
    mask = W.fixed_mask_face_x0(g)
    rng = np.random.default_rng(9)
    at = rng.permutation(g.n_node)[: g.n_node // 17]
    mask[at] |= rng.integers(1, 8, size=at.size).astype(np.uint8)
    dt = hexmg.F64 if dtype == torch.float64 else hexmg.F32
    grid = hexmg.Grid(*dims, levels, fixed_mask=torch.from_numpy(mask).cuda(), vcycle_both=1)
    grid.set_density(torch.from_numpy(W.random_field_density(g, seed=8, length_scale=3.0, lo=0.05)).cuda())
    r = torch.from_numpy(W.random_vector(g.n_dof, seed=7)).to("cuda", dtype)
    grid.set_coarse_cycle(dt, 0)
    ref = torch.empty_like(r)
    grid.vcycle(r, ref)
    # five products of some 200 terms on each of two or three levels, each up to a few
    # times the vector that it leaves; in binary32 no more than the oracle comparisons allow
    tol = min(1e4 * torch.finfo(dtype).eps, 1e-4)
    for level in range(1, levels - 1):
        grid.set_coarse_cycle(dt, level)
        z = torch.full_like(r, float("nan"))
        grid.vcycle(r, z)
        assert float((z - ref).norm()) <= tol * float(ref.norm()), level

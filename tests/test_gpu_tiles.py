"""Fused steps of the small levels (csrc/tile.hip): V-cycles with such levels inside against
the oracle, and solves that start on one (level 0) against the same solve launched
step by step, at sizes around the tile (4 x 4 x 2 nodes) and on both sides of the
size limit, with scattered supports and several right-hand sides."""
import numpy as np
import pytest

import workloads as W
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def case(dims, every=17):
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=8, length_scale=3.0, lo=0.05)
    mask = W.fixed_mask_face_x0(g)
    rng = np.random.default_rng(9)
    at = rng.permutation(g.n_node)[: max(1, g.n_node // every)]
    mask[at] |= rng.integers(1, 8, size=at.size).astype(np.uint8)
    return g, rho, mask


# (36, 32, 32) and (40, 32, 32): level 1 just below and just above the limit
@pytest.mark.parametrize("dims,levels", [((4, 4, 4), 3), ((8, 4, 12), 3), ((20, 12, 28), 3), ((36, 20, 4), 3),
                                         ((32, 16, 24), 4), ((36, 32, 32), 3), ((40, 32, 32), 3)])
def test_vcycle_oracle(dims, levels):
    from paper_2201_12931_amd import hexmg

    print(f"case tiles vcycle dims={dims} levels={levels}", flush=True)
    g, rho, mask = case(dims)
    h = mg.Hierarchy(*dims, rho, mask, levels)
    r = W.random_vector(g.n_dof, seed=7) * h.free[0]
    ref = h.vcycle(r)
    grid = hexmg.Grid(*dims, levels, fixed_mask=gpu(mask), vcycle_both=1)
    grid.set_density(gpu(rho))
    # the tolerances of the V-cycle's other comparisons with the oracle
    for dt, tol in ((torch.float64, 1e-10), (torch.float32, 1e-4)):
        z = torch.full((g.n_dof,), float("nan"), dtype=dt, device="cuda")
        grid.vcycle(gpu(r).to(dt), z)
        assert np.linalg.norm(z.cpu().numpy() - ref) <= tol * np.linalg.norm(ref), dt


@pytest.mark.parametrize("precision,tol", [("FP64", 1e-9), ("MIXED", 1e-3), ("MIXED32", 1e-3)])
@pytest.mark.parametrize("dims,levels,nrhs", [((4, 2, 2), 2, 1), ((6, 10, 14), 2, 3), ((20, 12, 8), 3, 2),
                                              ((22, 14, 12), 2, 1), ((18, 16, 16), 2, 1)])
def test_solve_equals_the_step_launches(precision, tol, dims, levels, nrhs):
    """Four iterations on either path: the same sums in another order.  A V-cycle differs
    by roundings (2^-52 or 2^-24, times the 1e2 to 1e3 terms of its chain of
    products and the growth over four iterations)."""
    from paper_2201_12931_amd import hexmg

    print(f"case tiles solve {precision} dims={dims} nrhs={nrhs}", flush=True)
    g, rho, mask = case(dims)
    f = W.point_loads(g, nrhs, seed=3)
    out = []
    for step in (False, True):
        grid = hexmg.Grid(*dims, levels, fixed_mask=gpu(mask), precision=getattr(hexmg, precision), max_nrhs=nrhs)
        grid.set_density(gpu(rho))
        if step:
            for l in range(levels):
                for dt in (hexmg.F64, hexmg.F32):
                    grid.set_kernel_choice(l, dt, hexmg.KERNEL_GATHER)
        u = torch.full((nrhs, g.n_dof), float("nan"), dtype=torch.float64, device="cuda")
        _, info = grid.solve(gpu(f), u, rtol=1e-30, maxit=4)
        out.append((u.cpu().numpy(), [i["compliance"] for i in info]))
    for k in range(nrhs):
        a, b = out[0][0][k], out[1][0][k]
        assert np.all(np.isfinite(a))
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b), k
        assert abs(out[0][1][k] - out[1][1][k]) <= tol * abs(out[1][1][k])

"""The explicit inverse of the coarsest operator (block sweeps on 64x64 tiles) at
the edges of its tiles: one-level grids, whose V-cycle is that inverse, of 24 to
2304 DOFs (single tile, exact multiples of 64, remainders)."""
import numpy as np
import pytest

import workloads as W
from oracle import fem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EPS = 2.0 ** -52


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 1), (6, 2, 2), (3, 3, 3), (4, 3, 3), (7, 3, 3), (12, 6, 6),
                                  (15, 7, 5)])
def test_one_level_vcycle_inverts_the_operator(dims):
    from paper_2201_12931_amd import hexmg

    g = W.Grid(*dims)
    print(f"case inverse dims={dims} n={g.n_dof}", flush=True)
    rho = W.iid_uniform_density(g, seed=5, lo=0.05)
    grid = hexmg.Grid(*dims, 1, precision=hexmg.FP64)
    grid.set_density(torch.from_numpy(rho).cuda())
    free = fem.free_dof_mask(W.fixed_mask_face_x0(g))
    A = fem.assemble_stiffness(*dims, fem.simp_modulus(rho)).toarray()
    A[~free] = 0.0
    A[:, ~free] = 0.0
    A[~free, ~free] = 1.0
    r = W.random_vector(g.n_dof, seed=6)
    z = torch.empty(g.n_dof, dtype=torch.float64, device="cuda")
    grid.vcycle(torch.from_numpy(r).cuda(), z)
    z = z.cpu().numpy()
    # an explicit inverse of relative error n eps kappa leaves a residual of that size
    lam = np.linalg.eigvalsh(A)
    assert np.linalg.norm(A @ z - r) <= g.n_dof * EPS * lam[-1] / lam[0] * np.linalg.norm(r)
    ref = np.linalg.solve(A, r)
    assert np.linalg.norm(z - ref) <= g.n_dof * EPS * lam[-1] / lam[0] * np.linalg.norm(ref)

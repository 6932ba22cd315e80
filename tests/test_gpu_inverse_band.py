"""The coarsest inverse swept from both ends of a banded operator: one-level grids
(whose V-cycle is that inverse) with narrow bands, so that most steps take two
pivots, and with an even or odd number of tiles left for the single ones."""
import numpy as np
import pytest

import workloads as W
from oracle import fem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EPS = 2.0 ** -52


# 64-wide tiles and the tiles that a band spans: 8/1, 9/1, 6/1, 12/2, 12/3, 27/3
@pytest.mark.parametrize("dims", [(1, 1, 40), (1, 1, 46), (1, 2, 19), (2, 3, 20), (3, 3, 15), (5, 4, 18)])
def test_banded_inverse(dims):
    from paper_2201_12931_amd import hexmg

    g = W.Grid(*dims)
    print(f"case banded inverse dims={dims} n={g.n_dof}", flush=True)
    rho = W.iid_uniform_density(g, seed=5, lo=0.3)
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
    bound = g.n_dof * EPS * lam[-1] / lam[0]
    assert np.linalg.norm(A @ z - r) <= bound * np.linalg.norm(r)
    ref = np.linalg.solve(A, r)
    assert np.linalg.norm(z - ref) <= bound * np.linalg.norm(ref)

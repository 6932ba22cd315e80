"""Supports among void elements so soft that omega / diag(A) overflows binary32:
a fully fixed node has a zero right-hand side and takes no part."""
import numpy as np
import pytest

import workloads as W
from oracle import fem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (MIXED32 reaches this rtol on the small grid only)
@pytest.mark.parametrize("precision,dims,levels", [("FP64", (8, 4, 4), 2), ("MIXED", (8, 4, 4), 2),
                                                   ("MIXED32", (8, 4, 4), 2), ("FP64", (48, 16, 16), 3),
                                                   ("MIXED", (48, 16, 16), 3)])
def test_void_corner_at_the_fixed_face(precision, dims, levels):
    from paper_2201_12931_amd import hexmg

    print(f"case void corner {precision} dims={dims}", flush=True)
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=5, length_scale=4.0, lo=0.3)
    rho[0] = 0.0  # the one element of the fixed corner node
    f = W.cantilever_line_load(g)
    emin = 1e-40
    free = fem.free_dof_mask(W.fixed_mask_face_x0(g))
    u_ref = fem.solve_direct(fem.assemble_stiffness(*dims, fem.simp_modulus(rho, Emin=emin)), f, free)
    grid = hexmg.Grid(*dims, levels, precision=getattr(hexmg, precision), Emin=emin)
    grid.set_density(torch.from_numpy(rho).cuda())
    u = torch.full((g.n_dof,), float("nan"), dtype=torch.float64, device="cuda")
    code, info = grid.solve(torch.from_numpy(f).cuda(), u, rtol=1e-8, maxit=200)
    assert code == 0, info
    # the residual test, amplified by the operator's condition number in the energy product
    assert info[0]["compliance"] == pytest.approx(fem.compliance(f, u_ref), rel=1e-6)

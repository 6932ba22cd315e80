"""CG's vector passes on both sides of the size up to which a thread's elements are
requested ahead (1 M unknowns): after a few iterations, in each precision and with
a right-hand side that stops at once, the recursive residual is the true one."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 989235 and 1078155 unknowns
@pytest.mark.parametrize("dims", [(88, 64, 56), (96, 64, 56)])
@pytest.mark.parametrize("precision", ["FP64", "MIXED", "MIXED32"])
@pytest.mark.parametrize("maxit", [1, 2, 3, 4])
def test_recursive_residual_is_the_true_one(dims, precision, maxit):
    from paper_2201_12931_amd import hexmg

    print(f"case vector passes {precision} dims={dims} maxit={maxit}", flush=True)
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=3, length_scale=4.0, lo=0.3)
    f = np.zeros((2, g.n_dof))
    f[1] = W.point_loads(g, 1, seed=5)[0]
    grid = hexmg.Grid(*dims, 4, precision=getattr(hexmg, precision), max_nrhs=2)
    grid.set_density(torch.from_numpy(rho).cuda())
    u = torch.full((2, g.n_dof), float("nan"), dtype=torch.float64, device="cuda")
    _, info = grid.solve(torch.from_numpy(f).cuda(), u, rtol=1e-30, maxit=maxit)
    assert info[0]["iterations"] == 0 and bool((u[0] == 0).all())
    assert info[1]["iterations"] == maxit and bool(torch.isfinite(u[1]).all())
    # |K| |u| is of the size of one unit of load per unknown (moduli in [0.03, 1], tip
    # deflections of a few units), in norm 1e3 |f|; ten roundings each, in the format K p is
    # formed in.  A lost or doubled update changes the residual by itself.
    eps = 2.0 ** -24 if precision == "MIXED32" else 2.0 ** -53
    a, b = info[1]["rel_res_true"], info[1]["rel_res_recursive"]
    assert abs(a - b) <= 1e4 * eps * maxit + 1e-9 * b

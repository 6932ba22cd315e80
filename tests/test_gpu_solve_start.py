"""x is written from zero by its first update instead of being cleared: solves into
a buffer of NaN, stopped after 0 to 5 iterations, one of two right-hand sides
zero, in each precision and on a one-level grid (one iteration); the reported
true residual and compliance against the oracle's operator."""
import numpy as np
import pytest

import workloads as W
from oracle import fem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precision", ["FP64", "MIXED", "MIXED32"])
@pytest.mark.parametrize("dims,levels", [((4, 2, 2), 1), ((20, 12, 8), 3)])
@pytest.mark.parametrize("maxit", [0, 1, 2, 3, 5])
def test_first_updates_into_nan(precision, dims, levels, maxit):
    from paper_2201_12931_amd import hexmg

    print(f"case start {precision} dims={dims} maxit={maxit}", flush=True)
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=3, length_scale=4.0, lo=0.05)
    free = fem.free_dof_mask(W.fixed_mask_face_x0(g))
    K = fem.assemble_stiffness(*dims, fem.simp_modulus(rho))
    f = np.zeros((2, g.n_dof))
    f[0] = W.cantilever_line_load(g)
    grid = hexmg.Grid(*dims, levels, precision=getattr(hexmg, precision), max_nrhs=2, rr_every=2)
    grid.set_density(gpu(rho))
    u = torch.full((2, g.n_dof), float("nan"), dtype=torch.float64, device="cuda")
    code, info = grid.solve(gpu(f), u, rtol=1e-30, maxit=maxit)
    u = u.cpu().numpy()
    assert np.all(u[1] == 0.0) and info[1]["iterations"] == 0
    assert np.all(np.isfinite(u[0])) and np.all(u[0][~free] == 0.0)
    assert info[0]["iterations"] == maxit or maxit > 1 and levels == 1  # exhausted in exact arithmetic
    r = f[0] - K @ u[0]
    nf = np.linalg.norm(f[0][free])
    # both sides form the residual from terms of the size |K| |u|
    noise = 60 * 2.0 ** -52 * np.linalg.norm((abs(K) @ np.abs(u[0]))[free]) / nf
    assert abs(info[0]["rel_res_true"] - np.linalg.norm(r[free]) / nf) <= noise + 1e-12 * info[0]["rel_res_true"]
    assert abs(info[0]["compliance"] - f[0] @ u[0]) <= 1e-13 * (np.abs(f[0]) @ np.abs(u[0])) + 1e-300
    if maxit == 0:
        assert np.all(u[0] == 0.0) and info[0]["rel_res_true"] == pytest.approx(1.0, rel=1e-14)


def test_streamed_final_residual_equals_the_separate_pass():
    """The true residual and compliance from the streaming product's own pass, for each
    of its shapes, one-plane and longer chunks, against the node-gather product's."""
    from paper_2201_12931_amd import hexmg

    dims, levels = (64, 24, 8), 3
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=4, length_scale=4.0, lo=0.05)
    f = gpu(W.point_loads(g, 2, seed=5))
    grid = hexmg.Grid(*dims, levels, precision=hexmg.FP64, max_nrhs=2)
    grid.set_density(gpu(rho))
    ref = None
    for choice in [None] + [(z, s) for s in range(3) for z in (1, 2, 3, 16)]:
        for l in range(levels):
            if choice is None:
                grid.set_kernel_choice(l, hexmg.F64, hexmg.KERNEL_GATHER)
            else:
                grid.set_kernel_choice(l, hexmg.F64, hexmg.KERNEL_STREAM, *choice)
        u = torch.empty_like(f)
        _, info = grid.solve(f, u, rtol=0.0, maxit=3)
        got = np.array([[i["rel_res_true"], i["compliance"]] for i in info])
        ref = got if ref is None else ref
        assert np.allclose(got, ref, rtol=1e-10, atol=0.0), choice

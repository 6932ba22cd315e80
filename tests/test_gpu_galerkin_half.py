"""Galerkin stencils stored by their symmetric half: every level's operator with
supports scattered over single components of interior and boundary nodes, on
grids whose node counts leave remainders of the 64-node blocks, several
right-hand sides, against the oracle's P~^T A P~ + (I - M)."""
import numpy as np
import pytest

import workloads as W
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims,levels", [((2, 2, 2), 2), ((4, 2, 6), 2), ((24, 8, 16), 4), ((64, 4, 4), 3)])
@pytest.mark.parametrize("every", [3, 17])
def test_operator_with_scattered_supports(dims, levels, every):
    from paper_2201_12931_amd import hexmg

    print(f"case galerkin half dims={dims} levels={levels} every={every}", flush=True)
    g = W.Grid(*dims)
    rho = W.random_field_density(g, seed=8, length_scale=3.0, lo=0.05)
    mask = W.fixed_mask_face_x0(g)
    rng = np.random.default_rng(9)
    at = rng.permutation(g.n_node)[: max(1, g.n_node // every)]
    mask[at] |= rng.integers(1, 8, size=at.size).astype(np.uint8)
    grid = hexmg.Grid(*dims, levels, coarse_op=hexmg.COARSE_GALERKIN, fixed_mask=gpu(mask), max_nrhs=2)
    grid.set_density(gpu(rho))
    h = mg.Hierarchy(*dims, rho, mask, levels, coarse_operator="galerkin", omega=0.5)
    for l in range(1, levels):
        n = h.A[l].shape[0]
        u = W.random_vector(n, seed=50 + l, nrhs=2)
        y = torch.empty((2, n), dtype=torch.float64, device="cuda")
        grid.apply_K(gpu(u), y, level=l)
        ref = (h.A[l] @ u.T).T
        # at most 81 products per row, from coefficients summed over fewer than 2^12 terms
        bound = 2.0 ** -52 * 2 ** 12 * (abs(h.A[l]) @ np.abs(u).T).T + 1e-300
        assert np.all(np.abs(y.cpu().numpy() - ref) <= bound), l
        y32 = torch.empty((2, n), dtype=torch.float32, device="cuda")
        grid.apply_K(gpu(u.astype(np.float32)), y32, level=l)
        bound32 = 2.0 ** -23 * 2 * 84 * (abs(h.A[l]) @ np.abs(u).T).T
        assert np.all(np.abs(y32.cpu().numpy() - ref) <= bound32), l

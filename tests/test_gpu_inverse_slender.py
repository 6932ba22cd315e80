"""Accuracy of the coarsest inverse on slender, ill-conditioned grids: the order in which
its blocks are swept must not lose digits against the natural order.  One-level
grids (whose V-cycle is that inverse) against block sweeps in the natural order in
numpy, both measured against a solve refined with residuals in extended precision."""
import numpy as np
import pytest
import scipy.linalg as sla

import workloads as W
from oracle import fem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BLOCK = 64


def sweeps_in_order(A):
    """-(A swept over every block) = A^-1, binary64, blocks from the first to the last."""
    n = len(A)
    m = np.eye(-(-n // BLOCK) * BLOCK)
    m[:n, :n] = A
    for k in range(0, len(m), BLOCK):
        K = slice(k, k + BLOCK)
        D = np.linalg.inv(m[K, K])
        C, X = m[:, K].copy(), D @ m[K]
        m = m - C @ X
        m[K], m[:, K], m[K, K] = X, C @ D, -D
    return -0.5 * (m + m.T)[:n, :n]


def refined_solve(A, B):
    d = 1.0 / np.sqrt(np.diag(A))
    c = sla.cho_factor(A * d[:, None] * d)
    step = lambda R: d[:, None] * sla.cho_solve(c, d[:, None] * R)
    X = step(B).astype(np.longdouble)
    for _ in range(6):
        X = X + step((B.astype(np.longdouble) - A.astype(np.longdouble) @ X).astype(np.float64))
    return X


def test_sweeps_from_both_ends_keep_the_accuracy():
    from paper_2201_12931_amd import hexmg

    ratios = []
    for dims in ((20, 1, 2), (24, 1, 2), (20, 2, 2)):
        g = W.Grid(*dims)
        free = fem.free_dof_mask(W.fixed_mask_face_x0(g))
        for seed in range(6):
            rho = W.random_field_density(g, seed=seed, length_scale=2.0, lo=0.05)
            A = fem.assemble_stiffness(*dims, fem.simp_modulus(rho, Emin=1e-3)).toarray()
            A[~free] = 0.0
            A[:, ~free] = 0.0
            A[~free, ~free] = 1.0
            r = W.random_vector(g.n_dof, seed=30 + seed)
            x = refined_solve(A, r[:, None])[:, 0]
            error = lambda z: float(np.linalg.norm((z - x).astype(np.float64)) / np.linalg.norm(x.astype(np.float64)))
            grid = hexmg.Grid(*dims, 1, Emin=1e-3)
            grid.set_density(torch.from_numpy(rho).cuda())
            z = torch.empty(g.n_dof, dtype=torch.float64, device="cuda")
            grid.vcycle(torch.from_numpy(r).cuda(), z)
            e, e0 = error(z.cpu().numpy()), error(sweeps_in_order(A) @ r)
            print(f"case slender inverse {dims} seed {seed}: error {e:.1e}, in order {e0:.1e}", flush=True)
            ratios.append(e / e0)
    # single cases spread by up to ten either way; a lost digit shows in the mean of 18
    assert np.exp(np.mean(np.log(ratios))) <= 4.0

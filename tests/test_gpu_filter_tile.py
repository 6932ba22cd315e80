"""The tiled filters (half-widths 1..3) against the oracle at the edges of their
tiles (32 x 8 columns), z-chunks and distance classes, beside the general kernel's
first half-width; and inputs that a zero weight must not let in."""
import numpy as np
import pytest

import workloads as W
from oracle import topopt as T

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EPS = 2.0 ** -52


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims", [(1, 1, 1), (31, 8, 4), (33, 7, 5), (32, 9, 33), (2, 1, 70), (97, 17, 6)])
@pytest.mark.parametrize("rmin", [1.2, 1.6, 2.0, 2.3, 2.9, 3.0, 3.7, 4.0, 4.2])
def test_filters_match_oracle(dims, rmin):
    from paper_2201_12931_amd import hexmg

    print(f"case filter tile dims={dims} rmin={rmin}", flush=True)
    H, Hs = T.filter_matrix(*dims, rmin)
    n = int(np.prod(dims))
    x = W.random_vector(n, seed=7)
    # every sum has at most m terms of one rounding each, on either side
    m = 2 * np.diff(H.indptr).max() + 8
    absH = abs(H)
    y = hexmg.density_filter(*dims, rmin, gpu(x)).cpu().numpy()
    assert np.all(np.abs(y - (H @ x) / Hs) <= m * EPS * (absH @ np.abs(x)) / Hs)
    ya = hexmg.density_filter(*dims, rmin, gpu(x), adjoint=True).cpu().numpy()
    assert np.all(np.abs(ya - H @ (x / Hs)) <= m * EPS * (absH @ np.abs(x / Hs)))
    rho = np.abs(W.random_vector(n, seed=8)) * 0.5
    s = hexmg.sensitivity_filter(*dims, rmin, gpu(rho), gpu(x), gamma=1e-3).cpu().numpy()
    den = np.maximum(1e-3, rho) * Hs
    assert np.all(np.abs(s - (H @ (rho * x)) / den) <= m * EPS * (absH @ np.abs(rho * x)) / den)


@pytest.mark.parametrize("rmin", [1.4, 2.0, 2.4, 3.0, 3.5])
def test_non_finite_inputs_reach_only_their_neighbours(rmin):
    from paper_2201_12931_amd import hexmg

    dims = (37, 11, 9)
    H, Hs = T.filter_matrix(*dims, rmin)
    n = int(np.prod(dims))
    x = W.random_vector(n, seed=9)
    e = 18 + 37 * (5 + 11 * 4)
    x[e] = np.nan
    near = np.zeros(n, bool)
    near[H.getrow(e).indices[H.getrow(e).data > 0]] = True
    for adjoint in (False, True):
        y = hexmg.density_filter(*dims, rmin, gpu(x), adjoint=adjoint).cpu().numpy()
        assert np.array_equal(np.isnan(y), near)

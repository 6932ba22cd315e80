"""Accuracy of the fused small-level steps in binary32 (csrc/tile.hip): V-cycles with such a
level inside are no further from the oracle's than the same cycles launched step by
step with the streaming kernel, whose element products are formed on differences."""
import numpy as np
import pytest

import workloads as W
from oracle import multigrid as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_fused_steps_keep_the_accuracy_of_the_step_launches():
    from paper_2201_12931_amd import hexmg

    logs = []
    for dims, levels in (((36, 32, 32), 3), ((24, 20, 28), 3), ((32, 16, 16), 3)):
        g = W.Grid(*dims)
        for seed in range(4):
            rho = W.random_field_density(g, seed=seed, length_scale=3.0, lo=0.05)
            h = mg.Hierarchy(*dims, rho, W.fixed_mask_face_x0(g), levels)
            # a body force: the corrections are smooth, and sums over an element's nodes cancel
            r = np.tile([0.0, 0.3, -1.0], g.n_node) * h.free[0]
            ref = h.vcycle(r)
            err = []
            for step in (False, True):
                grid = hexmg.Grid(*dims, levels, vcycle_both=1)
                grid.set_density(gpu(rho))
                grid.set_coarse_cycle(hexmg.F32, 0)
                grid.set_kernel_choice(0, hexmg.F32, hexmg.KERNEL_STREAM, 1, 6)  # the same on both sides
                if step:
                    for l in range(1, levels):
                        grid.set_kernel_choice(l, hexmg.F32, hexmg.KERNEL_STREAM, 1, 6)
                z = torch.empty(g.n_dof, dtype=torch.float32, device="cuda")
                grid.vcycle(gpu(r.astype(np.float32)), z)
                err.append(float(np.linalg.norm(z.cpu().numpy() - ref) / np.linalg.norm(ref)))
            print(f"case tiles accuracy {dims} seed {seed}: fused {err[0]:.2e}, steps {err[1]:.2e}", flush=True)
            logs.append(np.log(err[0] / err[1]))
    # the same precision throughout: the mean ratio of two rounding errors, within its
    # spread over 12 cases
    assert np.exp(np.mean(logs)) <= 1.0 + 2.0 * np.std(logs) / np.sqrt(len(logs))

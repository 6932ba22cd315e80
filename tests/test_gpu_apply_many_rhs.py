"""K u of more right-hand sides than one launch's grid takes (planes times
right-hand sides past 65535): the same results as one by one."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 13107: the most that the 4-plane chunks of a 17-plane level take in one launch
@pytest.mark.parametrize("precision,level,dtype,nrhs", [("FP64", 0, torch.float32, 13107), ("FP64", 0, torch.float64, 4000),
                                                        ("MIXED", 1, torch.float64, 8000), ("MIXED", 0, torch.float32, 3855),
                                                        ("MIXED", 0, torch.float32, 3856)])
def test_apply_many(precision, level, dtype, nrhs):
    from paper_2201_12931_amd import hexmg

    dims, levels = (2, 2, 16), 2
    print(f"case K u {precision} level {level} {dtype} nrhs={nrhs}", flush=True)
    g = W.Grid(*dims)
    grid = hexmg.Grid(*dims, levels, precision=getattr(hexmg, precision))
    grid.set_density(torch.from_numpy(W.random_field_density(g, seed=2, lo=0.05)).cuda())
    n = 3 * np.prod([d // 2**level + 1 for d in dims])
    u = torch.from_numpy(np.random.default_rng(4).standard_normal((nrhs, n))).to("cuda", dtype)
    y = torch.full_like(u, float("nan"))
    grid.apply_K(u, y, level=level)
    ref = torch.full_like(u, float("nan"))
    for k in range(0, nrhs, 1000):
        m = min(1000, nrhs - k)
        grid.apply_K(u[k:k + m].contiguous(), ref[k:k + m], level=level)
    assert torch.equal(y, ref)

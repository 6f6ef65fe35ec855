"""GPU checks of the sweep's token walk at the sizes where it can go wrong:
tiles one pixel short of, equal to and past the 32 x 32 tile, and grids on
which every pixel is active at once, so that more pixels wait for a lane than
a wave's ring holds and the rest wait for the next visit."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


def flooded(rng, Wd, Hd, K, L):
    """Every pixel holds excess; the sinks are a few pixels of one corner, so
    the flow of the whole grid crosses it through random n-links."""
    inst = W.tiny_random(rng, Wd, Hd, K, cmax=60, L=L, p_seed=0.0, lam_max=50)
    inst.cap_src = rng.integers(1, 200, size=(Hd, Wd)).astype(np.int32)
    corner = np.zeros((Hd, Wd), dtype=bool)
    corner[: max(1, Hd // 8), : max(1, Wd // 8)] = True
    inst.cap_snk0 = np.where(corner, rng.integers(500, 4000, size=(Hd, Wd)), 0).astype(np.int32)
    inst.snk_slope = np.where(corner, rng.integers(0, 40, size=(Hd, Wd)), 0).astype(np.int32)
    return inst


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("shape", [(31, 33), (32, 32), (33, 31), (64, 32), (65, 70)])
@pytest.mark.parametrize("opts", [{}, {"inner_iters": 1, "tail_inner_iters": 1}, {"tail_inner_iters": 4096}])
def test_flooded_grids(K, shape, opts):
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([K, shape[0], shape[1]])
    insts = [flooded(rng, shape[0], shape[1], K, 2) for _ in range(2)]
    for orientation in (0, 3):
        s = pmf.Solver(orientation=orientation, **opts)
        flows, status = s.solve(pmf.to_device(insts))
        torch.cuda.synchronize()
        assert int(status.cpu().max()) == 0
        f = flows.cpu().numpy()
        for i, inst in enumerate(insts):
            for k in range(inst.L):
                fo, mo = O.fifo_pr(inst, int(inst.lambdas[k]))
                assert int(f[2 * i + k]) == fo, (orientation, i, k)
                got = s.extract_cut(i, k).cpu().numpy().astype(bool)
                assert np.array_equal(got, np.asarray(mo, dtype=bool).reshape(inst.H, inst.W)), (orientation, i, k)
        s.close()

"""GPU check of the gap heuristic's statistic: between two global relabels a
pixel is stopped at most once, however often its tile is swept meanwhile."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,shape,L,orientation", [(4, (128, 96), 1, 0), (8, (128, 96), 1, 0), (8, (131, 97), 1, 3),
                                                   (4, (160, 128), 6, 0)])
def test_a_pixel_is_stopped_once_per_relabel(K, shape, L, orientation):
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([K, L, orientation])
    Wd, Hd = shape
    img = W.voronoi_image(Wd, Hd, 12, rng)
    inst = W.seed_instance(img, W.nlinks(img, K), K, Wd // 2, Hd // 2, 7, W.geometric_lambdas(1, 400, L), image=0)
    # one step per active pixel and visit, and the relabels far apart: many
    # visits of a tile between two of them
    s = pmf.Solver(gap=1, orientation=orientation, lambda_chunk=100, sweeps_per_relabel=2000, inner_iters=1,
                   tail_inner_iters=1)
    flows, status = s.solve(pmf.to_device([inst]))
    torch.cuda.synchronize()
    assert int(status.cpu().max()) == 0
    for k in range(L):
        assert int(flows[k]) == O.fifo_pr(inst, int(inst.lambdas[k]))[0]
    st = s.stats()
    s.close()
    print("stopped", st["gap_kills"], "in", st["global_relabels"], "relabels of", Wd * Hd, "pixels", flush=True)
    assert 0 < st["gap_kills"] <= st["global_relabels"] * Wd * Hd

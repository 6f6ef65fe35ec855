"""GPU checks of the tile listing of the separately launched supersteps at the
edges of its block sizes: instances of one trip of 256 tiles, one tile row
more, and just past one trip of 1024."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,shape", [(4, (512, 512)), (4, (515, 513)), (8, (544, 520)), (4, (1050, 1000))])
def test_listing_of_many_tiles(K, shape):
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([K, shape[0], shape[1]])
    inst = W.tiny_random(rng, shape[0], shape[1], K, cmax=60, L=2, p_seed=0.001, lam_max=50)
    want = [O.fifo_pr(inst, int(lam)) for lam in inst.lambdas]
    for use_graph in (0, 1):
        s = pmf.Solver(use_graph=use_graph)
        flows, status = s.solve(pmf.to_device([inst]))
        torch.cuda.synchronize()
        assert int(status.cpu().max()) == 0
        f = flows.cpu().numpy()
        for k, (fo, mo) in enumerate(want):
            assert int(f[k]) == fo, (use_graph, k)
            got = s.extract_cut(0, k).cpu().numpy().astype(bool)
            assert np.array_equal(got, np.asarray(mo, dtype=bool).reshape(inst.H, inst.W)), (use_graph, k)
        s.close()

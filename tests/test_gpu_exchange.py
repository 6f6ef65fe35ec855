"""GPU check of a sweep visit's exchanges with the neighbour tiles at the ends of
their ranges: as many as the options allow, with the largest capacities."""

import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("use_graph", [0, 1])
def test_many_exchanges_of_the_largest_capacities(K, use_graph):
    """Excess near 2^31 handed to and fro across tile borders up to 64 times
    in a visit: the words that count it stay in range."""
    import torch
    from helpers import headroom_instance
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([64, K])
    insts = [headroom_instance(rng, 70, 41, K, 2), headroom_instance(rng, 33, 66, K, 1)]
    for inst in insts:  # hardly any sink: excess wanders until it is given up
        inst.seed = np.where(np.arange(inst.W * inst.H).reshape(inst.H, inst.W) == 0, 2, inst.seed % 2).astype(np.uint8)
        inst.cap_snk0 = np.minimum(inst.cap_snk0, 5).astype(np.int32)
    want = [O.fifo_pr(inst, int(lam)) for inst in insts for lam in inst.lambdas]
    for orientation in (0, 3):
        s = pmf.Solver(orientation=orientation, use_graph=use_graph, tail_sweep_exchanges=64, tail_inner_iters=4096)
        flows, status = s.solve(pmf.to_device(insts))
        torch.cuda.synchronize()
        assert int(status.cpu().max()) == 0
        at = 0
        for i, inst in enumerate(insts):
            for k in range(inst.L):
                fo, mo = want[at]
                assert int(flows[at]) == fo, (orientation, i, k)
                got = s.extract_cut(i, k).cpu().numpy().astype(bool)
                assert np.array_equal(got, np.asarray(mo, dtype=bool).reshape(inst.H, inst.W)), (orientation, i, k)
                at += 1
        s.close()

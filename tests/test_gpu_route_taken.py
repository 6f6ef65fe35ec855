"""GPU checks that a work list takes the route its comment says, on both sides
of every line, with the results of separate launches on either.  A wait for
the device-driven solve stands behind one launch, a wait for launched
supersteps behind steps_per_sync of them."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


def row(tiles, K, L=1):
    """An image of `tiles` 32 x 32 tiles in one row, three pixels high."""
    rng = np.random.default_rng([tiles, K, L])
    return W.tiny_random(rng, tiles * 32, 3, K, cmax=40, L=L, lam_max=40, p_seed=0.05)


def few_of_many(route):
    return {"k8 of 640": [row(640, 8, 2)], "k8 of 641": [row(641, 8)],
            "k4 of 350": [row(350, 4, 2)], "k4 of 351": [row(351, 4)],
            "k4 of 640 and 1": [row(640, 4), row(1, 4)], "k4 of 640 and 60": [row(640, 4), row(60, 4)],
            "k4 of 640 and 61": [row(640, 4), row(61, 4)],
            "k4 of 640, k8 of 1": [row(640, 4, 2), row(1, 8)],
            "k4 of 641, k8 of 1": [row(641, 4), row(1, 8)]}[route]


@pytest.mark.parametrize("name,device", [("k8 of 640", True), ("k8 of 641", False), ("k4 of 350", True),
                                         ("k4 of 351", False), ("k4 of 640 and 1", True), ("k4 of 640 and 60", True),
                                         ("k4 of 640 and 61", False), ("k4 of 640, k8 of 1", True),
                                         ("k4 of 641, k8 of 1", False)])
def test_route(name, device):
    import torch
    from paper_1509_06004_amd import pmf
    insts = few_of_many(name)
    dev = pmf.to_device(insts)
    got = []
    for opts in ({}, {"use_graph": 0}):
        s = pmf.Solver(lambda_chunk=4, **opts)
        flows, status = s.solve(dev)
        torch.cuda.synchronize()
        assert int(status.cpu().max()) == 0
        st = s.stats()
        if opts == {}:
            assert (st["work_launches"] == st["host_syncs"]) == device, (st["work_launches"], st["host_syncs"])
        masks = [s.extract_cut(i, k).cpu().numpy().astype(bool) for i, inst in enumerate(insts) for k in range(inst.L)]
        got.append((flows.cpu().numpy(), masks))
        s.close()
    at = 0
    for inst in insts:
        for lam in inst.lambdas:
            fo, mo = O.fifo_pr(inst, int(lam))
            for f, m in got:
                assert int(f[at]) == fo, at
                assert np.array_equal(m[at], np.asarray(mo, dtype=bool).reshape(inst.H, inst.W)), at
            at += 1


def test_options_that_launch():
    """Options that need supersteps of their own are never left to the device."""
    import torch
    from paper_1509_06004_amd import pmf
    insts = [row(5, 4, 2), row(3, 8)]
    dev = pmf.to_device(insts)
    want = None
    for opts in ({}, {"use_graph": 0}, {"gap": 1}, {"timing": 1}, {"persist_tiles": 40}):
        s = pmf.Solver(**opts)
        flows, status = s.solve(dev)
        torch.cuda.synchronize()
        st = s.stats()
        s.close()
        want = flows.cpu() if want is None else want
        assert int(status.cpu().max()) == 0 and torch.equal(want, flows.cpu())
        assert (st["work_launches"] == st["host_syncs"]) == (opts == {}), opts

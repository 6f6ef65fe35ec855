"""GPU checks of the device-driven solve (every instance runs its own
supersteps inside one launch) against supersteps launched one by one
(use_graph = 0), which share the tile work but none of the scheduling: work
lists of one connectivity and of both, fewer and more instances than a word
of its bit map holds and than a handle has room for from the start, the
largest instance it takes and the smallest it leaves to the launches, and
sessions that stop after every superstep."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


def grids(name):
    rng = np.random.default_rng([5, len(name)])

    def tiny(Wd, Hd, K, L=2):
        return W.tiny_random(rng, Wd, Hd, K, cmax=40, L=L, lam_max=40, p_seed=0.05)
    if name == "k4":
        return [tiny(70, 50, 4), tiny(1, 1, 4), tiny(33, 97, 4, 5)]
    if name == "k8":
        return [tiny(70, 50, 8), tiny(1, 2, 8), tiny(33, 97, 8, 5)]
    if name == "mixed":
        return [tiny(64, 40, 8), tiny(40, 64, 4), tiny(9, 9, 8, 1), tiny(150, 33, 4, 4)]
    if name == "many":
        return [tiny(int(rng.integers(1, 40)), int(rng.integers(1, 40)), 4 if i % 3 else 8, 1) for i in range(130)]
    if name == "beyond the first room":
        return [tiny(3, 2, 4, 1) for _ in range(4200)]
    # 640 tiles in one row, and one more
    return [tiny(640 * 32 + (1 if name == "past the largest" else 0), 3, 4, 1)]


@pytest.mark.parametrize("name", ["k4", "k8", "mixed", "many", "beyond the first room", "the largest", "past the largest"])
def test_equals_separate_launches(name):
    import torch
    from paper_1509_06004_amd import pmf
    insts = grids(name)
    dev = pmf.to_device(insts)
    got = []
    for opts in ({}, {"use_graph": 0}, {"tile_w": 64, "tile_h": 16, "lambda_chunk": 2}):
        s = pmf.Solver(**opts)
        for _ in range(2):  # the second solve finds the first one's words
            flows, status = s.solve(dev)
        levels = []
        for i, inst in enumerate(insts):
            out = torch.empty((inst.H, inst.W), dtype=torch.uint8, device="cuda")
            assert pmf.pmf_extract_levels(s.handle, i, int(out.data_ptr())) == pmf.PMF_OK
            levels.append(out.reshape(-1))
        torch.cuda.synchronize()
        assert int(status.cpu().max()) == 0
        got.append((flows.cpu(), torch.cat(levels).cpu()))
        s.close()
    for f, lev in got[1:]:
        assert torch.equal(got[0][0], f) and torch.equal(got[0][1], lev)
    o = 0
    for inst in insts[:40]:
        for k in range(inst.L):
            assert int(got[0][0][o + k]) == O.fifo_pr(inst, int(inst.lambdas[k]))[0]
        o += inst.L


@pytest.mark.parametrize("step", [1, 3, 1000])
def test_session_stops_and_goes_on(step):
    import torch
    from paper_1509_06004_amd import pmf
    insts = grids("mixed")
    dev = pmf.to_device(insts)
    ref = pmf.Solver(use_graph=0)
    flows0, _ = ref.solve(dev)
    s = pmf.Solver()
    assert pmf.pmf_session_open(s.handle, 16, 64 << 20) == pmf.PMF_OK
    flows = torch.empty_like(flows0)
    status = torch.empty(len(insts), dtype=torch.int32, device="cuda")
    rc, ids = pmf.pmf_session_submit(s.handle, [d.c_struct() for d in dev], int(flows.data_ptr()), int(status.data_ptr()))
    assert rc == pmf.PMF_OK
    left = set(ids)
    for _ in range(20000):
        rc, done = pmf.pmf_session_step(s.handle, step)
        assert rc == pmf.PMF_OK
        left -= set(done)
        if not left:
            break
    torch.cuda.synchronize()
    assert not left and torch.equal(flows0, flows) and int(status.cpu().max()) == 0
    s.close()
    ref.close()

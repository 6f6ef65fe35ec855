"""GPU checks of the choice between the device-driven launch and separate
launches by the work list's average tiles per instance: both sides of the
line, the largest instance of a mostly small list, and a session that crosses
the line in mid-solve, in both directions."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


def tiny(rng, Wd, Hd, K, L=2):
    return W.tiny_random(rng, Wd, Hd, K, cmax=40, L=L, lam_max=40, p_seed=0.02)


def check(insts, flows, mask_of):
    o = 0
    for i, inst in enumerate(insts):
        for k, lam in enumerate(inst.lambdas):
            fo, mo = O.fifo_pr(inst, int(lam))
            assert int(flows[o + k]) == fo, (i, k)
            assert np.array_equal(mask_of(i, k), np.asarray(mo, dtype=bool).reshape(inst.H, inst.W)), (i, k)
        o += inst.L


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("shapes", [[(50 * 32, 7 * 32)], [(50 * 32, 7 * 32 + 1)], [(640 * 32, 3), (5, 4), (40, 30)]])
def test_batch_at_the_line(K, shapes):
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([K, len(shapes), shapes[0][1]])
    insts = [tiny(rng, w, h, K) for w, h in shapes]
    s = pmf.Solver(lambda_chunk=2)
    flows, status = s.solve(pmf.to_device(insts))
    torch.cuda.synchronize()
    assert int(status.cpu().max()) == 0
    check(insts, flows.cpu().numpy(), lambda i, k: s.extract_cut(i, k).cpu().numpy().astype(bool))
    s.close()


def test_session_crosses_the_line():
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng(414)
    big, small = [tiny(rng, 720, 576, 4, 4)], [tiny(rng, 60, 70, 4, 1) for _ in range(3)]
    o = pmf.pmf_default_options()
    h = pmf.pmf_create(o, int(torch.cuda.current_stream().cuda_stream))
    assert pmf.pmf_session_open(h, 8, 256 << 20) == pmf.PMF_OK
    runs = []

    def submit(insts):
        dev = pmf.to_device(insts)
        flows = torch.full((sum(d.L for d in dev),), -7, dtype=torch.int64, device="cuda")
        status = torch.full((len(dev),), -7, dtype=torch.int32, device="cuda")
        rc, ids = pmf.pmf_session_submit(h, [d.c_struct() for d in dev], int(flows.data_ptr()), int(status.data_ptr()))
        assert rc == pmf.PMF_OK
        runs.append((insts, dev, flows, status, ids))
        return set(ids)

    left = submit(big)
    for n in range(400):
        if n in (3, 9):
            left |= submit(small[: 1 + n // 4])
        rc, done = pmf.pmf_session_step(h, 4)
        assert rc == pmf.PMF_OK
        left.difference_update(done)
        if n > 9 and not left:
            break
    assert not left
    torch.cuda.synchronize()
    for insts, dev, flows, status, ids in runs:
        assert int(status.cpu().max()) == 0

        def mask(i, k):
            out = torch.empty((insts[i].H, insts[i].W), dtype=torch.uint8, device="cuda")
            assert pmf.pmf_extract_cut(h, ids[i], k, int(out.data_ptr())) == pmf.PMF_OK
            torch.cuda.synchronize()
            return out.cpu().numpy().astype(bool)
        check(insts, flows.cpu().numpy(), mask)
    pmf.pmf_destroy(h)

"""GPU checks of the memory a handle takes: with a workspace all of its device
memory is the workspace, with a budget no more than that, and the solve that
allocates nothing leaves a handle without any.  Limits that leave no room for
the device-driven solve's own words give the same results."""

import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu

MIB = 1 << 20
HANDLES = 48


def tiny(rng, Wd, Hd, K, L=1):
    return W.tiny_random(rng, Wd, Hd, K, cmax=40, L=L, lam_max=40, p_seed=0.05)


def solve(pmf, torch, handle, dev, noalloc=False):
    flows = torch.full((sum(d.L for d in dev),), -7, dtype=torch.int64, device="cuda")
    status = torch.full((len(dev),), -7, dtype=torch.int32, device="cuda")
    fn = pmf.pmf_solve_batch_noalloc if noalloc else pmf.pmf_solve_batch
    rc = fn(handle, [d.c_struct() for d in dev], int(flows.data_ptr()), int(status.data_ptr()))
    torch.cuda.synchronize()
    return rc, flows.cpu().numpy(), status.cpu().numpy()


def stream_bytes(pmf, torch):
    """Device memory that the runtime takes for HANDLES - 1 streams of its own
    (a handle has one, to capture into)."""
    lib = pmf.load_library()
    free0 = torch.cuda.mem_get_info()[0]
    streams = [ctypes.c_void_p() for _ in range(HANDLES - 1)]
    for s in streams:
        assert lib.hipStreamCreateWithFlags(ctypes.byref(s), ctypes.c_uint(1)) == 0
    taken = free0 - torch.cuda.mem_get_info()[0]
    for s in streams:
        assert lib.hipStreamDestroy(s) == 0
    return taken


@pytest.mark.parametrize("kind", ["workspace", "budget", "noalloc"])
def test_device_memory_of_handles(kind):
    """Many handles, each created and used once: the device's free memory
    falls by their workspaces or budgets (and streams) alone."""
    import torch
    from paper_1509_06004_amd import pmf
    inst = tiny(np.random.default_rng(7), 33, 20, 4)
    dev = pmf.to_device([inst])
    stream = int(torch.cuda.current_stream().cuda_stream)
    o = pmf.pmf_default_options()
    per = MIB
    if kind == "budget":
        o.mem_budget = per
    spaces = torch.empty((HANDLES, per), dtype=torch.uint8, device="cuda")

    def create(i):
        if kind == "workspace":
            return pmf.pmf_create(o, stream, int(spaces[i].data_ptr()), per)
        return pmf.pmf_create(o, stream)
    first = create(0)  # what the runtime sets up with a first call is not counted
    assert solve(pmf, torch, first, dev, kind == "noalloc")[0] == pmf.PMF_OK
    streams = stream_bytes(pmf, torch)
    free0 = torch.cuda.mem_get_info()[0]
    handles, flows = [], []
    for i in range(1, HANDLES):
        handles.append(create(i))
        rc, f, st = solve(pmf, torch, handles[-1], dev, kind == "noalloc")
        assert rc == pmf.PMF_OK and (st == 0).all()
        flows.append(int(f[0]))
    taken = free0 - torch.cuda.mem_get_info()[0] - streams
    for h in handles + [first]:
        pmf.pmf_destroy(h)
    # four readings of the free memory, each in steps of 2 MiB
    allowed = (HANDLES if kind == "budget" else 8) * MIB
    print(kind, "device memory taken by %d handles: %.1f MiB, %.1f MiB for their streams" %
          (HANDLES - 1, taken / MIB, streams / MIB), flush=True)
    assert taken <= allowed
    assert set(flows) == {O.fifo_pr(inst, int(inst.lambdas[0]))[0]}


@pytest.mark.parametrize("name", ["one pixel", "tiny images", "mixed", "a wide one"])
def test_workspaces_from_just_enough_to_ample(name):
    """The smallest workspace that a batch is accepted in, and larger ones: the
    words of the device-driven solve fit from some size on, and the results
    are those of a handle without limits at every size."""
    import torch
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([11, len(name)])
    insts = {"one pixel": [tiny(rng, 1, 1, 4)],
             "tiny images": [tiny(rng, 1 + i % 7, 1 + i % 5, 4 if i % 2 else 8) for i in range(70)],
             "mixed": [tiny(rng, 70, 41, 8, 3), tiny(rng, 9, 9, 4), tiny(rng, 33, 64, 4, 2)],
             "a wide one": [tiny(rng, 1300, 3, 4)]}[name]
    dev = pmf.to_device(insts)
    o = pmf.pmf_default_options()
    o.lambda_chunk = 1
    stream = int(torch.cuda.current_stream().cuda_stream)
    free = pmf.pmf_create(o, stream)
    rc, want, st = solve(pmf, torch, free, dev)
    assert rc == pmf.PMF_OK and (st == 0).all()
    pmf.pmf_destroy(free)
    at = 0
    for inst in insts:
        for k in range(inst.L):
            assert int(want[at + k]) == O.fifo_pr(inst, int(inst.lambdas[k]))[0]
        at += inst.L
    ample = 4 * MIB
    space = torch.empty(ample, dtype=torch.uint8, device="cuda")

    def accepted(size):
        h = pmf.pmf_create(o, stream, int(space.data_ptr()), size)
        rc, f, st = solve(pmf, torch, h, dev)
        pmf.pmf_destroy(h)
        assert rc in (pmf.PMF_OK, pmf.PMF_ENOMEM), rc
        if rc == pmf.PMF_OK:
            assert (st == 0).all() and (f == want).all(), size
        return rc == pmf.PMF_OK
    lo, hi = 256, ample
    assert accepted(hi)
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        lo, hi = (lo, mid) if accepted(mid) else (mid, hi)
    for more in (256, 1024, 2048, 4096, 16384, 65536):
        assert accepted(min(ample, hi + more))


@pytest.mark.parametrize("probes,narrow", [(1, None), (2, None), (64, None), (130, True), (300, False)])
def test_searches_within_budgets(probes, narrow):
    """A search of more than 256 change points under budgets given in probes
    of its image: room for 128 side by side but not for 256 narrows the rounds
    and leaves intervals for later ones, half a probe's room is too little."""
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng(4000)
    inst = W.tiny_random(rng, 33, 40, 4, cmax=3, L=1, p_seed=0.03, lam_max=50)
    inst.cap_src = rng.integers(0, 4000, size=(40, 33)).astype(np.int32)
    inst.cap_snk0 = rng.integers(0, 4, size=(40, 33)).astype(np.int32)
    inst.snk_slope = rng.integers(1, 4, size=(40, 33)).astype(np.int32)
    dev = pmf.to_device([inst])[0]
    free = pmf.Solver()
    want = pmf.pmf_parametric(free.handle, dev, 0, 4000)
    free.close()
    assert len(want[0]) > 256
    # a probe's state, its share of the control area and of the round's own data
    per = pmf.pmf_query_bytes([dev.c_struct()]) * 17 // 16 + 1024
    too_little = pmf.Solver(mem_budget=per // 2)
    with pytest.raises(pmf.PmfError) as exc:
        pmf.pmf_parametric(too_little.handle, dev, 0, 4000)
    assert exc.value.code == pmf.PMF_ENOMEM
    too_little.close()
    s = pmf.Solver(mem_budget=per * probes + 16384)
    try:
        got = pmf.pmf_parametric(s.handle, dev, 0, 4000)
    except pmf.PmfError as exc:
        # rounds of two probes an interval are not narrowed below 128
        assert exc.code == pmf.PMF_ENOMEM and narrow is None
    else:
        for g, w in zip(got, want):
            assert np.array_equal(np.asarray(g.cpu() if hasattr(g, "cpu") else g),
                                  np.asarray(w.cpu() if hasattr(w, "cpu") else w))
        assert s.stats()["device_bytes"] <= per * probes + 16384
    s.close()

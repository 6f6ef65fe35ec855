"""GPU checks of the breakpoint searches' table-driven kernels at the edges of
their tables and blocks: more open intervals than half a table (a round of
more than 64 masks), more changing intervals than one table, several probes of
one interval in a round, and grids short of, equal to and past one block."""

import math
from fractions import Fraction

import numpy as np
import pytest

from paper_1509_06004_amd import workload as W

pytestmark = pytest.mark.gpu


def scattered(rng, Wd, Hd, K, span, seeded):
    """Weak n-links and source capacities spread over `span`: nearly every
    pixel leaves the minimal set at a lambda of its own."""
    inst = W.tiny_random(rng, Wd, Hd, K, cmax=3, L=1, p_seed=0.03 if seeded else 0.0, lam_max=50)
    inst.cap_src = rng.integers(0, span, size=(Hd, Wd)).astype(np.int32)
    inst.cap_snk0 = rng.integers(0, 4, size=(Hd, Wd)).astype(np.int32)
    inst.snk_slope = rng.integers(1, 4, size=(Hd, Wd)).astype(np.int32)
    return inst


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("shape,span", [((17, 15), 2000), ((16, 16), 2000), ((19, 27), 4000), ((16, 16), 40)])
def test_probe_tables(K, shape, span):
    from helpers import check_breakpoints_oracle, host_threads
    from paper_1509_06004_amd import pmf
    rng = np.random.default_rng([K, shape[0], shape[1], span])
    inst = scattered(rng, shape[0], shape[1], K, span, seeded=span != 4000)
    lo, hi = 0, span
    s = pmf.Solver()
    dev = pmf.to_device([inst])[0]
    num, den, pa, pw, ex = pmf.pmf_breakpoints(s.handle, dev, lo, hi)
    check_breakpoints_oracle(inst, lo, hi, num, den, pa, pw, ex.cpu().numpy(), host_threads())
    bp, f, ex_i = pmf.pmf_parametric(s.handle, dev, lo, hi)
    s.close()
    xs = [Fraction(int(a), int(b)) for a, b in zip(num, den)]
    assert [int(c) for c in bp] == sorted({math.ceil(x) for x in xs})
    if span >= 2000:
        assert len(bp) > 64
    for c, fc in zip([lo] + [int(c) for c in bp], f):
        j = sum(1 for x in xs if x <= c)
        assert int(fc) == int(pa[j]) + int(pw[j]) * c, c
    ceil_of = np.array([lo] + [math.ceil(x) for x in xs] + [hi + 1], dtype=np.int64)
    assert (ceil_of[ex.cpu().numpy()] == ex_i.cpu().numpy()).all()


@pytest.mark.parametrize("mib", [4, 8, 24, 96])
def test_search_in_limited_memory(mib):
    """Rounds narrower than the widest, and intervals left for a later round,
    where the memory limit asks for it: the same change points and exits."""
    from paper_1509_06004_amd import pmf
    inst = scattered(np.random.default_rng(mib), 33, 40, 4, 4000, seeded=True)
    dev = pmf.to_device([inst])[0]
    free = pmf.Solver()
    want = pmf.pmf_parametric(free.handle, dev, 0, 4000)
    free.close()
    assert len(want[0]) > 256
    tight = pmf.Solver(mem_budget=mib << 20)
    try:
        got = pmf.pmf_parametric(tight.handle, dev, 0, 4000)
    except pmf.PmfError as exc:
        assert exc.code == pmf.PMF_ENOMEM and mib < 96
    else:
        assert all(np.array_equal(np.asarray(g.cpu() if hasattr(g, "cpu") else g),
                                  np.asarray(w.cpu() if hasattr(w, "cpu") else w)) for g, w in zip(got, want))
    tight.close()

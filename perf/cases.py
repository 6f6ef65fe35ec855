"""Performance cases: the work a program has this library do.

A case names an entry point (``call``), the images it is given and the lambda
schedules solved on them.  The images are the synthetic segmentation images of
``paper_1509_06004_amd.workload`` (Voronoi mosaics with noise, square
foreground seeds, the border ring as background seed), drawn from the seed.

``call`` is one of

* ``batch``: ``Solver.solve`` on every (image, seed) instance, then the nested
  masks of every instance as one byte per pixel (``pmf_extract_levels``);
* ``noalloc``: the same through ``pmf_solve_batch_noalloc``;
* ``session``: a serving request: submitted to an open session, stepped until
  every instance has finished, its masks read, its slots released;
* ``parametric``: every integer breakpoint over ``lam_lo..lam_hi``;
* ``breakpoints``: every real breakpoint over the same range.

A case with ``mix`` = 0 holds ``images`` images of W x H with ``seeds``
instances each and L geometric lambdas; with ``mix`` > 0 it holds ``images``
images of 64..W x 64..H pixels, each 4- or 8-connected with 1..``seeds``
instances of 10..L log-uniform lambdas (the shapes follow from ``mix``, the
contents from the seed).
"""

import math

import numpy as np
import torch

from paper_1509_06004_amd import pmf
from paper_1509_06004_amd import workload as wl


def _case(name, call, W, H, K, images=1, seeds=1, L=1, lam_lo=1, lam_hi=2000, mix=0):
    c = {"call": call, "W": W, "H": H, "K": K, "images": images, "seeds": seeds, "L": L, "lam_lo": lam_lo,
         "lam_hi": lam_hi, "mix": mix}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one cut of a thumbnail: the smallest call, all latency
        _case("one_cut_64", "batch", 64, 64, 4, lam_lo=100, lam_hi=100),
        # a small image of odd size, 8-connected, a short schedule
        _case("short_chain_97x61_k8", "batch", 97, 61, 8, L=3, lam_lo=20, lam_hi=400),
        # a folder of thumbnails segmented in one call, one cut each
        _case("thumbnails_128x96", "batch", 128, 96, 4, images=64, lam_lo=100, lam_hi=100),
        # one seed's whole schedule on a quarter-VGA image, in the buffer of
        # the solve that allocates nothing
        _case("noalloc_chain_320x240", "noalloc", 320, 240, 4, L=10),
        # one seed's whole schedule, one call at a time (the plain form)
        _case("chain_500x375", "batch", 500, 375, 4, L=20),
        # the benchmark workload: 25 seeds x 20 lambdas of one image
        _case("seeds25_500x375", "batch", 500, 375, 4, seeds=25, L=20),
        # the same, 8-connected
        _case("seeds25_500x375_k8", "batch", 500, 375, 8, seeds=25, L=20),
        # an uneven batch: many sizes, both connectivities, ragged schedules
        _case("uneven_24_images", "batch", 640, 480, 0, images=24, seeds=16, L=30, lam_hi=5000, mix=1),
        # one serving request: four seeds of a VGA image
        _case("request_640x480_k8", "session", 640, 480, 8, seeds=4, L=20),
        # the whole parametric solution of one seed, integer and real lambdas
        _case("parametric_500x375", "parametric", 500, 375, 4),
        _case("breakpoints_320x240", "breakpoints", 320, 240, 4),
        # the largest image: a full-HD frame, a few lambdas
        _case("frame_1920x1080", "batch", 1920, 1080, 4, L=4, lam_lo=40, lam_hi=400),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["batch", "batch", "batch", "batch", "noalloc", "session", "parametric", "breakpoints"])
    K = rng.choice([4, 8])
    lo = _log(rng, 1, 100)
    hi = lo + _log(rng, 50, 4000)
    if call in ("parametric", "breakpoints"):
        # a real breakpoint's denominator has to fit the scaled int32 solves
        W = _log(rng, 48, 500 if call == "parametric" else 320)
        H = _log(rng, 48, 375 if call == "parametric" else 240)
        return _case(None, call, W, H, K, lam_lo=lo, lam_hi=hi)
    if call == "noalloc":
        W, H = _log(rng, 40, 320), _log(rng, 40, 240)
        return _case(None, call, W, H, K, L=_log(rng, 1, 10), lam_lo=lo, lam_hi=hi)
    if call == "batch" and rng.random() < 0.25:
        return _case(None, call, rng.randint(96, 640), rng.randint(96, 480), 0, images=_log(rng, 2, 24),
                     seeds=_log(rng, 1, 16), L=rng.randint(10, 30), lam_hi=_log(rng, 200, 5000),
                     mix=rng.randint(2, 1 << 30))
    W, H = _log(rng, 40, 1920), _log(rng, 40, 1080)
    px = W * H
    # at most the pixel solves of the large listed cases, and images of more
    # than VGA size with a few lambdas only
    room = max(1, (30000000 if px < 640 * 480 else 6000000) // px)
    seeds = min(_log(rng, 1, 8 if call == "session" else 25), room)
    L = min(_log(rng, 1, 30), max(1, room // seeds))
    images = min(_log(rng, 1, 64), max(1, room // (seeds * L))) if call == "batch" and px < 30000 else 1
    return _case(None, call, W, H, K, images=images, seeds=seeds, L=L, lam_lo=lo, lam_hi=hi)


def _shapes(case):
    """(W, H, K, lambdas of each instance) of every image."""
    out = []
    if case["mix"]:
        g = np.random.default_rng([77, case["mix"]])
        for _ in range(case["images"]):
            W, H = int(g.integers(64, case["W"] + 1)), int(g.integers(64, case["H"] + 1))
            K = 4 if g.integers(0, 2) == 0 else 8
            lens = [int(g.integers(10, case["L"] + 1)) for _ in range(int(g.integers(1, case["seeds"] + 1)))]
            out.append((W, H, K, lens))
        return out
    return [(case["W"], case["H"], case["K"], [case["L"]] * case["seeds"])] * case["images"]


def _host(case, seed):
    insts = []
    for i, (W, H, K, lens) in enumerate(_shapes(case)):
        rng = np.random.default_rng([seed, i])
        img = wl.voronoi_image(W, H, int(rng.integers(8, 33)), rng)
        nl = wl.nlinks(img, K)
        for L in lens:
            if case["mix"]:
                lam = wl.loguniform_lambdas(rng, L, case["lam_hi"])
            else:
                lam = wl.geometric_lambdas(case["lam_lo"], case["lam_hi"], L)
            cx, cy = int(rng.integers(5, W - 5)), int(rng.integers(5, H - 5))
            insts.append(wl.seed_instance(img, nl, K, cx, cy, 7, lam, image=i))
    return insts


def prepare(case, seed):
    insts = pmf.to_device(_host(case, seed))
    state = {"case": case, "insts": insts, "solver": pmf.Solver()}
    if case["call"] == "session":
        # a resident session with room for two such requests
        need = pmf.pmf_query_bytes([d.c_struct() for d in insts])
        rc = pmf.pmf_session_open(state["solver"].handle, 2 * len(insts) + 2, 2 * need + (1 << 20))
        if rc != pmf.PMF_OK:
            raise pmf.PmfError(rc, "pmf_session_open")
    return state


def _check(rc, what):
    if rc != pmf.PMF_OK:
        raise pmf.PmfError(rc, what)


def _levels(handle, insts, ids):
    """Nested masks of every instance, one after another."""
    out = torch.empty(sum(d.W * d.H for d in insts), dtype=torch.uint8, device="cuda")
    at = int(out.data_ptr())
    for d, i in zip(insts, ids):
        _check(pmf.pmf_extract_levels(handle, i, at), "pmf_extract_levels")
        at += d.W * d.H
    return out


def _padded(a, size=4097):
    """A list of breakpoints in an array of the largest size the call takes."""
    out = np.zeros(size, dtype=np.int64)
    out[:len(a)] = a
    return out


def run(state):
    case, insts, solver = state["case"], state["insts"], state["solver"]
    call = case["call"]
    if call == "parametric":
        bp, f, ex = pmf.pmf_parametric(solver.handle, insts[0], case["lam_lo"], case["lam_hi"])
        return {"count": len(bp), "bp": _padded(bp), "f": _padded(f), "exit": ex}
    if call == "breakpoints":
        num, den, a, w, ex = pmf.pmf_breakpoints(solver.handle, insts[0], case["lam_lo"], case["lam_hi"])
        return {"count": len(num), "num": _padded(num), "den": _padded(den), "a": _padded(a), "w": _padded(w),
                "exit": ex}
    if call == "batch":
        flows, status = solver.solve(insts)
        return {"flows": flows, "status": status, "levels": _levels(solver.handle, insts, range(len(insts)))}
    structs = [d.c_struct() for d in insts]
    flows = torch.empty(sum(d.L for d in insts), dtype=torch.int64, device="cuda")
    status = torch.empty(len(insts), dtype=torch.int32, device="cuda")
    if call == "noalloc":
        _check(pmf.pmf_solve_batch_noalloc(solver.handle, structs, int(flows.data_ptr()), int(status.data_ptr())),
               "pmf_solve_batch_noalloc")
        return {"flows": flows, "status": status, "levels": _levels(solver.handle, insts, range(len(insts)))}
    rc, ids = pmf.pmf_session_submit(solver.handle, structs, int(flows.data_ptr()), int(status.data_ptr()))
    _check(rc, "pmf_session_submit")
    left = set(ids)
    while left:
        rc, done = pmf.pmf_session_step(solver.handle, 16)
        _check(rc, "pmf_session_step")
        left.difference_update(done)
    levels = _levels(solver.handle, insts, ids)
    for i in ids:
        _check(pmf.pmf_session_release(solver.handle, i), "pmf_session_release")
    return {"flows": flows, "status": status, "levels": levels}


def work(case):
    """Inputs read once (the n-links, zero sink capacities and slopes of an
    image are shared by its instances) and results written once."""
    total = 0
    for W, H, K, lens in _shapes(case):
        px = W * H
        total += px * (4 * K + 8)  # n-links, sink capacity at 0, slope
        for L in lens:
            total += px * 5 + 4 * L  # source capacity, seed, lambdas
            if case["call"] in ("parametric", "breakpoints"):
                total += 4 * px  # exit map
            else:
                total += px + 8 * L + 4  # levels, flows, status
    return {"bytes": float(total), "flops": 0.0}


def _cut(inst, lam):
    """Maximum flow and minimal source side of one lambda in 64-bit numpy: a
    push-relabel method on whole planes, one direction at a time, with exact
    distance labels recomputed every few rounds."""
    H, W, K = inst.H, inst.W, inst.K
    far = 1 << 40
    r = inst.nlink.astype(np.int64).copy()
    cs = np.where(inst.seed == 1, wl.INF, np.where(inst.seed == 2, 0, inst.cap_src)).astype(np.int64)
    ct = inst.cap_snk0.astype(np.int64) + inst.snk_slope.astype(np.int64) * lam
    ct = np.where(inst.seed == 1, 0, np.where(inst.seed == 2, wl.INF, ct))
    flow = int(np.minimum(cs, ct).sum())
    e, rt = cs - np.minimum(cs, ct), ct - np.minimum(cs, ct)

    def at(k):  # slices of p and of q = p + d_k
        dx, dy = wl.DX[k], wl.DY[k]
        p = (slice(max(0, -dy), H - max(0, dy)), slice(max(0, -dx), W - max(0, dx)))
        q = (slice(max(0, dy), H - max(0, -dy)), slice(max(0, dx), W - max(0, -dx)))
        return p, q

    pq = [at(k) for k in range(K)]
    while True:
        h = np.where(rt > 0, 1, far)
        while True:
            old = h.copy()
            for k in range(K):
                p, q = pq[k]
                h[p] = np.where(r[k][p] > 0, np.minimum(h[p], h[q] + 1), h[p])
            if (h == old).all():
                break
        h = np.minimum(h, far)
        if not ((e > 0) & (h < far)).any():
            break
        for _ in range(60):
            d = np.minimum(e, rt)
            e, rt, flow = e - d, rt - d, flow + int(d.sum())
            for k in range(K):
                p, q = pq[k]
                d = np.where((h[p] < far) & (h[p] == h[q] + 1), np.minimum(e[p], r[k][p]), 0)
                e[p] -= d
                e[q] += d
                r[k][p] -= d
                r[k ^ 1][q] += d
            low = np.where(rt > 0, 0, far)
            for k in range(K):
                p, q = pq[k]
                low[p] = np.where(r[k][p] > 0, np.minimum(low[p], h[q]), low[p])
            act = (e > 0) & (h < far)
            if not act.any():
                break
            h = np.where(act & (low >= h), np.minimum(low + 1, far), h)
    side = e > 0
    while True:
        old = side.copy()
        for k in range(K):
            p, q = pq[k]
            side[q] |= side[p] & (r[k][p] > 0)
        if (side == old).all():
            return flow, side


def exact(case, seed):
    """Flows and masks of the small cases (whole numbers; the larger ones take
    too long this way)."""
    if case["call"] not in ("batch", "noalloc") or case["mix"]:
        return None
    if case["W"] * case["H"] * case["images"] * case["seeds"] * case["L"] > 20000:
        return None
    flows, levels = [], []
    for inst in _host(case, seed):
        lev = np.zeros((inst.H, inst.W), dtype=np.uint8)
        for lam in inst.lambdas.tolist():
            f, m = _cut(inst, lam)
            flows.append(f)
            lev += m
        levels.append(lev.reshape(-1))
    return {"flows": np.array(flows, dtype=np.int64), "status": np.zeros(case["images"] * case["seeds"], dtype=np.int32),
            "levels": np.concatenate(levels)}

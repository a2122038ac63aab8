"""Performance cases: the calls a program that simulates threshold detection
makes through the public entry points, from the smallest to the largest.

Inputs are those of paper_2109_04528_amd.inputs.  Threshold detectors are used
on bright states (a detector that clicks does not say how many photons came),
so the FP64 cases take squeezed vacua of r ~ U[1, 1.5] (1.4 to 4.5 photons per
mode) with efficiencies from 0.7 to 1: the FP64 Torontonian then holds nine
digits or more up to 30 modes.  For dimmer states of many modes (r ~ U[.3, 1.2])
the sum cancels too far for an FP64 factor, and a program asks for the
double-double one: that is the input of the double-double cases.  General
Hermitian matrices (no Gaussian-state structure) take the complex path.

Kinds of case:
  eval       one Torontonian (host or device matrix; FP64 or double-double)
  batch      Torontonians of many matrices of uneven size in one call
  clicks     probabilities of given click patterns of one state
  click_all  probabilities of every click pattern of one state
  serve      a burst of submitted requests, drained and polled
"""
import math

import numpy as np
import torch

from paper_2109_04528_amd import (TOR_CHECK_HERMITIAN, TOR_FACTOR_DD, TOR_INPUT_DEVICE, TOR_OUTPUT_DEVICE,
                                  Context, inputs)
from paper_2109_04528_amd.flops import chol_flops, tor_flops


def _eval(name, n, form="state", factor="fp64", where="host", check=False):
    return {"name": name, "kind": "eval", "n": n, "form": form, "factor": factor, "where": where, "check": check}


def listed():
    return [
        # the first Torontonian anyone computes, and each early step of a
        # mode-by-mode sampler: all latency
        _eval("eval 10 host", 10),
        # a mid-size pattern of a state already on the GPU, an odd size
        _eval("eval 17 device", 17, where="device"),
        # ordinary: a 24-click event
        _eval("eval 24 host", 24),
        # the largest: the benchmark's 30 modes, the matrix in HBM
        _eval("eval 30 device", 30, where="device"),
        # general Hermitian input, the complex path: small and large, both odd
        _eval("eval 13 hermitian", 13, form="hermitian"),
        _eval("eval 27 hermitian", 27, form="hermitian", where="device"),
        # dim states of many modes: the double-double factor
        _eval("eval 23 double-double", 23, factor="dd"),
        # likelihoods of a data set of events, every event a matrix of its size
        {"name": "batch of 256", "kind": "batch", "count": 256, "n_lo": 8, "n_hi": 22, "where": "host"},
        # probabilities of the measured patterns of one state
        {"name": "clicks 200 of 26 modes", "kind": "clicks", "M": 26, "count": 200, "where": "host"},
        # the whole distribution of a small state, read back by the host
        {"name": "click_all 15 host", "kind": "click_all", "M": 15, "where": "host"},
        # the whole distribution of a large state, left on the GPU for sampling
        {"name": "click_all 25 device", "kind": "click_all", "M": 25, "where": "device"},
        # a service: a burst of events of mixed size
        {"name": "serve 48", "kind": "serve", "count": 48, "n_lo": 8, "n_hi": 25},
    ]


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "eval", "batch", "clicks", "click_all", "serve"])
    where = rng.choice(["host", "device"])
    if kind == "eval":
        # the work doubles with each mode, so a uniform size is uniform in the
        # logarithm of the work
        form = rng.choice(["state", "state", "state", "hermitian"])
        factor = "dd" if form == "state" and rng.random() < 0.25 else "fp64"
        top = 25 if factor == "dd" else 27 if form == "hermitian" else 30
        return {"kind": kind, "n": rng.randint(2, top), "form": form, "factor": factor, "where": where,
                "check": rng.random() < 0.25}
    if kind == "batch":
        lo = rng.randint(4, 16)
        return {"kind": kind, "count": int(round(2.0 ** rng.uniform(1, 8))), "n_lo": lo, "n_hi": lo + rng.randint(0, 8),
                "where": where}
    if kind == "clicks":
        return {"kind": kind, "M": rng.randint(6, 27), "count": int(round(2.0 ** rng.uniform(0, 8))), "where": where}
    if kind == "click_all":
        return {"kind": kind, "M": rng.randint(4, 18 if where == "host" else 26), "where": where}
    lo = rng.randint(6, 16)
    return {"kind": kind, "count": int(round(2.0 ** rng.uniform(1, 6))), "n_lo": lo, "n_hi": lo + rng.randint(2, 9)}


def _sizes(case):
    """Sizes of a batch's or a burst's matrices: uniform over the case's range, the same for every seed."""
    rng = np.random.default_rng(case["count"] * 64 + case["n_lo"])
    return [int(v) for v in rng.integers(case["n_lo"], case["n_hi"] + 1, case["count"])]


def _patterns(case):
    """Click patterns of a bright state: each mode clicks with probability 3/4 (the same for every seed)."""
    rng = np.random.default_rng(case["count"] * 64 + case["M"])
    return [int(sum(1 << q for q in range(case["M"]) if b[q])) for b in rng.random((case["count"], case["M"])) < 0.75]


def _bright(n, rng):
    return inputs.random_O(n, int(rng.integers(1 << 31)), 1.0, 1.5, float(rng.uniform(0.7, 1.0)))


def _matrices(case, seed):
    """The host matrices of a case."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "eval":
        if case["form"] == "hermitian":
            return [inputs.random_hpd_O(case["n"], int(rng.integers(1 << 31)), 0.3, 0.95)]
        if case["factor"] == "dd":
            return [inputs.random_O(case["n"], int(rng.integers(1 << 31)), 0.3, 1.2, 0.9)]
        return [_bright(case["n"], rng)]
    if kind in ("batch", "serve"):
        return [_bright(n, rng) for n in _sizes(case)]
    return [_bright(case["M"], rng)]


def prepare(case, seed):
    kind = case["kind"]
    mats = _matrices(case, seed)
    flags = 0
    if case.get("factor") == "dd":
        flags |= TOR_FACTOR_DD
    if case.get("check"):
        flags |= TOR_CHECK_HERMITIAN
    if case.get("where") == "device":
        flags |= TOR_INPUT_DEVICE
        if kind == "click_all":
            flags |= TOR_OUTPUT_DEVICE
        mats = [torch.from_numpy(O).cuda() for O in mats]
    state = {"kind": kind, "ctx": Context(flags=flags), "mats": mats}
    if kind == "clicks":
        state["patterns"] = _patterns(case)
    return state


def _gather(results):
    return {"tor": np.array([r.value for r in results]), "sum_abs": np.array([r.sum_abs for r in results]),
            "status": np.array([r.status for r in results]), "path": np.array([r.path for r in results])}


def run(state):
    kind, ctx, mats = state["kind"], state["ctx"], state["mats"]
    if kind == "eval":
        return _gather([ctx.eval(mats[0])])
    if kind == "batch":
        return _gather(ctx.eval_batch(mats))
    if kind == "clicks":
        probs, results = ctx.click_probs(mats[0], state["patterns"])
        return {"probs": probs, **_gather(results)}
    if kind == "click_all":
        probs, _, whole = ctx.click_all(mats[0])
        return {"probs": probs, **_gather([whole])}
    tickets = [ctx.submit(O) for O in mats]
    ctx.drain()
    return _gather([ctx.poll(t) for t in tickets])


def work(case):
    kind = case["kind"]
    if kind == "eval":
        n = case["n"]
        return {"bytes": 16 * n * (2 * n + 1), "flops": tor_flops(n, real=case["form"] == "state")}
    if kind in ("batch", "serve"):
        sizes = _sizes(case)
        return {"bytes": sum(16 * n * (2 * n + 1) + 16 for n in sizes), "flops": sum(tor_flops(n, real=True) for n in sizes)}
    M = case["M"]
    if kind == "clicks":
        sizes = [bin(p).count("1") for p in _patterns(case)]
        return {"bytes": 16 * M * (2 * M + 1) + 24 * len(sizes),
                "flops": chol_flops(2 * M) + sum(tor_flops(n, real=True) for n in sizes)}
    # every pattern: each subset's term once, and M additions per pattern
    return {"bytes": 16 * M * (2 * M + 1) + (8 << M), "flops": chol_flops(2 * M) + tor_flops(M, real=True) + (M << M)}


# --- the same values from the definition (Eq. 2), without the library ---------

_CHUNK = 21  # modes whose subsets are held at a time


def _dets(A, det, cat):
    """Determinants of every principal mode-submatrix below the nodes A (count x 2m x 2m, mode i in rows 2i and
    2i + 1) times det: bit i of the index, above the node's, says that mode i is in the subset."""
    while A.shape[1]:
        a, b, c, d = (A[:, i, j] for i in (0, 1) for j in (0, 1))
        pd = a * d - b * c
        B = A[:, 2:, 2:]
        if B.shape[1]:
            x, y = A[:, 2:, 0], A[:, 2:, 1]          # columns below the pivot block
            u, v = A[:, 0, 2:], A[:, 1, 2:]          # its rows
            s, t = (d[:, None] * u - b[:, None] * v) / pd[:, None], (a[:, None] * v - c[:, None] * u) / pd[:, None]
            B2 = B - x[:, :, None] * s[:, None, :] - y[:, :, None] * t[:, None, :]
            A = cat([B, B2])
        else:
            A = cat([B, B])
        det = cat([det, det * pd])
    return det.real


def _mode_order(O):
    n = O.shape[0] // 2
    p = np.arange(2 * n).reshape(2, n).T.reshape(-1)
    return (np.eye(2 * n) - O)[np.ix_(p, p)]


def _parity(count, xp_arange):
    """(-1)^|Z| of the masks 0..count-1."""
    z = xp_arange(count)
    s = 0
    for q in range(max(count.bit_length() - 1, 1)):
        s = s + ((z >> q) & 1)
    return 1 - 2 * (s % 2)


def _tor_exact(O, extended):
    """(Tor, sum of |t|).  extended: x87 numbers on the host (small sizes); else complex128 on torch's device."""
    n = O.shape[0] // 2
    C = _mode_order(O)
    if extended:
        A = C.astype(np.clongdouble)[None]
        t = 1 / np.sqrt(_dets(A, np.ones(1, np.clongdouble), np.concatenate))
        sign = _parity(1 << n, np.arange) * (-1) ** n
        return float((t * sign).sum()), float(t.sum())
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    top = max(0, n - _CHUNK)
    sign = _parity(1 << (n - top), lambda k: torch.arange(k, device=dev))
    whole, frac, total = 0, [], []
    for head in range(1 << top):  # the decisions on the first modes
        A, det = torch.from_numpy(C)[None], torch.ones(1, dtype=torch.complex128)
        for i in range(top):
            P, B = A[:, :2, :2], A[:, 2:, 2:]
            if (head >> i) & 1:
                B = B - A[:, 2:, :2] @ torch.linalg.solve(P, A[:, :2, 2:])
                det = det * torch.linalg.det(P)
            A = B
        t = _dets(A.to(dev), det.to(dev), torch.cat).rsqrt()
        lead = 1 - 2 * ((n + bin(head).count("1")) % 2)
        f = t.floor()  # whole parts add up exactly as integers
        whole += lead * int((f.to(torch.int64) * sign).sum())
        frac.append(lead * float(((t - f) * sign).sum()))
        total.append(float(t.sum()))
    return float(whole + math.fsum(frac)), math.fsum(total)


def _exact_results(mats, extended):
    got = [_tor_exact(O, extended and O.shape[0] <= 36) for O in mats]
    return {"tor": np.array([g[0] for g in got]), "sum_abs": np.array([g[1] for g in got]), "status": None, "path": None}


def exact(case, seed):
    kind = case["kind"]
    mats = _matrices(case, seed)
    if kind == "eval":
        if case["factor"] == "dd" and case["n"] > 18:
            return None  # 64 bits hold less than the double-double factor does
        return _exact_results(mats, case["n"] <= 18)
    if kind in ("batch", "serve"):
        return _exact_results(mats, False)
    M = case["M"]
    root = math.sqrt(np.linalg.det(np.eye(2 * M) - mats[0]).real)
    if kind == "clicks":
        sel = [[q for q in range(M) if (p >> q) & 1] for p in _patterns(case)]
        if sum(2.0 ** len(s) for s in sel) > 2.0 ** 31:
            return None
        r = _exact_results([inputs.click_submatrix(mats[0], s) for s in sel], False)
        return {"probs": r["tor"] * root, **r}
    if M > 18:
        return None  # the subset sums would have to be formed in more than 64 bits
    t = 1 / np.sqrt(_dets(_mode_order(mats[0]).astype(np.clongdouble)[None], np.ones(1, np.clongdouble), np.concatenate))
    total = float(t.sum())
    sign = _parity(1 << M, np.arange)
    g = t * sign
    for q in range(M):  # sums over the subsets of each mask
        g = g.reshape(-1, 2, 1 << q)
        g[:, 1] += g[:, 0]
        g = g.reshape(-1)
    tor = g * sign
    probs = (tor * root).astype(np.float64)
    if case["where"] == "device":
        probs = torch.from_numpy(probs)
    return {"probs": probs, "tor": np.array([float(tor[-1])]), "sum_abs": np.array([total]), "status": None, "path": None}

"""The work that a user of the library has it do, as calls through its public
entry points with the inputs they meet: single and batched encodes from one
vector to a million, encodes against list centroids, estimate scans of one
list and of a whole store with one and with many queries, the prefix and the
multi-stage scan, and the device fit.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from
a seed, ``run`` makes one pass, ``work`` says what a pass cannot do without
and ``exact`` gives the outputs in 64-bit arithmetic from plain torch.

Plans are given explicitly: the segments of a bit budget over a decaying
spectrum (16-dim units, at most 9 bits and 512 dims per segment, as the
library's defaults), M a dense orthonormal basis, c the mean.  Inside a
segment all dims have the segment's mean variance, as they do after the
random rotation that a fitted plan applies there.
"""
import heapq
import math

import numpy as np
import torch

import paper_2509_12086_amd as saq

DEV = "cuda:0"
ROWS = 131072          # rows per generated block
ROUNDS = 4             # the limit of Algorithm 1 that the configurations use


# -- cases -------------------------------------------------------------------

def listed():
    return [
        # the smallest served ingestion request: one 768-dim vector
        {"name": "encode_1x768_b4", "kind": "encode", "n": 1, "D": 768, "bpd": 4.0},
        # the median served request (512 vectors), a ragged size, the largest budget
        {"name": "encode_517x768_b6", "kind": "encode", "n": 517, "D": 768, "bpd": 6.0},
        # what a serving step hands over: the requests of three resident plans
        # in one batched call, in the launch mode that the server uses
        {"name": "batched_served_3x768", "kind": "batched", "D": 768, "grouped": True,
         "n0": 1900, "b0": 2.0, "n1": 517, "b1": 4.0, "n2": 63, "b2": 6.0},
        # a batch of text embeddings added to a store
        {"name": "encode_20011x1536_b4", "kind": "encode", "n": 20011, "D": 1536, "bpd": 4.0},
        # image features encoded against the centroids of their 1,024 lists
        {"name": "encode_ref_131072x960_b4", "kind": "encode_ref", "n": 131072, "D": 960,
         "bpd": 4.0, "K": 1024},
        # a whole dataset at once: 1M image features, the headline workload
        {"name": "encode_1000000x960_b4", "kind": "encode", "n": 1000000, "D": 960, "bpd": 4.0},
        # one query against one list of records held against its centroid
        {"name": "scan_list_1x9973x960", "kind": "scan", "nq": 1, "n": 9973, "D": 960, "bpd": 4.0,
         "prefix": 0, "ref": True},
        # one query against a whole store of text embeddings
        {"name": "scan_1x1000000x1536", "kind": "scan", "nq": 1, "n": 1000000, "D": 1536,
         "bpd": 4.0, "prefix": 0, "ref": False},
        # a batch of queries against a whole store (the scan the serving mix uses)
        {"name": "scan_64x1000000x768", "kind": "scan", "nq": 64, "n": 1000000, "D": 768,
         "bpd": 4.0, "prefix": 0, "ref": False},
        # a coarse pass over the leading two bits of long records, odd sizes
        {"name": "scan_prefix2_100x250007x3072", "kind": "scan", "nq": 100, "n": 250007,
         "D": 3072, "bpd": 4.0, "prefix": 2, "ref": False},
        # nearest-neighbour search with pruning: 10-nearest thresholds
        {"name": "multistage_8x500000x1536", "kind": "multistage", "nq": 8, "n": 500000,
         "D": 1536, "bpd": 4.0, "m": 4.0},
        # fitting a plan on rows that are on the device, the default sample size
        {"name": "fit_65536x960_b4", "kind": "fit", "n": 65536, "D": 960, "bpd": 4.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("encode", "encode", "encode", "encode_ref", "batched", "scan", "scan", "scan",
                       "multistage", "fit"))
    D = rng.choice((128, 768, 960, 1536, 3072, rng.randint(99, 3072)))
    bpd = rng.choice((2.0, 4.0, 6.0))
    if kind in ("encode", "encode_ref"):
        n = _log_int(rng, 1, min(1000000, 640000000000 // (D * D)))
        case = {"kind": kind, "n": n, "D": D, "bpd": bpd}
        if kind == "encode_ref":
            case["K"] = _log_int(rng, 1, 4096)
        return case
    if kind == "batched":
        case = {"kind": kind, "D": D, "grouped": rng.random() < 0.5}
        for i in range(rng.randint(1, 16)):
            case[f"n{i}"] = _log_int(rng, 1, min(16384, 40000000000 // (D * D)))
            case[f"b{i}"] = rng.choice((2.0, 4.0, 6.0))
        return case
    if kind == "scan":
        nq = _log_int(rng, 1, 130)
        n = _log_int(rng, 1000, min(1000000, 768000000 // D) if nq > 16 else 1000000)
        return {"kind": kind, "nq": nq, "n": n, "D": D, "bpd": bpd,
                "prefix": rng.choice((0, 0, 0, 1, 2, 4)), "ref": False}
    if kind == "multistage":
        n = _log_int(rng, 1000, min(1000000, 768000000 // D))
        return {"kind": kind, "nq": _log_int(rng, 1, 70), "n": n, "D": D, "bpd": 4.0,
                "m": rng.choice((2.0, 4.0))}
    D = rng.choice((128, 768, 960, rng.randint(99, 960)))
    return {"kind": "fit", "n": _log_int(rng, 4 * D, 65536), "D": D, "bpd": bpd}


# -- plans -------------------------------------------------------------------

# the plans fitted on the 1M x 960 image-feature mixture
FITTED = {(960, 2.0): ([224, 192, 160, 128, 256], [4, 3, 2, 1, 0]),
          (960, 4.0): ([80, 208, 176, 160, 96, 80, 64, 96], [7, 6, 5, 4, 3, 2, 1, 0])}


def _spectrum(D):
    """Per-dim variances, decreasing: an exponential over eight decay lengths,
    or at D = 960 close to the spectrum of the 1,024-cluster mixture."""
    x = np.arange(D) / D
    return 4.0 * (1.0 - x) ** 2 if D == 960 else np.exp(-8.0 * x)


def _segments(D, bpd):
    """(widths, bits) of the budget floor(bpd D): bits go one at a time to the
    16-dim unit whose modelled error 2^-b sum(variance) falls most per bit."""
    if (D, bpd) in FITTED:
        return FITTED[D, bpd]
    lam = _spectrum(D)
    units = [(a, min(D, a + 16)) for a in range(0, D, 16)]
    bits = [0] * len(units)
    left = int(bpd * D)
    heap = [(-lam[a:b].sum() / (b - a), i) for i, (a, b) in enumerate(units)]
    heapq.heapify(heap)
    while heap:
        gain, i = heapq.heappop(heap)
        w = units[i][1] - units[i][0]
        if w > left:
            continue
        left -= w
        bits[i] += 1
        if bits[i] < 9:
            heapq.heappush(heap, (gain / 2.0, i))
    widths, out = [], []
    for (a, b), k in zip(units, bits):
        if out and out[-1] == k and widths[-1] + (b - a) <= 512:
            widths[-1] += b - a
        else:
            widths.append(b - a)
            out.append(k)
    return widths, out


class _Shape:
    """A plan's numbers: segments, kept dims and their standard deviations,
    record sizes."""

    def __init__(self, D, bpd):
        self.D = D
        self.widths, self.bits = _segments(D, bpd)
        lam = _spectrum(D)
        var, pos = np.empty(D), 0
        keep = []
        for w, b in zip(self.widths, self.bits):
            var[pos:pos + w] = lam[pos:pos + w].mean()
            if b:
                keep.extend(range(pos, pos + w))
            pos += w
        self.var = var
        self.keep = np.asarray(keep, np.int64)
        self.dk = len(keep)
        self.segs = [(w, b) for w, b in zip(self.widths, self.bits) if b]
        self.code_bytes = sum(b * ((w + 7) // 8) for w, b in self.segs)
        self.n_factors = len(self.segs) + 1


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + what)
    return g


def _basis(D, seed):
    """A dense orthonormal D x D basis: two cosine transforms with random
    signs before each."""
    g = _gen(seed, 1)
    i = torch.arange(D, device=DEV, dtype=torch.float64)
    C = torch.cos(math.pi / D * (i[None, :] + 0.5) * i[:, None]) * math.sqrt(2.0 / D)
    C[0] *= math.sqrt(0.5)
    s = torch.randint(0, 2, (2, D), generator=g, device=DEV).double() * 2.0 - 1.0
    return (C * s[0]) @ (C * s[1])


def _plan_parts(shape, seed):
    """(basis FP64, M FP32 [dk x D], c FP32) of a case's plan."""
    Q = _basis(shape.D, seed)
    M = Q[torch.from_numpy(shape.keep).to(DEV)].float()
    c = torch.randn(shape.D, generator=_gen(seed, 2), device=DEV)
    return Q, M, c


def _plan(shape, M, c):
    return saq.Plan.from_parts(shape.widths, shape.bits, M.cpu().numpy(), c.cpu().numpy(),
                               variances=shape.var).upload(0)


def _rows(n, Q, sd, offset, g):
    """n rows offset + z Q with z ~ N(0, sd^2); offset: one row or one per row."""
    X = torch.empty((n, Q.shape[0]), dtype=torch.float32, device=DEV)
    Qf, sdf = Q.float(), torch.from_numpy(sd).to(DEV).float()
    for a in range(0, n, ROWS):
        b = min(n, a + ROWS)
        z = torch.randn((b - a, Q.shape[0]), generator=g, device=DEV) * sdf
        torch.addmm(offset if offset.dim() == 1 else offset[a:b], z, Qf, out=X[a:b])
    return X


# -- records for the scans ----------------------------------------------------

def _records(shape, n, seed):
    """Blocks (first row, [(codes, factor) per kept segment], norm2) of the
    records of n Gaussian vectors: the grid code of every segment, its rescale
    factor and the squared norm, from plain torch."""
    g = _gen(seed, 3)
    sd = torch.from_numpy(np.sqrt(shape.var)).to(DEV).float()
    keep = torch.from_numpy(shape.keep).to(DEV)
    for a in range(0, n, ROWS):
        z = torch.randn((min(n, a + ROWS) - a, shape.D), generator=g, device=DEV) * sd
        norm2 = (z.double() ** 2).sum(1).float()
        o, segs, col = z[:, keep], [], 0
        for w, b in shape.segs:
            x = o[:, col:col + w].double()
            v = x.abs().amax(1, keepdim=True)
            code = torch.floor((x + v) * (2.0 ** (b - 1) / v)).clamp_(0, 2 ** b - 1)
            u = code - (2 ** b - 1) / 2
            segs.append((code.int(), ((x * x).sum(1) / (u * x).sum(1)).float()))
            col += w
        yield a, segs, norm2


def _pack(shape, n, seed):
    """The packed records: codes uint8 [n, code_bytes], factors [n, n_factors]."""
    codes = torch.empty((n, shape.code_bytes), dtype=torch.uint8, device=DEV)
    factors = torch.empty((n, shape.n_factors), dtype=torch.float32, device=DEV)
    weight = 1 << torch.arange(8, device=DEV, dtype=torch.int32)
    for a, segs, norm2 in _records(shape, n, seed):
        b, pos = a + norm2.shape[0], 0
        for s, ((w, bits), (code, f)) in enumerate(zip(shape.segs, segs)):
            pb = (w + 7) // 8
            code = torch.nn.functional.pad(code, (0, 8 * pb - w)).view(b - a, pb, 8)
            for p in range(bits - 1, -1, -1):
                codes[a:b, pos:pos + pb] = (((code >> p) & 1) * weight).sum(2).to(torch.uint8)
                pos += pb
            factors[a:b, s] = f
        factors[a:b, -1] = norm2
    return codes, factors


def _queries(case, shape, seed):
    """(basis, M, c, ref or None, queries): queries around the reference that
    the records are held against."""
    Q, M, c = _plan_parts(shape, seed)
    ref = torch.randn(shape.D, generator=_gen(seed, 4), device=DEV) if case.get("ref") else None
    X = _rows(case["nq"], Q, np.sqrt(shape.var), c if ref is None else ref, _gen(seed, 5))
    return Q, M, c, ref, X


def _estimate64(case, shape, seed, M, center, X, n, bound=None):
    """Estimated squared distances [nq, n] in FP64; with bound = (tau, m) the
    multi-stage values (Section 4.3: a pair closes at the first stage whose
    lower bound exceeds its threshold)."""
    q = X.double() - center.double()
    qn = (q * q).sum(1)
    qp = q @ M.double().T.contiguous()
    out = torch.empty((X.shape[0], n), dtype=torch.float64, device=DEV)
    sig = None
    if bound is not None:
        lam = torch.from_numpy(shape.var[shape.keep]).to(DEV)
        col, sig = 0, []
        for w, _ in shape.segs:
            sig.append((qp[:, col:col + w] ** 2 * lam[col:col + w]).sum(1).sqrt())
            col += w
        sig = torch.stack(sig, 1)
        rest = sig.flip(1).cumsum(1).flip(1)                       # sum over s >= t
    prefix = case.get("prefix", 0)
    for a, segs, norm2 in _records(shape, n, seed):
        b = a + norm2.shape[0]
        base = norm2.double()[None, :] + qn[:, None]
        ip = torch.zeros_like(base)
        val, open_ = None, None
        if bound is not None:
            val, open_ = torch.zeros_like(base), torch.ones_like(base, dtype=torch.bool)
        col = 0
        for s, ((w, bits), (code, f)) in enumerate(zip(shape.segs, segs)):
            if bound is not None:
                lb = base - 2.0 * (ip + bound[1] * rest[:, s:s + 1])
                close = open_ & (lb > bound[0].double()[:, None])
                val[close] = lb[close]
                open_ &= ~close
            p = prefix if 0 < prefix < bits else bits
            u = (code >> (bits - p)).double() - (2 ** p - 1) / 2
            ip += (qp[:, col:col + w] @ u.T.contiguous()) * (f.double() * 2.0 ** (bits - p))[None, :]
            col += w
        full = base - 2.0 * ip
        out[:, a:b] = full if bound is None else torch.where(open_, full, val)
    return out


# -- the interface -------------------------------------------------------------

def _entries(case):
    k = 0
    while f"n{k}" in case:
        yield case[f"n{k}"], _Shape(case["D"], case[f"b{k}"])
        k += 1


def _encode_inputs(case, shape, seed, what=6):
    """(M, c, X, refs, ids) of an encode."""
    Q, M, c = _plan_parts(shape, seed)
    g = _gen(seed, what)
    if case["kind"] != "encode_ref":
        return M, c, _rows(case["n"], Q, np.sqrt(shape.var), c, g), None, None
    refs = _rows(case["K"], Q, 2.0 * np.sqrt(shape.var), c, _gen(seed, 7))
    ids = torch.randint(0, case["K"], (case["n"],), generator=g, device=DEV)
    X = _rows(case["n"], Q, np.sqrt(shape.var), refs[ids], g)
    return M, c, X, refs, ids.to(torch.int32)


def _out_buffers(shape, n):
    return (torch.empty((n, shape.code_bytes), dtype=torch.uint8, device=DEV),
            torch.empty((n, shape.n_factors), dtype=torch.float32, device=DEV))


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("encode", "encode_ref"):
        shape = _Shape(case["D"], case["bpd"])
        M, c, X, refs, ids = _encode_inputs(case, shape, seed)
        plan = _plan(shape, M, c)
        codes, factors = _out_buffers(shape, case["n"])
        return {"kind": kind, "plan": plan, "X": X, "refs": refs, "ids": ids, "codes": codes,
                "factors": factors, "ws": _bytes(plan.encode_workspace_bytes(case["n"]))}
    if kind == "batched":
        entries = []
        for i, (n, shape) in enumerate(_entries(case)):
            Q, M, c = _plan_parts(shape, seed + i)
            X = _rows(n, Q, np.sqrt(shape.var), c, _gen(seed + i, 6))
            entries.append((_plan(shape, M, c), X) + _out_buffers(shape, n))
        tuning = saq.BatchTuning(mode=saq.BATCH_GROUPED if case["grouped"] else saq.BATCH_FUSED)
        return {"kind": kind, "entries": entries, "tuning": tuning,
                "ws": _bytes(saq.batched_workspace_bytes(entries, tuning))}
    if kind in ("scan", "multistage"):
        shape = _Shape(case["D"], case["bpd"])
        _, M, c, ref, X = _queries(case, shape, seed)
        plan = _plan(shape, M, c)
        codes, factors = _pack(shape, case["n"], seed)
        state = {"kind": kind, "plan": plan, "Q": X, "ref": ref, "codes": codes, "factors": factors,
                 "out": torch.empty((case["nq"], case["n"]), device=DEV),
                 "ws": _bytes(plan.estimate_workspace_bytes(case["nq"]))}
        if kind == "scan":
            state["prefix"] = case["prefix"]
        else:
            state["tau"], state["m"] = _tau(case, shape, seed, M, c, X), case["m"]
            state["stage"] = torch.empty((case["nq"], case["n"]), dtype=torch.uint8, device=DEV)
        return state
    Q = _basis(case["D"], seed)
    X = _rows(case["n"], Q, np.sqrt(_spectrum(case["D"])),
              torch.randn(case["D"], generator=_gen(seed, 2), device=DEV), _gen(seed, 6))
    return {"kind": kind, "X": X, "params": saq.PlanParams(bits_per_dim=case["bpd"])}


def _tau(case, shape, seed, M, c, X):
    """Each query's 10th smallest estimate over the first 16,384 records."""
    n = min(case["n"], 16384)
    est = _estimate64(case, shape, seed, M, c, X, n)
    return torch.sort(est, dim=1)[0][:, min(9, n - 1)].float().contiguous()


def run(state):
    kind = state["kind"]
    if kind in ("encode", "encode_ref"):
        return saq.encode(state["plan"], state["X"], ROUNDS, state["codes"], state["factors"],
                          state["ws"], refs=state["refs"], ref_ids=state["ids"])
    if kind == "batched":
        return saq.encode_batched(state["entries"], ROUNDS, state["tuning"], state["ws"])
    if kind == "scan":
        return saq.estimate_dist(state["plan"], state["Q"], state["codes"], state["factors"],
                                 state["out"], state["ws"], prefix_bits=state["prefix"],
                                 ref=state["ref"])
    if kind == "multistage":
        return saq.estimate_multistage(state["plan"], state["Q"], state["codes"], state["factors"],
                                       state["tau"], state["m"], state["out"], state["stage"],
                                       state["ws"])
    plan = saq.Plan.fit_device(state["X"], state["params"])
    return {"widths": np.asarray(plan.widths), "bits": np.asarray(plan.bits),
            "arrays": plan.arrays()}


def _encode_work(n, shape):
    """Rows in, records out, M once; the projection and Algorithm 1's two
    trials per dim and round at six operations each."""
    return (n * (4 * shape.D + shape.code_bytes + 4 * shape.n_factors) + 4 * shape.D * shape.dk,
            n * shape.dk * (2 * shape.D + 12 * ROUNDS))


def work(case):
    kind = case["kind"]
    if kind == "batched":
        parts = [_encode_work(n, shape) for n, shape in _entries(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    D, n = case["D"], case["n"]
    if kind == "fit":
        # rows in, plan out; the covariance's upper triangle and a dense
        # symmetric eigen-decomposition (tridiagonalisation and QL: 9 D^3)
        return {"bytes": 4 * n * D + 8 * D * D, "flops": n * D * (D + 1) + 9 * D ** 3}
    shape = _Shape(D, case["bpd"])
    if kind in ("encode", "encode_ref"):
        b, f = _encode_work(n, shape)
        return {"bytes": b + (4 * case["K"] * D + 4 * n if kind == "encode_ref" else 0), "flops": f}
    nq = case["nq"]
    if kind == "multistage":
        # every pair reads at least the first segment
        w, bits = shape.segs[0]
        read, dims, outb = bits * ((w + 7) // 8) + 8, w, 5
    else:
        p = case["prefix"] or 16
        read = sum(min(b, p) * ((w + 7) // 8) for w, b in shape.segs) + 4 * shape.n_factors
        dims, outb = shape.dk, 4
    return {"bytes": n * read + nq * n * outb + 4 * nq * D + 4 * D * shape.dk,
            "flops": 2 * nq * n * dims + 2 * nq * D * shape.dk}


def _factors64(shape, O, norm2):
    """Algorithm 1's factors for projected rows O [n, dk] in FP64."""
    out = torch.empty((O.shape[0], shape.n_factors), dtype=torch.float64, device=DEV)
    col = 0
    for s, (w, b) in enumerate(shape.segs):
        o = O[:, col:col + w].T.contiguous()
        col += w
        cmax = 2 ** b - 1
        v = o.abs().amax(0)
        c = torch.floor((o + v) / (2.0 * v / 2 ** b)).clamp_(0, cmax)
        u = c - cmax / 2
        ip, nn = (u * o).sum(0), (u * u).sum(0)
        for _ in range(ROUNDS if b >= 2 else 0):
            moved = torch.zeros((), dtype=torch.bool, device=DEV)
            for i in range(w):
                x, ui = o[i], u[i]
                P = ip * ip
                A = nn * x * x - P
                Bv = 2.0 * x * nn * ip - 2.0 * ui * P
                up = (A + Bv > 0) & (ui < cmax / 2)
                dn = (A - Bv > 0) & (ui > -cmax / 2) & ~up
                sg = up.double() - dn.double()
                nn += sg * (2.0 * ui + sg)
                ip += sg * x
                ui += sg
                moved |= (up | dn).any()
            if not bool(moved):
                break
        out[:, s] = (o * o).sum(0) / ip
    out[:, -1] = norm2
    return out


def _encode64(shape, M, X, center):
    """Factors [n, n_factors] in FP64; center: one row or a function of a row range."""
    parts, step = [], 262144
    Mt = M.double().T.contiguous()
    for a in range(0, X.shape[0], step):
        b = min(X.shape[0], a + step)
        y = X[a:b].double() - (center(a, b) if callable(center) else center.double())
        parts.append(_factors64(shape, y @ Mt, (y * y).sum(1)))
    return torch.cat(parts)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batched":
        out = []
        for i, (n, shape) in enumerate(_entries(case)):
            Q, M, c = _plan_parts(shape, seed + i)
            X = _rows(n, Q, np.sqrt(shape.var), c, _gen(seed + i, 6))
            out.append((None, _encode64(shape, M, X, c)))
        return out
    if kind == "fit":
        return None            # M carries the fit's own random rotations
    shape = _Shape(case["D"], case["bpd"])
    if kind in ("encode", "encode_ref"):
        M, c, X, refs, ids = _encode_inputs(case, shape, seed)
        center = c if refs is None else (lambda a, b: refs[ids[a:b].long()].double())
        return None, _encode64(shape, M, X, center)
    _, M, c, ref, X = _queries(case, shape, seed)
    center = c if ref is None else ref
    if kind == "scan":
        return _estimate64(case, shape, seed, M, center, X, case["n"])
    tau = _tau(case, shape, seed, M, c, X)
    return _estimate64(case, shape, seed, M, center, X, case["n"], (tau, case["m"])), None

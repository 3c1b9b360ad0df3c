"""The plain scans where a query's components differ by orders of magnitude: an
estimate may be off by FP32 rounding of its own terms, not by that of a
component that the record does not meet.

Largest absolute error, with A = sum_s f_s sum_j |u_j q'_j| and 2^-24 of a value
for each rounding of it:
  integer passes (rows of M within 8 times each other's length): 5 roundings per
    pass and 5 more of ||o||^2 + ||q||^2 + 2 A, the queries' fixed point below
    one of them;
  split operands: a segment of 128 dims takes 8 16-dim products of up to 6 terms,
    at most two roundings each of 2 A, and 4 for the operands' splits: 100 of 2 A,
    and 5 of the scale."""
import numpy as np
import pytest

import oracle
import paper_2509_12086_amd as saq
from gpu_util import say, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [1, 4, 12, 40, 70])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("R", [1.0, 8.0, 64.0, 1024.0, 16384.0, 2.0 ** 30])
@pytest.mark.parametrize("where", ["one row", "a segment", "one row of a segment"])
def test_uneven_rows(where, R, bits, nq):
    """M is diagonal, one of its rows (or all of a segment's) R times as long as
    the others, and the records have no energy there."""
    D = 128
    widths = [128] if where == "one row" else [16, 112]
    long = slice(0, 16) if where == "a segment" else slice(0, 1)
    rng = np.random.default_rng(int(R) % 1000 + bits + nq)
    M = np.eye(D, dtype=np.float32)
    M[long] *= np.float32(R)
    plan = saq.Plan.from_parts(widths, [bits] * len(widths), M, np.zeros(D, np.float32)).upload(0)
    X = rng.standard_normal((161, D))
    X[:, : 16 if where != "one row" else 1] = 0.0
    X = (X / np.linalg.norm(X, axis=1, keepdims=True)).astype(np.float32)
    Q = rng.standard_normal((nq, D))
    Q = (Q / np.linalg.norm(Q, axis=1, keepdims=True)).astype(np.float32)
    enc = oracle.encode(X, M, np.zeros(D, np.float32), widths, plan.kept_bits, 4)
    fac = np.concatenate([enc.factors, enc.norm2[:, None]], axis=1).astype(np.float32)
    got = saq.estimate_dist(plan, to_dev(Q), to_dev(oracle.pack(enc.codes, widths, plan.kept_bits)), to_dev(fac))
    torch.cuda.synchronize()
    f64 = fac.astype(np.float64)
    ref = oracle.estimate(Q, M, np.zeros(D, np.float32), widths, plan.kept_bits, enc.codes, f64[:, :-1], f64[:, -1])
    qp = np.abs(Q.astype(np.float64) * np.diag(M))
    A, col = np.zeros((nq, len(X))), 0
    for s, w in enumerate(widths):
        u = np.abs(enc.codes[:, col:col + w] - (2 ** bits - 1) / 2) * f64[:, s:s + 1]
        A += qp[:, col:col + w] @ u.T
        col += w
    scale = f64[:, -1][None, :] + (Q.astype(np.float64) ** 2).sum(1)[:, None]
    split = R > 8
    tol = (100 * 2 * A + 5 * scale if split else (5 * len(widths) + 5) * (scale + 2 * A)) * 2.0 ** -24
    err = np.abs(got.cpu().numpy() - ref)
    say(f"  {where} R={R:g} {bits} bits nq={nq}: error {np.max(err / scale) * 2 ** 24:.2f} x 2^-24 of the scale, "
        f"{np.max(err / tol):.2f} of the bound")
    assert np.all(err <= tol)


@pytest.mark.parametrize("nq", [1, 4, 12, 40, 70])
@pytest.mark.parametrize("bits", [3, 8])
def test_small_components(bits, nq):
    """Segments whose spread halves from one to the next, seven times, and
    records with energy in one of them alone, their stored norms taking away
    ||q||^2, so that -2 <o, q> is the whole estimate: however small the segment's
    components, it is good to the roundings of its one pass (two with 8 planes)
    and of the queries' fixed point, a half unit of 2^-30 of a query's largest
    component weighted by 2^min(3, s) for every dim of segment s."""
    W, S = 48, 8
    rng = np.random.default_rng(bits + nq)
    sd = np.repeat(2.0 ** -np.arange(S), W)
    D = W * S
    plan = saq.Plan.from_parts([W] * S, [bits] * S, np.eye(D, dtype=np.float32), np.zeros(D, np.float32),
                               sd ** 2).upload(0)
    Q = (rng.standard_normal((nq, D)) * sd).astype(np.float32)
    _, qn2 = saq.project(plan, to_dev(Q))
    n = 130
    codes = rng.integers(0, 2 ** bits, (n, D)).astype(np.int32)
    packed = to_dev(oracle.pack(codes, plan.kept_widths, plan.kept_bits))
    top = np.max(np.abs(Q) * 2.0 ** np.minimum(np.repeat(np.arange(S), W), 3), axis=1)
    unit = 2.0 ** (np.frexp(top)[1] - 30)
    for s in range(S):
        cols = slice(s * W, (s + 1) * W)
        u = codes[:, cols] - (2 ** bits - 1) / 2
        f = rng.lognormal(0.0, 1.0, n).astype(np.float32)
        for q in range(nq):
            fac = np.zeros((n, S + 1), np.float32)
            fac[:, s] = f
            fac[:, -1] = -float(qn2[q])
            got = saq.estimate_dist(plan, to_dev(Q), packed, to_dev(fac))[q].cpu().numpy()
            fu = f.astype(np.float64)[:, None] * u
            ref = -2.0 * (fu @ Q[q, cols].astype(np.float64))
            fixed = 2.0 * np.abs(fu).sum(1) * 0.5 * unit[q] * 2.0 ** -min(s, 3)
            tol = 15 * 2.0 ** -24 * 2.0 * (np.abs(fu) @ np.abs(Q[q, cols])) + fixed
            assert np.all(np.abs(got - ref) <= tol), (s, q, np.max(np.abs(got - ref) / tol))


@pytest.mark.parametrize("nq", [3, 12, 40])
def test_queries_that_are_not_finite(nq):
    """A query with an infinite or NaN entry has NaN estimates, whichever kernel
    takes it, and its neighbours keep theirs to the bit; finite components whose
    squares overflow give infinities."""
    widths, bits = [80, 64, 99], [7, 9, 3]
    rng = np.random.default_rng(nq)
    D = sum(widths)
    plan = saq.Plan.from_parts(widths, bits, np.eye(D, dtype=np.float32), np.zeros(D, np.float32)).upload(0)
    codes = np.concatenate([rng.integers(0, 2 ** b, (150, w)) for w, b in zip(widths, bits)], 1).astype(np.int32)
    packed = to_dev(oracle.pack(codes, widths, bits))
    fac = to_dev((0.1 * rng.lognormal(0.0, 1.0, (150, 4))).astype(np.float32))
    Q = rng.standard_normal((nq, D)).astype(np.float32)
    want = saq.estimate_dist(plan, to_dev(Q), packed, fac)
    rest = [q for q in range(nq) if q != 1]
    for value, expect in ((np.nan, torch.isnan), (np.inf, torch.isnan), (-np.inf, torch.isnan),
                          (1e20, torch.isposinf), (1e30, torch.isposinf), (-1e32, torch.isposinf)):
        for where in (0, 100, D - 1):
            P = Q.copy()
            P[1, where] = value
            got = saq.estimate_dist(plan, to_dev(P), packed, fac)
            torch.cuda.synchronize()
            say(f"  nq={nq} {value} at {where}: {got[1, :3].tolist()}")
            assert bool(expect(got[1]).all())
            assert torch.equal(got[rest], want[rest])

"""Scans that unpack codes to split bf16 operands (the multi-stage scan and the
plain scan of many queries over narrow passes) at the segment widths and bits
where the unpacking can go wrong: around the 32-dim k-step and the 64-dim pairs
whose planes are fetched at once, and 1 to 16 bits around the 8 planes of one
transposition; odd plane and record sizes.

Thresholds of +inf keep every pair to the end, so the multi-stage scan's values
are full estimates.  Both sum FP32 terms with |f_s (c - h)| |q'_j| below
||o|| ||q||-sized products: W <= 300 kept dims of FP32 rounding 2^-24 each, and
the split products' 2^-22, stay under 2e-5 of ||o||^2 + ||q||^2."""
import numpy as np
import pytest

import oracle
import paper_2509_12086_amd as saq
from gpu_util import say, to_dev
from test_gpu_scan import _case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [([31, 32, 33], [1, 8, 9]), ([63, 64, 65], [8, 9, 7]), ([95, 96, 97], [16, 2, 10]),
          ([127, 128, 40], [9, 5, 15]), ([129, 160], [11, 3]), ([191, 72], [8, 12]), ([256, 24], [13, 6]),
          ([64] * 4, [14, 4, 16, 1])]


@pytest.mark.parametrize("widths,bits", SHAPES)
@pytest.mark.parametrize("nq", [1, 9, 33])
def test_multistage_unpacking(widths, bits, nq):
    _, codes, packed, fac, Q = _case(widths, bits, 161, nq, nq + widths[0])
    D = sum(widths)
    # every dim's spread: no kept segment's bound matters under +inf
    plan = saq.Plan.from_parts(widths, bits, np.eye(D, dtype=np.float32), np.zeros(D, np.float32),
                               np.ones(D)).upload(0)
    say(f"multi-stage W {widths} B {bits} nq={nq}")
    tau = torch.full((nq,), float("inf"), device="cuda:0")
    got, stage = saq.estimate_multistage(plan, to_dev(Q), to_dev(packed), to_dev(fac), tau, 4.0)
    torch.cuda.synchronize()
    assert bool((stage == len(widths)).all())
    _agrees(plan, codes, fac, Q, got)


@pytest.mark.parametrize("nq", [17, 40, 64])
@pytest.mark.parametrize("widths,bits", [([64, 65, 66, 63, 70], [9, 12, 16, 10, 9]), ([32] * 5, [9, 8, 16, 1, 11]),
                                         ([30, 17, 33, 9], [10, 8, 5, 16])])
def test_narrow_passes(widths, bits, nq):
    plan, codes, packed, fac, Q = _case(widths, bits, 161, nq, nq + widths[0])
    say(f"narrow passes W {widths} B {bits} nq={nq}")
    got = saq.estimate_dist(plan, to_dev(Q), to_dev(packed), to_dev(fac))
    torch.cuda.synchronize()
    _agrees(plan, codes, fac, Q, got)


def _agrees(plan, codes, fac, Q, got):
    f64 = fac.astype(np.float64)
    M, c, _ = plan.arrays()
    ref = oracle.estimate(Q, M, c, plan.kept_widths, plan.kept_bits, codes, f64[:, :-1], f64[:, -1])
    scale = f64[:, -1][None, :] + (Q.astype(np.float64) ** 2).sum(1)[:, None]
    err = np.max(np.abs(got.cpu().numpy() - ref) / scale)
    say(f"  error {err:.1e} of the scale")
    assert err < 2e-5


@pytest.mark.parametrize("nq", [3, 6, 14, 16])
@pytest.mark.parametrize("widths,bits", [([16] * 30, [4] * 30), ([24, 17, 16] * 12, [5, 9, 2] * 12)])
def test_narrow_passes_of_few_queries(widths, bits, nq):
    """Few queries whose digits do not fit in LDS take the same kernel as 32 of
    them: narrow passes are slow in the other one from the first query on.  The
    same kernel gives the same bits."""
    plan, codes, packed, fac, Q = _case(widths, bits, 161, 32, nq + len(widths))
    want = saq.estimate_dist(plan, to_dev(Q), to_dev(packed), to_dev(fac))
    got = saq.estimate_dist(plan, to_dev(Q[:nq]), to_dev(packed), to_dev(fac))
    torch.cuda.synchronize()
    assert torch.equal(got, want[:nq])
    _agrees(plan, codes, fac, Q, want)

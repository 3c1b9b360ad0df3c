"""Which kernel saq_project runs by sizes and alignment: the one for few rows only
where it is the faster, with norms or without; and the outputs do not depend on
the kernel or on how a row is staged, so they are the same bit by bit for the
same rows in every launch."""
import ctypes

import numpy as np
import pytest

import paper_2509_12086_amd as saq
from gpu_util import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(D, bits):
    return saq.Plan.from_parts([D // 2, D // 2], bits, np.eye(D, dtype=np.float32),
                               np.zeros(D, np.float32)).upload(0)


def _project(plan, X, norms):
    n, ld = X.shape[0], plan.D_kept
    out = torch.full((n, ld), float("nan"), device="cuda")
    nr = torch.full((n if norms else 1,), float("nan"), device="cuda")
    P = ctypes.c_void_p
    assert saq.lib().saq_project(plan._h, P(X.data_ptr()), n, P(out.data_ptr()), ld, 0,
                                 P(nr.data_ptr()) if norms else None, P(0)) == 0
    torch.cuda.synchronize()
    return out, nr


def _rows(n, D, shift):
    x = torch.randn(n * D + shift, generator=torch.Generator("cuda").manual_seed(n + D), device="cuda")
    return x[shift:].view(n, D)


# (dims, bits, rows, floats off a 16-byte boundary, whether the kernel for few rows runs)
ROUTES = [
    (64, [8, 4], 40, 0, False), (64, [8, 4], 4, 1, False), (96, [8, 4], 40, 0, True),
    (128, [8, 4], 2200, 0, False), (128, [8, 4], 300, 0, True), (128, [8, 4], 100, 1, False),
    (128, [8, 4], 4, 1, True), (3072, [8, 4], 450, 1, False), (3072, [8, 4], 100, 1, True),
    (768, [4, 4], 350, 0, False), (768, [8, 4], 350, 0, True),
]


@pytest.mark.parametrize("D,bits,n,shift,few", ROUTES)
def test_kernel_for_few_rows(D, bits, n, shift, few):
    from torch.profiler import ProfilerActivity, profile
    plan, X = _plan(D, bits), _rows(n, D, shift)
    for norms in (True, False):
        with profile(activities=[ProfilerActivity.CUDA]) as pr:
            _project(plan, X, norms)
        names = [e.name for e in pr.events() if "project" in e.name]
        say(f"  {D} x {n} +{shift} norms {norms}: {[v[-40:] for v in names]}")
        assert names and all(("project_few" in v) == few for v in names)


# Rows on each side of the lines between the tiles and between the ways a row is
# staged, for 4 column tiles of 64 (2 of 128) and 5 (3), with totals and without:
# 128, 512 and 720 small tiles, 340, 512, 704 and 1024 larger ones.
@pytest.mark.parametrize("D,bits", [(256, [8, 4]), (320, [8, 4]), (320, [4, 4])])
def test_same_bits_on_each_side_of_the_lines(D, bits):
    plan = _plan(D, bits)
    small, large = D // 64, (D + 127) // 128
    edges = {64 * (b // c) + d for b, c in ((128, small), (512, small), (720, small), (340, large),
                                            (512, large), (704, large), (1024, large)) for d in (0, 1)}
    X = _rows(max(edges), D, 0)
    want, norm = _project(plan, X, True)
    ref = X.double() @ torch.from_numpy(np.eye(D)).cuda()
    # o is exact to the dropped split products, 2^-22 of the row's largest term
    assert float((want.double() - ref).abs().max()) <= 2.0 ** -22 * float(X.abs().max())
    for n in sorted(edges):
        say(f"  {n} x {D}")
        for norms in (True, False):
            out, nr = _project(plan, X[:n], norms)
            assert torch.equal(out, want[:n])
            if norms:
                assert torch.equal(nr, norm[:n])

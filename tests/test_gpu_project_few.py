"""The projection of few rows (one workgroup per 32 x 32 block) against the
tiled projection of the same rows inside a large batch: every output element
and norm goes through the same operations, so the bits are equal.  Input
dimensions around the k-steps of 16, the 32-wide k-tiles, the rounds of 512
(FP64 totals) and 1,024 dims (the FP32 chain); kept dims around the blocks of
32; rows around 32 and 64; both accumulations (a segment of 8 or more bits
takes FP64 totals); all layouts, unaligned rows and per-row references."""
import numpy as np
import pytest

import paper_2509_12086_amd as saq
from gpu_util import say, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BIG = 40_000       # rows that take the tiled kernel


def _plan(D, dk, bits, seed):
    rng = np.random.default_rng(seed)
    M = rng.standard_normal((dk, D)).astype(np.float32) / np.float32(np.sqrt(D))
    c = rng.standard_normal(D).astype(np.float32)
    widths, b = ([dk, D - dk], [bits, 0]) if dk < D else ([dk], [bits])
    if dk == 0:
        widths, b = [D], [0]
    return saq.Plan.from_parts(widths, b, M, c).upload(0)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("D,dk", [(1, 1), (5, 3), (15, 15), (16, 0), (17, 17), (32, 31), (33, 33), (100, 64),
                                  (128, 97), (130, 130), (511, 40), (516, 33), (960, 130), (1024, 65)])
def test_few_rows_equal_the_tiled_projection(D, dk, bits):
    plan = _plan(D, dk, bits, D + dk)
    g = torch.Generator(device="cuda:0").manual_seed(D)
    X = torch.randn((BIG, D), generator=g, device="cuda:0")
    O, nrm = saq.project(plan, X)
    torch.cuda.synchronize()
    for n in (1, 31, 32, 33, 64, 65, 300):
        rows = X[:n].contiguous()
        o, m = saq.project(plan, rows)
        shifted = torch.empty(n * D + 1, device="cuda:0")[1:].view(n, D)     # 4-byte aligned only
        shifted.copy_(rows)
        o2, m2 = saq.project(plan, shifted)
        od, md = saq.project(plan, rows, layout=saq.LAYOUT_DIMS)
        ot, mt = saq.project(plan, rows, layout=saq.LAYOUT_TILES)
        torch.cuda.synchronize()
        for got in (m, m2, md, mt):
            assert torch.equal(got, nrm[:n]), n
        if dk == 0:
            continue
        assert torch.equal(o, O[:n]) and torch.equal(o2, O[:n]), n
        assert torch.equal(od[:, :n], O[:n].T), n
        flat = ot.transpose(1, 2).reshape(-1, dk)
        assert torch.equal(flat[:n], O[:n]), n
        # the slots past n hold copies of the last row
        assert torch.equal(flat[n:], O[n - 1].expand(flat.shape[0] - n, dk)), n
    say(f"D={D} kept={dk} bits={bits}: equal")


@pytest.mark.parametrize("D,dk", [(1025, 40), (1600, 33), (3072, 64)])
def test_long_rows(D, dk):
    plan = _plan(D, dk, 3, D)
    g = torch.Generator(device="cuda:0").manual_seed(D)
    X = torch.randn((BIG, D), generator=g, device="cuda:0")
    O, nrm = saq.project(plan, X)
    o, m = saq.project(plan, X[:70])
    torch.cuda.synchronize()
    assert torch.equal(o, O[:70]) and torch.equal(m, nrm[:70])


@pytest.mark.parametrize("D,bits", [(96, 4), (99, 9), (1030, 5)])
def test_references(D, bits):
    """Records against their references, few at a time and in one batch."""
    plan = _plan(D, 48, bits, D)
    g = torch.Generator(device="cuda:0").manual_seed(D)
    refs = torch.randn((7, D), generator=g, device="cuda:0")
    ids = torch.randint(-1, 8, (BIG,), generator=g, device="cuda:0").to(torch.int32)   # some out of range
    X = torch.randn((BIG, D), generator=g, device="cuda:0")
    codes, fac = saq.encode(plan, X, 4, refs=refs, ref_ids=ids)
    for n in (1, 40, 200):
        c, f = saq.encode(plan, X[:n].contiguous(), 4, refs=refs, ref_ids=ids[:n].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(c, codes[:n]), n
        assert torch.equal(f.view(torch.int32), fac[:n].view(torch.int32)) or \
            torch.equal(torch.nan_to_num(f, nan=-1.0), torch.nan_to_num(fac[:n], nan=-1.0)), n
        bad = (ids[:n] < 0) | (ids[:n] >= 7)
        assert torch.equal(torch.isnan(f[:, -1]), bad), n

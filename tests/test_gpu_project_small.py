"""The projection's 64 x 64 tiles, which middle-sized launches take, against the
larger tiles of the same rows inside a large batch: every output element and
norm goes through the same operations, so the bits are equal.  Input dimensions
around the k-steps of 16 and the 32-wide k-tiles; kept dims around the tiles of
64 and the 128-dim blocks of the pre-split matrix; ragged rows; both
accumulations (a segment of 8 bits takes FP64 totals); all layouts, per-row
references and grouped batches."""
import pytest

import paper_2509_12086_amd as saq
from gpu_util import say
from test_gpu_project_few import BIG, _plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _rows(dk, bits, refs=False):
    """The smallest row count past the one-block-per-workgroup kernel, and one
    below the larger tiles."""
    few = (512 if bits >= 8 else 450 if refs else 300) // ((dk + 31) // 32 + 1) * 32
    tile = 64 if bits >= 8 else 128
    limit = 128 if refs else 360 if bits >= 8 else 224
    top = (limit - 1) // max(1, (dk + 127) // 128) * tile
    assert few + 1 < top < BIG
    return few + 1, top - 3


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("D,dk", [(4, 4), (16, 0), (20, 20), (32, 32), (36, 36), (64, 64), (68, 65), (100, 97),
                                  (128, 128), (132, 129), (200, 192), (260, 193), (960, 200)])
def test_small_tiles_equal_the_large(D, dk, bits):
    plan = _plan(D, dk, bits, D + dk)
    g = torch.Generator(device="cuda:0").manual_seed(D)
    X = torch.randn((BIG, D), generator=g, device="cuda:0")
    O, nrm = saq.project(plan, X)
    for n in _rows(dk, bits):
        say(f"D={D} kept={dk} bits={bits} n={n}")
        rows = X[:n].contiguous()
        o, m = saq.project(plan, rows)
        od, md = saq.project(plan, rows, layout=saq.LAYOUT_DIMS)
        ot, mt = saq.project(plan, rows, layout=saq.LAYOUT_TILES)
        torch.cuda.synchronize()
        for got in (m, md, mt):
            assert torch.equal(got, nrm[:n])
        if dk == 0:
            continue
        assert torch.equal(o, O[:n])
        assert torch.equal(od[:, :n], O[:n].T)
        flat = ot.transpose(1, 2).reshape(-1, dk)
        assert torch.equal(flat[:n], O[:n])
        assert torch.equal(flat[n:], O[n - 1].expand(flat.shape[0] - n, dk))


@pytest.mark.parametrize("D,bits", [(96, 4), (100, 9)])
def test_references(D, bits):
    plan = _plan(D, 72, bits, D)
    g = torch.Generator(device="cuda:0").manual_seed(D)
    refs = torch.randn((7, D), generator=g, device="cuda:0")
    ids = torch.randint(-1, 8, (BIG,), generator=g, device="cuda:0").to(torch.int32)   # some out of range
    X = torch.randn((BIG, D), generator=g, device="cuda:0")
    codes, fac = saq.encode(plan, X, 4, refs=refs, ref_ids=ids)
    for n in _rows(72, bits, refs=True):
        say(f"references D={D} bits={bits} n={n}")
        c, f = saq.encode(plan, X[:n].contiguous(), 4, refs=refs, ref_ids=ids[:n].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(c, codes[:n])
        assert torch.equal(torch.nan_to_num(f, nan=-1.0), torch.nan_to_num(fac[:n], nan=-1.0))


@pytest.mark.parametrize("bits", [(4, 4, 4), (4, 8, 4)])
def test_grouped_batch(bits):
    g = torch.Generator(device="cuda:0").manual_seed(5)
    plans = [_plan(96 + 36 * i, 40 + 50 * i, b, 9 + i) for i, b in enumerate(bits)]
    Xs = [torch.randn((n, p.D), generator=g, device="cuda:0") for n, p in zip((2500, 3001, 70), plans)]
    say(f"grouped batch, bits {bits}")
    got = saq.encode_batched(list(zip(plans, Xs)), 4, saq.BatchTuning(mode=saq.BATCH_GROUPED))
    for p, X, (c, f) in zip(plans, Xs, got):
        c0, f0 = saq.encode(p, X, 4)
        torch.cuda.synchronize()
        assert torch.equal(c, c0) and torch.equal(f, f0)

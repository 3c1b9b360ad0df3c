"""Launches past the kernels for few rows and the 64 x 64 tiles: the 128- and
64-row projection tiles at input dimensions around the ends of their k-loop
(16-byte loads, then element loads; rows of odd length or 4-byte alignment take
the latter throughout), with and without a reference per record, and one
quantize workgroup per segment just past the line of the kernel for few vectors.
Every output goes through the same operations in all of them, so slices of a
large batch, its ends included, have the bits they get in small ones."""
import pytest

import paper_2509_12086_amd as saq
from gpu_util import say
from test_gpu_project_few import _plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 40_037


def _inputs(D, shift):
    g = torch.Generator(device="cuda:0").manual_seed(D)
    X = torch.randn(N * D + shift, generator=g, device="cuda:0")[shift:].view(N, D)
    refs = torch.randn((7, D), generator=g, device="cuda:0")
    ids = torch.randint(0, 7, (N,), generator=g, device="cuda:0").to(torch.int32)
    return X, refs, ids


SLICES = [(0, 100), (63, 129), (20_000, 20_200), (N - 37, N), (N - 133, N)]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("D", [16, 32, 48, 64, 80, 99, 100, 132, 200, 515])
def test_projection_k_loop(D, bits, shift):
    plan = _plan(D, min(D, 72), bits, D)
    X, _, _ = _inputs(D, shift)
    assert X.data_ptr() % 16 == 4 * shift
    O, nrm = saq.project(plan, X)
    for a, b in SLICES:
        o, m = saq.project(plan, X[a:b].clone())
        torch.cuda.synchronize()
        assert torch.equal(o, O[a:b]) and torch.equal(m, nrm[a:b]), (a, b)
    say(f"projection D={D} bits={bits} {4 * shift} bytes off: slices equal")


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("D", [33, 96, 99, 100, 514])
def test_references(D, bits, shift):
    plan = _plan(D, min(D, 72), bits, D)
    X, refs, ids = _inputs(D, shift)
    codes, fac = saq.encode(plan, X, 4, refs=refs, ref_ids=ids)
    for a, b in SLICES:
        c, f = saq.encode(plan, X[a:b].clone(), 4, refs=refs, ref_ids=ids[a:b].clone())
        torch.cuda.synchronize()
        assert torch.equal(c, codes[a:b]) and torch.equal(f, fac[a:b]), (a, b)
    say(f"references D={D} bits={bits} {4 * shift} bytes off: slices equal")


@pytest.mark.parametrize("widths,bits", [([512, 5], [7, 3]), ([511, 480], [12, 5]), ([300, 200, 16], [16, 9, 1])])
def test_quantize_at_the_line(widths, bits):
    """n vectors with n (kept dims + 60 per segment) just below and just above
    32,768 times the widest segment, against the walk over all segments that a
    call without norm2 takes."""
    dk = sum(widths)
    plan = saq.Plan.from_parts(widths, bits, torch.eye(dk).numpy(), torch.zeros(dk).numpy()).upload(0)
    line = 32768 * max(widths) // (dk + 60 * len(widths))
    g = torch.Generator(device="cuda:0").manual_seed(dk)
    O = torch.randn((line + 70, dk), generator=g, device="cuda:0")
    O[1] = 0.0
    for n in (line - 1, line + 1, line + 70):
        nrm = (O[:n].double() ** 2).sum(1).float()
        for rounds in (0, 2):
            c0, f0 = saq.quantize(plan, O[:n], rounds)
            c1, f1 = saq.quantize(plan, O[:n], rounds, norm2=nrm)
            torch.cuda.synchronize()
            assert torch.equal(c0, c1) and torch.equal(f0[:, :-1], f1[:, :-1]) and torch.equal(f1[:, -1], nrm), (n, rounds)
    say(f"quantize W {widths} B {bits}: equal around {line} vectors")

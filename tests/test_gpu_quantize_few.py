"""Quantization of few vectors (one wave per vector and segment) and of one
segment per workgroup, against the kernel that walks all segments of 64 vectors
per wave (the route without norm2, which the parity tests hold to the oracle):
the same operations in the same order, so every byte and factor is equal.
Sizes: segment widths around the 64-dim chunk and the widest the wave holds
(wider plans keep the other kernel), 1 to 16 bits, vectors around the
8 of a workgroup and the 64 of a tile, on both sides of the dispatch's line."""
import numpy as np
import pytest

import paper_2509_12086_amd as saq
from gpu_util import say, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [([1], [4]), ([1, 2, 3], [16, 1, 9]), ([63, 64, 65], [9, 4, 2]), ([127, 129], [8, 16]),
          ([512, 5], [7, 3]), ([511, 480], [12, 5]), ([640, 20], [6, 8]), ([16] * 9, [9, 8, 7, 6, 5, 4, 3, 2, 1])]


def _rows(n, dk, seed):
    rng = np.random.default_rng(seed)
    O = (rng.standard_normal((n, dk)) * rng.lognormal(0.0, 2.0, (n, 1))).astype(np.float32)
    O[rng.random((n, dk)) < 0.05] = 0.0
    if n > 2:
        O[1] = 0.0                                   # every segment zero
        O[2, : dk // 2] = np.float32(0.75)           # ties at the largest magnitude
    return O


@pytest.mark.parametrize("widths,bits", SHAPES)
def test_few_and_split_match_the_whole_walk(widths, bits):
    dk = sum(widths)
    plan = saq.Plan.from_parts(widths, bits, np.eye(dk, dtype=np.float32), np.zeros(dk, np.float32)).upload(0)
    for n in (1, 7, 8, 9, 64, 65, 130, 20000):
        if n * dk > 4_000_000:
            n = 4_000_000 // dk
        O = _rows(n, dk, n + dk)
        nrm = to_dev((O.astype(np.float64) ** 2).sum(1).astype(np.float32))
        od = to_dev(O)
        for rounds in (0, 1, 4, 16):
            c0, f0 = saq.quantize(plan, od, rounds)
            c1, f1 = saq.quantize(plan, od, rounds, norm2=nrm)
            torch.cuda.synchronize()
            assert torch.equal(c0, c1), (n, rounds)
            assert torch.equal(f0[:, :-1], f1[:, :-1]), (n, rounds)
            assert torch.equal(f1[:, -1], nrm), (n, rounds)
    say(f"W {widths[:4]} B {bits[:4]}: few and split equal the whole walk")


def test_layouts_and_strides():
    widths, bits = [70, 33, 5], [9, 5, 2]
    dk = sum(widths)
    plan = saq.Plan.from_parts(widths, bits, np.eye(dk, dtype=np.float32), np.zeros(dk, np.float32)).upload(0)
    for n in (1, 63, 65, 200):
        O = _rows(n, dk, n)
        nrm = to_dev((O.astype(np.float64) ** 2).sum(1).astype(np.float32))
        want = saq.quantize(plan, to_dev(O), 4)
        rows = torch.full((n, dk + 7), float("nan"), device="cuda:0")
        rows[:, :dk] = to_dev(O)
        dims = torch.full((dk, (n + 7) // 4 * 4), float("nan"), device="cuda:0")
        dims[:, :n] = to_dev(O).T
        tiles = torch.full(((n + 63) // 64, dk + 3, 64), float("nan"), device="cuda:0")
        flat = torch.full((((n + 63) // 64) * 64, dk), float("nan"), device="cuda:0")
        flat[:n] = to_dev(O)
        tiles[:, :dk] = flat.view(-1, 64, dk).transpose(1, 2)
        for buf, layout in ((rows, saq.LAYOUT_ROWS), (dims, saq.LAYOUT_DIMS), (tiles, saq.LAYOUT_TILES)):
            c, f = saq.quantize(plan, buf, 4, norm2=nrm, layout=layout, n=n)
            torch.cuda.synchronize()
            assert torch.equal(c, want[0]) and torch.equal(f[:, :-1], want[1][:, :-1]), (n, layout)

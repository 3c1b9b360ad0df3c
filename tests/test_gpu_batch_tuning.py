"""A grouped batched encode runs the launch shape that it is asked for: tiles of
64 or 128 rows and quantize workgroups of several waves also where the library
itself would take its kernels for few rows and few vectors (tile_rows 0,
quant_waves 1); the records are the same."""
import numpy as np
import pytest

import paper_2509_12086_amd as saq
from paper_2509_12086_amd import autotune
from gpu_util import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _kernels(f):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as pr:
        out = f()
        torch.cuda.synchronize()
    return [e.name for e in pr.events() if "kernel" in e.name], out


@pytest.mark.parametrize("D,rows", [(96, 100), (768, 63)])
def test_grouped_tuning_is_obeyed(D, rows):
    plan = saq.Plan.from_parts([D // 2, D // 2], [4, 3], np.eye(D, dtype=np.float32),
                               np.zeros(D, np.float32)).upload(0)
    X = torch.randn(rows, D, generator=torch.Generator("cuda").manual_seed(D), device="cuda")
    want = None
    tunings = [t for t in autotune.candidates([(plan, X)]) if t.mode == saq.BATCH_GROUPED]
    assert saq.BatchTuning(mode=saq.BATCH_GROUPED) in tunings
    for t in tunings:
        names, out = _kernels(lambda: saq.encode_batched([(plan, X)], 4, t))
        say(f"  {t}: {[n.split('kernel')[0][-24:] for n in names]}")
        if want is None:
            want = out
        assert all(torch.equal(a, b) for a, b in zip(out[0], want[0]))
        assert any("project_few" in n for n in names) == (t.tile_rows == 0)
        assert any("quantize_few" in n for n in names) == (t.quant_waves == 1)

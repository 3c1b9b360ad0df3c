"""The autotuner's choice from its timings: the fastest shape, unless the
library's own one is as fast within what two runs of a sample differ by."""
import paper_2509_12086_amd as saq
from paper_2509_12086_amd import autotune

OWN = saq.BatchTuning(mode=saq.BATCH_GROUPED)
ROW_MAJOR = saq.BatchTuning(mode=saq.BATCH_GROUPED, tile_rows=64, quant_waves=4, gemm_xcd_order=False)
FUSED = saq.BatchTuning(mode=saq.BATCH_FUSED, tile_rows=64)


def test_the_librarys_own_choice_is_a_candidate():
    c = autotune.candidates()
    assert OWN in c and len(c) == len({tuple(vars(t).values()) for t in c})


def test_pick():
    assert autotune.pick([(FUSED, 77.0), (ROW_MAJOR, 75.63), (OWN, 75.81)]) == OWN
    assert autotune.pick([(FUSED, 77.0), (ROW_MAJOR, 74.0), (OWN, 75.81)]) == ROW_MAJOR
    assert autotune.pick([(FUSED, 4.0), (ROW_MAJOR, 6.0), (OWN, 5.0)]) == FUSED
    assert autotune.pick([(FUSED, 4.0), (ROW_MAJOR, 6.0)]) == FUSED

"""Which batches take their steps in pairs, seen in the middle buffer their scratch holds (on the CPU)."""
import pytest

from paper_1710_07073_amd import lbm as L

BB, PER = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_PERIODIC


def _has_middle(shape, count, precision, nb, bc=(BB,) * 6):
    cols = L.make_columns([(shape, 1.5, bc, nb, 0.0, 0.0)] * count)
    pool, scratch = L.lbm_batch_bytes_required(cols, precision)
    state = 19 * count * shape[0] * shape[1] * shape[2] * (4 if precision == L.LBM_FP32_SHIFTED else 8)
    assert pool > 2 * state
    return scratch >= state


@pytest.mark.parametrize("shape,count,precision,nb,pairs", [
    ((64, 64, 256), 1, "f32", 1, True),      # 2^20 cells
    ((64, 64, 255), 1, "f32", 1, False),
    ((20, 20, 60), 100, "f32", 1, True),     # 1600 bytes a plane
    ((19, 19, 60), 100, "f32", 1, False),    # 1444
    ((14, 14, 60), 100, "f64", 1, True),     # 1568
    ((13, 13, 60), 150, "f64", 1, False),    # 1352
    ((16, 16, 60), 100, "f32", 0, True),     # 1024, no bubbles
    ((15, 17, 60), 100, "f32", 0, False),    # 1020
    ((11, 12, 60), 150, "f64", 0, True),     # 1056
    ((11, 11, 60), 150, "f64", 0, False)])   # 968
def test_pairs_by_size(shape, count, precision, nb, pairs):
    prec = L.LBM_FP32_SHIFTED if precision == "f32" else L.LBM_FP64_SHIFTED
    assert _has_middle(shape, count, prec, nb) == pairs
    assert not _has_middle(shape, count, prec, nb, (BB,) * 4 + (PER, PER))


def test_no_middle_buffer_that_keeps_a_batch_off_the_card():
    assert _has_middle((128, 128, 512), 100, L.LBM_FP32_SHIFTED, 1)      # 59 GiB a state
    assert not _has_middle((128, 128, 512), 120, L.LBM_FP32_SHIFTED, 1)  # 71 GiB

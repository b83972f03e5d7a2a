"""Which lattices may take their method steps in pairs, seen in the middle buffer their scratch holds (on the CPU)."""
import pytest

from paper_1710_07073_amd import lbm as L

BB, FS, PER = L.LBM_BC_BOUNCE_BACK, L.LBM_BC_FREE_SLIP, L.LBM_BC_PERIODIC
WALLS, TOP = (BB,) * 6, (BB,) * 5 + (FS,)


def _middle(shape, precision, bc, flags=0):
    desc = L.make_desc(shape, 1.5, L.LBM_FP32_SHIFTED if precision == "f32" else L.LBM_FP64_SHIFTED, bc, flags)
    pops, _, scratch = L.lbm_bytes_required(desc)
    return scratch >= pops


@pytest.mark.parametrize("shape,precision,bc,middle", [
    ((128, 128, 512), "f32", WALLS, True),
    ((256, 256, 768), "f32", WALLS, True),
    ((128, 128, 512), "f64", TOP, True),
    ((101, 67, 251), "f32", TOP, True),
    ((64, 64, 192), "f32", WALLS, True),
    ((64, 64, 191), "f32", WALLS, False),   # fewer than 3 2^18 cells
    ((64, 64, 96), "f64", WALLS, True),
    ((64, 64, 95), "f64", WALLS, False),    # fewer than 3 2^17
    ((8, 8, 20000), "f32", WALLS, False),   # narrow: a workgroup's planes are nearly empty
    ((8, 8, 20000), "f64", TOP, False),
    ((4, 400, 600), "f32", TOP, False),
    ((128, 128, 512), "f32", (BB,) * 4 + (PER, PER), False)])
def test_pairs_by_shape(shape, precision, bc, middle):
    assert _middle(shape, precision, bc) == middle
    assert not _middle(shape, precision, bc, L.LBM_FLAG_WRITE_U_ALL)

"""Kernels whose inner loops must stay in registers, checked in the built library."""
import pytest

from kernel_metadata import kernels


def _of(prefix):
    found = {n: k for n, k in kernels().items() if n.startswith(prefix)}
    assert found, prefix
    return found


def test_synthesis_sums_stay_in_registers():
    """A lane's sums over l (up to four ring pairs) are live through every step of the
    recurrences: in scratch memory they are read and written at every l (400 bytes a
    lane: 44 ms for nside 1024, lmax 3071)."""
    for name, k in _of("alm2ring_kernel").items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name


def test_unshared_tile_loop_spills():
    """The pair loop of one-grid TOD fills the 128 registers of four waves a SIMD; what
    its launches keep around it (the walk over the queues) may cost it a few spills a
    tile, as before launches could share tiles (at most 11 without a plate, 18 with
    one), and no scalar ones."""
    for name, k in _of("tile_kernel<0, 1, ").items():
        if name.endswith(", false>"):
            plate = name.split(", ")[4] == "true"
            assert k[".vgpr_spill_count"] <= (18 if plate else 11) and k[".sgpr_spill_count"] == 0, name


def test_pixel_path_stays_in_registers():
    """Each form of the pixel path (a sample a wave, four samples a wave) keeps its own
    registers: with both in one kernel the first spilled 8 to 10 in FP32."""
    for name, k in _of("conv_kernel<").items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name

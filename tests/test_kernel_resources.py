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

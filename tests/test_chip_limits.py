"""Host-side limits of the on-chip scaled solve: the LDS a problem of N knots asks for."""
import ctypes as C

import pytest

LIMITS = {6: 2128, 14: 768, 26: 360}  # longest horizons with r, u and w in 160 KiB less 256 bytes
CAP = 160 * 1024 - 256


def need(nx, n, all_vectors=False):
    from paper_2309_06427_amd import _lib
    f = _lib.load()._ZN3ssp8pcg4_ldsEiib
    f.restype = C.c_int64
    return f(nx, n, all_vectors)


@pytest.mark.parametrize("nx", sorted(LIMITS))
def test_lds_grows_with_the_horizon_up_to_the_largest(nx):
    """Only horizons up to the limit fit, also where N nx passes 2^31."""
    ns = [1, 2, 3, 4, 5, LIMITS[nx], LIMITS[nx] + 1, 10 ** 4, 10 ** 6, 2 ** 26, 2 ** 27, 2 ** 28, 2 ** 29, 2 ** 30, 2 ** 31 - 1]
    got = [need(nx, n) for n in ns]
    assert got == sorted(got)
    assert [v <= CAP for v in got] == [n <= LIMITS[nx] for n in ns]


def test_other_state_sizes_have_no_on_chip_form():
    assert all(need(nx, 10) == -1 for nx in range(1, 65) if nx not in LIMITS)

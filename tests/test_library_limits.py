"""Limits of the library's host side, on the CPU: what its descriptions need."""

import pytest

from test_library_cpu import make_desc, smcx, ws_size  # noqa: F401

STATIC = 64 << 20


@pytest.mark.parametrize("lattice,K,S,R,dims", [
    (0, 8, 3, 1, (332, 345, 281)), (0, 8, 2, 2, (225, 254, 266)), (0, 4, 3, 200, (43, 54, 56)),
    (0, 8, 3, 256, (38, 42, 55)), (0, 4, 2, 1024, (33, 23, 21)), (0, 4, 3, 1100, (29, 29, 15)),
    (1, 5, 4, 1, (230, 217, 311)), (1, 5, 3, 2, (205, 222, 161)),
])
def test_descriptions_that_just_fit_the_static_workspace(smcx, lattice, K, S, R, dims):  # noqa: F811
    """Their padded copies leave under 256 KiB for the tables and counters."""
    d, keep = make_desc(smcx, lattice=lattice, K=K, S=S, dims=(dims,) * R)
    rc, n = ws_size(smcx, d)
    assert rc == 0 and n <= STATIC, n - STATIC


@pytest.mark.parametrize("lattice,R", [(0, 1), (1, 3), (0, 2000)])
def test_small_descriptions_have_room_for_the_qsro_counters(smcx, lattice, R):  # noqa: F811
    """8192 waves count three 64-bit words each in the space of the padded copies."""
    d, keep = make_desc(smcx, lattice=lattice, K=2, S=1, dims=((4, 4, 4),) * R)
    rc, n = ws_size(smcx, d)
    assert rc == 0 and n >= 8192 * 24

"""Every number of lanes per trial with every counter width and lattice, in
resident and row sweeps, against the oracle.  The form that a case is meant for
is asked of the library, on the CPU too, so that a change of the rules cannot
move a case to another kernel unseen."""
import ctypes as C

import numpy as np
import pytest

from gpu_cases import gpu_vs_oracle, rand_occ, sym_V
from paper_2503_12591_amd import inputs as I
from test_library_cpu import make_desc, smcx  # noqa: F401

BCC, FCC = 0, 1
BITS = {4: 32, 5: 32, 6: 32, 7: 64, 8: 64}

# lattice, dims, link-cell edge, lanes per trial
RESIDENT = [
    (BCC, (12, 13, 9), 4, 16), (BCC, (16, 16, 16), 4, 8), (BCC, (20, 16, 21), 4, 4), (BCC, (28, 24, 28), 4, 2),
    (BCC, (36, 36, 36), 4, 2),   # more link cells than lanes at once
    (BCC, (10, 9, 9), 3, 16), (BCC, (12, 12, 11), 3, 8), (BCC, (14, 16, 12), 3, 4), (BCC, (24, 21, 18), 3, 2),
    (FCC, (8, 12, 13), 4, 16), (FCC, (16, 16, 12), 4, 8), (FCC, (20, 16, 21), 4, 4), (FCC, (28, 28, 24), 4, 4),
]
ROWS = [
    (BCC, (21, 16, 18), 4, 16), (BCC, (133, 16, 18), 4, 8), (BCC, (264, 12, 13), 4, 4), (BCC, (521, 12, 9), 4, 2),
    (BCC, (84, 84, 86), 4, 8),   # by the number of link cells
    (FCC, (21, 16, 18), 4, 16), (FCC, (133, 12, 13), 4, 8), (FCC, (264, 9, 8), 4, 4),
    (FCC, (100, 9, 8), 3, 8),
]


def form_of(smcx, lattice, dims, K, S, ell):  # noqa: F811
    d, keep = make_desc(smcx, lattice=lattice, K=K, S=S, dims=(dims,), ell=[ell])
    form = (C.c_int32 * 5)()
    assert smcx.lib().smcx_internal_forms(C.byref(d), form) == 0
    return list(form)


def shells(lattice, ell, K):
    """Link cells of 3 keep each mini-step apart with 4 shells on BCC."""
    return 4 if lattice == BCC and ell == 3 else 1 + K % 4


@pytest.mark.parametrize("K", sorted(BITS))
def test_forms_of_the_cases(smcx, K):  # noqa: F811
    for lattice, dims, ell, lanes in RESIDENT:
        form = form_of(smcx, lattice, dims, K, shells(lattice, ell, K), ell)
        assert form[0] == lanes and form[3] == BITS[K], (lattice, dims)
        assert (form[4] > 1) == (int(np.prod([n // ell for n in dims])) * lanes > 1024), (lattice, dims)
        if lattice == BCC and ell == 3:
            assert form[2] == 0, dims  # no shared windows: a barrier after every mini-step
    for lattice, dims, ell, lanes in ROWS:
        assert form_of(smcx, lattice, dims, K, shells(lattice, 4, K), ell)[2] == lanes, (lattice, dims)


def test_every_lane_count_is_among_the_cases():
    assert {(c[0], c[3]) for c in RESIDENT} == {(c[0], c[3]) for c in ROWS} == \
        {(BCC, 2), (BCC, 4), (BCC, 8), (BCC, 16), (FCC, 4), (FCC, 8), (FCC, 16)}


def sweep(lattice, dims, K, S, ell, mode):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    gpu_vs_oracle(lattice, dims, K, S, rand_occ(N, K, 3 * sum(dims) + K, equi=False), sym_V(S, K, 0.04, K + 2 * S),
                  I.beta_of_T([2200.0, 700.0]), seed=2 ** 40 + 17, mode=mode, ell=ell, first_sweep=5)


@pytest.mark.gpu
@pytest.mark.parametrize("K", sorted(BITS))
@pytest.mark.parametrize("lattice,dims,ell,lanes", RESIDENT)
def test_resident_lanes(smcx, lattice, dims, ell, lanes, K):  # noqa: F811
    S = shells(lattice, ell, K)
    assert form_of(smcx, lattice, dims, K, S, ell)[0] == lanes
    sweep(lattice, dims, K, S, ell, "persistent")


@pytest.mark.gpu
@pytest.mark.parametrize("K", sorted(BITS))
@pytest.mark.parametrize("lattice,dims,ell,lanes", ROWS)
def test_row_lanes(smcx, lattice, dims, ell, lanes, K):  # noqa: F811
    S = shells(lattice, 4, K)
    assert form_of(smcx, lattice, dims, K, S, ell)[2] == lanes
    sweep(lattice, dims, K, S, ell, "stream")

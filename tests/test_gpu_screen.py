"""Interaction tensors at the ends of what the integer screen takes, against
the oracle's sums in binary64."""
import numpy as np
import pytest

from gpu_cases import gpu_vs_oracle, rand_occ, sym_V
from paper_2503_12591_amd import inputs as I

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1

WINDOWS = [((9, 8, 10), "persistent", True), ((9, 8, 10), "stream", True), ((64, 60, 66), "stream", True),
           ((9, 8, 10), "stream", False), ((2, 3, 2), "persistent", True)]


def run(lattice, dims, K, V, mode, rows, T=(4000.0, 900.0)):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    gpu_vs_oracle(lattice, dims, K, len(V), rand_occ(N, K, K, equi=False), V, I.beta_of_T(list(T)), seed=K, mode=mode, ell=4,
                  rows=rows)


@pytest.mark.parametrize("dims,mode,rows", WINDOWS)
@pytest.mark.parametrize("lattice,K,value", [(BCC, 3, np.inf), (BCC, 6, -np.inf), (FCC, 5, np.inf), (BCC, 8, 1.7e308),
                                             (FCC, 4, 1e300)])
def test_infinite_differences(lattice, K, value, dims, mode, rows):
    """Terms of 0 times an infinite difference are no zeros (the sum is not a
    number, the trial not accepted), however alike two sites' neighbours are."""
    V = sym_V(2, K, 0.03, K)
    V[1, 0, 1] = V[1, 1, 0] = value
    V[1, 0, 0] = -value
    run(lattice, dims, K, V, mode, rows)


@pytest.mark.parametrize("dims,mode,rows", WINDOWS)
@pytest.mark.parametrize("lattice,K,value", [(BCC, 4, 1e36), (BCC, 4, 3e37), (FCC, 5, 1e40), (BCC, 6, 1e45), (BCC, 2, 1e60),
                                             (BCC, 7, np.inf)])
def test_differences_past_the_terms_range(lattice, K, value, dims, mode, rows):
    """Large differences (all of them infinite at 7 species) beside ordinary ones."""
    V = sym_V(2, K, 0.03, K)
    V[0, 0, 0] = V[1, K - 1, K - 1] = value
    if K == 7:
        V[:] = value
    run(lattice, dims, K, V, mode, rows)


def one_energy_per_shell(S, K, J):
    V = np.zeros((S, K, K))
    for s in range(S):
        V[s] = J[s] * (1.0 - np.eye(K))
    return V


@pytest.mark.parametrize("dims,mode,rows", WINDOWS)
@pytest.mark.parametrize("lattice,K,S,J", [
    (BCC, 4, 4, (1 / 64, 1 / 128, -1 / 256, 1 / 512)),   # whole units: the integer sum is the energy change
    (FCC, 5, 2, (1 / 64, -1 / 64)), (BCC, 8, 3, (0.25, 0.125, 3 / 64)), (BCC, 6, 1, (1 / 32,)),
    (BCC, 4, 4, (0.021, 0.011, -0.0047, 0.0023)),        # the binary64 sum decides where the integer sum is zero
    (FCC, 5, 4, (0.021, 0.011, -0.0047, 0.0023)), (BCC, 7, 2, (0.021, 0.011)), (FCC, 6, 3, (0.021, 0.011, 0.0031)),
    (BCC, 2, 2, (0.021, -0.011)), (BCC, 3, 2, (0.0, 0.0)),
])
def test_one_energy_per_shell(lattice, K, S, J, dims, mode, rows):
    """Many an energy change is zero though the neighbours differ."""
    run(lattice, dims, K, one_energy_per_shell(S, K, J), mode, rows, T=(1500.0, 300.0))

"""Resident sweeps at the limits of what they accept, against the oracle."""
import numpy as np
import pytest

from gpu_cases import gpu_vs_oracle, rand_occ, sym_V
from paper_2503_12591_amd import inputs as I

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1


@pytest.fixture(scope="module")
def smcx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2503_12591_amd import smcx as S
    S.lib()
    return S


def uniform(L, e):
    n = max(1, L // e)
    return [L // n + (1 if j < L % n else 0) for j in range(n)]


@pytest.mark.parametrize("lattice,dims,K,z", [
    (BCC, (30, 30, 64), 4, [60, 4]),    # offsets of the long cell lead the short one far past the lattice
    (FCC, (20, 20, 64), 5, [60, 4]),
    (BCC, (28, 34, 64), 7, [4, 56, 4]),
])
@pytest.mark.parametrize("mode", ["persistent", "auto"])
def test_strongly_uneven_cells_near_the_lds_limit(smcx, lattice, dims, K, z, mode):
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    cells = [uniform(dims[0], 4), uniform(dims[1], 4), z]
    gpu_vs_oracle(lattice, dims, K, 4, rand_occ(N, K, 17, equi=False), sym_V(4, K, 0.04, 6), I.beta_of_T([1500.0, 800.0]),
                  seed=2 ** 33 + 5, mode=mode, cells=cells)


def test_counters_past_32_bits_in_one_call(smcx):
    """One workgroup counts every trial of a call: 2^31 and more of them."""
    import torch
    L, n = 32, 2 ** 31 // (2 * 32 ** 3) + 7
    occ = torch.zeros(2 * L ** 3, dtype=torch.uint8, device="cuda")
    lat = smcx.Lattice(BCC, (L, L, L), 2, 1, occ)
    lat.set_epi(sym_V(1, 2, 0.03, 1))
    betas = torch.full((n, 1), 10.0, dtype=torch.float64, device="cuda")
    stats, _, ties = lat.sweep(n, 3, betas, mode="persistent")
    assert stats.tolist() == [n * 2 * L ** 3, 0, 0] and int(ties) == 0
    lat.close()

"""Sweeps of every species and shell count against the oracle, in every kind of
window: the last species held by the counters has no term of its own in the
screen (and at 6 species no whole field), so it is given the strongest
interactions, and half of the lattice starts as that species alone, where
a shell's counts reach their largest differences."""
import numpy as np
import pytest

from gpu_cases import gpu_vs_oracle, rand_occ, sym_V
from paper_2503_12591_amd import inputs as I

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1


@pytest.mark.parametrize("K", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("lattice", [BCC, FCC])
def test_every_species_and_shell_count(lattice, K):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    for S in (1, 2, 3, 4):
        V = sym_V(S, K, 0.03, 10 * K + S)
        V[:, K - 1, :] *= 8.0
        V[:, :, K - 1] *= 8.0
        for dims, mode, rows in (((9, 8, 10), "persistent", True), ((9, 8, 10), "stream", True),
                                 ((9, 8, 10), "stream", False), ((2, 3, 2), "persistent", True)):
            N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
            occ = rand_occ(N, K, K + S, equi=False)
            occ[: N // 2] = K - 1
            gpu_vs_oracle(lattice, dims, K, S, occ, V, I.beta_of_T([4000.0, 900.0, 12000.0]), seed=K, mode=mode, ell=4,
                          rows=rows)

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


@pytest.mark.parametrize("shift", [0, 1, 15])
@pytest.mark.parametrize("lattice,dims,K", [(BCC, (3, 3, 2), 4), (BCC, (16, 9, 7), 3), (FCC, (5, 7, 6), 8),
                                            (BCC, (200, 150, 180), 5)])
def test_species_check_at_init(lattice, dims, K, shift):
    """A byte that is not a species, at the ends and inside, at any address."""
    import torch
    from paper_2503_12591_amd import smcx
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    buf = torch.full((N + 32,), 255, dtype=torch.uint8, device="cuda")  # not species on either side
    occ = buf[shift:shift + N]
    occ[:] = torch.from_numpy(rand_occ(N, K, 3, equi=False)).cuda()
    smcx.Lattice(lattice, dims, K, 1, occ, ell=3).close()
    for at, v in [(0, K), (N - 1, K), (N // 2, 128), (17, 127), (N - 16, 255)]:
        keep = int(occ[at])
        occ[at] = v
        with pytest.raises(smcx.SmcxError):
            smcx.Lattice(lattice, dims, K, 1, occ, ell=3)
        occ[at] = keep

"""Local energies at the edges of their kernels' ranges, bit for bit against
the oracle: the smallest lattices, axes narrower than a tile, and site counts on
either side of the limits between them."""
import numpy as np
import pytest

from gpu_cases import rand_occ, say, sym_V
from oracle import oracle as O

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1


@pytest.mark.parametrize("lattice,dims,K,S", [
    (BCC, (2, 3, 2), 5, 2), (FCC, (2, 2, 3), 8, 2), (BCC, (3, 5, 2), 7, 4), (FCC, (9, 8, 7), 6, 4),
    (BCC, (64, 64, 64), 5, 4), (BCC, (64, 64, 65), 5, 4), (BCC, (64, 64, 65), 8, 2),   # 2^19 sites and more
    (FCC, (32, 64, 64), 8, 4), (FCC, (33, 64, 64), 6, 3), (FCC, (33, 64, 64), 7, 4),
    (BCC, (96, 64, 128), 8, 3), (BCC, (97, 64, 128), 6, 3),                            # 3 2^19 sites and more
    (FCC, (7, 210, 100), 8, 4), (BCC, (5, 420, 150), 5, 1), (BCC, (420, 5, 150), 6, 4),
    (BCC, (64, 64, 65), 4, 4), (FCC, (33, 64, 64), 2, 3), (BCC, (20, 120, 130), 6, 4), (BCC, (16, 150, 130), 7, 2),
    (BCC, (110, 90, 95), 6, 4),
])
def test_local_energies_at_the_limits(lattice, dims, K, S):
    import torch
    from paper_2503_12591_amd import smcx
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N = (2 if lattice == BCC else 4) * int(np.prod(dims))
    say(f"local energies lattice={lattice} dims={dims} K={K} S={S}")
    occ, V = rand_occ(N, K, 7, equi=False), sym_V(S, K, 0.05, 3)
    lat = smcx.Lattice(lattice, dims, K, S, occ)
    lat.set_epi(V)
    e = lat.local_energy().cpu().numpy()
    assert np.array_equal(e, O.local_energy(lattice, dims, K, S, occ, V))
    lat.close()

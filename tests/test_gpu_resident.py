"""Resident sweeps (persistent mode with the whole replica in LDS, several
lanes per trial) against the oracle, at the edges of their range: the smallest
lattices, every number of lanes per trial, more link cells than lanes, link
cells too small to share barriers between basis sites, every counter width,
lattices that just fit the LDS, partial sweeps and occupancies at odd
addresses."""
import numpy as np
import pytest

from gpu_cases import NTHREADS, gpu_vs_oracle, rand_occ, say, sym_V
from oracle import oracle as O
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


@pytest.mark.parametrize("lattice,dims,K,S,ell", [
    (BCC, (4, 4, 4), 4, 4, 4),        # one link cell, 16 lanes per trial
    (BCC, (5, 4, 7), 3, 2, 4),
    (BCC, (9, 8, 11), 8, 4, 4),       # 64-bit counters, uneven cells
    (BCC, (12, 13, 8), 5, 3, 4),      # 6-bit counters
    (BCC, (20, 20, 16), 4, 4, 4),     # 100 cells: 8 lanes
    (BCC, (24, 24, 16), 4, 2, 4),     # 144 cells: 4 lanes
    (BCC, (32, 24, 28), 4, 4, 4),     # 336 cells: 2 lanes
    (BCC, (28, 32, 24), 6, 3, 4),     # the same with 64-bit counters
    (BCC, (39, 38, 37), 4, 4, 4),     # 729 cells, two passes, near the LDS limit
    (BCC, (9, 10, 12), 4, 4, 3),      # cells of 3: a barrier per mini-step
    (BCC, (27, 30, 30), 4, 4, 3),     # the same in two passes
    (BCC, (7, 6, 9), 2, 1, 2),        # cells of 2 and 3
    (FCC, (4, 4, 4), 5, 4, 4),
    (FCC, (6, 5, 7), 7, 3, 3),
    (FCC, (16, 16, 12), 5, 4, 4),     # 48 cells: 16 lanes
    (FCC, (20, 20, 20), 5, 2, 4),     # 125 cells: 8 lanes
    (FCC, (24, 24, 20), 3, 4, 4),     # 180 cells: 4 lanes
    (FCC, (28, 28, 28), 4, 4, 4),     # 343 cells, two passes
    (FCC, (12, 9, 10), 5, 4, 5),
])
def test_resident_sweeps(smcx, lattice, dims, K, S, ell):
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    occ = rand_occ(N, K, 3 * sum(dims) + K, equi=False)
    V = sym_V(S, K, 0.04, K + 2 * S)
    gpu_vs_oracle(lattice, dims, K, S, occ, V, I.beta_of_T([2200.0, 700.0]), seed=2 ** 40 + 17, mode="persistent",
                  ell=ell, first_sweep=5)


@pytest.mark.parametrize("lattice,dims,K,S", [(BCC, (12, 9, 16), 4, 4), (FCC, (8, 9, 10), 5, 4)])
def test_resident_partial_ranges_and_odd_address(smcx, lattice, dims, K, S):
    import torch
    m = 2 if lattice == BCC else 4
    N = m * int(np.prod(dims))
    occ = rand_occ(N, K, 9)
    V = sym_V(S, K, 0.04, 8)
    b = I.beta_of_T([1100.0])
    say(f"resident partial ranges lattice={lattice} dims={dims}")
    buf = torch.zeros(N + 1, dtype=torch.uint8, device="cuda")
    buf[1:] = torch.from_numpy(occ).cuda()
    lat = smcx.Lattice(lattice, dims, K, S, buf[1:], ell=4)
    lat.set_epi(V)
    cells, nA = lat.schedule(0)
    for lo, hi in [(0, 3), (3, 8), (8, 13), (13, 14), (14, 77), (77, nA)]:
        lat.sweep_partial(2, lo, hi, 5, b, mode="persistent")
    ref = occ.copy()
    O.run(lattice, dims, K, S, cells, ref, V, 5, b, first_sweep=2, nthreads=NTHREADS)
    assert np.array_equal(lat.occupancy(), ref)
    assert int(buf[0]) == 0
    lat.close()


def test_resident_replicas_of_different_sizes(smcx):
    dims = np.array([[4, 5, 6], [16, 12, 20], [24, 20, 28], [9, 9, 9]], np.int32)
    K, S, n = 4, 4, 2
    occs = [rand_occ(int(2 * np.prod(d)), K, 70 + r) for r, d in enumerate(dims)]
    V = sym_V(S, K, 0.03, 4)
    betas = I.beta_of_T(np.array([400.0, 900.0, 1500.0, 2500.0]))
    say("resident replicas of different sizes")
    lat = smcx.Lattice(BCC, dims, K, S, np.concatenate(occs))
    lat.set_epi(V)
    stats, ties, tc = lat.sweep(n, 3, np.tile(betas, (n, 1)), mode="persistent")
    gpu = lat.occupancy()
    s = stats.cpu().numpy().reshape(-1, 3)
    tnp, _ = lat.ties_to_numpy(ties, tc)
    off = 0
    for r in range(len(dims)):
        cells, _ = lat.schedule(r)
        ref = occs[r].copy()
        res = O.run(BCC, dims[r], K, S, cells, ref, V, 3, [betas[r]] * n, replica=r, replay=tnp[tnp["replica"] == r],
                    nthreads=NTHREADS)
        assert np.array_equal(gpu[off:off + len(ref)], ref), f"replica {r}"
        assert s[r, 0] == res.stats[0] and s[r, 1] == res.stats[1]
        off += len(ref)
    lat.close()

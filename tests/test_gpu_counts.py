"""Bit-plane pair counts against the oracle where they can go wrong: rows at
and around whole words, the shortest lattices (periodic images with
multiplicity), every species count, lattices of several tiles, rows long
enough to be cut, occupancies at odd addresses, and the species check of the
batched call in every position."""
import numpy as np
import pytest

from gpu_cases import NTHREADS, rand_occ, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1


@pytest.fixture(scope="module")
def smcx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2503_12591_amd import smcx as S
    S.lib()
    return S


@pytest.mark.parametrize("lattice,dims,K,S,B", [
    (BCC, (2, 2, 2), 4, 3, 3), (BCC, (3, 2, 5), 3, 2, 2), (FCC, (2, 3, 2), 5, 1, 2), (FCC, (3, 3, 3), 8, 4, 2),
    (BCC, (31, 5, 4), 4, 4, 2), (BCC, (32, 4, 5), 4, 4, 2), (BCC, (33, 4, 5), 2, 4, 2), (BCC, (30, 6, 4), 5, 4, 1),
    (FCC, (31, 4, 4), 4, 4, 2), (FCC, (32, 5, 4), 5, 4, 2), (FCC, (33, 4, 4), 6, 3, 1), (FCC, (63, 4, 5), 5, 2, 1),
    (BCC, (64, 7, 6), 7, 4, 1), (BCC, (65, 6, 7), 8, 2, 1), (FCC, (65, 4, 4), 2, 4, 1), (FCC, (95, 5, 4), 7, 4, 1),
    (BCC, (16, 16, 16), 4, 4, 37), (BCC, (64, 64, 64), 4, 4, 3), (FCC, (40, 61, 50), 5, 4, 2),
    (BCC, (97, 120, 83), 3, 4, 1), (BCC, (10700, 5, 4), 4, 4, 1), (FCC, (4800, 4, 5), 5, 4, 1),
    (BCC, (10720, 4, 4), 4, 2, 1), (BCC, (11, 4, 5), 4, 4, 1700),
])
def test_counts(smcx, lattice, dims, K, S, B):
    import torch
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    say(f"counts lattice={lattice} dims={dims} K={K} S={S} B={B}")
    occs = np.stack([rand_occ(N, K, 31 * K + b, equi=False) for b in range(B)])
    buf = torch.zeros(B * N + 3, dtype=torch.uint8, device="cuda")
    for shift in (0, 3):
        buf[shift:shift + B * N] = torch.from_numpy(occs.reshape(-1)).cuda()
        C = smcx.energy_backward_counts(lattice, dims, K, S, buf[shift:shift + B * N].view(B, N)).cpu().numpy()
        for b in range(0, B, max(1, B // 5)):
            assert np.array_equal(C[b], O.pair_counts(lattice, dims, K, S, occs[b])), (shift, b)
        total = N * C.sum(axis=(2, 3))[:, 0] // N  # every configuration: all bonds of the first shell
        assert np.all(total == N * (8 if lattice == BCC else 12))


@pytest.mark.parametrize("lattice,dims,K,axis,width", [(BCC, (40, 48, 64), 4, 2, 8), (FCC, (40, 48, 32), 5, 2, 1),
                                                       (BCC, (96, 64, 32), 6, 1, 4), (FCC, (64, 64, 64), 3, 0, 32)])
def test_counts_of_layers(smcx, lattice, dims, K, axis, width):
    """Layers of one species: a workgroup may own bonds of a species it has no site of."""
    import torch
    m = 2 if lattice == BCC else 4
    say(f"counts of layers lattice={lattice} dims={dims} K={K}")
    pos = np.indices(dims[::-1])[2 - axis]  # z, y, x order
    occ = np.repeat(((pos // width) % K).astype(np.uint8).reshape(-1), m)
    C = smcx.energy_backward_counts(lattice, dims, K, 4, torch.from_numpy(occ[None]).cuda()).cpu().numpy()
    assert np.array_equal(C[0], O.pair_counts(lattice, dims, K, 4, occ))


@pytest.mark.parametrize("K", [2, 3, 4, 5, 7, 8])
def test_species_check(smcx, K):
    import torch
    dims, B, N = (35, 4, 5), 6, 2 * 35 * 4 * 5
    say(f"species check K={K}")
    good = np.stack([rand_occ(N, K, b, equi=False) for b in range(B)])
    smcx.energy_backward_counts(BCC, dims, K, 2, torch.from_numpy(good).cuda())
    for b, i, v in [(0, 0, K), (B - 1, N - 1, K), (2, 69, 127), (3, 333, 128), (4, 5, 255)]:
        bad = good.copy()
        bad[b, i] = v
        with pytest.raises(smcx.SmcxError):
            smcx.energy_backward_counts(BCC, dims, K, 2, torch.from_numpy(bad).cuda())


@pytest.mark.parametrize("lattice,dims,K,S", [(BCC, (512, 256, 240), 4, 4), (BCC, (420, 300, 260), 2, 2),
                                              (FCC, (500, 200, 260), 3, 2)])
def test_counts_with_large_workgroups(smcx, lattice, dims, K, S):
    """Tiles of a thousand words and more: 512 threads each."""
    import torch
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    say(f"counts with large workgroups lattice={lattice} dims={dims} K={K}")
    occ = rand_occ(N, K, 7 + K, equi=False)
    C = smcx.energy_backward_counts(lattice, dims, K, S, torch.from_numpy(occ[None]).cuda()).cpu().numpy()
    assert np.array_equal(C[0], O.pair_counts(lattice, dims, K, S, occ, NTHREADS))


def test_species_check_of_two_threads(smcx):
    """Each thread's calls, on a stream of its own, see their own batch's check."""
    import threading

    import torch
    dims, K, B, N = (35, 4, 5), 4, 6, 2 * 35 * 4 * 5
    say("species check of two threads")
    good = np.stack([rand_occ(N, K, b, equi=False) for b in range(B)])
    bad = good.copy()
    bad[3, 5] = K
    seen = {"good": 0, "bad": 0}

    def calls(name, occ):
        with torch.cuda.stream(torch.cuda.Stream()):
            occ = torch.from_numpy(occ).cuda()
            for _ in range(50):
                try:
                    smcx.energy_backward_counts(BCC, dims, K, 2, occ)
                except smcx.SmcxError:
                    seen[name] += 1

    threads = [threading.Thread(target=calls, args=a) for a in (("good", good), ("bad", bad))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert seen == {"good": 0, "bad": 50}

"""Row windows with several lanes per trial (stream mode of small lattices)
against the oracle: every number of lanes, rows that fill a wave only together,
uneven cells, long rows, every counter width, replicas of different sizes, and
mini-step ranges that cut a row group."""
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
    (BCC, (5, 8, 9), 4, 4, 4),          # one cell per row: rows of several cells share a wave
    (BCC, (9, 64, 60), 4, 2, 4),
    (BCC, (64, 60, 66), 4, 4, 4),       # 16 lanes per trial
    (BCC, (75, 76, 80), 3, 3, 4),       # 8 lanes, uneven cells
    (BCC, (130, 60, 64), 6, 3, 4),      # 8 lanes, 64-bit counters
    (BCC, (264, 40, 41), 4, 4, 4),      # 66 cells per row: fewer lanes so that a row fits a workgroup
    (BCC, (130, 121, 126), 4, 4, 4),    # 4 lanes
    (BCC, (131, 160, 162), 5, 2, 4),    # 2 lanes, 6-bit counters
    (BCC, (420, 36, 30), 4, 4, 4),      # rows of more than 40 chunks: a wave per row when staging
    (FCC, (12, 13, 14), 5, 4, 4),
    (FCC, (60, 50, 53), 5, 2, 3),       # 16 lanes, cells of 3 and 4
    (FCC, (100, 50, 53), 3, 4, 4),      # 16 lanes
    (FCC, (100, 90, 53), 7, 3, 4),      # 8 lanes, 64-bit counters
    (FCC, (120, 110, 112), 5, 4, 4),    # 4 lanes
])
def test_row_sweeps_with_several_lanes_per_trial(smcx, lattice, dims, K, S, ell):
    N = int(np.prod(dims)) * (2 if lattice == BCC else 4)
    occ = rand_occ(N, K, sum(dims) + K, equi=False)
    V = sym_V(S, K, 0.04, K + 2 * S)
    gpu_vs_oracle(lattice, dims, K, S, occ, V, I.beta_of_T([1300.0]), seed=2 ** 35 + 3, mode="stream", ell=ell,
                  first_sweep=4)


@pytest.mark.parametrize("lattice", [BCC, FCC])
def test_row_ranges_and_replicas_of_different_sizes(smcx, lattice):
    m = 2 if lattice == BCC else 4
    K, S = (4, 4) if lattice == BCC else (5, 4)
    V = sym_V(S, K, 0.03, 21)
    for dims in ([[20, 16, 24], [16, 28, 12]], [[17, 16, 18], [33, 21, 14]]):  # one decomposition, mixed
        dims = np.array(dims, np.int32)
        occs = [rand_occ(m * int(np.prod(d)), K, 90 + r) for r, d in enumerate(dims)]
        say(f"row ranges lattice={lattice} dims={dims.tolist()}")
        lat = smcx.Lattice(lattice, dims, K, S, np.concatenate(occs), ell=4)
        lat.set_epi(V)
        nA = [lat.schedule(r)[1] for r in range(2)]
        b = I.beta_of_T(np.array([800.0, 1500.0]))
        stats = None
        if nA[0] == nA[1] and [len(c) for c in lat.schedule(0)[0]] != []:
            for lo, hi in [(0, 3), (3, 11), (11, 40), (40, 41), (41, max(nA))]:
                stats, _, _ = lat.sweep_partial(3, lo, hi, 5, b, mode="stream", stats=stats)
        else:
            stats, _, _ = lat.sweep(1, 5, b.reshape(1, 2), first_sweep=3, mode="stream")
        gpu, s, off = lat.occupancy(), stats.cpu().numpy().reshape(-1, 3), 0
        for r in range(2):
            cells, _ = lat.schedule(r)
            ref = occs[r].copy()
            res = O.run(lattice, dims[r], K, S, cells, ref, V, 5, [b[r]], first_sweep=3, replica=r, nthreads=NTHREADS)
            assert np.array_equal(gpu[off:off + len(ref)], ref), f"replica {r}"
            assert s[r, 0] == res.stats[0] and s[r, 1] == res.stats[1]
            off += len(ref)
        lat.close()


@pytest.mark.parametrize("lattice,dims,K,S,rows", [
    (BCC, (17, 12, 13), 4, 4, True), (BCC, (46, 9, 10), 5, 2, True), (FCC, (14, 9, 10), 5, 4, True),
    (FCC, (31, 8, 9), 6, 2, True), (BCC, (17, 12, 13), 4, 4, False), (FCC, (14, 9, 10), 5, 4, False),
])
def test_stream_sweeps_at_odd_addresses(smcx, lattice, dims, K, S, rows):
    """Packing and unpacking an occupancy at any byte address, nothing beside it touched."""
    import torch
    N = (2 if lattice == BCC else 4) * int(np.prod(dims))
    occ = rand_occ(N, K, 5, equi=False)
    V = sym_V(S, K, 0.04, 8)
    b = I.beta_of_T([1100.0])
    say(f"odd addresses lattice={lattice} dims={dims} rows={rows}")
    for shift in (1, 2, 7):
        buf = torch.full((N + 32,), 3, dtype=torch.uint8, device="cuda")
        buf[shift:shift + N] = torch.from_numpy(occ).cuda()
        lat = smcx.Lattice(lattice, dims, K, S, buf[shift:shift + N], ell=4, rows=rows)
        lat.set_epi(V)
        cells, _ = lat.schedule(0)
        lat.sweep(1, 5, b, first_sweep=2, mode="stream")
        ref = occ.copy()
        O.run(lattice, dims, K, S, cells, ref, V, 5, b, first_sweep=2, nthreads=NTHREADS)
        assert np.array_equal(lat.occupancy(), ref)
        assert bool((buf[:shift] == 3).all()) and bool((buf[shift + N:] == 3).all())
        lat.close()

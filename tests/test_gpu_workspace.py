"""Regions of the workspace that calls share, and counters without slots."""
import numpy as np
import pytest

from gpu_cases import NTHREADS, rand_occ, say, sym_V
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


@pytest.mark.parametrize("lattice,dims,K", [(BCC, (8, 8, 8), 4), (FCC, (6, 7, 9), 5), (BCC, (4, 5, 4), 3)])
def test_qsro_and_pair_sweeps_in_turn_on_one_handle(smcx, lattice, dims, K):
    """qSRO sweeps count where pair-model sweeps hold their padded copies."""
    m, S = (2 if lattice == BCC else 4), 2
    occ = rand_occ(m * int(np.prod(dims)), K, 12, equi=False)
    V = sym_V(S, K, 0.04, 3)
    W = np.random.default_rng(4).normal(0, 0.05, (S, K))
    b = float(I.beta_of_T([1100.0])[0])
    calls = ["stream", "qsro", "persistent", "qsro", "plain", "stream", "qsro"]

    def run(shared):
        out, cur, lat = [], occ.copy(), None
        for j, call in enumerate(calls):
            say(f"in turn lattice={lattice} dims={dims} call={call} shared={shared}")
            if lat is None or not shared:
                lat = smcx.Lattice(lattice, dims, K, S, cur, ell=5)
                lat.set_epi(V)
                lat.set_qsro(V, W)
            if call == "qsro":
                stats, _, _ = lat.sweep_qsro(1, 5, [b], first_sweep=j)
            else:
                stats, _, _ = lat.sweep(1, 5, [b], first_sweep=j, mode=call)
            cur = lat.occupancy()
            out.append((cur.copy(), stats.tolist()))
            if not shared:
                lat.close()
        return out

    for (a, s), (a2, s2) in zip(run(True), run(False)):
        assert np.array_equal(a, a2) and s == s2
        assert s[0] == len(occ)


@pytest.mark.parametrize("mode,rows", [("stream", True), ("stream", False), ("persistent", True), ("plain", True)])
@pytest.mark.parametrize("R", [1024, 1025])
def test_counters_of_many_replicas(smcx, R, mode, rows):
    """More than 1024 replicas count straight into the caller's words."""
    dims, K, S, n = (5, 5, 6), 3, 2, 2 if mode != "plain" else 1
    N = 2 * int(np.prod(dims))
    occ = rand_occ(R * N, K, 8, equi=False)
    V = sym_V(S, K, 0.04, 2)
    b = float(I.beta_of_T([1000.0])[0])
    say(f"many replicas R={R} mode={mode} rows={rows}")
    lat = smcx.Lattice(BCC, np.array([dims] * R), K, S, occ, rows=rows)
    lat.set_epi(V)
    stats, ties, tc = lat.sweep(n, 3, np.full((n, R), b), mode=mode)
    gpu, s = lat.occupancy().reshape(R, N), stats.cpu().numpy().reshape(R, 3)
    tnp, _ = lat.ties_to_numpy(ties, tc)
    assert (s[:, 0] == n * N).all()
    for r in [0, 1, 2, 511, R - 2, R - 1]:
        cells, _ = lat.schedule(r)
        ref = occ[r * N:(r + 1) * N].copy()
        res = O.run(BCC, dims, K, S, cells, ref, V, 3, [b] * n, replica=r, replay=tnp[tnp["replica"] == r], nthreads=NTHREADS)
        assert np.array_equal(gpu[r], ref), f"replica {r}"
        assert s[r, 1] == res.stats[1]
    lat.close()

"""Sweeps whose padded copy passes 2 GiB: window addresses past 31 bits, in
every kind of window, against single mini-steps of the oracle.  Narrow rows
keep the sites few (a row of 5 cells takes 32 bytes of the copy)."""
import numpy as np
import pytest

from gpu_cases import NTHREADS, say, sym_V
from oracle import oracle as O
from paper_2503_12591_amd import inputs as I

pytestmark = pytest.mark.gpu
BCC = 0
DIMS = (5, 8300, 8300)


@pytest.mark.parametrize("ell,tile,rows,double_buffer,tau", [
    (4, (0, 0, 0), True, False, (16, 20)),    # row windows, one lane per trial
    (100, (1, 1, 1), True, False, (16, 40)),  # row windows, several lanes per trial
    (4, (0, 0, 0), False, False, (0, 3)),     # tile windows
    (4, (0, 0, 0), False, True, (3, 5)),      # tile windows, the next one streaming in
])
def test_windows_past_two_gib(ell, tile, rows, double_buffer, tau):
    import torch
    from paper_2503_12591_amd import smcx
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    K, S = 4, 2
    N = 2 * int(np.prod(DIMS, dtype=np.int64))
    say(f"padded copy of 2.2 GB ell={ell} rows={rows} double_buffer={double_buffer} tau={tau}")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    occ = torch.randint(0, K, (N,), generator=g, device="cuda", dtype=torch.uint8)
    ref = occ.cpu().numpy()
    V = sym_V(S, K, 0.04, 2)
    b = float(I.beta_of_T([1000.0])[0])
    lat = smcx.Lattice(BCC, DIMS, K, S, occ, ell=ell, tile=tile, rows=rows, double_buffer=double_buffer)
    assert lat.ws_bytes > 2 ** 31
    lat.set_epi(V)
    cells, _ = lat.schedule(0)
    stats, ties, tc = lat.sweep_partial(1, *tau, 7, [b], mode="stream")
    tnp, _ = lat.ties_to_numpy(ties, tc)
    s = stats.tolist()
    lat.close()
    res = O.run_ministeps(BCC, DIMS, K, S, cells, ref, V, 7, b, 1, *tau, replay=tnp, nthreads=NTHREADS)
    assert s[:2] == list(res.stats[:2])
    assert bool((occ == torch.from_numpy(ref).cuda()).all())

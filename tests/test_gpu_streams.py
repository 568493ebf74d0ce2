"""Calls on several streams and threads at a time."""
import numpy as np
import pytest

from gpu_cases import rand_occ, say, sym_V
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


@pytest.mark.parametrize("mode", ["stream", "persistent", "plain"])
def test_handles_on_two_streams_share_counters(smcx, mode):
    """Counters are added to, so two handles may count into the same words."""
    import torch
    say(f"shared counters mode={mode}")
    dims, K, S, n = (16, 12, 20), 4, 2, 30
    N = 2 * int(np.prod(dims))
    streams = [torch.cuda.Stream() for _ in range(2)]
    occs = [torch.from_numpy(rand_occ(N, K, 5 + i, equi=False)).cuda() for i in range(2)]
    lats = [smcx.Lattice(BCC, dims, K, S, o) for o in occs]
    for lat in lats:
        lat.set_epi(sym_V(S, K, 0.04, 3))
    betas = torch.full((1, 1), float(I.beta_of_T([900.0])[0]), dtype=torch.float64, device="cuda")

    def counters(shared):
        for lat, o, i in zip(lats, occs, range(2)):
            o.copy_(torch.from_numpy(rand_occ(N, K, 5 + i, equi=False)))
        stats = [torch.zeros(3, dtype=torch.int64, device="cuda") for _ in range(1 if shared else 2)]
        ties = torch.zeros(4096 * 24, dtype=torch.uint8, device="cuda")
        tc = torch.zeros(1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        for j in range(n):
            for i in range(2):
                with torch.cuda.stream(streams[i]):
                    lats[i].sweep(1, 9, betas, first_sweep=j, mode=mode, stats=stats[-1 if shared else i], ties=ties,
                                  tie_count=tc)
        torch.cuda.synchronize()
        return sum(stats).tolist()

    own = counters(shared=False)
    assert own[0] == 2 * n * N and own[1] > 0
    assert counters(shared=True) == own
    for lat in lats:
        lat.close()

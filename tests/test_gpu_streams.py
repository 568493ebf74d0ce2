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


def backward(smcx, occ, counts, dims, K, S, stream):
    """smcx_energy_backward on a given stream."""
    import ctypes as C
    d = np.asarray(dims, np.int32)
    return smcx.lib().smcx_energy_backward(BCC, d.ctypes.data_as(C.c_void_p), K, S, C.c_void_p(occ.data_ptr()), occ.shape[0],
                                           C.c_void_p(counts.data_ptr()), C.c_void_p(stream.cuda_stream))


def test_a_thread_that_counted_may_end_during_a_capture(smcx):
    """What a call leaves with its thread takes no HIP call to go away."""
    import threading

    import torch
    dims, K, S, B = (8, 8, 8), 4, 2, 5
    occ = torch.randint(0, K, (B, 1024), dtype=torch.uint8, device="cuda")
    counts = torch.zeros((B, S, K, K), dtype=torch.int64, device="cuda")
    x = torch.zeros(4, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    counted, end, rc = threading.Event(), threading.Event(), []

    def work():
        torch.cuda.set_device(0)
        rc.append(backward(smcx, occ, counts, dims, K, S, stream))
        counted.set()
        end.wait(30)

    t = threading.Thread(target=work)
    t.start()
    assert counted.wait(30) and rc == [0]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="global"):
        x.add_(1)
        end.set()
        t.join()
        x.add_(1)
    for n in (1, 2):
        g.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [2.0 * n] * 4


def test_counting_in_many_threads_at_once(smcx):
    """Every call hears of its own species only."""
    import threading

    import torch
    dims, K, S, B = (8, 9, 8), 4, 2, 3
    good = torch.randint(0, K, (B, 2 * 576), dtype=torch.uint8, device="cuda")
    bad = good.clone()
    bad[B - 1, 1000] = K
    streams = [torch.cuda.Stream() for _ in range(8)]
    outs = [torch.zeros((B, S, K, K), dtype=torch.int64, device="cuda") for _ in range(8)]
    torch.cuda.synchronize()
    rcs = [[] for _ in range(8)]

    def work(i):
        torch.cuda.set_device(0)
        for j in range(20):
            rcs[i].append(backward(smcx, bad if (i + j) % 3 == 0 else good, outs[i], dims, K, S, streams[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(8):
        assert rcs[i] == [-1 if (i + j) % 3 == 0 else 0 for j in range(20)]

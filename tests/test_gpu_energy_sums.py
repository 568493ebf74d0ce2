"""Energies and gradients from counts: the sums over terms and configurations
in their stated order, so equal to the same sums in numpy bit for bit, at the
edges of the kernels' tiles."""
import numpy as np
import pytest

from gpu_cases import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,K", [(1, 2), (3, 3), (4, 4), (2, 5), (4, 8)])
@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 33, 1023, 1024, 1025, 2500])
def test_sums_in_order(S, K, B):
    import torch
    from paper_2503_12591_amd import smcx
    g = np.random.default_rng(B * 100 + K)
    C = g.integers(0, 2 ** 40, size=(B, S, K, K))
    V, w = g.normal(size=(S, K, K)), g.normal(size=B)
    say(f"sums S={S} K={K} B={B}")
    Ct = torch.from_numpy(C).cuda()
    E = smcx.energy_of_counts(Ct, torch.from_numpy(V).cuda()).cpu().numpy()
    acc = np.zeros(B)
    for i in range(S * K * K):
        acc = acc + C.reshape(B, -1)[:, i].astype(np.float64) * V.reshape(-1)[i]
    assert np.array_equal(E, 0.5 * acc)
    grad = smcx.energy_grad(Ct, torch.from_numpy(w).cuda()).cpu().numpy()
    acc = np.zeros((S, K, K))
    for b in range(B):
        acc = acc + w[b] * C[b].astype(np.float64)
    assert np.array_equal(grad, 0.5 * acc)

"""Sweeps of 7 and 8 species (64-bit counters) at the edges of their launch
forms, against the oracle."""
import numpy as np
import pytest

from gpu_cases import gpu_vs_oracle, rand_occ, sym_V
from paper_2503_12591_amd import inputs as I

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1


@pytest.mark.parametrize("dims,K,S", [
    ((112, 112, 224), 7, 2),   # two lanes per trial, seven waves per CU
    ((140, 140, 144), 8, 4),   # one lane: two lanes would take ten
    ((24, 400, 400), 7, 4),    # short rows keep two lanes
])
def test_row_sweeps_at_the_two_lane_limit(dims, K, S):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N = 2 * int(np.prod(dims))
    gpu_vs_oracle(BCC, dims, K, S, rand_occ(N, K, sum(dims), equi=False), sym_V(S, K, 0.04, K), I.beta_of_T([1300.0]),
                  seed=2 ** 35 + 3, mode="stream", ell=4, first_sweep=4)


@pytest.mark.parametrize("dims,S", [((36, 36, 36), 3), ((34, 34, 34), 4), ((38, 38, 38), 1)])
def test_large_replicas_without_row_windows(dims, S):
    """Link cells of 3 at 4 shells, or tiles asked for: replicas that fit the
    LDS run resident or as tile launches."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N = 2 * int(np.prod(dims))
    gpu_vs_oracle(BCC, dims, 8, S, rand_occ(N, 8, sum(dims), equi=False), sym_V(S, 8, 0.04, 8), I.beta_of_T([1300.0]),
                  seed=2 ** 35 + 3, mode="auto", ell=3, first_sweep=4, rows=False)

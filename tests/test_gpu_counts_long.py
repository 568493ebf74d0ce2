"""Pair counts of lattices with an axis of more than 2^30 cells."""
import numpy as np
import pytest

from gpu_cases import say

pytestmark = pytest.mark.gpu
BCC, FCC = 0, 1
Z = {BCC: (8, 6), FCC: (12, 6)}


@pytest.mark.parametrize("lattice,dims", [
    (BCC, (2, 2 ** 30 + 77, 2)),
    (BCC, (2, 2, 2 ** 30 + 77)),
    (FCC, (2 ** 29 + 77, 2, 2)),   # the bytes of a row pass 2^31
])
def test_backward_counts_of_long_axes(lattice, dims):
    import torch
    from paper_2503_12591_amd import smcx
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m, K, S = (2 if lattice == BCC else 4), 2, 2
    N = m * int(np.prod(dims, dtype=np.int64))
    say(f"long axis lattice={lattice} dims={dims} sites={N}")
    occ = torch.zeros((1, N), dtype=torch.uint8, device="cuda")
    # sites of species 1 too far apart to be neighbours: the first, the last
    # cell of the long axis but a few, one in the middle
    axis = int(np.argmax(dims))
    stride = m * int(np.prod(dims[:axis], dtype=np.int64))
    at = [0, stride * (dims[axis] // 2), stride * (dims[axis] - 7)]
    for i in at:
        occ[0, i] = 1
    C = smcx.energy_backward_counts(lattice, dims, K, S, occ)[0].cpu().numpy()
    for s in range(S):
        z, n = Z[lattice][s], len(at)
        # the narrow axes hold images of a site: none of them is the site itself
        assert C[s].tolist() == [[z * (N - 2 * n), z * n], [z * n, 0]]
    del occ

"""Bit permutations at the edges of the tile kernel (rank 12, one tile; every
outer bit in the grid; tiles walked by a workgroup) and of the table kernel
(lower ranks, operands that are not 16-byte aligned): a permutation moves
values, so the result is exact."""
import numpy as np
import pytest
import torch

import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,seed,shift", [(1, 0, 0), (5, 1, 0), (11, 2, 0), (12, 3, 0), (12, -1, 0), (13, 4, 0),
                                             (13, 5, 1), (17, -1, 0), (20, 6, 0), (22, 7, 0), (23, 8, 0),
                                             (24, 9, 0), (23, 10, 1), (24, -2, 0)])
def test_permute_sizes(rank, seed, shift):
    print("permute", rank, seed, shift, flush=True)
    lin = list(range(rank))
    if seed == -1:
        lout = lin[::-1]           # full reversal
    elif seed == -2:
        lout = lin[1:] + lin[:1]   # rotation: most low bits kept
    else:
        lout = [int(x) for x in np.random.default_rng(seed).permutation(rank)]
    n = 1 << rank
    buf = torch.arange(2 * (n + shift), dtype=torch.float32, device="cuda").view(torch.complex64)
    X = buf[shift:]
    out = torch.zeros(n + shift, dtype=torch.complex64, device="cuda")[shift:]
    R.permute(X, lin, lout, out=out)
    e = torch.arange(n, device="cuda")
    src = torch.zeros_like(e)
    for i, l in enumerate(reversed(lout)):
        src |= ((e >> i) & 1) << (rank - 1 - lin.index(l))
    assert torch.equal(torch.view_as_real(out), torch.view_as_real(X[src]))

"""Fused small subtrees (one workgroup per subtree and copy, every tensor in
LDS): whole calls whose trees lie mostly or wholly inside them, against the
oracle.  FP32 amplitudes: normalised error <= 1e-4, the bound of every FP32
amplitude test.  Sizes: a tree of one step, trees that end inside a subtree,
trees with large steps between subtrees; several bitstrings and slices per
group and ragged groups; slice sets whose copies differ from their inputs'."""
import numpy as np
import pytest
import torch

import oracle
import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,depth,n_open,n_batch,sliced,limit", [
    (1, 2, 1, 0, 1, -1, 0),      # the smallest network
    (2, 2, 3, 4, 1, -1, 0),      # every qubit open
    (3, 3, 6, 2, 5, 2, 0),       # one subtree, slices x bitstrings
    (3, 4, 8, 6, 3, 3, 3),       # ragged slice groups
    (4, 4, 8, 0, 33, -1, 7),     # ragged bitstring groups
    (4, 4, 14, 3, 2, 2, 0),      # large steps above and below subtrees
    (4, 5, 10, 5, 2, 3, 0),
])
def test_small_subtrees_vs_statevector(rows, cols, depth, n_open, n_batch, sliced, limit):
    n = rows * cols
    print("chain", rows, cols, depth, n_open, n_batch, sliced, limit, flush=True)
    c = rqcgen.grid_rqc(rows, cols, depth, 17)
    openq = list(range(n - n_open, n))
    P = R.Plan(R.Network(R.Circuit.from_rqcgen(c), openq), seed=3, path_trials=32, n_sliced=sliced).bind()
    P.set_group_limit(limit, limit)
    bits = np.stack([rqcgen.random_bits(n - n_open, s) for s in range(n_batch)])
    ref = np.stack([oracle.amplitudes_sv(c, openq, b) for b in bits])
    for _ in range(3):  # captured, replayed, replayed
        got = R.to_complex(P.contract(bits))
        assert oracle.normalized_error(got.reshape(-1), ref.reshape(-1), n) < 1e-4
        torch.cuda.synchronize()
    direct = R.to_complex(P.contract_noalloc(bits))
    assert oracle.normalized_error(direct.reshape(-1), ref.reshape(-1), n) < 1e-4

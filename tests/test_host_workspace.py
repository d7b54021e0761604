"""The least workspace of a call (host only): fusing small subtrees never asks for
more than a launch per step takes, whose bytes are given here (leaves, labels,
scales and first-fit arena of the plan), and a budget of just that is accepted."""
import pytest

import paper_2110_14502_amd as R
import rqcgen


@pytest.mark.parametrize("rows,cols,depth,n_open,sliced,seed,n_batch,f32,f16", [
    (5, 6, 10, 5, 6, 3, 1, 271360, 234496),       # fused, in FP32: 52992 bytes more
    (5, 6, 11, 4, 6, 74, 1, 304640, 304640),
    (5, 6, 10, 5, 2, 58, 64, 250368, 250368),
    (6, 6, 10, 2, 6, 38, 64, 825600, 366848),
    (5, 5, 13, 5, 2, 59, 1, 78187776, 50385152),
])
def test_least_workspace(rows, cols, depth, n_open, sliced, seed, n_batch, f32, f16):
    n = rows * cols
    net = R.Network(R.Circuit.from_rqcgen(rqcgen.grid_rqc(rows, cols, depth, seed)), list(range(n - n_open, n)))
    P = R.Plan(net, n_sliced=sliced, seed=seed, path_trials=16)
    for prec, limit in ((R.F32, f32), (R.F16, f16)):
        lo, pref = P.workspace_bytes(0, n_batch, prec)
        assert lo <= limit and lo <= pref
    one = P.resident_bytes() + min(f32, P.workspace_bytes(1, 1, R.F32)[0])
    R.Plan(net, n_sliced=sliced, seed=seed, path_trials=16, hbm_budget_bytes=one)
    with pytest.raises(R.RqcError):
        R.Plan(net, n_sliced=sliced, seed=seed, path_trials=16, hbm_budget_bytes=one - 256)

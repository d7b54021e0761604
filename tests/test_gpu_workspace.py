"""Calls in the least workspace, where the subtrees' fused form does not fit and
every step has a launch of its own, and in the same buffer told to be larger:
each against the oracle (normalised error <= 1e-4 FP32, 2e-2 FP16: the bounds of
every amplitude test), captured and replayed, in turn.  A byte less is refused."""
import numpy as np
import pytest
import torch

import oracle
import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,lp,bound", [(R.F32, 0, 1e-4), (R.F16, 0, 2e-2), (R.F16, 4, 2e-2)])
@pytest.mark.parametrize("n_batch", [1, 3])
def test_least_workspace(prec, lp, bound, n_batch):
    print("least workspace", prec, lp, n_batch, flush=True)
    c = rqcgen.grid_rqc(5, 6, 10, 3)
    openq = list(range(25, 30))
    P = R.Plan(R.Network(R.Circuit.from_rqcgen(c), openq), n_sliced=6, seed=3, path_trials=16, lp_min_log2=lp).bind()
    bits = np.stack([rqcgen.random_bits(25, s) for s in range(n_batch)])
    ref = np.stack([oracle.amplitudes_tn(c, openq, b) for b in bits])
    lo, pref = P.workspace_bytes(0, n_batch, prec)
    buf = torch.empty(pref, dtype=torch.uint8, device="cuda")
    out = torch.empty(2 * n_batch * 32, dtype=torch.float64, device="cuda")
    for size in (lo, pref, lo + (1 << 16), lo, pref):
        got = R.to_complex(P.contract(bits, prec=prec, workspace=buf[:size], out=out))
        err = oracle.normalized_error(got.reshape(-1), ref.reshape(-1), 30)
        print(size, P.last_report, err, flush=True)
        assert err < bound and P.last_report["fp32_reruns"] == 0
    with pytest.raises(R.RqcError):
        P.contract(bits, prec=prec, workspace=buf[:lo - 1], out=out)


def test_tuning_in_the_least_workspace():
    c = rqcgen.grid_rqc(5, 6, 10, 3)
    openq = list(range(25, 30))
    P = R.Plan(R.Network(R.Circuit.from_rqcgen(c), openq), n_sliced=6, seed=3, path_trials=16).bind()
    bits = rqcgen.random_bits(25, 0)
    lo, pref = P.workspace_bytes(0, 1, R.F32)
    buf = torch.empty(pref, dtype=torch.uint8, device="cuda")
    print(P.autotune(R.F32, workspace=buf[:lo]), flush=True)
    ref = oracle.amplitudes_tn(c, openq, bits)
    lo, _ = P.workspace_bytes(0, 1, R.F32)
    for size in (lo, pref):
        got = R.to_complex(P.contract(bits, workspace=buf[:size]))[0]
        assert oracle.normalized_error(got, ref, 30) < 1e-4

"""A call's report reads the flags that this call wrote, also when the plan's kernel
and storage choices change between the call and its report (here by calibration,
which moves every step back to complex64 and so changes the program that the next
call uploads).  The FP16 slices that a storage-exponent bias drives out of range
are all counted and re-run in FP32 (normalised error below 1e-4, the bound of
every FP32 amplitude test); without a bias none is (2e-2, the FP16 bound)."""
import pytest
import torch

import oracle
import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias,reruns,bound", [(40, 8, 1e-4), (0, 0, 2e-2)])
def test_report_after_the_choices_changed(bias, reruns, bound):
    c = rqcgen.grid_rqc(5, 5, 8, 3)
    openq = list(range(21, 25))
    P = R.Plan(R.Network(R.Circuit.from_rqcgen(c), openq), n_sliced=3, seed=5, path_trials=32, lp_min_log2=4).bind()
    bits = rqcgen.random_bits(21, 9)
    P.set_scale_bias(bias)
    amps = P.contract(bits, prec=R.F16, sync=False)
    torch.cuda.synchronize()
    P.set_scale_bias(0)
    ws = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")  # not the call's own
    assert P.calibrate(bits, target_err=1e-12, workspace=ws)["reduced"] == 0
    report = P.report()
    print(report, flush=True)
    assert report["n_slices"] == 8 and report["fp32_reruns"] == reruns
    full = oracle.amplitudes_tn(c, openq, bits)
    assert oracle.normalized_error(R.to_complex(amps)[0], full, 25) < bound

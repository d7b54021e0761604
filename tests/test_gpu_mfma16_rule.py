"""The streamed form of the 16-bit matrix kernel is chosen, without tuning, only where
a launch has enough tiles to gain by it: 2^11 (sums of 2^5) or 2^12 (2^6) of 128 x 64
outputs, counted over the copies of the group.  The forms give the same bits, so
the values of two slices are the same in calls for two and for sixteen."""
import numpy as np
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


def test_streamed_form_by_tiles():
    c = rqcgen.grid_rqc(5, 6, 12, 3)
    openq = list(range(26, 30))
    P = R.Plan(R.Network(R.Circuit.from_rqcgen(c), openq), n_sliced=4, seed=4, path_trials=64).bind()
    bits = rqcgen.random_bits(26, 1)
    P.set_timing(4)
    seen, outs = set(), []
    for ids in (np.arange(2), np.arange(16)):
        outs.append(P.contract(bits, slice_ids=ids, prec=R.F16, per_slice=True)[1][:2].clone())
        for t in P.launch_timings():
            if t["kernel"] == R.KERN_MFMA16 and t["k"] in (5, 6):
                tiles = t["copies"] << (t["m"] + t["n"] - 13)
                seen.add((t["m"], t["n"], t["k"], tiles, bool(t["variant"] & R.VAR_STREAM)))
    P.set_timing(-1)
    print(sorted(seen), flush=True)
    streamed = [s for s in seen if s[4]]
    assert streamed and len(streamed) < len(seen)
    assert all(s[3] >= (1 << 11 if s[2] == 5 else 1 << 12) for s in streamed)
    assert torch.equal(outs[0], outs[1])

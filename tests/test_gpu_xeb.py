"""Batch statistics at the sizes where the split over workgroups changes:
one workgroup below 2^13 entries, partial sums above, ragged last workgroups,
more samples than entries, an unaligned buffer.  FP64 sums of positive terms
in another order: relative error <= n 2^-53, here at most 2e-11; checked at
1e-10."""
import numpy as np
import pytest
import torch

import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ns,shift", [(1, 0, 0), (1000, 7, 0), (131071, 131071, 0), (131072, 1, 0), (131073, 9000, 0),
                                        (190001, 3, 1), (5, 140000, 0), (1 << 18, 1 << 17, 0)])
def test_batch_statistics_sizes(n, ns, shift):
    print("xeb", n, ns, shift, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(2 * n + shift, dtype=torch.float64, device="cuda", generator=g) * 2.0 ** -18
    amps = buf[shift:]
    idx = torch.randint(0, n, (ns,), device="cuda", generator=g) if ns else None
    got = R.batch_xeb(amps, 36, samples=idx)
    p = amps.cpu().numpy().astype(np.longdouble).reshape(-1, 2)
    p = (p * p).sum(1)
    dim = np.longdouble(2.0) ** 36
    ref = {"sum_p": p.sum(), "sum_p2": (p * p).sum(), "xeb_all": dim * p.sum() / n - 1,
           "xeb_ideal_sampling": dim * (p * p).sum() / p.sum() - 1,
           "xeb_samples": dim * p[idx.cpu().numpy()].sum() / ns - 1 if ns else np.longdouble(0)}
    for k, v in ref.items():
        assert abs(got[k] - float(v)) <= 1e-10 * max(1.0, abs(float(v))), (k, got[k], v)
    if ns:
        idx[ns // 2] = n
        assert np.isnan(R.batch_xeb(amps, 36, samples=idx)["xeb_samples"])

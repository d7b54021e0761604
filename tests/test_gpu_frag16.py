"""The 16-bit long-sum GEMM on packed fragments at the edges of its tiles:
one tile with the shortest sum, split sums, rows and columns beyond one tile,
and operands that are 8- but not 16-byte aligned.  The products are exact in
FP32 on operands rounded to 16 bits, so the result is compared with the
complex128 product of the rounded operands: the FP32 sum of K terms is within
6 u sqrt(K) x RMS, u = 2^-24."""
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R
from test_gpu_split32 import _exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,dtype", [("f16", torch.float16), ("bf16", torch.bfloat16)])
@pytest.mark.parametrize("m,n,k,shift", [(8, 7, 8, 0), (8, 7, 13, 0), (10, 9, 8, 1), (9, 8, 11, 1), (12, 11, 9, 0)])
def test_long_sums_on_rounded_operands(prec, dtype, m, n, k, shift):
    print("frag16", prec, m, n, k, shift, flush=True)
    st = rqcgen.synthetic_step(m + k, n + k, k, 21)
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn((1 << (m + k)) + shift, dtype=torch.complex64, device="cuda", generator=g)[shift:]
    B = torch.randn((1 << (n + k)) + shift, dtype=torch.complex64, device="cuda", generator=g)[shift:]
    assert R.pair_workspace_bytes(st.labels_a, st.labels_b, st.labels_c, prec=R.PRECISIONS[prec])
    got = R.pair_contract(A, B, st.labels_a, st.labels_b, st.labels_c, prec=prec)
    rounded = [torch.view_as_complex(torch.view_as_real(x).to(dtype).to(torch.float64).contiguous()) for x in (A, B)]
    ref = _exact(st, *rounded)
    err = (got.to(torch.complex128) - ref).abs().max().item()
    assert err <= 6 * 2.0 ** -24 * 2.0 ** (k / 2) * ref.abs().square().mean().sqrt().item()

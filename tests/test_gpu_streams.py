"""Single-step calls on a stream that is not torch's current one.  Their temporary
workspace has to live on that stream: memory allocated under the current stream
is handed out again as soon as the call returns, while the kernels (held up here by
earlier work on their stream) have not even started.  The results are those of
the same call on the current stream, bit for bit."""
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


def _hold_up(side):
    """Tens of milliseconds of work on the stream."""
    with torch.cuda.stream(side):
        x = torch.randn(4096, 4096, device="cuda")
        for _ in range(40):
            x = torch.matmul(x, x) * 1e-2
    return x


@pytest.mark.parametrize("m,n,k,prec", [(9, 8, 10, R.BF16), (9, 8, 10, R.F32), (2, 2, 16, R.F32)])
def test_pair_workspace_on_another_stream(m, n, k, prec):
    print("[case]", m, n, k, prec, flush=True)
    st = rqcgen.synthetic_step(m + k, n + k, k, 3)
    labels = (st.labels_a, st.labels_b, st.labels_c)
    g = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn(1 << (m + k), dtype=torch.complex64, device="cuda", generator=g)
    B = torch.randn(1 << (n + k), dtype=torch.complex64, device="cuda", generator=g)
    need = R.pair_workspace_bytes(*labels, prec=prec)
    assert need
    ref = R.pair_contract(A, B, *labels, prec=prec)
    out = torch.zeros_like(ref)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    keep = _hold_up(side)
    R.pair_contract(A, B, *labels, C_out=out, prec=prec, stream=side.cuda_stream)
    # what the current stream allocates next must not be the workspace
    other = [torch.full((need,), 255, dtype=torch.uint8, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    assert torch.equal(torch.view_as_real(out).view(torch.int32), torch.view_as_real(ref).view(torch.int32))
    del other, keep


@pytest.mark.parametrize("n", [1 << 10, 1 << 18])
def test_batch_statistics_on_another_stream(n):
    print("[case]", n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    amps = torch.randn(2 * n, dtype=torch.float64, device="cuda", generator=g) * 2.0 ** -18
    ref = R.batch_xeb(amps, 36)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    keep = _hold_up(side)
    assert R.batch_xeb(amps, 36, stream=side.cuda_stream) == ref  # read after the kernels
    del keep

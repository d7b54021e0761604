"""Single steps captured into a graph and replayed on other contents of the same
buffers, with eager work and synchronisations between the replays: every replay gives
the eager call's bits.  The FP32 form on the FP16 matrix cores decides on the device
whether the operands suit it, so it has to decide anew in each replay."""
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,prec,batch", [(9, 8, 10, R.F32, 1), (9, 7, 14, R.F32, 1), (9, 8, 11, R.F32, 2),
                                              (9, 8, 10, R.BF16, 1), (2, 2, 16, R.F32, 1), (9, 4, 4, R.F32, 3)])
def test_replays_on_other_contents(m, n, k, prec, batch):
    print("[case]", m, n, k, prec, batch, flush=True)
    st = rqcgen.synthetic_step(m + k, n + k, k, 9)
    labels = (st.labels_a, st.labels_b, st.labels_c)
    kw = dict(batch=batch, stride_a=1 << (m + k), stride_b=1 << (n + k), stride_c=1 << (m + n), prec=prec)
    A = torch.randn(batch << (m + k), dtype=torch.complex64, device="cuda")
    B = torch.randn(batch << (n + k), dtype=torch.complex64, device="cuda")
    C = torch.empty(batch << (m + n), dtype=torch.complex64, device="cuda")
    need = R.pair_workspace_bytes(*labels, batch=batch, stride_a=kw["stride_a"], stride_b=kw["stride_b"], prec=prec)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    R.pair_contract(A, B, *labels, C_out=C, workspace=ws, **kw)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        R.pair_contract(A, B, *labels, C_out=C, workspace=ws, **kw)
    for turn in range(6):
        A.copy_(torch.randn(batch << (m + k), dtype=torch.complex64, device="cuda"))
        if turn % 2:
            A[torch.rand(A.shape, device="cuda") < 0.95] = 0  # not for the split form
        if turn == 4:
            B.mul_(2.0 ** -40)
        torch.cuda.synchronize()
        eager = R.pair_contract(A, B, *labels, **kw)
        C.fill_(9.0)
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(C).view(torch.int32), torch.view_as_real(eager).view(torch.int32)), turn
        if prec == R.F32 and turn % 2:
            full = R.pair_contract(A, B, *labels, **dict(kw, kernel=1)) if k >= 10 and n >= 7 else eager
            assert torch.equal(torch.view_as_real(full), torch.view_as_real(eager))

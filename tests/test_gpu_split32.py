"""FP32 long sums on the FP16 matrix cores (values as two halves): shapes at
the edges of its rule (one output tile, exchanged operands, split sums, a
batch with a shared operand) against complex128, and the operands that it
hands back to the FP32 kernel (a range above 2^18 inside one operand,
infinities, NaN, extreme scales), whose results have to be the FP32 kernel's
bit for bit.

Tolerance: two halves keep 2^-22 of a value of the largest ones' size, the sum
has K / 16 * 6 FP32 accumulations per product: max error <= 6 u sqrt(K / 2) x
RMS with u = 2^-24 (4 sigma and the two products per part), at K = 2^10: 8e-6."""
import numpy as np
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


def _case(m, n, k, seed, batch=1, shared_b=False):
    st = rqcgen.synthetic_step(m + k, n + k, k, seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn(batch << (m + k), dtype=torch.complex64, device="cuda", generator=g)
    B = torch.randn((1 if shared_b else batch) << (n + k), dtype=torch.complex64, device="cuda", generator=g)
    return st, A, B


def _index(have, want):
    r = len(have)
    e = torch.arange(1 << r, device="cuda")
    s = torch.zeros_like(e)
    for i, l in enumerate(reversed(want)):
        s |= ((e >> i) & 1) << (r - 1 - have.index(l))
    return s


def _exact(st, A, B):
    K = [x for x in st.labels_a if x in st.labels_b]
    M = [x for x in st.labels_a if x not in K]
    N = [x for x in st.labels_b if x not in K]
    a = A.to(torch.complex128)[_index(st.labels_a, M + K)].view(1 << len(M), -1)
    b = B.to(torch.complex128)[_index(st.labels_b, K + N)].view(1 << len(K), -1)
    return (a @ b).view(-1)[_index(M + N, st.labels_c)]


def _run(st, A, B, **kw):
    return R.pair_contract(A, B, st.labels_a, st.labels_b, st.labels_c, **kw)


@pytest.mark.parametrize("m,n,k,batch,shared_b", [
    (14, 7, 10, 1, False),   # shortest sum of any size, one column tile
    (7, 14, 10, 1, False),   # exchanged operands
    (8, 7, 10, 1, False),    # one output tile
    (8, 8, 14, 1, False),    # split sum
    (9, 7, 17, 1, False),    # widest split
    (13, 13, 8, 1, False),   # shortest sum, many tiles
    (11, 10, 10, 3, True),   # batch, shared B
    (9, 9, 11, 2, False),
])
def test_split_sums_vs_complex128(m, n, k, batch, shared_b):
    print("split32", m, n, k, batch, shared_b, flush=True)
    st, A, B = _case(m, n, k, 5, batch, shared_b)
    sa, sb, sc = 1 << (m + k), 0 if shared_b else 1 << (n + k), 1 << (m + n)
    need = R.pair_workspace_bytes(st.labels_a, st.labels_b, st.labels_c, batch=batch, stride_a=sa, stride_b=sb)
    assert need >= 12 * (sa + (1 << (n + k)))  # this form is taken
    got = _run(st, A, B, batch=batch, stride_a=sa, stride_b=sb)
    for j in range(batch):
        ref = _exact(st, A[j * sa:(j + 1) * sa], B[j * sb:j * sb + (1 << (n + k))])
        err = (got[j * sc:(j + 1) * sc].to(torch.complex128) - ref).abs().max().item()
        rms = ref.abs().square().mean().sqrt().item()
        assert err <= 6 * 2.0 ** -24 * (2.0 ** k / 2) ** 0.5 * rms, (j, err / rms)


@pytest.mark.parametrize("what", ["wide", "inf", "nan", "tiny", "huge", "wide_b"])
def test_operands_outside_the_split_take_the_fp32_kernel(what):
    print("split32 fallback", what, flush=True)
    st, A, B = _case(12, 10, 10, 9)
    if what == "wide":
        A[12345] *= 2.0 ** -24
    elif what == "wide_b":
        B[777] *= 2.0 ** 21
    elif what == "inf":
        A[5] = float("inf")
    elif what == "nan":
        B[6] = complex(0.0, float("nan"))
    elif what == "tiny":
        A *= 2.0 ** -110
    else:
        B *= 2.0 ** 105
    got = _run(st, A, B)
    ref = _run(st, A, B, kernel=1)
    assert torch.equal(torch.view_as_real(got).view(torch.int32), torch.view_as_real(ref).view(torch.int32))


def test_zero_operand_and_missing_workspace():
    st, A, B = _case(12, 10, 10, 11)
    assert _run(st, torch.zeros_like(A), B).abs().max().item() == 0.0
    # a workspace that is too small: the FP32 kernel, as without one
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda")
    got, ref = _run(st, A, B, workspace=ws), _run(st, A, B, kernel=1)
    assert (got - ref).abs().max().item() <= 2e-5 * ref.abs().square().mean().sqrt().item()

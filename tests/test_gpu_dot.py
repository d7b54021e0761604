"""The streaming dot products with the reads kept in flight (2 to 64 outputs,
rows on 16-byte boundaries): one round of the workgroup per split and several,
fewer splits than workgroups and more, row and column counts from 1 to 8.

The same operands one element (8 bytes) off such a boundary go to the kernel that
reads through registers, which sums in the same order: the same bits.  Both are
held to 2e-5 x RMS of the complex128 product (partial sums of at most 2^12
terms per split, added in FP32).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2110_14502_amd")

CASES = [
    # m, n, k, copies
    (3, 3, 16, 32),     # 2^9 terms per split: one round
    (3, 3, 17, 32),
    (3, 3, 18, 33),     # 8448 items
    (2, 2, 16, 32),
    (1, 3, 16, 32),
    (3, 1, 17, 20),
    (2, 3, 12, 700),
    (3, 2, 19, 5),
    (3, 3, 21, 1),      # 2^9 splits of 2^12: as many items as workgroups
    (1, 0, 18, 16),
    (0, 2, 16, 32),
    (1, 1, 17, 24),
    (3, 3, 15, 32),     # 2^8 terms per split: the register kernel both times
]


@pytest.mark.parametrize("m,n,k,copies", CASES)
def test_dot_copies(m, n, k, copies):
    print("[case]", m, n, k, copies, flush=True)
    rng = np.random.default_rng(m + 10 * n + 100 * k)
    M, N, K = list(range(m)), list(range(100, 100 + n)), list(range(200, 200 + k))
    lc = [int(x) for x in rng.permutation(M + N)]
    a = torch.randn(copies << (m + k), 2, generator=torch.Generator().manual_seed(k)).cuda()
    b = torch.randn((1 << (n + k)), 2, generator=torch.Generator().manual_seed(k + 1)).cuda()
    outs = []
    for shift in (0, 1):
        A = torch.zeros(a.shape[0] + 2, 2, device="cuda")[shift:shift + a.shape[0]]
        B = torch.zeros(b.shape[0] + 2, 2, device="cuda")[shift:shift + b.shape[0]]
        A.copy_(a)
        B.copy_(b)
        c = R.pair_contract(torch.view_as_complex(A), torch.view_as_complex(B), M + K, N + K, lc,
                            batch=copies, stride_a=1 << (m + k), stride_b=0)
        torch.cuda.synchronize()
        outs.append(torch.view_as_real(c).cpu())
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    got = torch.view_as_complex(outs[0]).numpy().reshape(copies, -1)
    bv = torch.view_as_complex(b.double()).reshape(1 << n, 1 << k)
    src = M + N
    for i in range(0, copies, max(1, copies // 7)):
        av = torch.view_as_complex(a[i << (m + k):(i + 1) << (m + k)].double()).reshape(1 << m, 1 << k)
        ref = (av @ bv.T).cpu().numpy().reshape([2] * (m + n))
        ref = ref.transpose([src.index(x) for x in lc]).reshape(-1)
        assert np.abs(got[i] - ref).max() <= 2e-5 * np.sqrt(np.mean(np.abs(ref) ** 2))

"""The row kernel with C's lowest address bits at any of a tile's row bits: which rows
a wave takes follows C's order.  Tiles of 256, 128 and fewer rows, sums whose rows
share a cache line of A and sums whose rows do not, one chunk of columns and several,
complex64 and 16-bit outputs.  Reference: the complex128 product; FP32 sums of 2^k
terms are within 2e-6 x RMS x 2^(k/2) at the largest of 2^16 outputs, a 16-bit output
adds 2^-11 (FP16) or 2^-8 (BF16) of the largest, five RMS."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2110_14502_amd")

T = {R.ST_C64: torch.float32, R.ST_F16: torch.float16, R.ST_BF16: torch.bfloat16}
ROUND = {R.ST_C64: 0.0, R.ST_F16: 5 * 2.0 ** -11, R.ST_BF16: 5 * 2.0 ** -8}


@pytest.mark.parametrize("store", [R.ST_C64, R.ST_F16, R.ST_BF16])
@pytest.mark.parametrize("m,n,k", [(10, 4, 4), (9, 2, 0), (9, 3, 2), (8, 5, 6), (7, 3, 4), (7, 1, 1), (6, 4, 3), (9, 7, 4)])
def test_orders_of_c(m, n, k, store):
    rng = np.random.default_rng(m + 10 * n + 100 * k)
    copies = 3
    M, N, K = list(range(m)), list(range(100, 100 + n)), list(range(200, 200 + k))  # label i of M: row bit i
    la, lb = M[::-1] + K, N[::-1] + K
    g = torch.Generator().manual_seed(m + n)
    a = torch.randn(copies, 1 << m, 1 << k, 2, generator=g)
    b = torch.randn(copies, 1 << n, 1 << k, 2, generator=g)
    prod = torch.matmul(torch.view_as_complex(a.double()), torch.view_as_complex(b.double()).transpose(1, 2).contiguous())
    prod = prod.numpy().reshape([copies] + [2] * (m + n))
    src = M[::-1] + N[::-1]
    lows = [x for x in ([0, 1], [6, 7], [7, 6, 5, 4], [4, 7], [6, 0], [100, 6], [5], [3, 6, 100, 2]) if max(
        [y for y in x if y < 100], default=0) < m]
    for low in lows + [[int(x) for x in rng.permutation(M + N)]]:
        lc = [int(x) for x in rng.permutation([x for x in M + N if x not in low])] + low[::-1]
        print("[case]", m, n, k, store, low, flush=True)
        C = torch.full((copies * (1 << (m + n)) + 2, 2), 7.0, dtype=T[store], device="cuda")
        R.pair_contract_stored(a.cuda(), b.cuda(), C[1:-1], la, lb, lc, R.ST_C64, R.ST_C64, store, R.KERN_ROWS, batch=copies,
                               stride_a=1 << (m + k), stride_b=1 << (n + k), stride_c=1 << (m + n))
        got = C.float().cpu().numpy().astype(np.float64)
        assert (got[0] == 7).all() and (got[-1] == 7).all()
        ref = prod.transpose([0] + [1 + src.index(x) for x in lc]).reshape(-1)
        err = np.abs(got[1:-1, 0] + 1j * got[1:-1, 1] - ref).max()
        assert err <= (2e-6 * 2.0 ** (k / 2) + ROUND[store]) * np.sqrt(np.mean(np.abs(ref) ** 2)), low

"""The forms of the 16-bit matrix kernel that a call chooses among by size and
storage (default, A streamed past a resident tile of B, operands exchanged) give
the same bits: sums of 32 to 128 terms, outputs of 64 to 256 columns, one row
tile and many, B in 16 bits and in complex64, 16-bit and complex64 outputs.
The smallest sizes that each rule names (2^13 and 2^16 rows) and one below."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2110_14502_amd")

T16 = {R.ST_F16: torch.float16, R.ST_BF16: torch.bfloat16}
MMA = {R.ST_F16: R.F16, R.ST_BF16: R.BF16}


@pytest.mark.parametrize("lp", [R.ST_F16, R.ST_BF16])
@pytest.mark.parametrize("m,n,k,copies", [(13, 7, 7, 2), (12, 7, 6, 3), (13, 6, 5, 3), (16, 6, 6, 1),
                                          (16, 7, 7, 1), (13, 8, 5, 1), (7, 7, 6, 1)])
def test_forms_agree(lp, m, n, k, copies):
    print("[case]", lp, m, n, k, copies, flush=True)
    rng = np.random.default_rng(m + 10 * n + 100 * k)
    M, N, K = list(range(m)), list(range(100, 100 + n)), list(range(200, 200 + k))
    lc = [int(x) for x in rng.permutation(M + N)]
    la = [x for x in lc if x < 100] + K
    lb = [x for x in lc if x >= 100] + K
    g = torch.Generator().manual_seed(m + n)
    A = (torch.randn(copies << (m + k), 2, generator=g) * 0.1).to(T16[lp]).cuda()
    B32 = (torch.randn(copies << (n + k), 2, generator=g) * 0.1).cuda()
    for sb, B in ((lp, B32.to(T16[lp])), (R.ST_C64, B32)):
        for sc in (lp, R.ST_C64):
            outs = []
            for v in (0, R.VAR_STREAM) + ((R.VAR_SWAP,) if n >= 7 else ()):
                C = torch.full((copies << (m + n), 2), 7.0, device="cuda",
                               dtype=torch.float32 if sc == R.ST_C64 else T16[lp])
                R.pair_contract_stored(A, B, C, la, lb, lc, lp, sb, sc, R.KERN_MFMA16,
                                       mma_prec=MMA[lp], batch=copies, stride_a=1 << (m + k),
                                       stride_b=1 << (n + k), stride_c=1 << (m + n), variant=v)
                torch.cuda.synchronize()
                outs.append(C.view(torch.int32 if sc == R.ST_C64 else torch.int16))
            assert all(torch.equal(o, outs[0]) for o in outs[1:]), (sb, sc)

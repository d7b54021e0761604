"""The FP32 matrix kernel that copies its chunks straight into LDS (complex64
operands, summed indices lowest): one tile and many, one chunk of summed terms
and many, several copies, fewer items than workgroups and more, C's lowest
index a row or a column, complex64 and 16-bit outputs; operands that it cannot
take (a base or a copy stride that is not a multiple of 16 bytes) go to the
register kernel.

The reference is the complex128 product of the operands.  The FP32 products of
2^k terms and their sums in the three-product form stay below 2e-5 x RMS (a 16-bit
output adds its rounding: 6e-3 / 4e-2 x RMS); the kernels sum in the same order,
so the per-tile kernel gives the same bits.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2110_14502_amd")

TOL = {R.ST_C64: 2e-5, R.ST_F16: 6e-3, R.ST_BF16: 4e-2}
TORCH = {R.ST_C64: torch.float32, R.ST_F16: torch.float16, R.ST_BF16: torch.bfloat16}


def _labels(m, n, k, low, seed):
    """Planner's layouts; `low`: the label of C's lowest index ('m' or 'n')."""
    rng = np.random.default_rng(seed)
    M, N, K = list(range(m)), list(range(100, 100 + n)), list(range(200, 200 + k))
    c = [int(x) for x in rng.permutation(M + N)]
    last = M[int(rng.integers(m))] if low == "m" else N[int(rng.integers(n))]
    c.remove(last)
    c.append(last)
    return [x for x in c if x < 100] + K, [x for x in c if x >= 100] + K, c


def _reference(A, B, la, lb, lc, m, n, k):
    """C in lc's order (labels most significant first)."""
    c = (A.reshape(1 << m, 1 << k) @ B.reshape(1 << n, 1 << k).T).reshape([2] * (m + n))
    src = la[:m] + lb[:n]
    return c.transpose([src.index(x) for x in lc]).reshape(-1)


CASES = [
    # m, n, k, copies, low, store_c, shift (elements), pad (elements of a copy)
    (7, 6, 4, 1, "m", R.ST_C64, 0, 0),
    (7, 6, 4, 1, "n", R.ST_C64, 0, 0),
    (7, 6, 5, 3, "n", R.ST_C64, 0, 0),
    (8, 7, 6, 5, "m", R.ST_C64, 0, 0),
    (7, 6, 7, 2, "n", R.ST_C64, 0, 0),
    (12, 7, 4, 9, "n", R.ST_C64, 0, 0),     # 576 items: a second item for some
    (11, 8, 5, 37, "m", R.ST_C64, 0, 0),    # 2368 items
    (9, 7, 8, 2, "n", R.ST_C64, 0, 0),      # long sums
    (7, 6, 11, 1, "m", R.ST_C64, 0, 0),
    (9, 8, 6, 3, "n", R.ST_F16, 0, 0),
    (9, 8, 6, 3, "m", R.ST_BF16, 0, 0),
    (8, 6, 5, 3, "n", R.ST_C64, 1, 0),      # base 8 bytes off a 16-byte boundary
    (8, 6, 5, 3, "n", R.ST_C64, 0, 1),      # odd copy strides
    (8, 6, 5, 3, "n", R.ST_C64, 0, 2),
]


@pytest.mark.parametrize("m,n,k,copies,low,sc,shift,pad", CASES)
def test_copy_kernel(m, n, k, copies, low, sc, shift, pad):
    print("[case]", m, n, k, copies, low, sc, shift, pad, flush=True)
    la, lb, lc = _labels(m, n, k, low, 7 * m + n + k)
    rng = np.random.default_rng(m + 10 * n + 100 * k)

    def operand(bits):
        step = (1 << bits) + pad
        x = rng.standard_normal((copies * step + shift, 2)).astype(np.float32)
        t = torch.from_numpy(x).cuda()
        v = (x[:, 0].astype(np.float64) + 1j * x[:, 1])[shift:]
        return t[shift:], [v[i * step:i * step + (1 << bits)] for i in range(copies)], step

    A, va, sa = operand(m + k)
    B, vb, sb = operand(n + k)
    size = 1 << (m + n)
    outs = []
    for variant in (0, R.VAR_PERSISTENT, R.VAR_TILES):
        # one guard element before and after each copy
        C = torch.full((copies * (size + 2), 2), 7.0, dtype=TORCH[sc], device="cuda")
        R.pair_contract_stored(A, B, C[1:], la, lb, lc, R.ST_C64, R.ST_C64, sc, R.KERN_MFMA,
                               batch=copies, stride_a=sa, stride_b=sb, stride_c=size + 2,
                               variant=variant)
        torch.cuda.synchronize()
        outs.append(C.cpu().reshape(copies, size + 2, 2))
    for o in outs[1:]:
        assert torch.equal(o.view(torch.int32 if sc == R.ST_C64 else torch.int16),
                           outs[0].view(torch.int32 if sc == R.ST_C64 else torch.int16))
    assert bool((outs[0][:, 0] == 7).all()) and bool((outs[0][:, -1] == 7).all())
    got = outs[0][:, 1:-1].float().numpy()
    for i in range(copies):
        ref = _reference(va[i], vb[i], la, lb, lc, m, n, k)
        d = got[i, :, 0] + 1j * got[i, :, 1] - ref
        assert np.abs(d).max() <= TOL[sc] * np.sqrt(np.mean(np.abs(ref) ** 2))

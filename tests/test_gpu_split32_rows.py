"""FP32 long sums on the FP16 matrix cores against the FP32 kernel (kernel=1), row by
row and column by column of C: operands that are dense and even take the split form,
whose error against complex128 has to be the FP32 kernel's; all others (few terms
per row, terms or rows of very different size, real operands, permutations) have
to give the FP32 kernel's bits.

Bound for the former: 1.25 times the FP32 kernel's error in every row and column.
The form adds 3/8 as many times as the FP32 kernel (0.8 of its error for even
terms, 1.0 where a term of three times the others ends the sum); the root mean
square of a row's 2^10 complex errors scatters by 2 %, the ratio by 3 %, so 1.25 is
more than eight of these."""
import pytest
import torch

import rqcgen
import paper_2110_14502_amd as R
from test_gpu_split32 import _index

pytestmark = pytest.mark.gpu

M, N, K = 11, 10, 10


def _normal(rows, g):
    return torch.randn(rows, 1 << K, dtype=torch.complex64, device="cuda", generator=g)


def _unit(rows, g):
    x = torch.rand(rows, 1 << K, device="cuda", generator=g) * 6.283185307
    return torch.polar(torch.ones_like(x), x)


def _sparse(terms):
    def make(rows, g):
        x = _normal(rows, g)
        keep = torch.rand(rows, 1 << K, device="cuda", generator=g).argsort(1) < terms
        return x * keep
    return make


def _outlier(c, base):
    def make(rows, g):
        x = base(rows, g)
        x[:, -1] *= c
        return x
    return make


def _scaled_rows(bits):
    def make(rows, g):
        e = torch.randint(0, bits + 1, (rows, 1), device="cuda", generator=g)
        return _normal(rows, g) * torch.pow(2.0, -e.float())
    return make


def _growing(bits, base):
    def make(rows, g):
        return base(rows, g) * torch.pow(2.0, bits * (torch.arange(1 << K, device="cuda") / (1 << K) - 1))
    return make


def _identity(rows, g):
    x = torch.zeros(rows, 1 << K, dtype=torch.complex64, device="cuda")
    x[torch.arange(rows), torch.randperm(1 << K, generator=g, device="cuda")[:rows]] = 1
    return x


def _one_large(rows, g):
    x = _unit(rows, g) * 2.0 ** -18
    x[3, 5] = 1.0
    return x


def _real(rows, g):
    return _normal(rows, g).real + 0j


def _constant(rows, g):
    return torch.full((rows, 1 << K), 1.2345678 + 0.7654321j, dtype=torch.complex64, device="cuda")


def _half(rows, g):
    x = _normal(rows, g)
    x[:, 1 << (K - 1):] = 0
    return x


KEEP = {"normal": (_normal, _normal), "unit modulus": (_unit, _unit), "scaled rows": (_scaled_rows(4), _scaled_rows(4)),
        "outlier of 3": (_outlier(3, _unit), _outlier(3, _unit)), "growing by 2": (_growing(1, _unit), _growing(1, _unit)),
        "zero rows": (lambda r, g: _normal(r, g) * (torch.arange(r, device="cuda") % 16 > 0)[:, None], _normal)}
BACK = {"one term": (_sparse(1), _normal), "8 terms": (_sparse(8), _sparse(8)), "64 terms": (_normal, _sparse(64)),
        "a quarter": (_sparse(1 << (K - 2)), _sparse(1 << (K - 2))), "three quarters": (_sparse(768), _normal),
        "half": (_half, _normal), "permutation": (_normal, _identity), "real": (_real, _real), "constant": (_constant, _normal),
        "real and complex": (_real, _normal), "outlier of 16": (_outlier(16, _unit), _outlier(16, _unit)),
        "growing by 16": (_growing(4, _normal), _growing(4, _normal)), "rows to 2^-16": (_scaled_rows(16), _normal),
        "one large element": (_one_large, _unit), "large element of B": (_unit, _one_large)}


def _call(make_a, make_b, seed):
    st = rqcgen.synthetic_step(M + K, N + K, K, seed)
    ks = [x for x in st.labels_a if x in st.labels_b]
    ms, ns = [x for x in st.labels_a if x not in ks], [x for x in st.labels_b if x not in ks]
    g = torch.Generator(device="cuda").manual_seed(seed)
    a, b = make_a(1 << M, g).contiguous(), make_b(1 << N, g).contiguous()
    A = a.view(-1)[_index(ms + ks, st.labels_a)]
    B = b.view(-1)[_index(ns + ks, st.labels_b)]
    got, ref = [R.pair_contract(A, B, st.labels_a, st.labels_b, st.labels_c, kernel=k)[_index(st.labels_c, ms + ns)].view(1 << M, 1 << N)
                for k in (-1, 1)]
    return got, ref, a.to(torch.complex128) @ b.to(torch.complex128).T.contiguous()


@pytest.mark.parametrize("what", sorted(KEEP))
def test_even_operands_have_the_fp32_error(what):
    print("split32 rows", what, flush=True)
    got, ref, exact = _call(*KEEP[what], 31)
    assert not torch.equal(got, ref)  # the split form ran
    for dim in (0, 1):
        e = [(x - exact).abs().square().mean(dim).sqrt() for x in (got, ref)]
        assert bool((e[0] <= 1.25 * e[1]).all()), (dim, (e[0] / e[1]).max().item())


@pytest.mark.parametrize("what", sorted(BACK))
def test_uneven_operands_get_the_fp32_bits(what):
    print("split32 rows", what, flush=True)
    got, ref, _ = _call(*BACK[what], 32)
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(ref))


@pytest.mark.parametrize("m,n,shared", [(10, 9, None), (9, 10, "a"), (10, 9, "b"), (8, 7, None)])
def test_copies_of_a_batch(m, n, shared):
    """All copies in one call, of scales from 1 to 2^-30 (each has its own): within 6
    u sqrt(K / 2) x RMS of complex128 as single calls are, and all of them the FP32
    kernel's bits where one has a sparse row."""
    print("split32 batch", m, n, shared, flush=True)
    nb, k = 3, 11
    st = rqcgen.synthetic_step(m + k, n + k, k, 8)
    ks = [x for x in st.labels_a if x in st.labels_b]
    ms, ns = [x for x in st.labels_a if x not in ks], [x for x in st.labels_b if x not in ks]
    g = torch.Generator(device="cuda").manual_seed(4)
    na, nbb = (1 if shared == "a" else nb), (1 if shared == "b" else nb)
    A = torch.randn(na, 1 << (m + k), dtype=torch.complex64, device="cuda", generator=g)
    B = torch.randn(nbb, 1 << (n + k), dtype=torch.complex64, device="cuda", generator=g)
    scale = torch.tensor([1.0, 2.0 ** -30, 2.0 ** -9], device="cuda")[:, None]
    (B if shared == "a" else A).mul_(scale)
    args = dict(batch=nb, stride_a=0 if shared == "a" else A.shape[1], stride_b=0 if shared == "b" else B.shape[1],
                stride_c=(1 << (m + n)) + 6)

    def run(kernel):
        C = torch.full((nb, args["stride_c"]), 5.0, dtype=torch.complex64, device="cuda")
        R.pair_contract(A.view(-1), B.view(-1), st.labels_a, st.labels_b, st.labels_c, C_out=C.view(-1), kernel=kernel, **args)
        assert bool((C[:, 1 << (m + n):] == 5.0).all())
        return C[:, :1 << (m + n)]

    got, ref = run(-1), run(1)
    assert not torch.equal(got, ref)
    for j in range(nb):
        a = A[0 if shared == "a" else j].to(torch.complex128)[_index(st.labels_a, ms + ks)].view(1 << m, -1)
        b = B[0 if shared == "b" else j].to(torch.complex128)[_index(st.labels_b, ks + ns)].view(1 << k, -1)
        exact = (a @ b).view(-1)[_index(ms + ns, st.labels_c)]
        rms = exact.abs().square().mean().sqrt().item()
        assert (got[j] - exact).abs().max().item() <= 6 * 2.0 ** -24 * (2.0 ** k / 2) ** 0.5 * rms, j
    row = _index(ms + ks, st.labels_a).argsort()[:1 << k]  # row 0 of A
    A[-1, row[1:]] = 0
    assert torch.equal(torch.view_as_real(run(-1)), torch.view_as_real(run(1)))

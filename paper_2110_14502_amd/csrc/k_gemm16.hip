// FP16 / BF16 matrix-core GEMM for long sums (two-phase reduced-precision
// contraction, Sections 5.4 and 5.5).
#include "frag_gemm.h"

namespace rqc {

// ---------------------------------------------------------------------------
// When a step sums over many indices its arithmetic outweighs its operand
// traffic by orders of magnitude, and the 16-bit matrix cores (16 times the
// FP32 rate) are limited by how fast operands reach them, not by HBM.  Such
// a step runs in two phases: each operand is permuted into fragments of
// 16-bit real and imaginary parts (this file), then multiplied by the GEMM of
// frag_gemm.h, which writes C in its own layout through per-row and per-column
// offset tables.  The extra traffic (read 8 B, write 4 B per operand element)
// is small against 8 MNK flops.
// (m, n, k) = (14, 13, 13) in BF16: 8.65 ms with packed (re, im) words, B's real
// expansion formed per lane and operands staged through registers (GEMM 7.82
// ms, 1125 TFLOP/s); 7.23 ms now (GEMM 6.75, 1300 TFLOP/s; a vendor BF16
// product of 16384^3 reaches 1353 on this card).
// ---------------------------------------------------------------------------
template <int LP>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  if constexpr (LP == ST_F16) {
    h2 v;
    v.x = (_Float16)a;
    v.y = (_Float16)b;
    return __builtin_bit_cast(uint32_t, v);
  } else {
    b2 v;
    v.x = (__bf16)a;
    v.y = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
  }
}

template <int LP>
__global__ __launch_bounds__(256) void k_pack16(const float2* in, char* out, PermTiles p,
                                                uint32_t n_iter) {
  permute_tiles(in, p, blockIdx.x, n_iter, [&](int64_t o, float2 a, float2 b, float2 c, float2 e) {
    char* dst = out + frag_at(o);
    *reinterpret_cast<uint2*>(dst) = make_uint2(pack2<LP>(a.x, b.x), pack2<LP>(c.x, e.x));
    *reinterpret_cast<uint2*>(dst + kFragBytes) = make_uint2(pack2<LP>(a.y, b.y), pack2<LP>(c.y, e.y));
  });
}

hipError_t launch_pack16(const void* in, char* out, int rank, const int8_t* src_of_out, int lp_kind,
                         hipStream_t s) {
  PermTiles t;
  uint32_t grid, n_iter;
  if (!plan_permute_tiles(rank, src_of_out, t, grid, n_iter)) return hipErrorInvalidValue;
  t.aligned = (reinterpret_cast<uintptr_t>(in) & 15) == 0;
  const float2* src = static_cast<const float2*>(in);
  if (lp_kind == ST_F16)
    hipLaunchKernelGGL(k_pack16<ST_F16>, dim3(grid), dim3(256), 0, s, src, out, t, n_iter);
  else if (lp_kind == ST_BF16)
    hipLaunchKernelGGL(k_pack16<ST_BF16>, dim3(grid), dim3(256), 0, s, src, out, t, n_iter);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Split-K partials summed in split order (the result does not depend on
// timing) and written to C in its layout: one thread per output element.
__global__ __launch_bounds__(256) void k_gemm16_reduce(FragDesc d) {
  if (d.hdr && d.hdr->flag) return;  // the FP32 kernel takes the product
  const uint64_t per = uint64_t(1) << (d.m + d.n);
  const uint64_t total = per * (uint64_t)d.copies;
  const int S = 1 << d.ksplit;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t copy = e >> (d.m + d.n), rc = e & (per - 1);
    const uint64_t r = rc >> d.n, c = rc & ((uint64_t(1) << d.n) - 1);
    const float2* p = d.P + ((copy << d.ksplit) << (d.m + d.n)) + rc;
    float2 v = p[0];
    for (int s = 1; s < S; ++s) {
      const float2 w = p[(uint64_t)s << (d.m + d.n)];
      v.x += w.x;
      v.y += w.y;
    }
    int64_t o = (int64_t)copy * d.sC;
    for (int b = 0; b < d.m; ++b)
      if ((r >> b) & 1) o += int64_t(1) << d.crow[b];
    for (int b = 0; b < d.n; ++b)
      if ((c >> b) & 1) o += int64_t(1) << d.ccol[b];
    reinterpret_cast<float2*>(d.C)[o] = v;
  }
}

hipError_t launch_gemm16(const FragDesc& d, int lp_kind, hipStream_t s) {
  hipError_t e = hipErrorInvalidValue;
  if (lp_kind == ST_F16) e = launch_frag_gemm<1, ST_F16>(d, s);
  if (lp_kind == ST_BF16) e = launch_frag_gemm<1, ST_BF16>(d, s);
  return e != hipSuccess || !d.ksplit ? e : launch_gemm16_reduce(d, s);
}

hipError_t launch_gemm16_reduce(const FragDesc& d, hipStream_t s) {
  const uint64_t total = (uint64_t)d.copies << (d.m + d.n);
  const uint64_t blocks = (total + 255) / 256;
  hipLaunchKernelGGL(k_gemm16_reduce, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0,
                     s, d);
  return hipGetLastError();
}

}  // namespace rqc

// FP32 contraction with long sums on the FP16 matrix cores: every FP32 value
// as the sum of two FP16 values, three products per FP32 product.
#include "frag_gemm.h"

namespace rqc {

// ---------------------------------------------------------------------------
// The FP32 matrix cores peak at 157 TFLOP/s, the FP16 ones at 2.5 PFLOP/s.  A
// long sum in FP32 is bound by the former, so it is computed as
//     a = a_h + a_l,  b = b_h + b_l  (FP16 halves of the scaled FP32 values),
//     a b ~ a_h b_h + a_h b_l + a_l b_h   (FP32 accumulation),
// with a complex product as three real ones, in the form that needs only two
// accumulators:
//     X = (ar + ai) br,  Y = X + ar (bi - br),  X = X - ai (br + bi):
// X is Re C and Y is Im C.  18 FP16 flops per complex multiply-add against 6
// on the FP32 cores, at 16 times their rate.
//
// Precision.  The operand is scaled by one power of two so that its largest
// component lies in (2^13, 2^14]; two halves then keep 22-23 bits of every
// component above 2^-16 of the largest, and 2^-25 absolute below.  The packing
// kernel checks every element: if one would lose more than 2^-20 of its own
// magnitude (a range above 2^18 inside one operand), or the operand holds an
// infinity or a NaN, or its largest value lies outside 2^+-100, a flag sends
// the whole product to the FP32 kernel (launched behind this one; it returns
// at once when the flag is clear).  The sum itself has 6 accumulations per 16
// terms against 16 on the FP32 cores, and no a_l b_l term (2^-24 at most), so
// for the sums that take this path (256 terms and more) the error against 64
// bits is smaller than the FP32 kernel's.  Measured on complex normal operands
// (2-norm, this form / FP32 kernel): 3.3e-7 / 4.1e-7 at 2^8 terms, 4.5e-7 to
// 6.2e-7 / 8.1e-7 at 2^10, 1.25e-6 / 1.62e-6 at 2^12, 1.9e-6 / 3.2e-6 at 2^14
// (with split sums, which add shorter partials, 0.5e-6).
//
// Steps: (1) largest components, per workgroup; (2) packing: each operand is
// permuted (the tile walk of the permutation kernel) into fragments of its high
// and low parts, three planes (ar + ai, ar, -ai; br, bi - br, br + bi); (3) the
// GEMM of frag_gemm.h, which writes C in its own layout.
// (m, n, k) = (14, 12, 12): 13.80 ms on the FP32 cores, 4.92 here (maxima 0.14,
// packing 0.30, GEMM 4.47: 1110 TFLOP/s executed, 447 algorithmic).
// ---------------------------------------------------------------------------
constexpr int kAbsParts = kSplitParts;  // workgroups of the maximum; 256 threads read four each
static_assert(kAbsParts == 1024, "k_split_pack reads four partial maxima per thread");

// Largest |component| (as bits; NaN and infinity compare above all finite
// values) over n float4 per workgroup; clears the operand's flag.
__global__ __launch_bounds__(256) void k_split_absmax(const uint4* x, uint64_t n, uint32_t* part,
                                                      int32_t* flag) {
  uint32_t m = 0;
#pragma unroll 4
  for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += kAbsParts * 256ull) {
    const uint4 v = x[i];
    const uint32_t a = max(v.x & 0x7fffffffu, v.y & 0x7fffffffu);
    const uint32_t b = max(v.z & 0x7fffffffu, v.w & 0x7fffffffu);
    m = max(m, max(a, b));
  }
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  __shared__ uint32_t w[4];
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    part[blockIdx.x] = max(max(w[0], w[1]), max(w[2], w[3]));
    if (blockIdx.x == 0) *flag = 0;
  }
}

// Two halves of four scaled values; the four high halves and the four low
// halves as 8-byte words.
struct Halves {
  uint2 hi, lo;
};
__device__ __forceinline__ Halves split4(float a, float b, float c, float e) {
  const float x[4] = {a, b, c, e};
  h2 h[2], l[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const _Float16 hi = (_Float16)x[i];
    const _Float16 lo = (_Float16)(x[i] - (float)hi);
    h[i >> 1][i & 1] = hi;
    l[i >> 1][i & 1] = lo;
  }
  return Halves{make_uint2(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1])),
                make_uint2(__builtin_bit_cast(uint32_t, l[0]), __builtin_bit_cast(uint32_t, l[1]))};
}

// Packs one operand.  B: the right operand's planes.
template <bool B>
__global__ __launch_bounds__(256) void k_split_pack(const float2* in, char* out, int64_t plane,
                                                    PermTiles p, uint32_t n_iter,
                                                    const uint32_t* part, int32_t* flag,
                                                    int32_t* scale_exp) {
  __shared__ uint32_t red[4];
  const int tid = threadIdx.x;
  const uint4 q = reinterpret_cast<const uint4*>(part)[tid];
  uint32_t mx = max(max(q.x, q.y), max(q.z, q.w));
  for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = max(max(red[0], red[1]), max(red[2], red[3]));
  const float big = __uint_as_float(mx);
  // (a NaN fails both comparisons)
  if (mx != 0 && !(big > 0x1p-100f && big < 0x1p100f)) {
    if (tid == 0) *flag = 1;
    return;
  }
  const int sh = mx ? 14 - ceil_log2(big) : 0;
  if (blockIdx.x == 0 && tid == 0) *scale_exp = sh;
  const float sc = ldexpf(1.f, sh);
  int wide = 0;  // an element that two halves do not hold to 2^-20
  permute_tiles(in, p, n_iter, [&](int64_t o, float2 a, float2 b, float2 c, float2 e) {
    const float2 v[4] = {a, b, c, e};
    float re[4], im[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re[i] = v[i].x * sc;
      im[i] = v[i].y * sc;
      const float rr = re[i] - (float)(_Float16)re[i], ri = im[i] - (float)(_Float16)im[i];
      const float er = fabsf(rr - (float)(_Float16)rr), ei = fabsf(ri - (float)(_Float16)ri);
      if (fmaxf(er, ei) > 0x1p-20f * fmaxf(fabsf(re[i]), fabsf(im[i]))) wide = 1;
    }
    char* dst = out + frag_at(o);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (B) x[i] = t == 0 ? re[i] : (t == 1 ? im[i] - re[i] : re[i] + im[i]);
        else x[i] = t == 0 ? re[i] + im[i] : (t == 1 ? re[i] : -im[i]);
      }
      const Halves h = split4(x[0], x[1], x[2], x[3]);
      *reinterpret_cast<uint2*>(dst + t * plane) = h.hi;
      *reinterpret_cast<uint2*>(dst + t * plane + kFragBytes) = h.lo;
    }
  });
  if (wide) *flag = 1;
}

hipError_t launch_split_pack(const void* in, char* out, int rank, const int8_t* src_of_out,
                             int64_t plane, bool right, uint32_t* part, int32_t* flag,
                             int32_t* scale_exp, hipStream_t s) {
  PermTiles t;
  uint32_t grid, n_iter;
  if (rank < kPermBits || !plan_permute_tiles(rank, src_of_out, t, grid, n_iter))
    return hipErrorInvalidValue;
  t.aligned = 1;  // (the maximum reads 16-byte words: the caller checks)
  const float2* src = static_cast<const float2*>(in);
  hipLaunchKernelGGL(k_split_absmax, dim3(kAbsParts), dim3(256), 0, s,
                     static_cast<const uint4*>(in), uint64_t(1) << (rank - 1), part, flag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (right)
    hipLaunchKernelGGL(k_split_pack<true>, dim3(grid), dim3(256), 0, s, src, out, plane, t, n_iter,
                       part, flag, scale_exp);
  else
    hipLaunchKernelGGL(k_split_pack<false>, dim3(grid), dim3(256), 0, s, src, out, plane, t, n_iter,
                       part, flag, scale_exp);
  return hipGetLastError();
}

hipError_t launch_split_gemm(const FragDesc& d, hipStream_t s) {
  const hipError_t e = launch_frag_gemm<0, ST_F16>(d, s);
  return e != hipSuccess || !d.ksplit ? e : launch_gemm16_reduce(d, s);
}

}  // namespace rqc

// FP32 contraction with long sums on the FP16 matrix cores: every FP32 value
// as the sum of two FP16 values, three products per FP32 product.
#include <algorithm>

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
// Precision.  Each copy of an operand is scaled by one power of two so that its
// largest component lies in (2^13, 2^14]; two halves then keep 22-23 bits of every
// component above 2^-16 of the largest, and 2^-25 absolute below, and there is no
// a_l b_l term (2^-24 at most).  The sum itself has 6 accumulations per 16 terms
// against 16 on the FP32 cores.  So over many comparable terms the error against
// 64 bits is below the FP32 kernel's, and over few, or where a few dominate, above
// it (1.9-2.0 times with up to a quarter of the terms nonzero).  Therefore the
// operands are looked at, row by row of A and column by column of B, and a flag
// sends the whole call to the FP32 kernel (launched behind this one; it returns
// at once when the flag is clear) unless every one is dense and even, with
// moduli r over the 2^k terms and r0 their root mean square:
//   (mean r)^2 >= 11/16 r0^2 and mean log r^2 >= log r0^2 - 1, at 2^8 terms - 1.15
//   (complex normal values: 0.785 and -0.577; an eighth of the terms missing, or
//   normal values that drift by a factor of four over the sum, fail one of them);
//   largest r^2 <= 28 r0^2, at 2^8 terms 20 (exceeded by normal values once in
//   10^12 and in 10^8 to 10^9);
//   real and imaginary parts at least 1/64 of r0^2 each (the form does not keep
//   an exactly zero part of C, as the FP32 kernel does for real operands);
//   the modulus of the mean value squared at most 3/4 r0^2 (the rounding errors of
//   nearly equal terms all add up: 0.1 to 1.5 times the FP32 kernel's);
//   r0 at least 2^-14 of the operand's largest component.
// It is raised also by an element that loses more than 2^-18 of itself (one below
// 2^-21 of the largest; what smaller losses add is 2^-25 of r0 and less, and a
// tighter limit met a normal value in one product of 2^27 elements in a hundred), an
// infinity, a NaN, or a largest component outside 2^+-100.  Rows and columns that are zero are
// exact and pass.
// Error against 64 bits of the rows and columns of C over the FP32 kernel's (median):
// complex normal operands 0.80 at 2^8 terms, 0.77 at 2^10, 0.39 at 2^12 (with split
// sums); terms growing by a factor of two over the sum 0.93 to 0.97; one term of four
// times the others in both operands, the last of the sum, 1.02 at 2^8 terms, 0.82 at
// 2^10.  The largest of operands that pass: 1.19, equal moduli growing by a factor of
// four over 2^8 terms (single rows reach 1.3 there, and 1.5 with a last term of 4.4 times).
//
// Steps, each one launch for all copies: (1) largest components and
// zeros, per workgroup; (2) packing: the operands are permuted (the tile walk of the permutation kernel)
// into fragments of their high and low parts, three planes (ar + ai, ar, -ai; br, bi
// - br, br + bi); (3) the look at rows and columns, from the packed high parts;
// (4) the GEMM of frag_gemm.h, which writes C in its own layout.
// (m, n, k) = (14, 12, 12): 13.9 ms on the FP32 cores (12.2 with operands that are
// copied straight into LDS), 4.85 here (first look 0.11, packing 0.31, rows and
// columns 0.11, GEMM 4.3 to 4.5: 1110 TFLOP/s executed, 447 algorithmic); 14.4 where
// an operand is sent back.  Bound by the matrix cores at the clock the power limit
// allows; small products by the launches (77 us for one tile).
// ---------------------------------------------------------------------------
struct SplitOp {
  const char* in;
  char* out;
  int64_t stride_in, stride_out, plane;  // bytes
  struct SplitStat* part;
  int32_t* exps;
  int32_t rank, copies, parts_log2;
  uint32_t n_iter;
  PermTiles t;
};
struct SplitArgs {
  SplitOp op[2];  // A, B
  int32_t* flag;
  int32_t k;
};

// What a first look at every element tells: the largest |re| and |im| (as bits; NaN
// and infinity compare above all finite values) and the number of zeros.
struct SplitStat {
  uint32_t re, im, zeros, pad;
};
__device__ __forceinline__ SplitStat stat_join(const SplitStat& a, const SplitStat& b) {
  return SplitStat{max(a.re, b.re), max(a.im, b.im), a.zeros + b.zeros, 0};
}
// Over 256 threads; the same in every thread.
__device__ __forceinline__ SplitStat stat_block(SplitStat v) {
  __shared__ SplitStat w[4];
  for (int o = 32; o > 0; o >>= 1)
    v = stat_join(v, SplitStat{(uint32_t)__shfl_xor((int)v.re, o, 64), (uint32_t)__shfl_xor((int)v.im, o, 64),
                               (uint32_t)__shfl_xor((int)v.zeros, o, 64), 0});
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = v;
  __syncthreads();
  return stat_join(stat_join(w[0], w[1]), stat_join(w[2], w[3]));
}

// Per workgroup and copy; clears the flag.
__global__ __launch_bounds__(256) void k_split_first(SplitArgs a) {
  const int which = (int)blockIdx.y < a.op[0].copies ? 0 : 1;
  const SplitOp& q = a.op[which];
  const int copy = (int)blockIdx.y - (which ? a.op[0].copies : 0);
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *a.flag = 0;
  if (blockIdx.x >> q.parts_log2) return;
  const uint4* x = reinterpret_cast<const uint4*>(q.in + copy * q.stride_in);
  const uint64_t n = uint64_t(1) << (q.rank - 1), step = uint64_t(256) << q.parts_log2;
  SplitStat m{0, 0, 0, 0};
#pragma unroll 4
  for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += step) {
    const uint4 v = x[i];
    const uint32_t r0 = v.x & 0x7fffffffu, i0 = v.y & 0x7fffffffu, r1 = v.z & 0x7fffffffu, i1 = v.w & 0x7fffffffu;
    m = stat_join(m, SplitStat{max(r0, r1), max(i0, i1), (uint32_t)((r0 | i0) == 0) + (uint32_t)((r1 | i1) == 0), 0});
  }
  m = stat_block(m);
  if (threadIdx.x == 0) q.part[(copy << q.parts_log2) + blockIdx.x] = m;
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

// Packs both operands: the workgroups of A's copies, then of B's.
__global__ __launch_bounds__(256) void k_split_pack(SplitArgs a) {
  const uint32_t n_a = (uint32_t)a.op[0].copies << a.op[0].t.gbits;
  const int which = blockIdx.x < n_a ? 0 : 1;
  const SplitOp& q = a.op[which];
  const uint32_t at = blockIdx.x - (which ? n_a : 0);
  const int copy = (int)(at >> q.t.gbits);
  const int tid = threadIdx.x;
  SplitStat m{0, 0, 0, 0};
  for (int i = tid; i < 1 << q.parts_log2; i += 256) m = stat_join(m, q.part[(copy << q.parts_log2) + i]);
  m = stat_block(m);
  const uint32_t mx = max(m.re, m.im);
  const float big = __uint_as_float(mx);
  // (A NaN fails both comparisons.)  More than an eighth of the elements zero means
  // rows with as many, and a real or imaginary operand fails the look in every row:
  // those are not packed.
  if (mx != 0 && (!(big > 0x1p-100f && big < 0x1p100f) || m.re == 0 || m.im == 0 ||
                  m.zeros > 1u << (q.rank - 3))) {
    if (tid == 0) *a.flag = 1;
    return;
  }
  const int sh = mx ? 14 - ceil_log2(big) : 0;
  const uint32_t block = at & ((1u << q.t.gbits) - 1);
  if (block == 0 && tid == 0) q.exps[copy] = sh;
  const float sc = ldexpf(1.f, sh);
  int wide = 0;  // an element that two halves do not hold to 2^-18
  char* const out = q.out + copy * q.stride_out;
  const int64_t plane = q.plane;
  permute_tiles(reinterpret_cast<const float2*>(q.in + copy * q.stride_in), q.t, block, q.n_iter,
                [&](int64_t o, float2 e0, float2 e1, float2 e2, float2 e3) {
    const float2 v[4] = {e0, e1, e2, e3};
    float re[4], im[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re[i] = v[i].x * sc;
      im[i] = v[i].y * sc;
      const float rr = re[i] - (float)(_Float16)re[i], ri = im[i] - (float)(_Float16)im[i];
      const float er = fabsf(rr - (float)(_Float16)rr), ei = fabsf(ri - (float)(_Float16)ri);
      if (fmaxf(er, ei) > 0x1p-18f * fmaxf(fabsf(re[i]), fabsf(im[i]))) wide = 1;
    }
    char* dst = out + frag_at(o);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (which) x[i] = t == 0 ? re[i] : (t == 1 ? im[i] - re[i] : re[i] + im[i]);
        else x[i] = t == 0 ? re[i] + im[i] : (t == 1 ? re[i] : -im[i]);
      }
      const Halves h = split4(x[0], x[1], x[2], x[3]);
      *reinterpret_cast<uint2*>(dst + t * plane) = h.hi;
      *reinterpret_cast<uint2*>(dst + t * plane + kFragBytes) = h.lo;
    }
  });
  if (wide) *a.flag = 1;
}

// The look at rows and columns: a workgroup takes 8 rows of one copy of A, or 8
// columns of B, its waves every 8th group of 64 terms; a lane reads 8 terms of one
// row at a time.  Bound by the reads of a third of the packed bytes.
constexpr int kSplitLookWaves = 8;
struct RowSums {
  float re, im, re2, im2, r, lg, top;  // sums of re, im, re^2, im^2, r and log2 r^2; largest r^2
  __device__ __forceinline__ void add(const RowSums& o) {
    re += o.re, im += o.im, re2 += o.re2, im2 += o.im2, r += o.r, lg += o.lg;
    top = fmaxf(top, o.top);
  }
};
__global__ __launch_bounds__(64 * kSplitLookWaves) void k_split_look(SplitArgs a) {
  if (*a.flag) return;
  const int b0 = a.op[0].rank - a.k - 3;  // log2 workgroups per copy of A
  const uint32_t n_a = (uint32_t)a.op[0].copies << b0;
  const int which = blockIdx.x < n_a ? 0 : 1;
  const SplitOp& q = a.op[which];
  const uint32_t at = blockIdx.x - (which ? n_a : 0);
  const int bits = q.rank - a.k - 3;
  const int copy = (int)(at >> bits);
  const uint32_t grp = at & ((1u << bits) - 1);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Fragments of 16 terms: [8-term half][32 rows][8 terms] of the high parts, then
  // of the low ones.
  const char* src = q.out + copy * q.stride_out + ((int64_t)(grp >> 2) << (a.k + 7)) +
                    (int64_t)(lane >> 4) * 2 * kFragBytes + ((lane >> 3) & 1) * (kFragBytes / 2) +
                    ((grp & 3) * 8 + (lane & 7)) * 16;
  RowSums v{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int c = wave; c < 1 << (a.k - 6); c += kSplitLookWaves) {
    const frag_u4 w1 = *reinterpret_cast<const frag_u4*>(src + q.plane + (int64_t)c * 8 * kFragBytes);
    const frag_u4 w2 = *reinterpret_cast<const frag_u4*>(src + 2 * q.plane + (int64_t)c * 8 * kFragBytes);
    const frag_h8 x1 = __builtin_bit_cast(frag_h8, w1), x2 = __builtin_bit_cast(frag_h8, w2);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // A: ar, -ai; B: bi - br, br + bi.
      const float y1 = (float)x1[i], y2 = (float)x2[i];
      const float re = which ? 0.5f * (y2 - y1) : y1, im = which ? 0.5f * (y1 + y2) : y2;
      const float r2 = re * re + im * im;
      v.re += re;
      v.im += im;
      v.re2 += re * re;
      v.im2 += im * im;
      v.r += __builtin_amdgcn_sqrtf(r2);
      v.lg += __builtin_amdgcn_logf(fmaxf(r2, 0x1p-14f));
      v.top = fmaxf(v.top, r2);
    }
  }
  for (int o = 8; o < 64; o <<= 1)
    v.add(RowSums{__shfl_xor(v.re, o, 64), __shfl_xor(v.im, o, 64), __shfl_xor(v.re2, o, 64), __shfl_xor(v.im2, o, 64), __shfl_xor(v.r, o, 64),
                  __shfl_xor(v.lg, o, 64), __shfl_xor(v.top, o, 64)});
  __shared__ RowSums part[kSplitLookWaves][8];
  if (lane < 8) part[wave][lane] = v;
  __syncthreads();
  if (tid >= 8) return;
  v = part[0][tid];
  for (int w = 1; w < kSplitLookWaves; ++w) v.add(part[w][tid]);
  const float K = ldexpf(1.f, a.k), S = v.re2 + v.im2;  // S: K times the mean r^2
  const float lg = a.k > 8 ? 1.4427f : 1.6591f, top = a.k > 8 ? 28.f : 20.f;  // (base 2)
  const bool even = v.r * v.r * 16.f >= 11.f * K * S && v.lg >= K * (__builtin_amdgcn_logf(S / K) - lg) &&
                    v.top * K <= top * S && fminf(v.re2, v.im2) * 64.f >= S &&
                    (v.re * v.re + v.im * v.im) * 4.f <= 3.f * K * S && S >= K;
  if (S != 0.f && !even) *a.flag = 1;
}

hipError_t launch_split_pack(const SplitOperand& A, const SplitOperand& B, int k, SplitHdr* hdr,
                             hipStream_t s) {
  SplitArgs a{};
  a.flag = &hdr->flag;
  a.k = k;
  uint32_t parts = 0, pack = 0, look = 0, copies = 0;
  for (int i = 0; i < 2; ++i) {
    const SplitOperand& x = i ? B : A;
    SplitOp& q = a.op[i];
    uint32_t grid;
    if (x.copies < 1 || x.copies > kSplitCopies || k < 8 || x.rank - k < 5 ||
        ((uintptr_t)x.in | (uintptr_t)(8 * x.stride_in)) % 16 ||
        !plan_permute_tiles(x.rank, x.src_of_out, q.t, grid, q.n_iter))
      return hipErrorInvalidValue;
    q.t.aligned = 1;
    q.in = static_cast<const char*>(x.in);
    q.out = x.out;
    q.stride_in = 8 * x.stride_in, q.stride_out = x.stride_out, q.plane = x.plane;
    q.part = static_cast<SplitStat*>(x.part);
    q.exps = i ? hdr->exp_b : hdr->exp_a;
    q.rank = x.rank, q.copies = x.copies;
    // Eight 16-byte words and more per thread of the maximum; at most 1024
    // workgroups for all copies (a packing workgroup that walks one tile only
    // does not repay its start: (8, 7, 13) x 32 took 1.80 ms with one, 0.92
    // with 16).
    q.parts_log2 = x.rank - 12 < 10 ? x.rank - 12 : 10;
    static_assert(kSplitParts * sizeof(SplitStat) == kSplitPartBytes && kSplitParts == 1 << 10, "partial results");
    while (q.parts_log2 > 0 && (x.copies << q.parts_log2) > 1024) --q.parts_log2;
    for (; q.t.gbits > 0 && (x.copies << q.t.gbits) > 1024; --q.t.gbits) q.n_iter *= 2;
    parts = std::max(parts, 1u << q.parts_log2);
    copies += (uint32_t)x.copies;
    pack += (uint32_t)x.copies << q.t.gbits;
    look += (uint32_t)x.copies << (x.rank - k - 3);
  }
  hipLaunchKernelGGL(k_split_first, dim3(parts, copies), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_split_pack, dim3(pack), dim3(256), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_split_look, dim3(look), dim3(64 * kSplitLookWaves), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_split_gemm(const FragDesc& d, hipStream_t s) {
  const hipError_t e = launch_frag_gemm<0, ST_F16>(d, s);
  return e != hipSuccess || !d.ksplit ? e : launch_gemm16_reduce(d, s);
}

}  // namespace rqc

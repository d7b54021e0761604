// FP32 contraction with long sums on the FP16 matrix cores: every FP32 value
// as the sum of two FP16 values, three products per FP32 product.
#include "permute_tiles.h"

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
// permuted (the tile walk of the permutation kernel) into the fragments the
// matrix instructions read: for a block of 32 rows and 16 summed indices, 1 KB
// [8-term half][row][8 terms] of the high parts, then of the low parts, three
// planes (ar + ai, ar, -ai; br, bi - br, br + bi); (3) the GEMM: fragments go
// from memory to LDS and from LDS to registers as straight 16-byte copies,
// without padding or bank conflicts; C is written in its own layout.
// The GEMM is bound by the matrix cores under the card's power limit: its
// matrix pipe is busy 0.52-0.54 of the cycles at a clock of 1.65 GHz, and data
// from the nearest cache instead of memory make it 9% faster.  (m, n, k) = (14,
// 12, 12): 13.80 ms on the FP32 cores, 5.31 here (maxima 0.14, packing 0.30,
// GEMM 4.86: 1020 TFLOP/s executed, 415 algorithmic).
// ---------------------------------------------------------------------------
typedef _Float16 s32_h8 __attribute__((ext_vector_type(8)));
typedef unsigned int s32_u4 __attribute__((ext_vector_type(4)));

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

// Packs one operand.  The permutation's output order is the fragments': terms
// 0-2, rows 0-4, term 3, term 4, ..., rows 5, ...  B: the right operand's
// planes.
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
    // Output element o: fragment o >> 9, byte 2 (o & 511) of its halves.
    char* dst = out + ((o >> 9) << 11) + 2 * (o & 511);
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
      *reinterpret_cast<uint2*>(dst + t * plane + 1024) = h.lo;
    }
  });
  if (wide) *flag = 1;
}

// ---------------------------------------------------------------------------
// The GEMM.  Tile 256 rows x 128 columns, 8 waves as 4 x 2, each 64 x 64 as
// 2 x 2 blocks of v_mfma_f32_32x32x16_f16 on two accumulator sets (X, Y); 32
// summed indices per LDS chunk (48 KB), two LDS buffers and two register sets
// (two chunks in flight), one barrier per chunk.  The chunks of the three
// planes form one stream.  Per 16 terms a wave reads 8 fragments (8 KB) for 12
// matrix instructions.  Workgroup order as in the 16-bit GEMM: contiguous
// ranges per XCD, tiles in groups of 8 row tiles; split sums for outputs with
// few tiles.
// ---------------------------------------------------------------------------
constexpr int kS32Frag = 1024;                       // bytes of one fragment half
constexpr int kS32Blk = 4 * kS32Frag;                // one row block of a chunk: 2 x (hi, lo)
constexpr int kS32ABuf = kSplitM / 32 * kS32Blk;     // 32 KB
constexpr int kS32BBuf = kSplitN / 32 * kS32Blk;     // 16 KB

constexpr int kS32Buf = kS32ABuf + kS32BBuf;

// 16 bytes per lane from memory to LDS: lane i's go to LDS byte dst + 16 i (dst
// uniform).  In assembly because the compiler waits for every copy in flight
// before any LDS read when it places the waits itself; the kernel's own wait
// before the barrier covers them.  No vector register is written; M0, the LDS
// address, has no other use in this kernel and must be set one wait state ahead.
__device__ __forceinline__ void s32_copy(const char* src, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(
                   __builtin_amdgcn_readfirstlane(dst)),
               "v"(src)
               : "memory");
}

__device__ __forceinline__ floatx16 s32_mfma(s32_u4 a, s32_u4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(s32_h8, a),
                                                __builtin_bit_cast(s32_h8, b), c, 0, 0, 0);
}

__global__ __launch_bounds__(512, 1) void k_split_gemm(SplitDesc d) {
  __shared__ __attribute__((aligned(16))) char lds[3 * kS32Buf];
  __shared__ int64_t roff[kSplitM];
  __shared__ int64_t coff[kSplitN];
  if (d.hdr->flag_a | d.hdr->flag_b) return;  // the FP32 kernel takes the product
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const uint64_t T = gridDim.x;
  uint64_t L = blockIdx.x;
  if ((T & 7) == 0) L = (L & 7) * (T >> 3) + (L >> 3);
  const int rbits = d.m - 8, cbits = d.n - 7;
  const uint64_t l = L & ((uint64_t(1) << (rbits + cbits)) - 1);
  const uint64_t ks = L >> (rbits + cbits);
  const int gr = rbits < 3 ? rbits : 3;
  const uint64_t grp = l >> (gr + cbits);
  const uint64_t in = l & ((uint64_t(1) << (gr + cbits)) - 1);
  const uint64_t rt = (grp << gr) | (in & ((uint64_t(1) << gr) - 1));
  const uint64_t ct = in >> gr;

  if (tid < kSplitM) {
    const uint64_t r = (rt << 8) | (uint64_t)tid;
    int64_t o = 0;
    if (d.ksplit)
      o = (int64_t)r << d.n;
    else
      for (int b = 0; b < d.m; ++b)
        if ((r >> b) & 1) o += int64_t(1) << d.crow[b];
    roff[tid] = o;
  } else if (tid < kSplitM + kSplitN) {
    const uint64_t c = (ct << 7) | (uint64_t)(tid - kSplitM);
    int64_t o = 0;
    if (d.ksplit)
      o = (int64_t)c;
    else
      for (int b = 0; b < d.n; ++b)
        if ((c >> b) & 1) o += int64_t(1) << d.ccol[b];
    coff[tid - kSplitM] = o;
  }

  // Chunk q of the stream: plane q >> lg, chunk q & (n_kc - 1) of this split.
  const int lg = __builtin_amdgcn_readfirstlane(d.k - 5 - d.ksplit);
  const int n_kc = 1 << lg, n_q = 3 << lg;
  const int64_t blk = int64_t(kS32Blk) << (d.k - 5);  // bytes of a 32-row block over the whole sum
  // Half `sub` (16 terms) of chunk q: 16 KB of A and 8 KB of B, copied straight
  // into LDS in pieces of 1 KB (a block's high or low parts), three per wave.
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  const int64_t piece = (int64_t)(wv >> 1) * blk + (int64_t)(ks << lg) * kS32Blk + (wv & 1) * kS32Frag;
  const char* At = d.A + (int64_t)(rt * (kSplitM / 32)) * blk + piece + lane * 16;
  const char* Bt = d.B + (int64_t)(ct * (kSplitN / 32)) * blk + piece + lane * 16;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds +
                        (uint32_t)((wv >> 1) * kS32Blk + (wv & 1) * kS32Frag);
  auto fetch = [&](int q, int sub, int buf) {
    const int64_t at = (int64_t)(q & (n_kc - 1)) * kS32Blk + sub * 2 * kS32Frag;
    const char* a = At + (q >> lg) * d.plane_a + at;
    const char* b = Bt + (q >> lg) * d.plane_b + at;
    const uint32_t l = lds0 + (uint32_t)(buf * kS32Buf + sub * 2 * kS32Frag);
    s32_copy(a, l);
    s32_copy(a + 4 * blk, l + 4 * kS32Blk);
    s32_copy(b, l + kS32ABuf);
  };
  fetch(0, 0, 0);
  fetch(0, 1, 0);
  fetch(1, 0, 1);
  fetch(1, 1, 1);
  fetch(2, 0, 2);

  floatx16 X[2][2], Y[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) X[i][j][r] = 0.f;

  s32_u4 a0[2][2], b0[2][2], a1[2][2], b1[2][2];  // fragments [block][hi, lo] of 16 terms
  auto frags = [&](int buf, int sub, s32_u4 (&a)[2][2], s32_u4 (&b)[2][2]) {
    const char* As = lds + buf * kS32Buf + wr * 2 * kS32Blk + lane * 16;
    const char* Bs = lds + buf * kS32Buf + kS32ABuf + wc * 2 * kS32Blk + lane * 16;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i][s] = *reinterpret_cast<const s32_u4*>(As + i * kS32Blk + (2 * sub + s) * kS32Frag);
        b[i][s] = *reinterpret_cast<const s32_u4*>(Bs + i * kS32Blk + (2 * sub + s) * kS32Frag);
      }
  };
  auto products = [&](const s32_u4 (&a)[2][2], const s32_u4 (&b)[2][2], floatx16 (&acc)[2][2]) {
#pragma unroll
    for (int s = 0; s < 3; ++s)  // a_h b_h, a_l b_h, a_h b_l
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = s32_mfma(a[i][s == 1 ? 1 : 0], b[j][s == 2 ? 1 : 0], acc[i][j]);
  };
  // Chunk q sits in LDS buffer q mod 3.  Its first half is read during chunk
  // q - 1 and its second half at its own start, so no wave starts a chunk by
  // waiting for LDS, and the halves of a buffer fall free at different
  // barriers: at chunk q's, the second half of chunk q - 1 (taken by chunk q +
  // 2) and the first half of chunk q itself (taken by chunk q + 3).  Either
  // way a copy has two chunks' time to land: the barrier waits for all but the
  // six copies issued one chunk ago.
  int buf = 0;
  auto plane = [&](int q0, floatx16 (&acc)[2][2]) {
    for (int q = q0; q < q0 + n_kc; ++q) {
      if (q + 2 < n_q) __builtin_amdgcn_s_waitcnt(0x0F76);  // vmcnt(6)
      else __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): fewer were issued
      __builtin_amdgcn_s_barrier();
      const int nb = buf == 2 ? 0 : buf + 1;
      if (q + 2 < n_q) fetch(q + 2, 1, nb == 2 ? 0 : nb + 1);
      if (q + 3 < n_q) fetch(q + 3, 0, buf);
      frags(buf, 1, a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      products(a0, b0, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (q + 1 < n_q) frags(nb, 0, a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      products(a1, b1, acc);
      __builtin_amdgcn_sched_barrier(0);
      buf = nb;
    }
  };
  // Chunk 0: its first half has landed for every wave before it is read (all
  // but the six youngest copies).
  __builtin_amdgcn_s_waitcnt(0x0F76);
  __syncthreads();
  frags(0, 0, a0, b0);
  plane(0, X);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) Y[i][j] = X[i][j];
  plane(n_kc, Y);
  plane(2 * n_kc, X);

  typedef float f2v __attribute__((ext_vector_type(2)));
  const int sh = -(d.hdr->exp_a + d.hdr->exp_b);
  f2v* Cf = d.ksplit ? reinterpret_cast<f2v*>(d.P) + ((int64_t)ks << (d.m + d.n))
                     : reinterpret_cast<f2v*>(d.C);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t co = coff[wc * 64 + j * 32 + (lane & 31)];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wr * 64 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const f2v v = {ldexpf(X[i][j][r], sh), ldexpf(Y[i][j][r], sh)};
        __builtin_nontemporal_store(v, Cf + roff[row] + co);
      }
    }
}

hipError_t launch_split_pack(const void* in, char* out, int rank, const int8_t* src_of_out,
                             int64_t plane, bool right, uint32_t* part, int32_t* flag,
                             int32_t* scale_exp, hipStream_t s) {
  PermTiles t;
  uint32_t grid, n_iter;
  if (rank < kPermBits || !plan_permute_tiles(rank, src_of_out, t, grid, n_iter))
    return hipErrorInvalidValue;
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

hipError_t launch_split_gemm(const SplitDesc& d, hipStream_t s) {
  // Three chunks at least are loaded ahead and planes start at LDS buffer 0:
  // an even number of chunks per split.
  if (d.m < 8 || d.n < 7 || d.k > 24 || d.ksplit < 0 || d.k - 5 - d.ksplit < 1 || (d.ksplit && !d.P))
    return hipErrorInvalidValue;
  const uint64_t tiles = uint64_t(1) << (d.m - 8 + d.n - 7 + d.ksplit);
  if (tiles > 0x7fffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_gemm, dim3((unsigned)tiles), dim3(512), 0, s, d);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !d.ksplit) return e;
  Gemm16Desc r{};
  r.C = d.C;
  r.m = d.m, r.n = d.n, r.k = d.k;
  r.copies = 1;
  r.ksplit = d.ksplit;
  r.P = d.P;
  for (int b = 0; b < 40; ++b) r.crow[b] = d.crow[b], r.ccol[b] = d.ccol[b];
  return launch_gemm16_reduce(r, s);
}

}  // namespace rqc

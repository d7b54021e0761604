// The matrix-core GEMM on packed fragments shared by the two-phase contractions
// (k_gemm16.hip: FP16 / BF16; k_split32.hip: FP32 as two FP16 halves).
#pragma once

#include "permute_tiles.h"

namespace rqc {

typedef _Float16 frag_h8 __attribute__((ext_vector_type(8)));
typedef __bf16 frag_b8 __attribute__((ext_vector_type(8)));
typedef unsigned int frag_u4 __attribute__((ext_vector_type(4)));

// Byte offset of element o (a multiple of 4, in the packing order: terms 0-2,
// rows 0-4, term 3, term 4, ..., rows 5, ...) in the first part's fragments;
// the second part lies kFragBytes further.
constexpr int kFragBytes = 1024;
__device__ __forceinline__ int64_t frag_at(int64_t o) { return ((o >> 9) << 11) + 2 * (o & 511); }

// ---------------------------------------------------------------------------
// GEMM of the two-phase contractions on packed fragments.  The packing kernels
// write each operand as the fragments the matrix instructions read: for a
// block of 32 rows (columns of B) and 16 summed indices, 1 KB [8-term
// half][row][8 terms] of one part of the values, then of the other; blocks of
// a row over the whole sum back to back.  Fragments go from memory to LDS and
// from LDS to registers as straight 16-byte copies, without padding, bank
// conflicts or vector instructions.
//
// Tile 256 rows x 128 columns, 8 waves as 4 x 2, each 64 x 64 as
// 2 x 2 blocks of v_mfma_f32_32x32x16_f16 on two accumulator sets (X, Y); 32
// summed indices per LDS chunk (48 KB), three LDS buffers (144 KB: one workgroup per CU), one
// barrier per chunk; the copies of the chunks ahead go out one by one between
// the matrix instructions (together at the start of a chunk they held up its
// LDS reads: 13-15% slower).  Bound by the matrix cores at the clock the power
// limit allows (1.65 GHz).  The chunks of all planes form one stream.  Per 16 terms a
// wave reads 8 fragments (8 KB) for 12 (MODE 0) or 16 (MODE 1) matrix
// instructions.
//
// Workgroup order: blocks are dealt round-robin to the 8 XCDs, so block b is
// remapped to a contiguous range of tiles per XCD; inside a copy, tiles are
// walked in groups of 4 row tiles, row tiles fastest, so the workgroups of an
// XCD that run together share 4 row panels of A and 8 column panels of B in
// that XCD's L2 (4 x 32 KB + 8 x 16 KB a chunk; groups of 8: 2% slower).  When the output has too few tiles to fill the GPU, the sum is
// split 2^ksplit ways: each split writes FP32 partials to a plain buffer and a
// second kernel adds them in split order.
// ---------------------------------------------------------------------------
constexpr int kFragBlk = 4 * kFragBytes;                // one row block of a chunk: 2 x (hi, lo)
constexpr int kFragABuf = kGemm16M / 32 * kFragBlk;     // 32 KB
constexpr int kFragBBuf = kGemm16N / 32 * kFragBlk;     // 16 KB

constexpr int kFragBuf = kFragABuf + kFragBBuf;

template <int LP>
__device__ __forceinline__ floatx16 frag_mfma(frag_u4 a, frag_u4 b, floatx16 c) {
  if constexpr (LP == ST_F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(frag_h8, a),
                                                  __builtin_bit_cast(frag_h8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(frag_b8, a),
                                                   __builtin_bit_cast(frag_b8, b), c, 0, 0, 0);
}

// MODE 0 (FP32 as two FP16 halves): fragments (high, low), three planes, per
// block pair a_h b_h + a_l b_h + a_h b_l into X, Y, X by plane, with Y = X after
// the first.  MODE 1 (16-bit complex): fragments (re, im), one plane,
// X += ar br - ai bi, Y += ar bi + ai br.
template <int MODE, int LP>
__global__ __launch_bounds__(512, 1) void k_frag_gemm(FragDesc d) {
  __shared__ __attribute__((aligned(16))) char lds[3 * kFragBuf];
  __shared__ int64_t roff[kGemm16M];
  __shared__ int64_t coff[kGemm16N];
  if (MODE == 0 && d.hdr->flag) return;  // the FP32 kernel takes the product
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const uint64_t T = gridDim.x;
  uint64_t L = blockIdx.x;
  if ((T & 7) == 0) L = (L & 7) * (T >> 3) + (L >> 3);
  const int rbits = d.m - 8, cbits = d.n - 7;
  const uint64_t l = L & ((uint64_t(1) << (rbits + cbits)) - 1);
  const uint64_t ks = (L >> (rbits + cbits)) & ((uint64_t(1) << d.ksplit) - 1);
  const int64_t copy = (int64_t)(L >> (rbits + cbits + d.ksplit));
  const int gr = rbits < 2 ? rbits : 2;
  const uint64_t grp = l >> (gr + cbits);
  const uint64_t in = l & ((uint64_t(1) << (gr + cbits)) - 1);
  const uint64_t rt = (grp << gr) | (in & ((uint64_t(1) << gr) - 1));
  const uint64_t ct = in >> gr;

  if (tid < kGemm16M) {
    const uint64_t r = (rt << 8) | (uint64_t)tid;
    int64_t o = 0;
    if (d.ksplit)
      o = (int64_t)r << d.n;
    else
      for (int b = 0; b < d.m; ++b)
        if ((r >> b) & 1) o += int64_t(1) << d.crow[b];
    roff[tid] = o;
  } else if (tid < kGemm16M + kGemm16N) {
    const uint64_t c = (ct << 7) | (uint64_t)(tid - kGemm16M);
    int64_t o = 0;
    if (d.ksplit)
      o = (int64_t)c;
    else
      for (int b = 0; b < d.n; ++b)
        if ((c >> b) & 1) o += int64_t(1) << d.ccol[b];
    coff[tid - kGemm16M] = o;
  }

  // Chunk q of the stream: plane q >> lg, chunk q & (n_kc - 1) of this split.
  const int lg = __builtin_amdgcn_readfirstlane(d.k - 5 - d.ksplit);
  const int n_kc = 1 << lg, n_q = (MODE == 0 ? 3 : 1) << lg;
  const int64_t blk = int64_t(kFragBlk) << (d.k - 5);  // bytes of a 32-row block over the whole sum
  // Half `sub` (16 terms) of chunk q: 16 KB of A and 8 KB of B, copied straight
  // into LDS in pieces of 1 KB (a block's high or low parts), three per wave.
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  const int64_t piece = (int64_t)(wv >> 1) * blk + (int64_t)(ks << lg) * kFragBlk + (wv & 1) * kFragBytes;
  const char* At = d.A + copy * d.sA + (int64_t)(rt * (kGemm16M / 32)) * blk + piece + lane * 16;
  const char* Bt = d.B + copy * d.sB + (int64_t)(ct * (kGemm16N / 32)) * blk + piece + lane * 16;
  const uint32_t lds0 = lds_address(lds) +
                        (uint32_t)((wv >> 1) * kFragBlk + (wv & 1) * kFragBytes);
  // Copy j of half `sub` of chunk q: blocks 0-3 and 4-7 of A, then B.
  auto copy1 = [&](int q, int sub, int buf, int j) {
    const int64_t at = (int64_t)(q & (n_kc - 1)) * kFragBlk + sub * 2 * kFragBytes;
    const uint32_t l = lds0 + (uint32_t)(buf * kFragBuf + sub * 2 * kFragBytes);
    if (j < 2)
      lds_copy16(At + (MODE == 0 ? (q >> lg) * d.plane_a : 0) + at + j * 4 * blk, l + j * 4 * kFragBlk);
    else
      lds_copy16(Bt + (MODE == 0 ? (q >> lg) * d.plane_b : 0) + at, l + kFragABuf);
  };
  auto fetch = [&](int q, int sub, int buf) {
    for (int j = 0; j < 3; ++j) copy1(q, sub, buf, j);
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
      for (int r = 0; r < 16; ++r) X[i][j][r] = Y[i][j][r] = 0.f;

  frag_u4 a0[2][2], b0[2][2], a1[2][2], b1[2][2];  // fragments [block][hi, lo] of 16 terms
  auto frags = [&](int buf, int sub, frag_u4 (&a)[2][2], frag_u4 (&b)[2][2]) {
    const char* As = lds + buf * kFragBuf + wr * 2 * kFragBlk + lane * 16;
    const char* Bs = lds + buf * kFragBuf + kFragABuf + wc * 2 * kFragBlk + lane * 16;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i][s] = *reinterpret_cast<const frag_u4*>(As + i * kFragBlk + (2 * sub + s) * kFragBytes);
        b[i][s] = *reinterpret_cast<const frag_u4*>(Bs + i * kFragBlk + (2 * sub + s) * kFragBytes);
      }
  };
  // One block of 16 terms into X (and, MODE 1, Y), in groups of four matrix
  // instructions with `between(g)` after group g.
  auto products = [&](const frag_u4 (&a)[2][2], const frag_u4 (&b)[2][2], floatx16 (&acc)[2][2],
                      auto between) {
    if constexpr (MODE == 0) {
#pragma unroll
      for (int s = 0; s < 3; ++s) {  // a_h b_h, a_l b_h, a_h b_l
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = frag_mfma<LP>(a[i][s == 1 ? 1 : 0], b[j][s == 2 ? 1 : 0], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        between(s);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      frag_u4 neg[2];  // -ai
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) neg[i][w] = a[i][1][w] ^ 0x80008000u;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (s == 0) X[i][j] = frag_mfma<LP>(a[i][0], b[j][0], X[i][j]);
            if (s == 1) Y[i][j] = frag_mfma<LP>(a[i][0], b[j][1], Y[i][j]);
            if (s == 2) X[i][j] = frag_mfma<LP>(neg[i], b[j][1], X[i][j]);
            if (s == 3) Y[i][j] = frag_mfma<LP>(a[i][1], b[j][0], Y[i][j]);
          }
        __builtin_amdgcn_sched_barrier(0);
        if (s < 3) between(s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Chunk q sits in LDS buffer q mod 3.  Its first half is read during chunk
  // q - 1 and its second half at its own start, so no wave starts a chunk by
  // waiting for LDS, and the halves of a buffer fall free at different
  // barriers: at chunk q's, the second half of chunk q - 1 (taken by chunk q +
  // 2) and the first half of chunk q itself (taken by chunk q + 3).  Every wave
  // waits for its own LDS reads before that barrier (lgkmcnt(0); the last ones
  // were issued twelve and more matrix instructions ago): the first half's are
  // used only behind it, where other waves already copy into the same bytes.
  // Either way a copy has two chunks' time to land: the barrier waits for all
  // but the six copies issued one chunk ago.
  int buf = 0;
  auto plane = [&](int q0, floatx16 (&acc)[2][2]) {
    for (int q = q0; q < q0 + n_kc; ++q) {
      asm volatile("" ::: "memory");  // the reads above are issued before the wait
      if (q + 2 < n_q) __builtin_amdgcn_s_waitcnt(0x0076);  // vmcnt(6) lgkmcnt(0)
      else __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0): fewer copies were issued
      plain_barrier();
      const int nb = buf == 2 ? 0 : buf + 1;
      frags(buf, 1, a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      const int b2 = nb == 2 ? 0 : nb + 1;
      products(a0, b0, acc, [&](int j) {
        if (q + 2 < n_q) copy1(q + 2, 1, b2, j);
      });
      if (q + 1 < n_q) frags(nb, 0, a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      products(a1, b1, acc, [&](int j) {
        if (q + 3 < n_q) copy1(q + 3, 0, buf, j);
      });
      buf = nb;
    }
  };
  // Chunk 0: its first half has landed for every wave before it is read (all
  // but the six youngest copies).
  __builtin_amdgcn_s_waitcnt(0x0F76);
  __syncthreads();
  frags(0, 0, a0, b0);
  plane(0, X);
  if constexpr (MODE == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) Y[i][j] = X[i][j];
    plane(n_kc, Y);
    plane(2 * n_kc, X);
  }

  typedef float f2v __attribute__((ext_vector_type(2)));
  const int sh = MODE == 0 ? -(d.hdr->exp_a[d.sA ? copy : 0] + d.hdr->exp_b[d.sB ? copy : 0]) : 0;
  f2v* Cf = d.ksplit ? reinterpret_cast<f2v*>(d.P) + ((copy << d.ksplit | (int64_t)ks) << (d.m + d.n))
                     : reinterpret_cast<f2v*>(d.C) + copy * d.sC;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t co = coff[wc * 64 + j * 32 + (lane & 31)];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wr * 64 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        f2v v = {X[i][j][r], Y[i][j][r]};
        if (MODE == 0) v = f2v{ldexpf(v[0], sh), ldexpf(v[1], sh)};
        __builtin_nontemporal_store(v, Cf + roff[row] + co);
      }
    }
}

// Launches the GEMM (and nothing else: a split sum's partials are added by
// launch_gemm16_reduce).
template <int MODE, int LP>
inline hipError_t launch_frag_gemm(const FragDesc& d, hipStream_t s) {
  // Five half chunks are fetched ahead.
  const int chunks = d.k - 5 - d.ksplit;
  if (d.m < 8 || d.n < 7 || d.m > 40 || d.n > 40 || d.k > 32 || d.copies < 1 || d.ksplit < 0 ||
      chunks < (MODE == 0 ? 0 : 2) || (d.ksplit && !d.P))
    return hipErrorInvalidValue;
  const uint64_t tiles = (uint64_t)d.copies << (d.m - 8 + d.n - 7 + d.ksplit);
  if (tiles > 0x7fffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_frag_gemm<MODE, LP>), dim3((unsigned)tiles), dim3(512), 0, s, d);
  return hipGetLastError();
}

}  // namespace rqc

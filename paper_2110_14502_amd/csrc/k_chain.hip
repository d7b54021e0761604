// Fused evaluation of small subtrees of the contraction tree.
#include "kernels_dev.h"

namespace rqc {

// ---------------------------------------------------------------------------
// A circuit's tree holds dozens of steps whose tensors are a few kilobytes.
// As launches of their own they cost 6-9 us each (one workgroup: descriptor
// and table reads, one tile, the scale epilogue) and run one after the other:
// 0.17 ms of a 4x4 call, 0.8 ms of a 32-slice 6x6 call.  Here one workgroup
// evaluates a whole subtree for one copy (slice, bitstring): the leaves are
// bound (Section 5.1) straight into LDS, every intermediate stays there, and
// only the subtree's root is written to memory; subtrees that do not depend
// on each other run side by side in one launch.  A step inside is bound by
// the LDS round trips of its chain (descriptor, operands, maximum, barrier),
// not by bandwidth or arithmetic.  Measured (whole calls): 4x4 256 -> 99 us,
// 24 bitstrings of a 5x5 circuit 715 -> 334 us, 16 FP16 slices of a 5x5
// circuit 703 -> 300 us, 32 slices of the 6x6 circuit 10.58 -> 9.70 ms in
// FP32 and 6.00 -> 5.23 ms in FP16.
//
// The arithmetic is the row kernel's, instruction for instruction (its 16 x 8
// tiles, its deal of the summed indices over the lanes and its order of
// products, the power-of-two normalisation of scale_of), so a step gives the
// same bits here as in a launch of its own; k_rows.hip explains the operands.
// The tiles of a step go round-robin over the four waves.
// ---------------------------------------------------------------------------
typedef float chain_f4 __attribute__((ext_vector_type(4)));

// Maximum over the wave, valid in lane 63 (VALU lane moves only: a shuffle
// through LDS would add six LDS round trips to every step).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max(float v) {
  // Lanes without a source read 0, the identity for absolute values.
  const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false);
  return fmaxf(v, __int_as_float(o));
}
__device__ __forceinline__ float wave_max_63(float v) {
  v = dpp_max<0x111, 0xf>(v);  // row_shr:1
  v = dpp_max<0x112, 0xf>(v);  // row_shr:2
  v = dpp_max<0x114, 0xf>(v);  // row_shr:4
  v = dpp_max<0x118, 0xf>(v);  // row_shr:8
  v = dpp_max<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_max<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// This wave's tiles of one step: C = A B with sums in chunks of 2^KB terms.
// Rows and columns past the step's read the last valid one and are not
// stored, as in the row kernel.
template <int KB>
__device__ __forceinline__ void chain_tiles(const ChainStep& s, int m, int n, int k, int shift,
                                            const float2* pool, float* dst_lds, float* dst_mem,
                                            bool to_mem, int wave, int lane, float& lmax, int& bad) {
  constexpr int K = 1 << KB, NJ = K >= 2 ? K / 2 : 1;
  const int g = lane >> 4, lc = lane & 15, q = lc & 1;
  const int R = 1 << m, N = 1 << n, nkc = 1 << (k - KB);
  const int tr = m > 4 ? m - 4 : 0, tn = n > 3 ? n - 3 : 0;
  // The lane's part of the output address: row bits 2 and 3, column bits 0-2.
  int at_lane = 0;
  if (g & 1) at_lane += 1 << s.rpos[2];
  if (g & 2) at_lane += 1 << s.rpos[3];
  if (lc & 2) at_lane += 1 << s.cpos[0];
  if (lc & 4) at_lane += 1 << s.cpos[1];
  if (lc & 8) at_lane += 1 << s.cpos[2];
  const int r1 = 1 << s.rpos[0], r2 = 1 << s.rpos[1];
  for (int tile = wave; tile < (1 << (tr + tn)); tile += 4) {
    const int rt = tile & ((1 << tr) - 1), ct = tile >> tr;
    const int row = rt * 16 + lc, col = ct * 8 + (lc >> 1);
    const float2* pa = pool + s.lds_a + ((row < R ? row : R - 1) << k);
    const float2* pb = pool + s.lds_b + ((col < N ? col : N - 1) << k);
    chain_f4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int kc = 0; kc < nkc; ++kc) {
      if constexpr (K <= 2) {
        const float2 av = pa[K == 2 ? g >> 1 : 0], b = pb[K == 2 ? g >> 1 : 0];
        float af = (g & 1) ? av.y : av.x;
        if (K == 1 && g >= 2) af = 0.f;
        const float bop = (g & 1) == 0 ? (q == 0 ? b.x : b.y) : (q == 0 ? -b.y : b.x);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af, bop, acc, 0, 0, 0);
      } else {
        float2 av[NJ / 2], bv[NJ / 2];
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
          av[j] = pa[kc * K + g * (NJ / 2) + j];
          bv[j] = pb[kc * K + g * (NJ / 2) + j];
        }
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j].x, q == 0 ? bv[j].x : bv[j].y, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j].y, q == 0 ? -bv[j].y : bv[j].x, acc, 0, 0, 0);
        }
      }
    }
    int at = at_lane;
    for (int b = 0; b < tr; ++b)
      if ((rt >> b) & 1) at += 1 << s.rpos[4 + b];
    for (int b = 0; b < tn; ++b)
      if ((ct >> b) & 1) at += 1 << s.cpos[3 + b];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (rt * 16 + 4 * g + i < R && col < N) {
        const float v = shift ? ldexpf(acc[i], -shift) : acc[i];
        const int e = 2 * (at + ((i & 1) ? r1 : 0) + ((i & 2) ? r2 : 0)) + q;
        if (to_mem) dst_mem[e] = v;
        else dst_lds[e] = v;
        const float x = fabsf(v);
        if (!(x <= 3.4e38f)) bad = 1;
        else lmax = fmaxf(lmax, x);
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_chain(ChainArgs a) {
  extern __shared__ __attribute__((aligned(16))) float2 pool[];  // tensors
  __shared__ ChainStep steps[kChainMaxSteps];
  __shared__ uint32_t smax[kChainMaxSlots];  // max-abs (as bits) per tensor
  __shared__ int sexp[kChainMaxSlots];
  const ChainComp& comp = a.comps[blockIdx.x];
  const int cs = comp.dep_s ? a.gs : 1, cb = comp.dep_b ? a.gb : 1;
  const int copy = blockIdx.y;
  if (copy >= cs * cb) return;
  const int js = copy % cs, jb = copy / cs;
  const int tid = threadIdx.x;
  const int n_steps = comp.n_steps, n_in = comp.n_inputs;

  // The program, and the slots of the computed tensors.
  {
    const int* src = reinterpret_cast<const int*>(a.steps + comp.step0);
    const int words = n_steps * (int)(sizeof(ChainStep) / 4);
    for (int i = tid; i < words; i += 256) reinterpret_cast<int*>(steps)[i] = src[i];
    for (int i = n_in + tid; i < n_in + n_steps; i += 256) smax[i] = 0u;
  }
  // Inputs: 16 threads each, 16 inputs at a time (leaves hold at most 16
  // elements, so all leaves of a pass are in flight together).
  for (int i = tid >> 4; i < n_in; i += 16) {
    const ChainInput& in = a.inputs[comp.input0 + i];
    const int l16 = tid & 15, ne = 1 << in.rank;
    float2* dst = pool + in.lds;
    if (in.leaf) {
      int64_t base = in.src;
      for (int s = 0; s < in.nsel; ++s) {
        const int w = in.sel_src[s];
        const int v = w >= 0 ? (int)((a.slice_ids[js] >> w) & 1ull)
                             : (a.closed[(int64_t)jb * a.n_closed + (-w - 1)] & 1);
        if (v) base += int64_t(1) << in.sel_pos[s];
      }
      for (int e = l16; e < ne; e += 16) {
        int64_t at = base;
        for (int b = 0; b < in.rank; ++b)
          if ((e >> b) & 1) at += int64_t(1) << in.pos[b];
        dst[e] = reinterpret_cast<const float2*>(a.res)[at];
      }
      if (l16 == 0) {
        smax[i] = __float_as_uint(in.max_const);
        sexp[i] = 0;
      }
    } else {
      const char* base = (in.resident ? a.res : a.arena) + in.src;
      const float2* src = reinterpret_cast<const float2*>(base) + js * in.s_stride + jb * in.b_stride;
      for (int e = l16; e < ne; e += 16) dst[e] = src[e];
      if (l16 == 0) {
        const char* sb = in.resident ? a.res : a.scale;
        const int ci = js * in.es + jb * in.eb;
        smax[i] = in.m_off < 0 ? __float_as_uint(in.max_const)
                               : reinterpret_cast<const uint32_t*>(sb + in.m_off)[ci];
        sexp[i] = in.e_off < 0 ? 0 : reinterpret_cast<const int*>(sb + in.e_off)[ci];
      }
    }
  }
  __syncthreads();

  int bad = 0;
  float* out = reinterpret_cast<float*>(reinterpret_cast<float2*>(a.arena + comp.dst) +
                                        js * comp.s_stride + jb * comp.b_stride);
  const int wave = tid >> 6, lane = tid & 63;
  for (int st = 0; st < n_steps; ++st) {
    const ChainStep& s = steps[st];
    const int m = __builtin_amdgcn_readfirstlane(s.m), n = __builtin_amdgcn_readfirstlane(s.n);
    const int k = __builtin_amdgcn_readfirstlane(s.k);
    const int slot = n_in + st, sa = s.slot_a, sb = s.slot_b;
    const bool last = st + 1 == n_steps;
    const float mA = __uint_as_float(smax[sa]), mB = __uint_as_float(smax[sb]);
    int t = 0;
    if (mA > 0.f && mB > 0.f && mA <= 3.0e38f && mB <= 3.0e38f)
      t = k + 1 + ceil_log2(mA) + ceil_log2(mB) - kC64Target;
    float lmax = 0.f;
    float* dst = reinterpret_cast<float*>(pool + s.lds_c);
    switch (k) {
      case 0: chain_tiles<0>(s, m, n, k, t, pool, dst, out, last, wave, lane, lmax, bad); break;
      case 1: chain_tiles<1>(s, m, n, k, t, pool, dst, out, last, wave, lane, lmax, bad); break;
      case 2: chain_tiles<2>(s, m, n, k, t, pool, dst, out, last, wave, lane, lmax, bad); break;
      case 3: chain_tiles<3>(s, m, n, k, t, pool, dst, out, last, wave, lane, lmax, bad); break;
      default: chain_tiles<4>(s, m, n, k, t, pool, dst, out, last, wave, lane, lmax, bad); break;
    }
    lmax = wave_max_63(lmax);
    if ((tid & 63) == 63 && lmax > 0.f) atomicMax(&smax[slot], __float_as_uint(lmax));
    if (tid == 0) sexp[slot] = sexp[sa] + sexp[sb] + t;
    __syncthreads();
  }
  // The root's scale: this workgroup is the copy's only writer.
  if (tid == 0) {
    const int ci = js * comp.es + jb * comp.eb;
    reinterpret_cast<uint32_t*>(a.scale + comp.m_off)[ci] = smax[n_in + n_steps - 1];
    reinterpret_cast<int*>(a.scale + comp.e_off)[ci] = sexp[n_in + n_steps - 1];
  }
  if (bad) {
    if (comp.dep_s) a.flag[js] = 1;
    else
      for (int i = 0; i < a.gs; ++i) a.flag[i] = 1;  // shared by every slice
  }
}

hipError_t launch_chain(const ChainArgs& a, int n_comps, int max_copies, int lds_elems, hipStream_t s) {
  if (n_comps <= 0) return hipSuccess;
  if (max_copies < 1 || max_copies > 65535 || lds_elems < 0 || lds_elems > kChainMaxElems)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_chain, dim3((unsigned)n_comps, (unsigned)max_copies), dim3(256),
                     sizeof(float2) * (size_t)lds_elems, s, a);
  return hipGetLastError();
}

}  // namespace rqc

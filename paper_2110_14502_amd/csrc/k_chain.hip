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
// not by bandwidth or arithmetic.  Measured (whole calls, before / one step
// after the other / levels side by side): 4x4 256 / 99 / 90 us, 24 bitstrings of
// a 5x5 circuit 715 / 334 / 303, 16 FP16 slices of a 5x5 circuit 703 / 300 / 274;
// 32 slices of the 6x6 circuit 10.58 -> 9.70 ms in FP32 and 6.00 -> 5.23 in FP16.
//
// The arithmetic is the row kernel's, instruction for instruction (its 16 x 8
// tiles, its deal of the summed indices over the lanes and its order of
// products, the power-of-two normalisation of scale_of), so a step gives the
// same bits here as in a launch of its own; k_rows.hip explains the operands.
//
// The steps come in levels of independent ones (the tree's depth, not its
// size, sets the number of barriers); the tiles of a level go round-robin over
// the eight waves.
// ---------------------------------------------------------------------------
static_assert(kChainMaxSteps <= 512, "one thread clears each step's slot");
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

constexpr int kChainThreads = 512, kChainWaves = kChainThreads / 64;

typedef __attribute__((address_space(1))) float chain_global;  // keeps stores global, not generic
typedef __attribute__((address_space(3))) float chain_lds;

// Tiles first, first + 8, ... of one step: C = A B.  Rows and columns past the
// step's read the last valid one and are not stored, as in the row kernel.
// One loop serves every sum of four terms and more: a workgroup meets each
// line of this code once or twice, and fetching instructions costs it more
// than running them (a form specialised on the chunk size took 1.6 us a step).
__device__ __forceinline__ void chain_tiles(const ChainStep& s, int m, int n, int k, int shift,
                                            const float2* pool, chain_global* dst_mem, bool to_mem,
                                            int first, int tiles, int lane, float& lmax, int& bad) {
  const int g = lane >> 4, lc = lane & 15, q = lc & 1;
  const int R = 1 << m, N = 1 << n;
  const int tr = m > 4 ? m - 4 : 0, tn = n > 3 ? n - 3 : 0;
  // Sums in chunks of 2^kb terms, 2^kb / 4 of them per lane quarter.
  const int kb = k < 4 ? k : 4, ks = kb - 2, per = 1 << ks;
  // The lane's part of the output address: row bits 2 and 3, column bits 0-2.
  int at_lane = 0;
  if (g & 1) at_lane += 1 << s.rpos[2];
  if (g & 2) at_lane += 1 << s.rpos[3];
  if (lc & 2) at_lane += 1 << s.cpos[0];
  if (lc & 4) at_lane += 1 << s.cpos[1];
  if (lc & 8) at_lane += 1 << s.cpos[2];
  const int r1 = 1 << s.rpos[0], r2 = 1 << s.rpos[1];
  for (int tile = first; tile < tiles; tile += kChainWaves) {
    const int rt = tile & ((1 << tr) - 1), ct = tile >> tr;
    const int row = rt * 16 + lc, col = ct * 8 + (lc >> 1);
    const float2* pa = pool + s.lds_a + ((row < R ? row : R - 1) << k);
    const float2* pb = pool + s.lds_b + ((col < N ? col : N - 1) << k);
    chain_f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (k < 2) {
      const int kk = k ? g >> 1 : 0;
      const float2 av = pa[kk], b = pb[kk];
      float af = (g & 1) ? av.y : av.x;
      if (k == 0 && g >= 2) af = 0.f;
      const float bop = (g & 1) == 0 ? (q == 0 ? b.x : b.y) : (q == 0 ? -b.y : b.x);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af, bop, acc, 0, 0, 0);
    } else {
      // Term `it` of this lane's quarters, chunk by chunk; the next one is
      // read while this one is multiplied.
      const int its = 1 << (k - 2);
      int at = g << ks;
      float2 av = pa[at], bv = pb[at];
#pragma unroll 1
      for (int it = 0; it < its; ++it) {
        const float2 a = av, b = bv;
        const int nx = it + 1 < its ? it + 1 : it;
        at = ((nx >> ks) << kb) + (g << ks) + (nx & (per - 1));
        av = pa[at];
        bv = pb[at];
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, q == 0 ? b.x : b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, q == 0 ? -b.y : b.x, acc, 0, 0, 0);
      }
    }
    int at = at_lane;
    for (int b = 0; b < tr; ++b)
      if ((rt >> b) & 1) at += 1 << s.rpos[4 + b];
    for (int b = 0; b < tn; ++b)
      if ((ct >> b) & 1) at += 1 << s.cpos[3 + b];
    chain_lds* dst = (chain_lds*)(pool + s.lds_c);
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ldexpf(acc[i], -shift);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (rt * 16 + 4 * g + i < R && col < N) {
        const int e = 2 * (at + ((i & 1) ? r1 : 0) + ((i & 2) ? r2 : 0)) + q;
        if (to_mem) dst_mem[e] = v[i];
        else dst[e] = v[i];
        const float x = fabsf(v[i]);
        if (!(x <= 3.4e38f)) bad = 1;
        else lmax = fmaxf(lmax, x);
      }
    }
  }
}

__global__ __launch_bounds__(kChainThreads) void k_chain(ChainArgs a) {
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
    const uint4* src = reinterpret_cast<const uint4*>(a.steps + comp.step0);
    const int words = n_steps * (int)(sizeof(ChainStep) / 16);
    for (int i = tid; i < words; i += kChainThreads) reinterpret_cast<uint4*>(steps)[i] = src[i];
    if (tid < n_steps) smax[n_in + tid] = 0u;
  }
  // Small inputs: 16 threads each, 32 inputs at a time.  A descriptor is read
  // whole, then all selector bits, then the value: three memory round trips
  // (field by field a leaf took a dozen).
  const uint64_t sid = a.slice_ids[js];
  const uint8_t* cbits = a.closed + (int64_t)jb * a.n_closed;
  for (int i = tid >> 4; i < comp.n_small; i += kChainThreads / 16) {
    uint4 w[6];
    const uint4* src = reinterpret_cast<const uint4*>(a.inputs + comp.input0 + i);
#pragma unroll
    for (int j = 0; j < 6; ++j) w[j] = src[j];
    ChainInput in;
    __builtin_memcpy(&in, w, sizeof in);
    const int e = tid & 15;
    int64_t at = js * in.s_stride + jb * in.b_stride + e;
    if (in.leaf) {
      uint32_t c[4], off = 0;
#pragma unroll
      for (int s = 0; s < 4; ++s) c[s] = cbits[in.sel_src[s] < 0 ? -in.sel_src[s] - 1 : 0];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t v = in.sel_src[s] < 0 ? c[s] : (uint32_t)(sid >> in.sel_src[s]);
        if (s < in.nsel) off += (v & 1u) << ((in.sel_pos >> (8 * s)) & 255u);
      }
#pragma unroll
      for (int b = 0; b < kChainLeafBits; ++b)
        off += (((uint32_t)e >> b) & 1u) << ((in.pos >> (8 * b)) & 255u);
      at = off;
    }
    const char* base = (in.resident ? a.res : a.arena) + in.src;
    const char* sb = in.resident ? a.res : a.scale;
    const int ci = js * in.es + jb * in.eb;
    if (e < (1 << in.rank)) pool[in.lds + e] = reinterpret_cast<const float2*>(base)[at];
    if (e == 0) {
      smax[i] = in.m_off < 0 ? __float_as_uint(in.max_const)
                             : reinterpret_cast<const uint32_t*>(sb + in.m_off)[ci];
      sexp[i] = in.e_off < 0 ? 0 : reinterpret_cast<const int*>(sb + in.e_off)[ci];
    }
  }
  // Larger inputs (computed tensors): all threads, four elements each.
  for (int i = comp.n_small; i < n_in; ++i) {
    const ChainInput& in = a.inputs[comp.input0 + i];
    const char* base = (in.resident ? a.res : a.arena) + in.src;
    const float2* src = reinterpret_cast<const float2*>(base) + js * in.s_stride + jb * in.b_stride;
    const int ne = 1 << in.rank;
    float2 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (tid + j * kChainThreads < ne) v[j] = src[tid + j * kChainThreads];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (tid + j * kChainThreads < ne) pool[in.lds + tid + j * kChainThreads] = v[j];
    if (tid == 0) {
      const char* sb = in.resident ? a.res : a.scale;
      const int ci = js * in.es + jb * in.eb;
      smax[i] = in.m_off < 0 ? __float_as_uint(in.max_const)
                             : reinterpret_cast<const uint32_t*>(sb + in.m_off)[ci];
      sexp[i] = in.e_off < 0 ? 0 : reinterpret_cast<const int*>(sb + in.e_off)[ci];
    }
  }
  __syncthreads();

  int bad = 0;
  chain_global* out = (chain_global*)(reinterpret_cast<float2*>(a.arena + comp.dst) +
                                      js * comp.s_stride + jb * comp.b_stride);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  int mine = wave;  // this wave's first tile of the next step
  for (int st = 0; st < n_steps; ++st) {
    const ChainStep& s = steps[st];
    const int m = __builtin_amdgcn_readfirstlane(s.m), n = __builtin_amdgcn_readfirstlane(s.n);
    const int k = __builtin_amdgcn_readfirstlane(s.k);
    const int tiles = __builtin_amdgcn_readfirstlane(s.tiles);
    if (mine < tiles) {
      const int slot = n_in + st, sa = s.slot_a, sb = s.slot_b;
      const bool last = st + 1 == n_steps;
      const float mA = __uint_as_float(smax[sa]), mB = __uint_as_float(smax[sb]);
      int t = 0;
      if (mA > 0.f && mB > 0.f && mA <= 3.0e38f && mB <= 3.0e38f)
        t = k + 1 + ceil_log2(mA) + ceil_log2(mB) - kC64Target;
      float lmax = 0.f;
      chain_tiles(s, m, n, k, t, pool, out, last, mine, tiles, lane, lmax, bad);
      lmax = wave_max_63(lmax);
      if (lane == 63 && lmax > 0.f) atomicMax(&smax[slot], __float_as_uint(lmax));
      if (mine == 0 && lane == 0) sexp[slot] = sexp[sa] + sexp[sb] + t;
    }
    mine = (mine - tiles) & (kChainWaves - 1);
    if (__builtin_amdgcn_readfirstlane(s.level_end)) {
      __syncthreads();
      mine = wave;
    }
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
  hipLaunchKernelGGL(k_chain, dim3((unsigned)n_comps, (unsigned)max_copies), dim3(kChainThreads),
                     sizeof(float2) * (size_t)lds_elems, s, a);
  return hipGetLastError();
}

}  // namespace rqc

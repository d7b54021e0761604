// FP32 matrix-core contraction kernel (fused permute + complex GEMM).
#include "kernels_dev.h"

namespace rqc {

// ---------------------------------------------------------------------------
// MFMA contraction (FP32 matrix cores, v_mfma_f32_32x32x2_f32): 128 rows x
// 64 complex columns per tile, 16 complex k per LDS chunk, double buffered;
// 4 waves in a 2x2 grid, each 64 rows x 64 real columns.  The operand
// offsets come from LDS tables built once per workgroup; the output tile is
// staged through LDS in two halves of 64 rows (inside the operand buffers)
// and stored in C's address order.
//
// Persistent: the (copy, tile) items, column tiles fastest, are walked in
// steps of one item per workgroup, the workgroups of an XCD taking
// consecutive items, so that the tiles in flight on an XCD share rows of A.
// A workgroup loads the first chunk of its next tile while its current
// tile's last chunk is multiplied, and writes it to LDS before the current
// tile's output stores go out, so that those stores drain during the next
// tile's products; the scale and the running max-abs are flushed when the
// copy changes.  62 KB of LDS; two workgroups per CU.
// ---------------------------------------------------------------------------
constexpr unsigned kMfmaGrid = 256 * 2;

// ---------------------------------------------------------------------------
// Arithmetic of one 16-k chunk for one wave (64 rows x 32 complex columns of
// the tile), in two forms:
//
// 4M: the real 2x2 expansion of B (kernels_dev.h): A_r (64 x 32 real k) times
//     B_r (32 real k x 64 real columns) on four 32x32 accumulators; 8 real
//     flops executed per complex multiply-add.
// 3M: three real products per complex product (Gauss):
//         P1 = Ar Br,  P2 = Ai Bi,  P3 = (Ar + Ai)(Br + Bi),
//         Re C = P1 - P2,  Im C = P3 - P1 - P2,
//     on six 32x32 accumulators (two row blocks x three products); each
//     MFMA takes two complex k (one per half wave), so a chunk is 48 MFMAs
//     instead of 64: 6 real flops executed per complex multiply-add, with
//     half the LDS reads.  The sums Ar + Ai and Br + Bi are formed in
//     registers from the same LDS planes.
// ---------------------------------------------------------------------------
template <bool M3>
struct Acc32 {
  floatx16 v[M3 ? 6 : 4];
};

template <bool M3>
__device__ __forceinline__ void acc_zero(Acc32<M3>& acc) {
#pragma unroll
  for (int i = 0; i < (M3 ? 6 : 4); ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc.v[i][r] = 0.f;
}

// Abuf_cb / Bbuf_cb: the chunk's LDS buffers ([k][re|im][row] floats and
// [k][col] complex values).
template <bool M3>
__device__ __forceinline__ void chunk_mfma(const float* Abuf_cb, const float2* Bbuf_cb, int lane,
                                           int wm, int wn, Acc32<M3>& acc) {
  if constexpr (!M3) {
    const int lrow = lane & 31;
    const int cpart = lane >> 5;         // A_r column parity: 0 re, 1 im
    const int dpart = lane & 1;          // C_r column parity
    const int ncol = (lane & 31) >> 1;   // complex column inside a 16-col block
    const bool bswap = cpart != dpart;
    const float bsign = (cpart == 1 && dpart == 0) ? -1.f : 1.f;
    const float* As = Abuf_cb + cpart * kAPlane + wm * 64 + lrow;
    const float2* Bs = Bbuf_cb + wn * 32 + ncol;
    // Operands of step k+1 are read from LDS while the MFMAs of step k run.
    float a0 = As[0], a1 = As[32];
    float2 b0 = Bs[0], b1 = Bs[16];
#pragma unroll
    for (int k = 0; k < kTK; ++k) {
      float a0n = 0.f, a1n = 0.f;
      float2 b0n = make_float2(0.f, 0.f), b1n = make_float2(0.f, 0.f);
      if (k + 1 < kTK) {
        a0n = As[(k + 1) * kAStride];
        a1n = As[(k + 1) * kAStride + 32];
        b0n = Bs[(k + 1) * kBStride];
        b1n = Bs[(k + 1) * kBStride + 16];
      }
      const float v0 = bsign * (bswap ? b0.y : b0.x);
      const float v1 = bsign * (bswap ? b1.y : b1.x);
      acc.v[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, v0, acc.v[0], 0, 0, 0);
      acc.v[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, v1, acc.v[1], 0, 0, 0);
      acc.v[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, v0, acc.v[2], 0, 0, 0);
      acc.v[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, v1, acc.v[3], 0, 0, 0);
      a0 = a0n;
      a1 = a1n;
      b0 = b0n;
      b1 = b1n;
    }
  } else {
    // Lane half h takes complex k = 2 kk + h; rows / columns lane & 31.
    const int h = lane >> 5, l = lane & 31;
    const float* As = Abuf_cb + h * kAStride + wm * 64 + l;
    const float2* Bs = Bbuf_cb + h * kBStride + wn * 32 + l;
    float ar0 = As[0], ai0 = As[kAPlane], ar1 = As[32], ai1 = As[kAPlane + 32];
    float2 b = Bs[0];
#pragma unroll
    for (int kk = 0; kk < kTK / 2; ++kk) {
      float nr0 = 0.f, ni0 = 0.f, nr1 = 0.f, ni1 = 0.f;
      float2 nb = make_float2(0.f, 0.f);
      if (kk + 1 < kTK / 2) {
        const int o = 2 * (kk + 1) * kAStride;
        nr0 = As[o];
        ni0 = As[o + kAPlane];
        nr1 = As[o + 32];
        ni1 = As[o + kAPlane + 32];
        nb = Bs[2 * (kk + 1) * kBStride];
      }
      // Keep the next step's LDS reads ahead of this step's products (left
      // to itself the scheduler sinks them below the products and waits for
      // them right away).
      __builtin_amdgcn_sched_barrier(0);
      const float bs = b.x + b.y, as0 = ar0 + ai0, as1 = ar1 + ai1;
      acc.v[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar0, b.x, acc.v[0], 0, 0, 0);
      acc.v[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai0, b.y, acc.v[1], 0, 0, 0);
      acc.v[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(as0, bs, acc.v[2], 0, 0, 0);
      acc.v[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar1, b.x, acc.v[3], 0, 0, 0);
      acc.v[4] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai1, b.y, acc.v[4], 0, 0, 0);
      acc.v[5] = __builtin_amdgcn_mfma_f32_32x32x2f32(as1, bs, acc.v[5], 0, 0, 0);
      ar0 = nr0;
      ai0 = ni0;
      ar1 = nr1;
      ai1 = ni1;
      b = nb;
    }
  }
}

// Writes this wave's 64 x 32 complex accumulators into the staged half Cs
// ([row][real column] floats, kCStride per row).
template <bool M3>
__device__ __forceinline__ void stage_acc(float* Cs, const Acc32<M3>& acc, int lane, int wn) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      if constexpr (!M3) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int col = wn * 64 + j * 32 + (lane & 31);
          Cs[row * kCStride + col] = acc.v[2 * i + j][r];
        }
      } else {
        const float p1 = acc.v[3 * i][r], p2 = acc.v[3 * i + 1][r], p3 = acc.v[3 * i + 2][r];
        const int col = 2 * (wn * 32 + (lane & 31));
        *reinterpret_cast<float2*>(Cs + row * kCStride + col) = make_float2(p1 - p2, p3 - p1 - p2);
      }
    }
}

// LDS of the persistent kernel: buffer b holds A's chunk at b * kPersPair
// and B's right after it; the output staging area starts at buffer 1 and
// runs past it, so that buffer 0 can take the next tile's first chunk while
// the current tile's output is staged.
constexpr int kPersPair = kABuf + 2 * kBBuf;
constexpr int kPersFloats = kPersPair + kCHalf;
static_assert(kPersFloats >= 2 * kPersPair && kPersPair % 4 == 0, "persistent LDS layout");

template <int SA, int SB, int SC, bool M3>
__global__ __launch_bounds__(256, 2) void k_mfma32(StepDesc d, uint64_t n_items) {
  __shared__ float lds[kPersFloats + 16];
  __shared__ TileTab tcs;
  __shared__ OuterTab ot;
  float* Abuf = lds;                                      // [2][kTK][2][kAPlane], pair stride
  float2* Bbuf = reinterpret_cast<float2*>(lds + kABuf);  // [2][kTK][kBStride], pair stride
  float* red = lds + kPersFloats;
  if (d.run_if && !d.run_if->flag) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // Per-thread element offsets of the A (2048) and B (1024) chunk tiles.
  int64_t gA[8];
  int lA[8];
  int64_t gB[4];
  int lB[4];
  // The C tile bit that carries row bit 6 (which half of the tile).
  int hb = 0;
  for (int b = 0; b < d.tC.nbits; ++b)
    if (d.tC.role[b] == 0 && d.tC.cbit[b] == 6) hb = b;
  {
    TileTab* ta = reinterpret_cast<TileTab*>(lds);
    TileTab* tb = ta + 1;
    build_tab(d.tA, 1, 0, kAStride, *ta);
    build_tab(d.tB, 0, 1, kBStride, *tb);
    build_tab_skip(d.tC, hb, kCStride, 2, tcs);
    build_outer(d, ot);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      gA[j] = ta->g[lane] + ta->g[64 + wave + 4 * j];
      lA[j] = ta->c[lane] + ta->c[64 + wave + 4 * j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      gB[j] = tb->g[lane] + tb->g[64 + wave + 4 * j];
      lB[j] = tb->c[lane] + tb->c[64 + wave + 4 * j];
    }
    __syncthreads();
  }
  const int64_t g_half = int64_t(1) << d.tC.gpos[hb];
  const int64_t g_lane = tcs.g[lane];
  const int c_lane = tcs.c[lane];
  // Vector stores when C's two lowest address bits are the two lowest
  // C-order bits of the staged half.
  const bool vec_c = d.tC.nbits > 2 && hb > 1 && d.tC.gpos[0] == 0 && d.tC.gpos[1] == 1;
  const int64_t g_lo4 = tcs.g[(tid & 15) << 2];
  int c_lo4[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) c_lo4[i] = tcs.c[((tid & 15) << 2) + i];

  const int n_kc = 1 << d.n_ko;
  // Tile counts are powers of two: item t is copy t >> tb, row tile
  // (t & tmask) >> n_no, column tile t & cmask.
  const int tb = d.n_ro + d.n_no;
  const uint64_t tmask = (uint64_t(1) << tb) - 1, cmask = (uint64_t(1) << d.n_no) - 1;
  // Step i of the walk covers items i*G .. i*G + G - 1, dealt so that the
  // workgroups of one XCD (blocks go round-robin to the 8 XCDs) take
  // consecutive items: they share rows of A in that XCD's L2.
  const uint64_t G = gridDim.x;
  uint64_t t = (G & 7) == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;

  auto item_offsets = [&](uint64_t it, int64_t& oA, int64_t& oB, int64_t& oC) {
    const int copy = (int)(it >> tb);
    const uint64_t bid = it & tmask;
    outer_offsets(d, ot, bid >> d.n_no, bid & cmask, copy % d.gs_c, copy / d.gs_c, oA, oB, oC);
  };
  float2 ra[8], rb[4];
  auto load_chunk = [&](int64_t oA, int64_t oB, int kc) {
    int64_t kA, kB;
    k_offsets(d, ot, kc, kA, kB);
#pragma unroll
    for (int j = 0; j < 8; ++j) ra[j] = load_c<SA>(d.A, oA + kA + gA[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) rb[j] = load_c<SB>(d.B, oB + kB + gB[j]);
  };
  auto store_chunk = [&](int buf) {
    float* An = Abuf + buf * kPersPair;
    float2* Bn = Bbuf + buf * (kPersPair / 2);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      An[lA[j]] = ra[j].x;
      An[lA[j] + kAPlane] = ra[j].y;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) Bn[lB[j]] = rb[j];
  };

  // The scale of a copy is read when its first tile is prefetched (before
  // those loads are issued), not at the top of the tile, where the wait for
  // it would also wait for the previous tile's output stores.
  Scale sc{0, 0}, nsc{0, 0};
  if (t < n_items) {
    int64_t oA, oB, oC;
    const int copy = (int)(t >> tb);
    nsc = compute_scale(d, copy % d.gs_c, copy / d.gs_c);
    item_offsets(t, oA, oB, oC);
    load_chunk(oA, oB, 0);
    store_chunk(0);
  }
  __syncthreads();
  int cur = -1;
  int cjs = 0, cjb = 0;
  bool wexp = false;
  float lmax = 0.f;
  int bad = 0;
  for (; t < n_items; t += G) {
    const int copy = (int)(t >> tb);
    const uint64_t bid = t & tmask;
    const int js = copy % d.gs_c, jb = copy / d.gs_c;
    if (copy != cur) {
      if (cur >= 0) finish_scale<256>(d, cjs, cjb, lmax, bad, red, wexp, sc);
      sc = nsc;
      lmax = 0.f;
      bad = 0;
      wexp = false;
      cur = copy;
      cjs = js;
      cjb = jb;
    }
    wexp = wexp || bid == 0;
    int64_t oA, oB, oC;
    outer_offsets(d, ot, bid >> d.n_no, bid & cmask, js, jb, oA, oB, oC);
    const bool next_tile = t + G < n_items;

    Acc32<M3> acc;
    acc_zero(acc);

    // Every chunk but the last: the next chunk is loaded while this one is
    // multiplied.  The products run at raised wave priority, so that the
    // other workgroup's epilogue on this CU does not hold back their issue.
    for (int kc = 0; kc + 1 < n_kc; ++kc) {
      const int cb = kc & 1;
      load_chunk(oA, oB, kc + 1);
      __builtin_amdgcn_s_setprio(1);
      chunk_mfma<M3>(Abuf + cb * kPersPair, Bbuf + cb * (kPersPair / 2), lane, wm, wn, acc);
      __builtin_amdgcn_s_setprio(0);
      store_chunk(cb ^ 1);
      __syncthreads();
    }
    // The last chunk: meanwhile the next tile's first chunk is loaded, and
    // the scale inputs of its copy before it (unconditionally: loads and
    // uses under one condition keep the compiler's wait counts exact).
    ScaleIn nin{0, 0, 0.f, 0.f};
    if (next_tile) {
      const int cn = (int)((t + G) >> tb);
      nin = load_scale(d, cn % d.gs_c, cn / d.gs_c);
      int64_t pA, pB, pC;
      item_offsets(t + G, pA, pB, pC);
      load_chunk(pA, pB, 0);
    }
    {
      const int cb = (n_kc - 1) & 1;
      __builtin_amdgcn_s_setprio(1);
      chunk_mfma<M3>(Abuf + cb * kPersPair, Bbuf + cb * (kPersPair / 2), lane, wm, wn, acc);
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    // The next tile's first chunk goes to buffer 0 (free since the barrier
    // above) before this tile's output stores are issued: the vector memory
    // counter completes in issue order, so a wait for these loads placed
    // after the stores would also wait for the stores to finish.
    if (next_tile) {
      store_chunk(0);
      nsc = scale_of(d, nin);
    }

    // Epilogue: two halves of 64 rows staged from buffer 1 on; the first
    // barrier also publishes buffer 0.
    float* Cs = lds + kPersPair;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (wm == h) stage_acc<M3>(Cs, acc, lane, wn);
      __syncthreads();
      if (vec_c)
        store_half4<SC>(d, Cs, tcs, oC + g_lo4 + (h ? g_half : 0), c_lo4, tid, sc, lmax, bad);
      else
        store_half<SC, 8>(d, Cs, tcs, oC + g_lane + (h ? g_half : 0), c_lane, wave, sc, lmax, bad);
      __syncthreads();
    }
  }
  if (cur >= 0) finish_scale<256>(d, cjs, cjb, lmax, bad, red, wexp, sc);
}

// ---------------------------------------------------------------------------
// The persistent walk for complex64 operands in the planner's layout (the
// summed indices lowest in A and B): chunks are copied straight into LDS, 16
// bytes (two summed terms of a row) per lane, instead of passing through
// registers.  The arithmetic is k_mfma32's three-product form in the same
// order: the same bits.
//
// What bounds it: the FP32 matrix products (64 cycles each) and, for short sums,
// memory at the same time.  The FP32 products run on the vector ALUs: every
// other vector instruction costs about 6 cycles of product time, and 17 where the
// next product waits for its result.  So a step of six products has three
// further vector instructions, the sums for the three-product form, made a step
// ahead; LDS addresses are constants beside two bases per operand, copies take
// a scalar base, a tile's first products a zero sum, and outer indices are
// worked out in scalar registers.
//
// LDS holds blocks of 8 rows, each [4][8 rows][2 pairs of terms]: the copying
// lanes choose what lands where by their source address (two lanes read 32
// consecutive bytes), and odd blocks swap the two pairs, so that the rows a wave
// reads at one step meet two to a bank.  Three buffers: the copies of the chunk
// after next go out one a step; a chunk's last step waits for the next chunk,
// meets the one barrier and reads its first operands, among its products.
//
// Output: each wave stages its 64 x 32 block itself, 16 rows at a time, in the
// buffer of the last chunk, two elements per lane and store.  74 KB of LDS, two
// workgroups per CU.
//
// Measured against k_mfma32 (and the per-tile kernel where that was the choice):
// 2^(14+6) x 2^(7+6), 37 copies 390 -> 308 us; 2^(16+7) x 2^(7+7), 32 copies
// 2232 -> 1936; 2^(9+10) x 2^(8+10), 32 copies 234 -> 206 (125 TFLOP/s
// executed of 157); 2^(8+13) x 2^(7+13), 32 copies 1232 -> 901.
// ---------------------------------------------------------------------------
constexpr int kDmaA = kTM * 128, kDmaB = kTN * 128;  // bytes of a chunk (16 terms of 8 bytes per row)
constexpr int kDmaBuf = kDmaA + kDmaB;
constexpr int kDmaLdc = 33;                          // complex values per staged row
static_assert(4 * 16 * kDmaLdc * 8 <= kDmaBuf, "the staged rows of four waves fit one buffer");

// IF: only where d.run_if is flagged (a form of its own: the test at its start alone
// made (14, 7, 6) x 37 6% slower).
template <int SC, bool IF>
__global__ __launch_bounds__(256, 2) void k_mfma32_copy(StepDesc d, uint32_t n_items) {
  if (IF && !d.run_if->flag) return;
  __shared__ __attribute__((aligned(16))) char lds[3 * kDmaBuf];
  __shared__ int64_t cg[72];  // C offset of a staged element: low six bits, then the rest
  __shared__ int32_t cc[72];  // its place in the staging area
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l = lane & 31, h = lane >> 5;
  const OuterReg ot = outer_reg(d);

  // Byte offsets of the copies: block i = 4 wave + j of A's rows, 2 wave + j of
  // B's columns.
  uint32_t gA[4], gB[2];
  {
    const int p = (lane >> 4) * 2 + (lane & 1), r = (lane >> 1) & 7;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = (4 * wave + j) * 8 + r;
      gA[j] = 16 * (p ^ (j & 1));
      for (int b = 4; b < d.tA.nbits; ++b)
        if ((row >> d.tA.cbit[b]) & 1) gA[j] += 8u << d.tA.gpos[b];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = (2 * wave + j) * 8 + r;
      gB[j] = 16 * (p ^ (j & 1));
      for (int b = 4; b < d.tB.nbits; ++b)
        if ((col >> d.tB.cbit[b]) & 1) gB[j] += 8u << d.tB.gpos[b];
    }
  }
  // Staged elements: row bits 0-3 and column bits 0-4 in C's address order;
  // the other tile bits select the pass and the wave.
  int64_t rw[3] = {0, 0, 0}, cw = 0;  // C weights of row bits 4, 5, 6 and column bit 5
  bool vec_c = false;                 // C's address bit 0 is staged bit 0: stores of two elements
  {
    int64_t g = 0;
    int c = 0, n = 0;
    const int v = tid < 64 ? tid : tid - 64, b0 = tid < 64 ? 0 : 6, b1 = tid < 64 ? 6 : 9;
    for (int b = 0; b < d.tC.nbits; ++b) {
      const int role = d.tC.role[b], cb = d.tC.cbit[b], gp = d.tC.gpos[b];
      if (role == 0 && cb >= 4) {
        if (cb == 4) rw[0] = int64_t(1) << gp;
        if (cb == 5) rw[1] = int64_t(1) << gp;
        if (cb == 6) rw[2] = int64_t(1) << gp;
        continue;
      }
      if (role == 1 && cb == 5) {
        cw = int64_t(1) << gp;
        continue;
      }
      if (gp == 0) vec_c = true;
      if (n >= b0 && n < b1 && ((v >> (n - b0)) & 1)) {
        g += int64_t(1) << gp;
        c += role == 0 ? kDmaLdc << cb : 1 << cb;
      }
      ++n;
    }
    if (tid < 72) {
      cg[tid] = g;
      cc[tid] = c;
    }
  }
  __syncthreads();
  const int64_t g_wave = (wm ? rw[2] : 0) + (wn ? cw : 0);
  const int lo = vec_c ? (lane & 31) << 1 : lane;
  const int64_t g_lo = cg[lo];
  const int c_lo = cc[lo], c_lo1 = vec_c ? cc[lo + 1] : 0;

  // Items as in k_mfma32: step i of the walk covers items i G .. i G + G - 1,
  // consecutive ones on one XCD.
  const int n_ko = __builtin_amdgcn_readfirstlane(d.n_ko), n_kc = 1 << n_ko;
  const int tb = d.n_ro + d.n_no;
  const uint32_t tmask = (1u << tb) - 1, cmask = (1u << d.n_no) - 1;
  const uint32_t G = gridDim.x;
  uint32_t t = (G & 7) == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  auto item_offsets = [&](uint32_t it, int64_t& oA, int64_t& oB, int64_t& oC) {
    const int copy = (int)(it >> tb);
    const uint32_t bid = it & tmask;
    const int js = copy % d.gs_c, jb = copy / d.gs_c;
    int64_t cr = 0, cn = 0;
    oA = js * d.sA_s + jb * d.sA_b;
    oB = js * d.sB_s + jb * d.sB_b;
    outer_sum(ot.rn, bid >> d.n_no, oA, cr);
    outer_sum(ot.rn >> 16, bid & cmask, oB, cn);
    oC = js * d.sC_s + jb * d.sC_b + cr + cn;
  };

  // The next chunk to copy: chunk fk of item ft (whose operands start at iA,
  // iB), at fA, fB.
  uint32_t ft = t;
  int fk = -1;
  int64_t iA = 0, iB = 0;
  const float2 *fA = nullptr, *fB = nullptr;
  const uint32_t l0 = lds_address(lds);
  auto fetch1 = [&](int j, uint32_t at) {  // at: LDS address of the buffer
    if (j < 4) lds_copy16(fA, gA[j], at + (uint32_t)((4 * wave + j) * 1024));
    else lds_copy16(fB, gB[j - 4], at + (uint32_t)(kDmaA + (2 * wave + j - 4) * 1024));
  };
  auto advance = [&]() {
    if (ft >= n_items) return;
    if (++fk == n_kc) {
      fk = 0;
      ft += G;
      if (ft >= n_items) return;
      int64_t oC;
      item_offsets(ft, iA, iB, oC);
    }
    int64_t kA = iA, kB = iB;
    outer_sum(ot.k, (uint32_t)fk, kA, kB);
    fA = static_cast<const float2*>(d.A) + kA;
    fB = static_cast<const float2*>(d.B) + kB;
  };
  auto fetch = [&](int buf) {
    if (ft < n_items)
#pragma unroll
      for (int j = 0; j < 6; ++j) fetch1(j, l0 + (uint32_t)(buf * kDmaBuf));
    advance();
  };

  // Lane half h takes summed term 2 kk + h of row (column) l at step kk.
  const int at_l = (l >> 3) * 1024 + (l & 7) * 32 + h * 8, sw = ((l >> 3) & 1) * 16;
  const int a_at = wm * 8192 + at_l, b_at = kDmaA + wn * 4096 + at_l;
  float2 a0, a1, b;    // the operands of the step at hand
  float as0, as1, bs;  // and their sums
  int aE, aO, bE, bO;  // LDS offsets of a chunk's even and odd steps
  auto at_buf = [&](int buf) {
    aE = buf * kDmaBuf + a_at + sw;
    aO = buf * kDmaBuf + a_at + 16 - sw;
    bE = buf * kDmaBuf + b_at + sw;
    bO = buf * kDmaBuf + b_at + 16 - sw;
  };
  auto rd = [&](int at) { return *reinterpret_cast<const float2*>(lds + at); };

  Scale sc{0, 0}, nsc{0, 0};
  bool stored = false;  // output was stored since chunk c + 1's copies were issued
  if (t < n_items) {
    const int copy = (int)(t >> tb);
    nsc = compute_scale_s(d, copy % d.gs_c, copy / d.gs_c);
    int64_t oC;
    item_offsets(t, iA, iB, oC);
    advance();
    fetch(0);
    fetch(1);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    plain_barrier();
    at_buf(0);
    a0 = rd(aE);
    a1 = rd(aE + 4096);
    b = rd(bE);
    as0 = a0.x + a0.y;
    as1 = a1.x + a1.y;
    bs = b.x + b.y;
  }
  int buf = 0, cur = -1, cjs = 0, cjb = 0, bad = 0;
  bool wexp = false;
  float lmax = 0.f;
  for (; t < n_items; t += G) {
    const int copy = (int)(t >> tb);
    const uint32_t bid = t & tmask;
    const int js = copy % d.gs_c, jb = copy / d.gs_c;
    if (copy != cur) {
      if (cur >= 0) finish_scale<256>(d, cjs, cjb, lmax, bad, red, wexp, sc);
      sc = nsc;
      lmax = 0.f;
      bad = 0;
      wexp = false;
      cur = copy;
      cjs = js;
      cjb = jb;
    }
    wexp = wexp || bid == 0;
    if (t + G < n_items) {
      const int cn = (int)((t + G) >> tb);
      if (cn != copy) nsc = compute_scale_s(d, cn % d.gs_c, cn / d.gs_c);
    }
    Acc32<true> acc;
    auto mma = [&](int i, float x, float y, bool zero) {
      if (zero) {  // a tile's first products take a zero sum
        floatx16 z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = 0.f;
        acc.v[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, z, 0, 0, 0);
      } else {
        acc.v[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc.v[i], 0, 0, 0);
      }
    };
    for (int kc = 0; kc < n_kc; ++kc) {
      const int nb = buf == 2 ? 0 : buf + 1;
      const uint32_t fat = __builtin_amdgcn_readfirstlane(l0 + (uint32_t)((buf == 0 ? 2 : buf - 1) * kDmaBuf));
      // ft < n_items (below 2^31), as a scalar: chunk c + 2's copies go out one a step.
      const uint32_t more = (ft - n_items) >> 31;
      __builtin_amdgcn_s_setprio(1);
      auto step = [&](int kk, bool zero) {
        float2 na0, na1, nb0;
        if (kk + 1 < kTK / 2) {
          const int o = ((kk + 1) >> 1) * 256;
          na0 = rd((kk & 1 ? aE : aO) + o);
          na1 = rd((kk & 1 ? aE : aO) + o + 4096);
          nb0 = rd((kk & 1 ? bE : bO) + o);
        }
        // The scheduling barriers keep the reads ahead of four products and the
        // sums for the next step among this step's.
        __builtin_amdgcn_sched_barrier(0);
        mma(0, a0.x, b.x, zero);
        __builtin_amdgcn_sched_barrier(0);
        if (kk < 6 && more) fetch1(kk, fat);
        if (kk == 6) advance();
        if (kk + 1 == kTK / 2) {
          // Every read of this chunk is done and chunk c + 1 has landed: its
          // copies are older than chunk c + 2's six and, after a tile's end,
          // than that tile's stores (16 at the least; the count completes in
          // order, so a wait past them would wait for them too).
          asm volatile("" ::: "memory");
          if (!more) __builtin_amdgcn_s_waitcnt(0x0070);          // vmcnt(0) lgkmcnt(0)
          else if (stored) __builtin_amdgcn_s_waitcnt(0x4076);    // vmcnt(22) lgkmcnt(0)
          else __builtin_amdgcn_s_waitcnt(0x0076);                // vmcnt(6) lgkmcnt(0)
          plain_barrier();
          at_buf(nb);
          na0 = rd(aE);
          na1 = rd(aE + 4096);
          nb0 = rd(bE);
          __builtin_amdgcn_sched_barrier(0);
        }
        mma(1, a0.y, b.y, zero);
        mma(2, as0, bs, zero);
        mma(3, a1.x, b.x, zero);
        mma(4, a1.y, b.y, zero);
        __builtin_amdgcn_sched_barrier(0);
        float nas0 = na0.x + na0.y, nas1 = na1.x + na1.y, nbs = nb0.x + nb0.y;
        asm volatile("" : "+v"(nas0), "+v"(nas1), "+v"(nbs));
        __builtin_amdgcn_sched_barrier(0);
        mma(5, as1, bs, zero);
        a0 = na0;
        a1 = na1;
        b = nb0;
        as0 = nas0;
        as1 = nas1;
        bs = nbs;
      };
      if (kc == 0) step(0, true);
      else step(0, false);
#pragma unroll
      for (int kk = 1; kk < kTK / 2; ++kk) step(kk, false);
      __builtin_amdgcn_s_setprio(0);
      stored = false;
      if (kc + 1 < n_kc) buf = nb;
    }
    // The last chunk's buffer is free (the barrier in its last step).
    int64_t oA, oB, oC;
    item_offsets(t, oA, oB, oC);
    float2* Cs = reinterpret_cast<float2*>(lds + buf * kDmaBuf) + wave * 16 * kDmaLdc;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        // Rows 32 i + 16 hf .. + 15: lane (h, l) holds rows 8 (r / 4) + 4 h + r
        // mod 4 of column l.
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float p1 = acc.v[3 * i][8 * hf + r], p2 = acc.v[3 * i + 1][8 * hf + r];
          const float p3 = acc.v[3 * i + 2][8 * hf + r];
          Cs[(8 * (r >> 2) + 4 * h + (r & 3)) * kDmaLdc + l] = make_float2(p1 - p2, p3 - p1 - p2);
        }
        __builtin_amdgcn_wave_barrier();
        const int64_t at = oC + g_wave + (i ? rw[1] : 0) + (hf ? rw[0] : 0) + g_lo;
        if (vec_c) {
          float2 x[8];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int c = cc[64 + 2 * u + (lane >> 5)];
            x[2 * u] = Cs[c_lo + c];
            x[2 * u + 1] = Cs[c_lo1 + c];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float2(&pair)[2] = *reinterpret_cast<float2(*)[2]>(&x[2 * u]);
            store_out2<SC>(d, at + cg[64 + 2 * u + (lane >> 5)], pair, sc);
          }
          if (d.track) track_out<SC, 8>(x, lmax, bad);
        } else {
          float2 x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = Cs[c_lo + cc[64 + u]];
#pragma unroll
          for (int u = 0; u < 8; ++u) store_out<SC>(d, at + cg[64 + u], x[u], sc, lmax, bad);
        }
      }
    // Every wave is done with the buffer before copies go into it.
    plain_barrier();
    stored = true;
    buf = buf == 2 ? 0 : buf + 1;
  }
  if (cur >= 0) finish_scale<256>(d, cjs, cjb, lmax, bad, red, wexp, sc);
}

// Whether a step's tiles can be copied in 16-byte pairs: the chunk's summed
// bits are A's and B's address bits 0-3, in order, a tile's offsets fit 32 bits,
// and the operands (with every copy stride) keep 16-byte alignment.
bool mfma32_copies(const StepDesc& d) {
  if ((d.variant & (kVarTiles | kVar4M)) || (uint64_t)d.copies << (d.n_ro + d.n_no) >= (uint64_t(1) << 31))
    return false;
  for (const TileMap* m : {&d.tA, &d.tB})
    for (int b = 0; b < m->nbits; ++b) {
      if (b < 4 && (m->role[b] != 2 || m->gpos[b] != b || m->cbit[b] != b)) return false;
      if (b >= 4 && m->gpos[b] > 28) return false;
    }
  return ((reinterpret_cast<uintptr_t>(d.A) | reinterpret_cast<uintptr_t>(d.B)) & 15) == 0 &&
         ((d.sA_s | d.sA_b | d.sB_s | d.sB_b) & 1) == 0;
}

// ---------------------------------------------------------------------------
// Long sums (K >= 256): one tile per workgroup, three workgroups per CU.  The
// per-tile overheads the persistent walk hides are small against hundreds of
// chunks, and the third resident wave per SIMD keeps the matrix cores busier
// in the chunk loop.  Same tiling and arithmetic; the output table is built in
// the operand buffers after the last chunk.  51.8 KB of LDS.
// ---------------------------------------------------------------------------
template <int SA, int SB, int SC, bool M3>
__global__ __launch_bounds__(256, M3 ? 2 : 3) void k_mfma32_tiles(StepDesc d) {
  if (d.run_if && !d.run_if->flag) return;
  __shared__ float lds[kMainFloats + 16];
  __shared__ OuterTab ot;
  __shared__ TileMap maps[3];  // A, B, C
  float* Abuf = lds;
  float2* Bbuf = reinterpret_cast<float2*>(lds + 2 * kABuf);
  float* red = lds + kMainFloats;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // XCD-aware block order: consecutive logical tiles share the row tile of A
  // and land on the same XCD (blocks are dealt round-robin to the 8 XCDs).
  uint64_t bid = blockIdx.x;
  const uint64_t nblk = gridDim.x;
  if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
  const uint64_t cmask = (uint64_t(1) << d.n_no) - 1;
  const uint64_t no = bid & cmask, ro = bid >> d.n_no;

  int64_t gA[8];
  int lA[8];
  int64_t gB[4];
  int lB[4];
  {
    TileTab* ta = reinterpret_cast<TileTab*>(lds);
    TileTab* tb = ta + 1;
    stage_maps(d, maps);
    build_outer(d, ot);
    __syncthreads();
    build_tab(maps[0], 1, 0, kAStride, *ta);
    build_tab(maps[1], 0, 1, kBStride, *tb);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      gA[j] = ta->g[lane] + ta->g[64 + wave + 4 * j];
      lA[j] = ta->c[lane] + ta->c[64 + wave + 4 * j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      gB[j] = tb->g[lane] + tb->g[64 + wave + 4 * j];
      lB[j] = tb->c[lane] + tb->c[64 + wave + 4 * j];
    }
  }
  int hb = 0;
  for (int b = 0; b < maps[2].nbits; ++b)
    if (maps[2].role[b] == 0 && maps[2].cbit[b] == 6) hb = b;
  const int64_t g_half = int64_t(1) << maps[2].gpos[hb];

  const int n_kc = 1 << d.n_ko;
  float2 ra[8], rb[4];
  for (int copy = blockIdx.y; copy < d.copies; copy += gridDim.y) {
    const int js = copy % d.gs_c, jb = copy / d.gs_c;
    int64_t oA, oB, oC;
    outer_offsets(d, ot, ro, no, js, jb, oA, oB, oC);
    auto load_chunk = [&](int kc) {
      int64_t kA, kB;
      k_offsets(d, ot, kc, kA, kB);
#pragma unroll
      for (int j = 0; j < 8; ++j) ra[j] = load_c<SA>(d.A, oA + kA + gA[j]);
#pragma unroll
      for (int j = 0; j < 4; ++j) rb[j] = load_c<SB>(d.B, oB + kB + gB[j]);
    };
    auto store_chunk = [&](int buf) {
      float* An = Abuf + buf * kABuf;
      float2* Bn = Bbuf + buf * kBBuf;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        An[lA[j]] = ra[j].x;
        An[lA[j] + kAPlane] = ra[j].y;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) Bn[lB[j]] = rb[j];
    };
    Acc32<M3> acc;
    acc_zero(acc);
    // The copy's scale inputs are read before the first chunk, whose wait
    // covers them; they are used only in the epilogue.
    ScaleIn sin = load_scale(d, js, jb);
    load_chunk(0);
    __syncthreads();  // the tables (or the previous copy's output) are done with
    store_chunk(0);
    __syncthreads();
    for (int kc = 0; kc < n_kc; ++kc) {
      const int cb = kc & 1;
      const bool more = kc + 1 < n_kc;
      if (more) load_chunk(kc + 1);
      __builtin_amdgcn_s_setprio(1);
      chunk_mfma<M3>(Abuf + cb * kABuf, Bbuf + cb * kBBuf, lane, wm, wn, acc);
      __builtin_amdgcn_s_setprio(0);
      if (more) store_chunk(cb ^ 1);
      __syncthreads();
    }

    // Epilogue: the C table and two halves of 64 rows in the operand buffers.
    float* Cs = lds;
    TileTab* tcs = reinterpret_cast<TileTab*>(lds + kCHalf);
    build_tab_skip(maps[2], hb, kCStride, 2, *tcs);
    asm volatile("" : "+v"(sin.eA), "+v"(sin.eB), "+v"(sin.mA), "+v"(sin.mB));
    const Scale sc = scale_of(d, sin);
    float lmax = 0.f;
    int bad = 0;
    __syncthreads();
    const int64_t g_lane = tcs->g[lane];
    const int c_lane = tcs->c[lane];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (wm == h) stage_acc<M3>(Cs, acc, lane, wn);
      __syncthreads();
      const int64_t gl = g_lane + (h ? g_half : 0);
#pragma unroll 4
      for (int j = 0; j < 16; ++j) {
        const int hi = 64 + wave + 4 * j;
        const int c = c_lane + tcs->c[hi];
        store_out<SC>(d, oC + gl + tcs->g[hi], make_float2(Cs[c], Cs[c + 1]), sc, lmax, bad);
      }
      __syncthreads();
    }
    finish_scale<256>(d, js, jb, lmax, bad, red, ro == 0 && no == 0, sc);
  }
}

#define RQC_MFMA_CASE(a, b, c)                                                          \
  if (sa == a && sb == b && sc == c) {                                                  \
    if (tiles_kernel && m3)                                                             \
      hipLaunchKernelGGL((k_mfma32_tiles<a, b, c, true>), grid, dim3(256), 0, s, d);   \
    else if (tiles_kernel)                                                              \
      hipLaunchKernelGGL((k_mfma32_tiles<a, b, c, false>), grid, dim3(256), 0, s, d);  \
    else if (m3)                                                                        \
      hipLaunchKernelGGL((k_mfma32<a, b, c, true>), grid, dim3(256), 0, s, d, n_items); \
    else                                                                                \
      hipLaunchKernelGGL((k_mfma32<a, b, c, false>), grid, dim3(256), 0, s, d, n_items); \
    return hipGetLastError();                                                           \
  }

hipError_t launch_mfma32_kernel(const StepDesc& d, int sa, int sb, int sc, dim3 grid,
                                hipStream_t s) {
  if (d.rt != 7 || d.nt != 6 || d.kt != 4) return hipErrorInvalidValue;
  const uint64_t n_items = (uint64_t)grid.x * (uint64_t)d.copies;
  // Operands that can be copied straight into LDS: k_mfma32_copy at every length
  // of the sum (figures there; the smallest calls, 2^(9+6) x 2^(7+6), take 25 us
  // either way).  Others, sums of 256 or more complex terms: one tile per
  // workgroup (grid = tiles x copies as given); shorter sums: the persistent walk.
  const bool tiles_kernel = d.variant & kVarTiles ? true : (d.variant & kVarPersistent ? false : d.n_ko >= 4);
  const bool m3 = (d.variant & kVar4M) == 0;
  if (sa == ST_C64 && sb == ST_C64 && mfma32_copies(d)) {
    grid = dim3((unsigned)(n_items < kMfmaGrid ? n_items : kMfmaGrid), 1);
    auto* kern = sc == ST_F16 ? k_mfma32_copy<ST_F16, false> : sc == ST_BF16 ? k_mfma32_copy<ST_BF16, false>
                 : d.run_if ? k_mfma32_copy<ST_C64, true> : k_mfma32_copy<ST_C64, false>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, d, (uint32_t)n_items);
    return hipGetLastError();
  }
  if (!tiles_kernel) grid = dim3((unsigned)(n_items < kMfmaGrid ? n_items : kMfmaGrid), 1);
  RQC_MFMA_CASE(ST_C64, ST_C64, ST_C64)
  RQC_MFMA_CASE(ST_C64, ST_C64, ST_F16)
  RQC_MFMA_CASE(ST_C64, ST_C64, ST_BF16)
  RQC_MFMA_CASE(ST_F16, ST_C64, ST_F16)
  RQC_MFMA_CASE(ST_F16, ST_C64, ST_C64)
  RQC_MFMA_CASE(ST_BF16, ST_C64, ST_BF16)
  RQC_MFMA_CASE(ST_BF16, ST_C64, ST_C64)
  RQC_MFMA_CASE(ST_C64, ST_F16, ST_F16)
  RQC_MFMA_CASE(ST_C64, ST_F16, ST_C64)
  RQC_MFMA_CASE(ST_C64, ST_BF16, ST_BF16)
  RQC_MFMA_CASE(ST_C64, ST_BF16, ST_C64)
  RQC_MFMA_CASE(ST_F16, ST_F16, ST_F16)
  RQC_MFMA_CASE(ST_F16, ST_F16, ST_C64)
  RQC_MFMA_CASE(ST_BF16, ST_BF16, ST_BF16)
  RQC_MFMA_CASE(ST_BF16, ST_BF16, ST_C64)
  return hipErrorInvalidValue;
}
#undef RQC_MFMA_CASE

}  // namespace rqc

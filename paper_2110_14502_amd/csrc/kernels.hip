// Step dispatch and the small kernels of the path: slice / bitstring
// instantiation of the leaves (Section 5.1), the FP64 cross-slice reduction
// (Section 6.4), fills, and the unfused permute used as a baseline.
#include "permute_tiles.h"

namespace rqc {

hipError_t launch_step(const StepDesc& d0, int kernel, int sa, int sb, int sc, int lp_kind,
                       hipStream_t s) {
  StepDesc d = d0;
  d.sb_store = sb;
  d.sc_store = sc;
  const uint64_t tiles = (uint64_t)d.n_row_tiles * (uint64_t)d.n_col_tiles;
  const unsigned gy = (unsigned)(d.copies < 65535 ? d.copies : 65535);
  const dim3 grid((unsigned)tiles, gy);
  switch (kernel) {
    case KERN_MFMA16: return launch_mfma16_kernel(d, sa, sb, sc, lp_kind, grid, s);
    case KERN_MFMA: return launch_mfma32_kernel(d, sa, sb, sc, grid, s);
    case KERN_ROWS: return launch_rows_kernel(d, sa, grid, s);
    case KERN_SIMT: return launch_simt_kernel(d, sa, sb, sc, tiles, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Leaf instantiation: fix sliced wires to the bits of the slice id and closed
// selectors to the requested bits (Section 5.1), producing one copy per
// (slice, bitstring) of the group that the leaf depends on.
// ---------------------------------------------------------------------------
// Blocks past the jobs clear the call's flags and the group's scale arrays
// (three launches of 1-4 us with 4-5 us gaps between them before).
__global__ void k_prologue(const LeafJob* jobs, int n_jobs, const float2* store, float2* dst,
                           const uint64_t* slice_ids, const uint8_t* closed, int n_closed, int gs,
                           int gb, int32_t* flags, int64_t n_flags, int32_t* scale,
                           int64_t n_scale) {
  if ((int)blockIdx.x >= n_jobs) {
    const int64_t i0 = (blockIdx.x - n_jobs) * (int64_t)blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)(gridDim.x - n_jobs) * blockDim.x;
    for (int64_t i = i0; i < n_flags; i += step) flags[i] = 0;
    for (int64_t i = i0; i < n_scale; i += step) scale[i] = 0;
    return;
  }
  const LeafJob& J = jobs[blockIdx.x];
  const int ne = 1 << J.rank;
  const int cs = J.dep_s ? gs : 1;
  const int cb = J.dep_b ? gb : 1;
  const int total = ne * cs * cb;
  for (int t = threadIdx.x; t < total; t += blockDim.x) {
    const int e = t % ne;
    const int cp = t / ne;
    const int js = cp % cs, jb = cp / cs;
    int64_t src = J.src;
    for (int i = 0; i < J.rank; ++i)
      if ((e >> i) & 1) src += int64_t(1) << J.pos[i];
    for (int s = 0; s < J.nsel; ++s) {
      int v;
      if (J.sel_src[s] >= 0) v = (int)((slice_ids[js] >> J.sel_src[s]) & 1ull);
      else v = closed[(int64_t)jb * n_closed + (-J.sel_src[s] - 1)] & 1;
      if (v) src += int64_t(1) << J.sel_pos[s];
    }
    dst[J.dst + (int64_t)js * J.out_s + (int64_t)jb * J.out_b + e] = store[src];
  }
}

hipError_t launch_prologue(const LeafJob* jobs_dev, int n_jobs, const void* leaf_store,
                           void* dst_base, const uint64_t* slice_ids, const uint8_t* closed_bits,
                           int n_closed, int gs, int gb, int32_t* flags, int64_t n_flags,
                           int32_t* scale, int64_t n_scale, hipStream_t s) {
  const int64_t n = n_flags > n_scale ? n_flags : n_scale;
  int64_t fill = (n + 255) / 256;
  if (fill > 4096) fill = 4096;
  if (n_jobs + fill <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_prologue, dim3((unsigned)(n_jobs + fill)), dim3(256), 0, s, jobs_dev, n_jobs,
                     reinterpret_cast<const float2*>(leaf_store), reinterpret_cast<float2*>(dst_base),
                     slice_ids, closed_bits, n_closed, gs, gb, flags, n_flags, scale, n_scale);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Cross-slice sum in FP64, fixed order (slice 0, 1, ... of the group; groups
// in call order), skipping slices flagged for an FP32 re-run.
// ---------------------------------------------------------------------------
template <int S>
__global__ void k_slice_sum(const void* root, const int32_t* rexp, int64_t rs, int64_t rb,
                            int32_t res, int32_t reb, int n_elems, int gs, int gb, int dep_s,
                            int dep_b, const int32_t* flags, double* out, double* per_slice,
                            int64_t ps_row0, int64_t n_batch_total, int64_t b0, int first) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)n_elems * gb) return;
  const int e = (int)(t % n_elems);
  const int jb = (int)(t / n_elems);
  const int jbs = dep_b ? jb : 0;
  double sr = 0.0, si = 0.0;
  // Eight slices' values, exponents and flags are read together (their
  // latencies overlap; one slice at a time took 16 us for 32 slices) and added
  // in slice order.
  constexpr int B = 8;
  for (int j0 = 0; j0 < gs; j0 += B) {
    float2 v[B];
    int ex[B], skip[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int js = j0 + i < gs ? j0 + i : gs - 1;
      const int jss = dep_s ? js : 0;
      v[i] = load_c<S>(root, jss * rs + jbs * rb + e);
      ex[i] = rexp ? rexp[jss * res + jbs * reb] : 0;
      skip[i] = flags ? flags[js] : 0;
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int js = j0 + i;
      if (js >= gs) break;
      double vr = 0.0, vi = 0.0;
      if (!skip[i]) {
        vr = ldexp((double)v[i].x, ex[i]);
        vi = ldexp((double)v[i].y, ex[i]);
      }
      sr += vr;
      si += vi;
      if (per_slice && !skip[i]) {
        const int64_t o = (((ps_row0 + js) * n_batch_total + (b0 + jb)) * n_elems + e) * 2;
        per_slice[o] = vr;
        per_slice[o + 1] = vi;
      }
    }
  }
  const int64_t o = ((b0 + jb) * (int64_t)n_elems + e) * 2;
  if (first) {
    out[o] = sr;
    out[o + 1] = si;
  } else {
    out[o] += sr;
    out[o + 1] += si;
  }
}

hipError_t launch_slice_sum(const void* root, int root_store, const int32_t* root_exp,
                            int64_t root_s, int64_t root_b, int32_t re_s, int32_t re_b, int dep_s,
                            int dep_b, int n_elems, int gs, int gb, const int32_t* flags,
                            double* out, double* per_slice, int64_t ps_row0,
                            int64_t n_batch_total, int64_t b0, int first, hipStream_t s) {
  const int64_t n = (int64_t)n_elems * gb;
  const dim3 grid((unsigned)((n + 255) / 256));
  if (root_store == ST_C64)
    hipLaunchKernelGGL(k_slice_sum<ST_C64>, grid, dim3(256), 0, s, root, root_exp, root_s, root_b,
                       re_s, re_b, n_elems, gs, gb, dep_s, dep_b, flags, out, per_slice, ps_row0,
                       n_batch_total, b0, first);
  else if (root_store == ST_F16)
    hipLaunchKernelGGL(k_slice_sum<ST_F16>, grid, dim3(256), 0, s, root, root_exp, root_s, root_b,
                       re_s, re_b, n_elems, gs, gb, dep_s, dep_b, flags, out, per_slice, ps_row0,
                       n_batch_total, b0, first);
  else
    hipLaunchKernelGGL(k_slice_sum<ST_BF16>, grid, dim3(256), 0, s, root, root_exp, root_s, root_b,
                       re_s, re_b, n_elems, gs, gb, dep_s, dep_b, flags, out, per_slice, ps_row0,
                       n_batch_total, b0, first);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small utility kernel: adds an FP32 re-run to the sums that skipped it
// ---------------------------------------------------------------------------
__global__ void k_add_f64(double* d, const double* s, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    d[i] += s[i];
}

static dim3 fill_grid(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return dim3((unsigned)b);
}

hipError_t launch_add_f64(double* dst, const double* src, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_add_f64, fill_grid(n), dim3(256), 0, s, dst, src, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Bit permutation (the separate-permutation baseline; the packing kernels of
// the two-phase contractions share the tile walk): tiles staged through
// LDS so that both the reads (low input bits) and the writes (low output
// bits) are contiguous.  Bound by HBM.
//
// k_permute_tiles (rank >= 12, 16-byte aligned operands): tiles of 2^12
// elements, the lowest six or more bits of the input and of the output, so
// that reads and writes come in runs of 512 bytes and more.  The host sorts
// the bits; a thread's four groups of four elements keep their offsets and
// LDS slots in registers, a tile only moves two uniform bases, and the next
// tile is read before the current one is written.
// Rank 26, random order: 345 us through tables (2^10-element tiles, 3.1 TB/s),
// 226 us here (4.74 TB/s, the rate of a plain copy).
// k_permute serves everything else, tiles of 2^10 elements through tables.
// ---------------------------------------------------------------------------
struct PermDesc {
  int32_t rank;
  int8_t src_of_out[48];  // input bit feeding output bit i
};

__global__ __launch_bounds__(256) void k_permute(const float2* in, float2* out, PermDesc p,
                                                 int lo_in, int lo_out, uint64_t n_blocks) {
  // Tile = the lowest `lo_in` input bits  U  the lowest `lo_out` output bits.
  // The tile's element offsets (relative to the tile base) and LDS slots are
  // tabulated once per workgroup; workgroups stride over the tiles (a grid
  // has at most 2^32 work-items), each tile base a sum over its set bits.
  __shared__ float2 tile[1024 + 32];
  __shared__ int64_t toff_in[1024];   // input offset of tile element t (input order)
  __shared__ int16_t tslot[1024];     // its slot in output order
  __shared__ int64_t toff_out[1024];  // output offset of tile element t (output order)
  __shared__ int64_t bin[48], bout[48];  // input / output offset of outer bit i
  const int r = p.rank;
  int out_of_in[48];
  for (int i = 0; i < r; ++i) out_of_in[p.src_of_out[i]] = i;
  // Tile bits, as output bit indices: the low output bits plus the output
  // bits fed by the low input bits.
  uint64_t tmask = 0;
  for (int i = 0; i < lo_out && i < r; ++i) tmask |= 1ull << i;
  for (int i = 0; i < lo_in && i < r; ++i) tmask |= 1ull << out_of_in[i];
  int tb[20], nt = 0;
  for (int i = 0; i < r; ++i)
    if ((tmask >> i) & 1) tb[nt++] = i;
  int no = 0;
  for (int i = 0; i < r; ++i)
    if (!((tmask >> i) & 1)) {
      if ((int)threadIdx.x == no) {
        bout[no] = int64_t(1) << i;
        bin[no] = int64_t(1) << p.src_of_out[i];
      }
      ++no;
    }
  const int nte = 1 << nt;
  // Tile bits sorted by their input bit: element t of the read phase.
  int tin[20];
  for (int i = 0; i < nt; ++i) tin[i] = p.src_of_out[tb[i]];
  for (int i = 0; i < nt; ++i) {
    int best = i;
    for (int j = i + 1; j < nt; ++j)
      if (tin[j] < tin[best]) best = j;
    const int x = tin[i];
    tin[i] = tin[best];
    tin[best] = x;
  }
  // Slot bit of read-order bit i: the position of its output bit in tb.
  int sbit[20];
  for (int i = 0; i < nt; ++i) {
    const int ob_i = out_of_in[tin[i]];
    sbit[i] = 0;
    for (int j = 0; j < nt; ++j)
      if (tb[j] == ob_i) sbit[i] = j;
  }
  for (int t = threadIdx.x; t < nte; t += blockDim.x) {
    int64_t a = 0;
    int slot = 0;
    for (int i = 0; i < nt; ++i)
      if ((t >> i) & 1) {
        a |= int64_t(1) << tin[i];
        slot |= 1 << sbit[i];
      }
    toff_in[t] = a;
    tslot[t] = (int16_t)slot;
    int64_t o = 0;
    for (int j = 0; j < nt; ++j)
      if ((t >> j) & 1) o |= int64_t(1) << tb[j];
    toff_out[t] = o;
  }
  __syncthreads();
  for (uint64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
    int64_t base_in = 0, base_out = 0;
    for (uint64_t b = blk; b; b &= b - 1) {
      const int i = __builtin_ctzll(b);
      base_in += bin[i];
      base_out += bout[i];
    }
    for (int t = threadIdx.x; t < nte; t += blockDim.x) {
      const int sl = tslot[t];
      tile[sl + (sl >> 5)] = in[base_in + toff_in[t]];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nte; t += blockDim.x)
      out[base_out + toff_out[t]] = tile[t + (t >> 5)];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_permute_tiles(const float2* in, float2* out, PermTiles p,
                                                       uint32_t n_iter) {
  permute_tiles(in, p, blockIdx.x, n_iter, [&](int64_t o, float2 a, float2 b, float2 c, float2 e) {
    float4* q = reinterpret_cast<float4*>(out + o);
    q[0] = make_float4(a.x, a.y, b.x, b.y);
    q[1] = make_float4(c.x, c.y, e.x, e.y);
  });
}

hipError_t launch_permute(const void* in, void* out, int rank, const int8_t* src_pos_of_out_bit,
                          hipStream_t s) {
  PermDesc p;
  p.rank = rank;
  for (int i = 0; i < rank; ++i) p.src_of_out[i] = src_pos_of_out_bit[i];
  const float2* src = reinterpret_cast<const float2*>(in);
  float2* dst = reinterpret_cast<float2*>(out);
  PermTiles t;
  uint32_t tgrid, n_iter;
  if ((reinterpret_cast<uintptr_t>(in) & 15) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0 &&
      plan_permute_tiles(rank, src_pos_of_out_bit, t, tgrid, n_iter)) {
    t.aligned = 1;
    hipLaunchKernelGGL(k_permute_tiles, dim3(tgrid), dim3(256), 0, s, src, dst, t, n_iter);
    return hipGetLastError();
  }
  // The lo_in lowest input bits and the lo_out lowest output bits: both grown
  // alternately while the union fits ten bits.
  int out_of_in[48];
  for (int i = 0; i < rank; ++i) out_of_in[(int)p.src_of_out[i]] = i;
  auto tile_bits = [&](int li, int lo) {
    uint64_t m = 0;
    for (int i = 0; i < lo; ++i) m |= 1ull << i;
    for (int i = 0; i < li; ++i) m |= 1ull << out_of_in[i];
    return __builtin_popcountll(m);
  };
  int lo_in = 0, lo_out = 0;
  for (bool grew = true; grew;) {
    grew = false;
    if (lo_out < rank && tile_bits(lo_in, lo_out + 1) <= 10) ++lo_out, grew = true;
    if (lo_in < rank && tile_bits(lo_in + 1, lo_out) <= 10) ++lo_in, grew = true;
  }
  const uint64_t blocks = 1ull << (rank - tile_bits(lo_in, lo_out));
  // Eight workgroups per CU, each walking many tiles (its tables are built
  // once).
  const uint64_t grid = blocks < 2048 ? blocks : 2048;
  hipLaunchKernelGGL(k_permute, dim3((unsigned)grid), dim3(256), 0, s, src, dst, p, lo_in, lo_out,
                     blocks);
  return hipGetLastError();
}

}  // namespace rqc

namespace rqc {

// ---------------------------------------------------------------------------
// Statistics of an amplitude batch in FP64 (fixed summation order, so the result
// does not depend on timing): sum |a|^2, sum |a|^4, and the linear cross-entropy
// values derived from them; optionally the mean |a|^2 over sampled entries of the
// batch (bounds-checked: an index outside the batch makes that result NaN).
//
// Batches of 2^17 amplitudes and more are read by many workgroups
// (rqc_batch_xeb_ws): each writes four partial sums, and one workgroup adds
// them in workgroup order; the split depends on the batch size alone.  One
// workgroup reads 56 GB/s (601 us for 2^21 amplitudes, 33 MB; 32 us split), and
// up to 2^16 amplitudes stay in its reach: whole calls 30 us either way at 2^16, 36
// against 31 us at 2^17, 24 against 29 us at 2^10.
// ---------------------------------------------------------------------------
constexpr int kStatThreads = 1024;

struct Stats {
  double s1, s2, s3;  // sum p, sum p^2, sum p over samples
  int bad;            // a sample index outside the batch
};

// Sums over entries first, first + stride, ... and the samples likewise.
__device__ __forceinline__ Stats stat_range(const double* amps, uint64_t n, const uint64_t* samples,
                                            uint64_t n_samples, uint64_t first, uint64_t stride) {
  typedef double d2v __attribute__((ext_vector_type(2)));
  Stats v{0.0, 0.0, 0.0, 0};
  // Amplitudes are read as aligned 16-byte pairs where the buffer allows it,
  // eight in flight per thread.
  uint64_t i = first;
  if ((reinterpret_cast<uintptr_t>(amps) & 15) == 0) {
    const d2v* q = reinterpret_cast<const d2v*>(amps);
    for (; i + 7 * stride < n; i += 8 * stride) {
      d2v a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = q[i + u * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double p = a[u][0] * a[u][0] + a[u][1] * a[u][1];
        v.s1 += p;
        v.s2 += p * p;
      }
    }
  }
  for (; i < n; i += stride) {
    const double re = amps[2 * i], im = amps[2 * i + 1];
    const double p = re * re + im * im;
    v.s1 += p;
    v.s2 += p * p;
  }
  for (uint64_t j = first; j < n_samples; j += stride) {
    const uint64_t i = samples[j];
    if (i >= n) {
      v.bad = 1;
      continue;
    }
    const double re = amps[2 * i], im = amps[2 * i + 1];
    v.s3 += re * re + im * im;
  }
  return v;
}

// Sum over the workgroup in a fixed tree order; valid in thread 0.
template <int T>
__device__ __forceinline__ Stats stat_reduce(Stats v) {
  __shared__ double r1[T], r2[T], r3[T];
  __shared__ int bad_any[T];
  const int t = threadIdx.x;
  r1[t] = v.s1;
  r2[t] = v.s2;
  r3[t] = v.s3;
  bad_any[t] = v.bad;
  __syncthreads();
  for (int w = T / 2; w > 0; w >>= 1) {
    if (t < w) {
      r1[t] += r1[t + w];
      r2[t] += r2[t + w];
      r3[t] += r3[t + w];
      bad_any[t] |= bad_any[t + w];
    }
    __syncthreads();
  }
  return Stats{r1[0], r2[0], r3[0], bad_any[0]};
}

__device__ __forceinline__ void stat_write(const Stats& v, uint64_t n, double dim, uint64_t n_samples,
                                           double* out) {
  out[0] = v.s1;
  out[1] = v.s2;
  out[2] = n ? dim * v.s1 / (double)n - 1.0 : 0.0;  // all entries taken as samples
  out[3] = v.s1 > 0.0 ? dim * v.s2 / v.s1 - 1.0 : 0.0;  // entries drawn with p = |a|^2
  out[4] = n_samples == 0 ? 0.0
           : (v.bad ? __builtin_nan("") : dim * v.s3 / (double)n_samples - 1.0);
}

__global__ __launch_bounds__(kStatThreads) void k_batch_stats(const double* amps, uint64_t n,
                                                               double dim, const uint64_t* samples,
                                                               uint64_t n_samples, double* out) {
  const Stats v =
      stat_reduce<kStatThreads>(stat_range(amps, n, samples, n_samples, threadIdx.x, kStatThreads));
  if (threadIdx.x == 0) stat_write(v, n, dim, n_samples, out);
}

__global__ __launch_bounds__(256) void k_batch_stats_part(const double* amps, uint64_t n,
                                                          const uint64_t* samples,
                                                          uint64_t n_samples, double* part) {
  const Stats v = stat_reduce<256>(stat_range(amps, n, samples, n_samples,
                                              (uint64_t)blockIdx.x * 256 + threadIdx.x,
                                              (uint64_t)gridDim.x * 256));
  if (threadIdx.x == 0) {
    double* p = part + 4 * (uint64_t)blockIdx.x;
    p[0] = v.s1;
    p[1] = v.s2;
    p[2] = v.s3;
    p[3] = v.bad ? 1.0 : 0.0;
  }
}

__global__ __launch_bounds__(256) void k_batch_stats_sum(const double* part, int n_part, uint64_t n,
                                                         double dim, uint64_t n_samples, double* out) {
  Stats v{0.0, 0.0, 0.0, 0};
  for (int i = threadIdx.x; i < n_part; i += 256) {
    v.s1 += part[4 * i];
    v.s2 += part[4 * i + 1];
    v.s3 += part[4 * i + 2];
    v.bad |= part[4 * i + 3] != 0.0;
  }
  v = stat_reduce<256>(v);
  if (threadIdx.x == 0) stat_write(v, n, dim, n_samples, out);
}

// Workgroups of the split form: 2048 amplitudes (32 KB) or samples each, at
// most four per CU; 0 below 2^17.
static int stat_blocks(uint64_t n, uint64_t n_samples) {
  const uint64_t most = n > n_samples ? n : n_samples;
  if (most < (uint64_t(1) << 17)) return 0;
  const uint64_t b = (most + 2047) / 2048;
  return (int)(b < 1024 ? b : 1024);
}

uint64_t batch_stats_workspace(uint64_t n, uint64_t n_samples) {
  return 32 * (uint64_t)stat_blocks(n, n_samples);
}

hipError_t launch_batch_stats(const double* amps, uint64_t n, int n_qubits, const uint64_t* samples,
                              uint64_t n_samples, double* out, void* ws, hipStream_t s) {
  const double dim = ldexp(1.0, n_qubits);
  const int blocks = ws ? stat_blocks(n, n_samples) : 0;
  if (blocks == 0) {
    hipLaunchKernelGGL(k_batch_stats, dim3(1), dim3(kStatThreads), 0, s, amps, n, dim, samples,
                       n_samples, out);
    return hipGetLastError();
  }
  double* part = static_cast<double*>(ws);
  hipLaunchKernelGGL(k_batch_stats_part, dim3((unsigned)blocks), dim3(256), 0, s, amps, n, samples,
                     n_samples, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_batch_stats_sum, dim3(1), dim3(256), 0, s, part, blocks, n, dim, n_samples, out);
  return hipGetLastError();
}

}  // namespace rqc

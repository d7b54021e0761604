// Tile walk of a bit permutation (k_permute_tiles and the packing kernels):
// the host's choice of the tile and the device loop, which hands groups of
// four consecutive output elements to a writer.
#pragma once

#include "kernels_dev.h"

namespace rqc {

constexpr int kPermBits = 12;                              // tile bits
constexpr int kPermGroups = (1 << kPermBits) / (4 * 256);  // groups of four elements per thread
struct PermTiles {
  int32_t n_outer;
  int32_t gbits;            // 2^gbits workgroups walk the tiles
  int32_t aligned;          // the input is 16-byte aligned
  int8_t tin[kPermBits];    // input address bit of read-order bit i (ascending)
  int8_t slot[kPermBits];   // output-order bit of read-order bit i
  int8_t tout[kPermBits];   // output address bit of output-order bit i (ascending)
  int8_t oin[48], oout[48]; // input / output address bit of outer bit i
};

// LDS element of output-order index s: two elements of padding per 32.
__device__ __forceinline__ int perm_pad(int s) { return s + 2 * (s >> 5); }

// 256 threads, workgroup `block` of the 2^gbits; put(o, a, b, c, e) stores output
// elements o .. o + 3.
template <class Put>
__device__ __forceinline__ void permute_tiles(const float2* in, const PermTiles& p, uint32_t block,
                                              uint32_t n_iter, Put put) {
  __shared__ __attribute__((aligned(16))) float2 tile[(1 << kPermBits) + 2 * (1 << (kPermBits - 5))];
  __shared__ int64_t step_in[32], step_out[32];
  const int tid = threadIdx.x;
  // Tile of iteration i: outer bits block + 2^gbits i; i -> i + 1 moves the
  // bases by step[ctz(i + 1)].
  const int gbits = p.gbits;
  if (tid < p.n_outer - gbits) {
    int64_t si = int64_t(1) << p.oin[gbits + tid], so = int64_t(1) << p.oout[gbits + tid];
    for (int j = 0; j < tid; ++j) {
      si -= int64_t(1) << p.oin[gbits + j];
      so -= int64_t(1) << p.oout[gbits + j];
    }
    step_in[tid] = si;
    step_out[tid] = so;
  }
  int64_t base_in = 0, base_out = 0;
  for (int b = 0; b < gbits; ++b)
    if ((block >> b) & 1u) {
      base_in += int64_t(1) << p.oin[b];
      base_out += int64_t(1) << p.oout[b];
    }
  // Group g of this thread: read-order elements 4 (tid + 256 g) .. + 3, and
  // the same indices in output order.
  int64_t off_in = 0, off_out = 0;
  int slot_t = 0;
#pragma unroll
  for (int b = 0; b < 8; ++b)
    if ((tid >> b) & 1) {
      off_in += int64_t(1) << p.tin[2 + b];
      off_out += int64_t(1) << p.tout[2 + b];
      slot_t += perm_pad(1 << p.slot[2 + b]);
    }
  int64_t gin[kPermGroups], gout[kPermGroups];
  int gslot[kPermGroups], eslot[4];
#pragma unroll
  for (int g = 0; g < kPermGroups; ++g) {
    gin[g] = gout[g] = 0;
    gslot[g] = 0;
#pragma unroll
    for (int b = 0; b < 2; ++b)
      if ((g >> b) & 1) {
        gin[g] += int64_t(1) << p.tin[10 + b];
        gout[g] += int64_t(1) << p.tout[10 + b];
        gslot[g] += perm_pad(1 << p.slot[10 + b]);
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    eslot[e] = ((e & 1) ? perm_pad(1 << p.slot[0]) : 0) + ((e & 2) ? perm_pad(1 << p.slot[1]) : 0);
  float4 v[kPermGroups][2];
  auto load = [&]() {
#pragma unroll
    for (int g = 0; g < kPermGroups; ++g) {
      const float2* q = in + base_in + off_in + gin[g];
      if (p.aligned) {
        const float4* src = reinterpret_cast<const float4*>(q);
        v[g][0] = src[0];
        v[g][1] = src[1];
      } else {
        const float2 a = q[0], b = q[1], c = q[2], e = q[3];
        v[g][0] = make_float4(a.x, a.y, b.x, b.y);
        v[g][1] = make_float4(c.x, c.y, e.x, e.y);
      }
    }
  };
  load();
  __syncthreads();
  for (uint32_t i = 0; i < n_iter; ++i) {
#pragma unroll
    for (int g = 0; g < kPermGroups; ++g) {
      const int s = slot_t + gslot[g];
      tile[s + eslot[0]] = make_float2(v[g][0].x, v[g][0].y);
      tile[s + eslot[1]] = make_float2(v[g][0].z, v[g][0].w);
      tile[s + eslot[2]] = make_float2(v[g][1].x, v[g][1].y);
      tile[s + eslot[3]] = make_float2(v[g][1].z, v[g][1].w);
    }
    __syncthreads();
    const int64_t bo = base_out + off_out;
    if (i + 1 < n_iter) {
      const int b = __builtin_ctz(i + 1);
      base_in += step_in[b];
      base_out += step_out[b];
      load();
    }
#pragma unroll
    for (int g = 0; g < kPermGroups; ++g) {
      const float4* src = reinterpret_cast<const float4*>(tile + perm_pad(4 * (tid + 256 * g)));
      const float4 a = src[0], c = src[1];
      put(bo + gout[g], make_float2(a.x, a.y), make_float2(a.z, a.w), make_float2(c.x, c.y),
          make_float2(c.z, c.w));
    }
    __syncthreads();
  }
}

// The tile: the lo_in lowest input bits and the lo_out lowest output bits,
// both grown alternately while the union holds at most kPermBits bits, so a
// permutation that keeps its low bits still gets full tiles.  From rank 12 on
// the union always fills up (each step adds at most one bit), with at least
// six low bits of both sides.  At most 1024 workgroups (four per CU), each
// walking n_iter tiles.  src_of_out: input bit of each output bit.
inline bool plan_permute_tiles(int rank, const int8_t* src_of_out, PermTiles& t, uint32_t& grid,
                               uint32_t& n_iter) {
  if (rank < kPermBits || rank > 48) return false;
  int out_of_in[48];
  for (int i = 0; i < rank; ++i) out_of_in[(int)src_of_out[i]] = i;
  auto tile_mask = [&](int li, int lo) {  // as output bits
    uint64_t m = 0;
    for (int i = 0; i < lo; ++i) m |= 1ull << i;
    for (int i = 0; i < li; ++i) m |= 1ull << out_of_in[i];
    return m;
  };
  int lo_in = 0, lo_out = 0;
  for (bool grew = true; grew;) {
    grew = false;
    if (lo_out < rank && __builtin_popcountll(tile_mask(lo_in, lo_out + 1)) <= kPermBits) ++lo_out, grew = true;
    if (lo_in < rank && __builtin_popcountll(tile_mask(lo_in + 1, lo_out)) <= kPermBits) ++lo_in, grew = true;
  }
  const uint64_t m = tile_mask(lo_in, lo_out);
  if (__builtin_popcountll(m) != kPermBits || lo_in < 2 || lo_out < 2) return false;
  int no = 0, nb = 0, inb[kPermBits];
  for (int i = 0; i < rank; ++i) {
    if ((m >> i) & 1) {
      t.tout[nb] = (int8_t)i;
      inb[nb++] = src_of_out[i];
    } else {
      t.oin[no] = src_of_out[i];
      t.oout[no++] = (int8_t)i;
    }
  }
  t.n_outer = no;
  for (int i = 0; i < kPermBits; ++i) {  // read order: by input bit
    int at = 0;
    for (int j = 0; j < kPermBits; ++j) at += inb[j] < inb[i];
    t.tin[at] = (int8_t)inb[i];
    t.slot[at] = (int8_t)i;
  }
  t.gbits = no < 10 ? no : 10;
  grid = 1u << t.gbits;
  n_iter = 1u << (no - t.gbits);
  return true;
}

}  // namespace rqc

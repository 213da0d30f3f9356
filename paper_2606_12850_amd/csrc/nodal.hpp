// The points of a node and their sum: device maps shared by the kernels that
// work node by node on element-local values.
#pragma once
#include "semx_internal.hpp"

namespace semx {
namespace {

constexpr int kNodeT = 256;  // lanes of a node kernel's blocks

// ---------------------------------------------------------------------------
// Nodal sums.  One lane per node, all its components; row y of the grid is
// model y.  What bounds them is latency: a node's loads depend on its point
// numbers, so the numbers come from the lattice where the mesh is one (one
// round trip: every load of a node is issued at once), and from the tables,
// four points at a time, elsewhere (three round trips).  Blocks are dealt so
// that an XCD takes one contiguous eighth, the share of the mesh whose
// element kernels it ran.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t xcd_block(uint32_t nblk) {
  const uint32_t per = (nblk + kNumXcd - 1) / kNumXcd;
  return (blockIdx.x % kNumXcd) * per + blockIdx.x / kNumXcd;
}

__device__ __forceinline__ uint32_t div(uint32_t x, const FastDiv& d) { return (__umulhi(x, d.m) + x) >> d.s; }

// Any mesh: the points of node g from the tables.
struct TableMap {
  const int32_t* ptr;
  const int32_t* idx;
  int64_t nglob;
  uint32_t nblk;

  __device__ __forceinline__ bool locate(int64_t& g) {
    g = (int64_t)xcd_block(nblk) * kNodeT + threadIdx.x;
    return g < nglob;
  }
  template <class T, int NC>
  __device__ __forceinline__ void sum(const T* __restrict__ pm, int64_t g, T s[NC]) const {
    const int32_t b = ptr[g], e = ptr[g + 1];
    for (int32_t k = b; k < e; k += 4) {
      T v[4][NC];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const T* p = pm + (int64_t)idx[min(k + q, e - 1)] * NC;
#pragma unroll
        for (int c = 0; c < NC; ++c) v[q][c] = p[c];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (k + q < e) {
#pragma unroll
          for (int c = 0; c < NC; ++c) s[c] += v[q][c];
        }
    }
  }
  // fn(point) for the node's points in their order
  template <class F>
  __device__ __forceinline__ void each(int64_t g, F fn) const {
    for (int32_t k = ptr[g]; k < ptr[g + 1]; ++k) fn(idx[k]);
  }
};

// A box of nex x ney x nez elements on one node lattice, x fastest: node
// (gx, gy, gz) belongs to one or two elements per axis, and colours are the
// parities of the element indices (checked when the mesh is laid out), so an
// axis takes its even element first.  Point numbers are sums of one offset
// per axis.  A block covers tx x (256 / tx) nodes of one z plane.
struct LatticeMap {
  Lattice L;
  int ox[2], oy[2], oz[2];
  bool x2, y2, z2;

  __device__ __forceinline__ bool axis(int g, int ne, int se, int si, int o[2]) const {
    const int N = L.n - 1;
    const int e = (int)div((uint32_t)g, L.dn), i = g - e * N;
    const bool two = i == 0 && e > 0 && e < ne;
    const int lo = (e - 1) * se + N * si, hi = e * se + i * si;  // lo: the last point of the element below
    const bool low_only = e == ne;                               // the last node of the axis
    const bool odd = (e & 1) != 0;
    o[0] = low_only || (two && odd) ? lo : hi;
    o[1] = odd ? hi : lo;
    return two;
  }
  __device__ __forceinline__ bool locate(int64_t& g) {
    const uint32_t t = xcd_block(L.ntiles);
    if (t >= L.ntiles) return false;
    const uint32_t gz = div(t, L.dplane), r = t - gz * (L.ntx * L.nty);
    const uint32_t by = div(r, L.drow), bx = r - by * L.ntx;
    const int gx = (int)(bx << L.txs) + ((int)threadIdx.x & ((1 << L.txs) - 1));
    const int gy = (int)(by << (8 - L.txs)) + ((int)threadIdx.x >> L.txs);
    if (gx >= L.Gx || gy >= L.Gy) return false;
    const int n3 = L.n * L.n * L.n;
    x2 = axis(gx, L.nex, n3, 1, ox);
    y2 = axis(gy, L.ney, L.nex * n3, L.n, oy);
    z2 = axis((int)gz, L.nez, L.nex * L.ney * n3, L.n * L.n, oz);
    g = gx + (int64_t)L.Gx * (gy + (int64_t)L.Gy * gz);
    return true;
  }
  template <class T, int NC>
  __device__ __forceinline__ void sum(const T* __restrict__ pm, int64_t, T s[NC]) const {
    T v[2][2][2][NC];
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
          for (int c = 0; c < NC; ++c) v[z][y][x][c] = 0;
          if ((!z || z2) && (!y || y2) && (!x || x2)) {
            const T* p = pm + (int64_t)(oz[z] + oy[y] + ox[x]) * NC;
#pragma unroll
            for (int c = 0; c < NC; ++c) v[z][y][x][c] = p[c];
          }
        }
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int c = 0; c < NC; ++c) s[c] += v[z][y][x][c];
  }
  template <class F>
  __device__ __forceinline__ void each(int64_t, F fn) const {
    for (int z = 0; z <= (z2 ? 1 : 0); ++z)
      for (int y = 0; y <= (y2 ? 1 : 0); ++y)
        for (int x = 0; x <= (x2 ? 1 : 0); ++x)
          fn((z ? oz[1] : oz[0]) + (y ? oy[1] : oy[0]) + (x ? ox[1] : ox[0]));
  }
};

__device__ __forceinline__ bool has_bit(const uint32_t* __restrict__ bits, int64_t g) {
  return bits && ((bits[g >> 5] >> (g & 31)) & 1u);
}

inline uint32_t node_blocks(int64_t n) { return (uint32_t)((n + kNodeT - 1) / kNodeT); }

// Calls fn(map, grid) with the context's node map.
template <class F>
hipError_t with_map(const semx_ctx* c, F fn) {
  if (c->lattice.n > 0) {
    const uint32_t nb = (c->lattice.ntiles + kNumXcd - 1) / kNumXcd * kNumXcd;
    LatticeMap m;
    m.L = c->lattice;
    fn(m, dim3(nb, (unsigned)c->nmodels));
  } else {
    const uint32_t nblk = node_blocks(c->nglob);
    fn(TableMap{c->d_nptr.as<int32_t>(), c->d_nidx.as<int32_t>(), c->nglob, nblk},
       dim3((nblk + kNumXcd - 1) / kNumXcd * kNumXcd, (unsigned)c->nmodels));
  }
  return hipGetLastError();
}

}  // namespace
}  // namespace semx

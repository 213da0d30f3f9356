// Node tables and nodal sums: the points of every node, and the assembly of
// element-local values by the nodes that own them (Sec. IV-C asks for an
// assembly without conflicting updates).
//
// The element kernels store the forces of their own points, and one lane per
// node value adds its node's points: no two writers meet, and a force pass is
// one launch over the whole mesh and one gather instead of one launch per
// colour.  The points are added in the order in which a pass colour by colour
// would reach the node, so the sums are those of that pass to the bit.
#include <algorithm>

#include "newmark.hpp"
#include "nodal.hpp"

namespace semx {
namespace {

constexpr int kT = kNodeT;
constexpr int kScanItems = 16;  // per lane
constexpr int kScanTile = kT * kScanItems;

__global__ __launch_bounds__(kT) void count_points_kernel(int64_t npt, const int32_t* __restrict__ ibool,
                                                          int32_t* __restrict__ count) {
  for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < npt; t += (int64_t)gridDim.x * kT)
    atomicAdd(count + ibool[t], 1);
}

__global__ __launch_bounds__(kT) void zero_int_kernel(int64_t n, int32_t* __restrict__ p) {
  for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kT) p[t] = 0;
}

__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* tmp, int32_t* total) {
  const int t = threadIdx.x;
  tmp[t] = v;
  __syncthreads();
  for (int d = 1; d < kT; d <<= 1) {
    const int32_t x = t >= d ? tmp[t - d] : 0;
    __syncthreads();
    tmp[t] += x;
    __syncthreads();
  }
  const int32_t incl = tmp[t];
  *total = tmp[kT - 1];
  __syncthreads();
  return incl - v;
}

// sums[b] = sum of tile b of x
__global__ __launch_bounds__(kT) void tile_sum_kernel(int64_t n, const int32_t* __restrict__ x,
                                                      int32_t* __restrict__ sums) {
  __shared__ int32_t tmp[kT];
  int32_t s = 0;
  const int64_t t0 = blockIdx.x * (int64_t)kScanTile + threadIdx.x * (int64_t)kScanItems;
  for (int e = 0; e < kScanItems; ++e)
    if (t0 + e < n) s += x[t0 + e];
  int32_t total;
  block_exclusive_scan(s, tmp, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// exclusive scan of the tile sums, one workgroup
__global__ __launch_bounds__(kT) void scan_sums_kernel(int nb, int32_t* __restrict__ sums) {
  __shared__ int32_t tmp[kT];
  int32_t carry = 0;
  for (int b0 = 0; b0 < nb; b0 += kT) {
    const int b = b0 + threadIdx.x;
    const int32_t v = b < nb ? sums[b] : 0;
    int32_t total;
    const int32_t ex = block_exclusive_scan(v, tmp, &total);
    if (b < nb) sums[b] = carry + ex;
    carry += total;
  }
}

// ptr[t] = exclusive scan of x over [0, n), ptr[n] = total; cursor = ptr (may
// be x: a lane reads its items before it writes them)
__global__ __launch_bounds__(kT) void scan_tiles_kernel(int64_t n, const int32_t* x,
                                                        const int32_t* __restrict__ sums, int32_t* __restrict__ ptr,
                                                        int32_t* cursor) {
  __shared__ int32_t tmp[kT];
  const int64_t t0 = blockIdx.x * (int64_t)kScanTile + threadIdx.x * (int64_t)kScanItems;
  int32_t v[kScanItems], s = 0;
  for (int e = 0; e < kScanItems; ++e) {
    v[e] = t0 + e < n ? x[t0 + e] : 0;
    s += v[e];
  }
  int32_t total;
  int32_t at = sums[blockIdx.x] + block_exclusive_scan(s, tmp, &total);
  for (int e = 0; e < kScanItems; ++e) {
    if (t0 + e < n) {
      ptr[t0 + e] = at;
      cursor[t0 + e] = at;
    }
    at += v[e];
    if (t0 + e == n - 1) ptr[n] = at;
  }
}

__global__ __launch_bounds__(kT) void place_points_kernel(int64_t npt, const int32_t* __restrict__ ibool,
                                                          int32_t* __restrict__ cursor, int32_t* __restrict__ idx) {
  for (int64_t t = blockIdx.x * (int64_t)kT + threadIdx.x; t < npt; t += (int64_t)gridDim.x * kT)
    idx[atomicAdd(cursor + ibool[t], 1)] = (int32_t)t;
}

// Each node's points in ascending order of their element's rank: by insertion
// where they are few, as on any ordinary mesh; the points of a node that very many
// elements share (the axis of a fan) come in no order and go through a heap, so
// that the lane ends in n log n.
constexpr int32_t kInsertion = 32;
__global__ __launch_bounds__(kT) void sort_points_kernel(int64_t nglob, int n3, const int32_t* __restrict__ rank,
                                                         const int32_t* __restrict__ ptr, int32_t* __restrict__ idx) {
  auto before = [&](int32_t x, int32_t y) {
    const int32_t rx = rank[x / n3], ry = rank[y / n3];
    return rx != ry ? rx < ry : x < y;
  };
  for (int64_t g = blockIdx.x * (int64_t)kT + threadIdx.x; g < nglob; g += (int64_t)gridDim.x * kT) {
    const int32_t b = ptr[g], e = ptr[g + 1];
    if (e - b > kInsertion) {
      int32_t* h = idx + b;
      auto sift = [&](int32_t at, int32_t n) {
        const int32_t v = h[at];
        for (int32_t k; (k = 2 * at + 1) < n; at = k) {
          if (k + 1 < n && before(h[k], h[k + 1])) ++k;
          if (!before(v, h[k])) break;
          h[at] = h[k];
        }
        h[at] = v;
      };
      for (int32_t i = (e - b) / 2 - 1; i >= 0; --i) sift(i, e - b);
      for (int32_t n = e - b - 1; n > 0; --n) {
        const int32_t top = h[0];
        h[0] = h[n];
        h[n] = top;
        sift(0, n);
      }
      continue;
    }
    for (int32_t i = b + 1; i < e; ++i) {
      const int32_t v = idx[i];
      int32_t j = i - 1;
      for (; j >= b && before(v, idx[j]); --j) idx[j + 1] = idx[j];
      idx[j + 1] = v;
    }
  }
}

// f = sum of the node's points (from the prior f at the nodes of srcbits)
template <class T, int NC, class MAP>
__global__ __launch_bounds__(kT) void gather_kernel(MAP m, int64_t nglob, int64_t npt, const T* __restrict__ part,
                                                    const uint32_t* __restrict__ srcbits, T* __restrict__ f) {
  int64_t g;
  if (!m.locate(g)) return;
  T* fg = f + ((int64_t)blockIdx.y * nglob + g) * NC;
  T s[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) s[c] = 0;
  if (has_bit(srcbits, g)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) s[c] = fg[c];
  }
  m.template sum<T, NC>(part + (int64_t)blockIdx.y * npt * NC, g, s);
#pragma unroll
  for (int c = 0; c < NC; ++c) fg[c] = s[c];
}

// The time loop's Newmark pass on element-local forces: f^n of the node is
// summed in registers (from f at the nodes of srcbits, which holds the source
// force there) and applied at once, so it is neither written nor read back.
template <class T, int NC, class MAP, int MODE>
__global__ __launch_bounds__(kT) void newmark_parts_kernel(MAP m, int64_t nglob, int64_t npt, T dt,
                                                           const T* __restrict__ part,
                                                           const uint32_t* __restrict__ srcbits,
                                                           const T* __restrict__ f, const T* __restrict__ minv,
                                                           T* __restrict__ u, T* __restrict__ v, T* __restrict__ seg_u,
                                                           T* __restrict__ seg_a) {
  static_assert((MODE & ~kSeg) == (kCorrect | kPredict), "a step of the loop");
  int64_t g;
  if (!m.locate(g)) return;
  const int64_t at = (int64_t)blockIdx.y * nglob + g;
  T uu[NC], vv[NC], s[NC];
  const T mi = minv[at];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    uu[c] = u[at * NC + c];
    vv[c] = v[at * NC + c];
    s[c] = 0;
  }
  if (has_bit(srcbits, g)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) s[c] = f[at * NC + c];
  }
  m.template sum<T, NC>(part + (int64_t)blockIdx.y * npt * NC, g, s);
  const T hdt = (T)0.5 * dt, hdt2 = (T)0.5 * dt * dt;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const T acc = newmark_entry<MODE, T>(mi, s[c], (T)0, dt, hdt, hdt2, uu[c], vv[c]);
    u[at * NC + c] = uu[c];
    v[at * NC + c] = vv[c];
    if constexpr ((MODE & kSeg) != 0) {
      if (seg_u) seg_u[at * NC + c] = uu[c];
      if (seg_a) seg_a[at * NC + c] = acc;
    }
  }
}

template <class MAP>
__global__ __launch_bounds__(kT) void mass_kernel(MAP m, int n3, int64_t nspec, int64_t nglob,
                                                  const int32_t* __restrict__ order, const double* __restrict__ rho,
                                                  const double* __restrict__ wdet, double* __restrict__ mass) {
  int64_t g;
  if (!m.locate(g)) return;
  const double* __restrict__ rm = rho + (int64_t)blockIdx.y * nspec * n3;
  double s = 0.0;
  m.each(g, [&](int32_t t) {
    const int32_t pos = t / n3;
    s = fma(rm[(int64_t)order[pos] * n3 + (t - pos * n3)], wdet[t], s);  // the same bits on every map
  });
  mass[(int64_t)blockIdx.y * nglob + g] = s;
}

}  // namespace

int build_node_points(semx_ctx* c) {
  if (c->lattice.n > 0) {  // the points follow from the node's place
    dev_free(c->d_nptr);
    dev_free(c->d_nidx);
    return SEMX_OK;
  }
  // rank of each position: its place colour by colour (or itself)
  std::vector<int32_t> rank(c->nspec);
  for (int64_t t = 0; t < c->nspec; ++t) rank[c->h_clist.empty() ? t : c->h_clist[t]] = (int32_t)t;
  const int64_t npt = c->nspec * c->n3, nglob = c->nglob;
  const int nb = (int)((nglob + kScanTile - 1) / kScanTile);
  DevBuf count, sums, drank;
  int rc = dev_alloc(c, c->d_nptr, sizeof(int32_t) * (nglob + 1));
  if (!rc) rc = dev_alloc(c, c->d_nidx, sizeof(int32_t) * npt);
  if (!rc) rc = dev_alloc(c, count, sizeof(int32_t) * nglob);
  if (!rc) rc = dev_alloc(c, sums, sizeof(int32_t) * nb);
  if (!rc) rc = dev_alloc(c, drank, sizeof(int32_t) * c->nspec);
  if (!rc) {
    const int32_t* ib = c->d_ibool.as<int32_t>();
    zero_int_kernel<<<grid_1d(nglob, 4096), kT, 0, c->stream>>>(nglob, count.as<int32_t>());
    count_points_kernel<<<grid_1d(npt, 8192), kT, 0, c->stream>>>(npt, ib, count.as<int32_t>());
    tile_sum_kernel<<<nb, kT, 0, c->stream>>>(nglob, count.as<int32_t>(), sums.as<int32_t>());
    scan_sums_kernel<<<1, kT, 0, c->stream>>>(nb, sums.as<int32_t>());
    // the tile scan reads a tile of `count` before it overwrites it with the cursors
    scan_tiles_kernel<<<nb, kT, 0, c->stream>>>(nglob, count.as<int32_t>(), sums.as<int32_t>(), c->d_nptr.as<int32_t>(),
                                                count.as<int32_t>());
    place_points_kernel<<<grid_1d(npt, 8192), kT, 0, c->stream>>>(npt, ib, count.as<int32_t>(), c->d_nidx.as<int32_t>());
    hipError_t e = hipMemcpyAsync(drank.p, rank.data(), sizeof(int32_t) * c->nspec, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) {
      sort_points_kernel<<<grid_1d(nglob, 8192), kT, 0, c->stream>>>(nglob, c->n3, drank.as<int32_t>(),
                                                                     c->d_nptr.as<int32_t>(), c->d_nidx.as<int32_t>());
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) rc = hip_fail(c, e, "node tables");
  }
  dev_free(count);
  dev_free(sums);
  dev_free(drank);
  return rc;
}

namespace {

template <class T, int NC>
hipError_t gather_t(const semx_ctx* c, T* f, const uint32_t* srcbits, hipStream_t s) {
  return with_map(c, [&](auto m, dim3 grid) {
    gather_kernel<T, NC, decltype(m)><<<grid, kT, 0, s>>>(m, c->nglob, c->nspec * c->n3, c->d_part.as<T>(), srcbits, f);
  });
}

template <class T, int NC, int MODE>
hipError_t newmark_t(const semx_ctx* c, T dt, const T* minv, const uint32_t* srcbits, T* seg_u, T* seg_a,
                     hipStream_t s) {
  return with_map(c, [&](auto m, dim3 grid) {
    newmark_parts_kernel<T, NC, decltype(m), MODE><<<grid, kT, 0, s>>>(
        m, c->nglob, c->nspec * c->n3, dt, c->d_part.as<T>(), srcbits, c->d_f.as<T>(), minv, c->d_u.as<T>(),
        c->d_v.as<T>(), seg_u, seg_a);
  });
}

// Division by an invariant divisor as a multiplication and a shift (Granlund
// and Montgomery 1994, Fig. 4.1); nodal.hpp's div() applies it.
FastDiv fast_div(uint32_t d) {
  uint32_t s = 0;
  while ((uint64_t(1) << s) < d) ++s;
  return {(uint32_t)(((uint64_t(1) << 32) * ((uint64_t(1) << s) - d)) / d + 1), s};
}

}  // namespace

void find_lattice(semx_ctx* c, const std::vector<std::array<int32_t, 4>>& aff) {
  c->lattice = Lattice{};
  const int N = c->n - 1;
  const int64_t nspec = c->nspec;
  if (c->kind_launches.size() != 1 || c->ncolors == 0 || c->user_colors || aff[0][0] != 0 || aff[0][1] != 1) return;
  const int64_t Gx = aff[0][2], gy = aff[0][3];
  if (Gx < 2 || (Gx - 1) % N != 0 || gy % Gx != 0) return;
  const int64_t Gy = gy / Gx;
  if (Gy < 2 || (Gy - 1) % N != 0) return;
  const int64_t nex = (Gx - 1) / N, ney = (Gy - 1) / N;
  if (nspec % (nex * ney) != 0) return;
  const int64_t nez = nspec / (nex * ney), Gz = nez * N + 1;
  if (Gx * Gy * Gz != c->nglob) return;
  for (int64_t e = 0; e < nspec; ++e) {
    const int64_t ex = e % nex, ey = (e / nex) % ney, ez = e / (nex * ney);
    if (aff[e][0] != N * (ex + Gx * (ey + Gy * ez)) || aff[e][1] != 1 || aff[e][2] != Gx || aff[e][3] != Gx * Gy) return;
  }
  // the order in which a node's elements are added: colours by parity
  for (int k = 0; k < c->ncolors; ++k)
    for (int32_t t = c->color_ptr[k]; t < c->color_ptr[k + 1]; ++t) {
      const int64_t e = c->elem_order[t], ex = e % nex, ey = (e / nex) % ney, ez = e / (nex * ney);
      const int64_t par = (ex & 1) + (nex > 1 ? 2 : 1) * ((ey & 1) + (ney > 1 ? 2 : 1) * (ez & 1));
      if (par != k) return;
    }
  Lattice L{};
  L.n = c->n;
  L.Gx = (int)Gx;
  L.Gy = (int)Gy;
  L.nex = (int)nex;
  L.ney = (int)ney;
  L.nez = (int)nez;
  L.dn = fast_div((uint32_t)N);
  // the widest tile (up to a wave's 64 nodes along x) that leaves the fewest
  // of its lanes outside the box
  int64_t least = INT64_MAX;
  for (int txs = 6; txs >= 2; --txs) {
    const int64_t tx = int64_t(1) << txs, ty = kT / tx, lanes = (Gx + tx - 1) / tx * tx * ((Gy + ty - 1) / ty * ty);
    if (least == INT64_MAX || lanes * 20 < least * 19) {
      least = lanes;
      L.txs = (uint32_t)txs;
    }
  }
  const int64_t tx = int64_t(1) << L.txs, ty = kT / tx;
  L.ntx = (uint32_t)((Gx + tx - 1) / tx);
  L.nty = (uint32_t)((Gy + ty - 1) / ty);
  if ((int64_t)L.ntx * L.nty * Gz >= INT32_MAX) return;
  L.ntiles = (uint32_t)(L.ntx * L.nty * Gz);
  L.drow = fast_div(L.ntx);
  L.dplane = fast_div(L.ntx * L.nty);
  c->lattice = L;
}

hipError_t launch_gather(const semx_ctx* c, float* f, const uint32_t* srcbits, hipStream_t s) {
  return c->ncomp == 1 ? gather_t<float, 1>(c, f, srcbits, s) : gather_t<float, 3>(c, f, srcbits, s);
}

hipError_t launch_gather64(const semx_ctx* c, double* f, const uint32_t* srcbits, hipStream_t s) {
  return gather_t<double, 3>(c, f, srcbits, s);
}

hipError_t launch_newmark_parts(const semx_ctx* c, const uint32_t* srcbits, float* seg_u, float* seg_a,
                                hipStream_t s) {
  const float dt = (float)c->dt;
  const float* minv = c->d_minv.as<float>();
  constexpr int kStep = kCorrect | kPredict;
  if (c->ncomp == 1) return newmark_t<float, 1, kStep>(c, dt, minv, srcbits, nullptr, nullptr, s);
  if (seg_u || seg_a) return newmark_t<float, 3, kStep | kSeg>(c, dt, minv, srcbits, seg_u, seg_a, s);
  return newmark_t<float, 3, kStep>(c, dt, minv, srcbits, nullptr, nullptr, s);
}

hipError_t launch_newmark_parts64(const semx_ctx* c, const uint32_t* srcbits, hipStream_t s) {
  return newmark_t<double, 3, kCorrect | kPredict>(c, c->dt, c->d_minv64.as<double>(), srcbits, nullptr, nullptr, s);
}

hipError_t launch_mass(const semx_ctx* c, const double* rho, double* mass, hipStream_t s) {
  return with_map(c, [&](auto m, dim3 grid) {
    mass_kernel<decltype(m)><<<grid, kT, 0, s>>>(m, c->n3, c->nspec, c->nglob, c->d_order.as<int32_t>(), rho,
                                                 c->d_wdet.as<double>(), mass);
  });
}

}  // namespace semx

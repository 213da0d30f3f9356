// Element force kernel with one lane per line of points (T = float: NC = 3
// elastic, NC = 1 acoustic; T = double: elastic): element-local forces for the
// nodal sum.
//
// The per-point kernels (one lane per GLL point) read n values per component
// and direction from LDS for each point and fetch D with them; at NGLL 5 they
// are bound by vector instructions (316 a point, 62 % of the ALU time of a
// force pass at 64^3 elements) before they are bound by memory.  Here a lane
// owns a whole line of n points: a derivative of the line is a small product
// whose coefficients are the same for every lane (scalar registers).
//
//   home layout: lane c = (i, j) of its element holds the points k = 0..n-1
//     (the zeta line): gather, pointwise stage, result; the zeta derivative
//     and its transpose stay in registers;
//   xi lines (lane (j, k)) and eta lines (lane (i, k)): the same lane number
//     read across; values cross through LDS, each written once and read once
//     per direction (45 LDS accesses a point, against some 110 before).
//
// A workgroup takes as many elements as fill its wavefronts (5 elements of 25
// lines in two waves at NGLL 5: 125 of 128 lanes); where an element's lines
// fit one wave (NGLL 2-4, 8) the workgroup is that wave and its barriers cost
// nothing.  LDS lines are padded to an odd stride so that the lines of a wave
// start on different banks.
#pragma once
#include "elem_common.hpp"

namespace semx {
namespace {

template <class T, int NG>
struct LineShape {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr int N2 = NG * NG;
  static constexpr int N3 = NG * NG * NG;
  static constexpr int P = NG | 1;          // LDS stride of a xi line
  static constexpr int ESZ = P * NG * NG;   // LDS words of one field of one element
  // elements per workgroup (NGLL 10: one in 100 of 128 lanes; three in 300 of
  // 320 leave two workgroups a compute unit and took 79 instead of 59 us per
  // apply at 16^3 elements), lanes
  static constexpr int EPW = NG == 2 ? 16 : NG == 3 ? 7 : NG == 4 ? 4 : NG == 5 ? 5 : NG == 6 ? (F64 ? 3 : 5)
                             : NG == 7 ? (F64 ? 1 : 5) : NG == 9 ? (F64 ? 1 : 3) : 1;
  static constexpr int BLK = (EPW * N2 + 63) / 64 * 64;
};

// D on a line, from the tables of line_table(): the upper half of its rows,
// the left half of the middle row (odd n; D is centro-antisymmetric, so these
// are all of it), and the halves A[i][j] = (D[i][j] - D[i][n-1-j]) / 2, B[i][j] =
// (D[i][j] + D[i][n-1-j]) / 2.
//
// y = D x takes the rows as they are.  The even-odd form (the sums and
// differences of mirrored points times A and B) has a quarter fewer operations,
// but its parts cancel: forces of 5-30 nodes per wavelength came out up to 1.5
// times as far from FP64 as the per-point kernels' (NGLL 5; 2.4 times at 40 nodes
// and more), which the rows do not (0.88-1.03 times).  Terms are added from the
// far end of the line, the large ones last, but at NGLL 3, where the small ones
// go last.  z = D^T q holds fluxes, which do not cancel so: it takes the even-odd
// form from NGLL 6, the rows below (1.00 against 1.03-1.05 times the error at
// NGLL 4 and 5).  All in even-odd form an apply took 0-2 % less up to NGLL 6, 2-5 %
// to 9, 3-10 % from 10.
template <class T, int NG>
struct LineD {
  static constexpr int H = NG / 2;
  static constexpr bool ODD = NG & 1;
  const T* __restrict__ t;
  __device__ __forceinline__ T D(int i, int j) const { return t[i * NG + j]; }
  __device__ __forceinline__ T mid(int j) const { return t[H * NG + j]; }
  __device__ __forceinline__ T A(int i, int j) const { return t[H * (NG + 1) + i * H + j]; }
  __device__ __forceinline__ T B(int i, int j) const { return t[H * (NG + 1) + H * H + i * H + j]; }

  // x = D x
  __device__ __forceinline__ void apply(T x[NG]) const {
    T y[NG];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      T s, r;
      if constexpr (NG == 3) {
        s = D(i, 0) * x[0];
        r = D(i, NG - 1) * x[0];
#pragma unroll
        for (int j = 1; j < NG; ++j) {
          s += D(i, j) * x[j];
          r += D(i, NG - 1 - j) * x[j];
        }
      } else {
        s = D(i, NG - 1) * x[NG - 1];
        r = D(i, NG - 1) * x[0];
#pragma unroll
        for (int j = NG - 2; j >= 0; --j) {
          s += D(i, j) * x[j];
          r += D(i, j) * x[NG - 1 - j];
        }
      }
      y[i] = s;
      y[NG - 1 - i] = -r;
    }
    if constexpr (ODD) {
      T s = mid(0) * (x[0] - x[NG - 1]);
#pragma unroll
      for (int j = 1; j < H; ++j) s += mid(j) * (x[j] - x[NG - 1 - j]);
      y[H] = s;
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) x[i] = y[i];
  }

  // q = D^T q
  __device__ __forceinline__ void apply_t(T q[NG]) const {
    T z[NG];
    if constexpr (NG <= 5) {
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        T s = D(0, j) * q[0];
#pragma unroll
        for (int i = 1; i < H; ++i) s += D(i, j) * q[i];
        if constexpr (ODD) {
          if (j < H) s += mid(j) * q[H];
          if (j > H) s -= mid(NG - 1 - j) * q[H];
        }
#pragma unroll
        for (int i = H - 1; i >= 0; --i) s -= D(i, NG - 1 - j) * q[NG - 1 - i];
        z[j] = s;
      }
    } else {
      T e[H], o[H];
#pragma unroll
      for (int i = 0; i < H; ++i) {
        e[i] = q[i] + q[NG - 1 - i];
        o[i] = q[i] - q[NG - 1 - i];
      }
#pragma unroll
      for (int j = 0; j < H; ++j) {
        T s = B(0, j) * o[0], r = A(0, j) * e[0];
#pragma unroll
        for (int i = 1; i < H; ++i) {
          s += B(i, j) * o[i];
          r += A(i, j) * e[i];
        }
        if constexpr (ODD) r += mid(j) * q[H];
        z[j] = s + r;
        z[NG - 1 - j] = s - r;
      }
      if constexpr (ODD) {
        T s = D(0, H) * o[0];
#pragma unroll
        for (int i = 1; i < H; ++i) s += D(i, H) * o[i];
        z[H] = s;
      }
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) q[i] = z[i];
  }
};

// Geometry of the points of one zeta line.  kTrilinear: along the line the
// first two columns of J are linear in zeta and the third is constant.
template <class T, int GEO>
struct LineGeom {
  T g[GEO == kStored ? 1 : GEO == kRegular ? 9 : 15];

  __device__ __forceinline__ void load(const LineArgs<T>& a, int pos, T rx, T ry) {
    if constexpr (GEO == kRegular) {
#pragma unroll
      for (int d = 0; d < 9; ++d) g[d] = a.gam_el[(size_t)pos * 9 + d];
    } else if constexpr (GEO == kTrilinear) {
      const float4* src = reinterpret_cast<const float4*>(a.tri + (size_t)pos * 24);
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        const float4 lo = src[2 * ax], hi = src[2 * ax + 1];  // c0 c1 c2 c3, c4 c5 c6 c7
        const float b0 = hi.y + hi.w * ry;
        g[5 * ax + 0] = lo.y + hi.x * ry;            // dx/dxi   = g0 + g1 zeta
        g[5 * ax + 1] = b0;
        g[5 * ax + 2] = lo.z + hi.x * rx;            // dx/deta  = g2 + g3 zeta
        g[5 * ax + 3] = hi.z + hi.w * rx;
        g[5 * ax + 4] = lo.w + hi.z * ry + rx * b0;  // dx/dzeta
      }
    }
  }
  // Mg and scale as in geom_map_from (G: the point's Gamma on the stored path)
  __device__ __forceinline__ void at(T rz, const T G[9], T Mg[9], T& scale) const {
    scale = 1;
    if constexpr (GEO == kStored) {
#pragma unroll
      for (int d = 0; d < 9; ++d) Mg[d] = G[d];
    } else if constexpr (GEO == kRegular) {
#pragma unroll
      for (int d = 0; d < 9; ++d) Mg[d] = g[d];
    } else {
      T J[3][3];
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        J[ax][0] = g[5 * ax + 0] + g[5 * ax + 1] * rz;
        J[ax][1] = g[5 * ax + 2] + g[5 * ax + 3] * rz;
        J[ax][2] = g[5 * ax + 4];
      }
      Mg[0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
      Mg[3] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
      Mg[6] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
      Mg[1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
      Mg[4] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
      Mg[7] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
      Mg[2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
      Mg[5] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
      Mg[8] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
      const T det = J[0][0] * Mg[0] + J[0][1] * Mg[3] + J[0][2] * Mg[6];
      const T id = __builtin_amdgcn_rcpf(det);
      scale = id * id;
    }
  }
};

// Weighted fluxes of one point in place of its reference derivatives d[c][dir].
template <class T>
__device__ __forceinline__ void point_flux(T d[3][3], const T Mg[9], T scale, T lamw, T muw) {
  T gr[3][3];
  apply_map(d, Mg, gr);
  const T ls = lamw * scale, ms = muw * scale, ms2 = 2 * ms;
  const T ltr = ls * (gr[0][0] + gr[1][1] + gr[2][2]);
  T sg[3][3];
  sg[0][0] = ltr + ms2 * gr[0][0];
  sg[1][1] = ltr + ms2 * gr[1][1];
  sg[2][2] = ltr + ms2 * gr[2][2];
  sg[0][1] = sg[1][0] = ms * (gr[0][1] + gr[1][0]);
  sg[0][2] = sg[2][0] = ms * (gr[0][2] + gr[2][0]);
  sg[1][2] = sg[2][1] = ms * (gr[1][2] + gr[2][1]);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int q = 0; q < 3; ++q) d[c][q] = sg[c][0] * Mg[q * 3 + 0] + sg[c][1] * Mg[q * 3 + 1] + sg[c][2] * Mg[q * 3 + 2];
}

template <class T>
__device__ __forceinline__ void scalar_flux(T d[3], const T Mg[9], T scale, T w) {
  T g[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) g[b] = d[0] * Mg[0 * 3 + b] + d[1] * Mg[1 * 3 + b] + d[2] * Mg[2 * 3 + b];
  const T s = w * scale;
#pragma unroll
  for (int q = 0; q < 3; ++q) d[q] = s * (g[0] * Mg[q * 3 + 0] + g[1] * Mg[q * 3 + 1] + g[2] * Mg[q * 3 + 2]);
}

template <class T, int NG, int NC, int GEO, bool AFF, class X>
__global__ __launch_bounds__((LineShape<T, NG>::BLK)) void force_line_kernel(LineArgs<T> a, X aux) {
  using S = LineShape<T, NG>;
  constexpr int N2 = S::N2, N3 = S::N3, P = S::P, EPW = S::EPW;
  constexpr int AS = EPW * S::ESZ;  // words of one field
  __shared__ T s[2 * NC * AS];

  if (run_aux(aux)) return;  // uniform over the block
  const int ngrp = ((int)a.count + EPW - 1) / EPW;
  const int grp = xcd_group(ngrp, aux_lead(aux));
  if (grp >= ngrp) return;  // uniform over the block
  // spare lanes repeat the last line (the same values to the same places),
  // spare elements of the last group the last element; neither stores a result
  const int l = min((int)threadIdx.x, EPW * N2 - 1);
  const int e = l / N2, c = l - e * N2;
  const int i = c % NG, j = c / NG;
  const int el = grp * EPW + e;
  const bool act = (int)threadIdx.x < EPW * N2 && el < (int)a.count;
  const int pos = (int)a.pos0 + min(el, (int)a.count - 1);

  const int model = blockIdx.y;
  const T* __restrict__ u = a.u + (size_t)model * a.nglob * NC;
  const T* __restrict__ mat = a.mat + ((size_t)model * a.nspec + pos) * 2 * N3 + c;
  const LineD<T, NG> D{a.dtab};

  // the line's nodes, u and material; the element's geometry
  T uc[NC][NG], lam[NG], mu[NC == 3 ? NG : 1];
  if constexpr (AFF) {
    const int4 r = *reinterpret_cast<const int4*>(a.aff + (size_t)pos * 4);
    const T* p = u + (int64_t)(r.x + i * r.y + j * r.z) * NC;
    const int64_t step = (int64_t)r.w * NC;
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int q = 0; q < NC; ++q) uc[q][k] = p[k * step + q];
  } else {
    const int32_t* ib = a.ibool + (size_t)pos * N3 + c;
    int node[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) node[k] = ldnt(ib + k * N2);
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int q = 0; q < NC; ++q) uc[q][k] = u[(int64_t)node[k] * NC + q];
  }
  LineGeom<T, GEO> geo;
  geo.load(a, pos, GEO == kTrilinear ? a.xi[i] : (T)0, GEO == kTrilinear ? a.xi[j] : (T)0);
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    lam[k] = ldnt(mat + k * N2);
    if constexpr (NC == 3) mu[k] = ldnt(mat + N3 + k * N2);
  }
  const T* __restrict__ gp = GEO == kStored ? a.gam_pt + (size_t)pos * 9 * N3 + c : nullptr;
  // Gamma of the next PD points of the line (a stored-path pass is bound by
  // the bytes in flight)
  constexpr int PD = NG <= 5 && !S::F64 ? NG : 2;
  T Gn[PD][9];
  if constexpr (GEO == kStored) {
#pragma unroll
    for (int k = 0; k < PD; ++k)
#pragma unroll
      for (int d = 0; d < 9; ++d) Gn[k][d] = ldnt(gp + d * N3 + k * N2);
  }

  T* const sz = s + e * S::ESZ + i + P * j;       // home: + k P n
  T* const sx = s + e * S::ESZ + P * c;           // xi line (j, k) = c: + b
  T* const sy = s + e * S::ESZ + i + P * NG * j;  // eta line (i, k = j): + b P
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int k = 0; k < NG; ++k) sz[q * AS + k * P * NG] = uc[q][k];
  __syncthreads();

  // ---- forward contractions: xi and eta derivatives take the place of u ----
  {
    // eta derivatives go to the second field at once (in double at NGLL 9 an
    // apply at 729000 points 28.5 -> 26.3 us against all lines first); xi
    // derivatives take the place of u and wait for its last reader
    T x[NC][NG];
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int b = 0; b < NG; ++b) x[q][b] = sx[q * AS + b];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      T y[NG];
#pragma unroll
      for (int b = 0; b < NG; ++b) y[b] = sy[q * AS + b * P];
      D.apply(y);
#pragma unroll
      for (int b = 0; b < NG; ++b) sy[(NC + q) * AS + b * P] = y[b];
      D.apply(uc[q]);  // zeta derivatives
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      D.apply(x[q]);
#pragma unroll
      for (int b = 0; b < NG; ++b) sx[q * AS + b] = x[q][b];
    }
  }
  __syncthreads();

  // ---- pointwise: geometry map, stress, weighted fluxes in place ----
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    T G[9];
    if constexpr (GEO == kStored) {
#pragma unroll
      for (int d = 0; d < 9; ++d) G[d] = Gn[k % PD][d];
      if (k + PD < NG) {
#pragma unroll
        for (int d = 0; d < 9; ++d) Gn[k % PD][d] = ldnt(gp + d * N3 + (k + PD) * N2);
      }
    }
    T Mg[9], scale;
    geo.at(GEO == kTrilinear ? a.xi[k] : (T)0, G, Mg, scale);
    T d[NC][3];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      d[q][0] = sz[q * AS + k * P * NG];
      d[q][1] = sz[(NC + q) * AS + k * P * NG];
      d[q][2] = uc[q][k];
    }
    if constexpr (NC == 3) point_flux(d, Mg, scale, lam[k], mu[k]);
    else scalar_flux(d[0], Mg, scale, lam[k]);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      sz[q * AS + k * P * NG] = d[q][0];
      sz[(NC + q) * AS + k * P * NG] = d[q][1];
      uc[q][k] = d[q][2];
    }
  }
  __syncthreads();

  // ---- transpose contractions, each line in place ----
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    T x[NG], y[NG];
#pragma unroll
    for (int b = 0; b < NG; ++b) {
      x[b] = sx[q * AS + b];
      y[b] = sy[(NC + q) * AS + b * P];
    }
    D.apply_t(x);
    D.apply_t(y);
#pragma unroll
    for (int b = 0; b < NG; ++b) {
      sx[q * AS + b] = x[b];
      sy[(NC + q) * AS + b * P] = y[b];
    }
    D.apply_t(uc[q]);
  }
  __syncthreads();

  if (!act) return;
  T* out = a.part + (((size_t)model * a.nspec + pos) * N3 + c) * NC;
#pragma unroll
  for (int k = 0; k < NG; ++k)
#pragma unroll
    for (int q = 0; q < NC; ++q)
      out[k * N2 * NC + q] = -(uc[q][k] + (sz[q * AS + k * P * NG] + sz[(NC + q) * AS + k * P * NG]));
}

template <class T, int NG, int NC, int GEO>
hipError_t launch_line(bool aff, const LineArgs<T>& a, hipStream_t s) {
  using S = LineShape<T, NG>;
  const int64_t ngrp = (a.count + S::EPW - 1) / S::EPW;
  const unsigned nb = (unsigned)((ngrp + kNumXcd - 1) / kNumXcd * kNumXcd);
  with_aux(a.aux, S::BLK, kNumXcd, [&](auto aux, unsigned lead) {
    const dim3 grid(nb + lead, (unsigned)a.nmodels);
    if (aff) force_line_kernel<T, NG, NC, GEO, true><<<grid, S::BLK, 0, s>>>(a, aux);
    else force_line_kernel<T, NG, NC, GEO, false><<<grid, S::BLK, 0, s>>>(a, aux);
  });
  return hipGetLastError();
}

template <class T, int NG, int NC>
hipError_t launch_line_n(int geo, bool aff, const LineArgs<T>& a, hipStream_t s) {
  switch (geo) {
    case kRegular: return launch_line<T, NG, NC, kRegular>(aff, a, s);
    case kStored: return launch_line<T, NG, NC, kStored>(aff, a, s);
    case kTrilinear:
      if constexpr (sizeof(T) == 4) return launch_line<T, NG, NC, kTrilinear>(aff, a, s);
    default: return hipErrorInvalidValue;
  }
}

// MAXN: largest NGLL of the instantiation
template <class T, int NC, int MAXN>
hipError_t launch_line_any(int n, int geo, int64_t naff, const LineArgs<T>& a, hipStream_t s) {
  if (!a.part || !a.dtab) return hipErrorInvalidValue;
  return split_affine(naff, a, [&](const LineArgs<T>& b, bool aff) -> hipError_t {
    switch (n) {
      case 2: return launch_line_n<T, 2, NC>(geo, aff, b, s);
      case 3: return launch_line_n<T, 3, NC>(geo, aff, b, s);
      case 4: return launch_line_n<T, 4, NC>(geo, aff, b, s);
      case 5: return launch_line_n<T, 5, NC>(geo, aff, b, s);
      case 6: return launch_line_n<T, 6, NC>(geo, aff, b, s);
      case 7: return launch_line_n<T, 7, NC>(geo, aff, b, s);
      case 8: return launch_line_n<T, 8, NC>(geo, aff, b, s);
      case 9: return launch_line_n<T, 9, NC>(geo, aff, b, s);
      case 10: return launch_line_n<T, 10, NC>(geo, aff, b, s);
      case 11:
        if constexpr (MAXN >= 11) return launch_line_n<T, 11, NC>(geo, aff, b, s);
        return hipErrorInvalidValue;
      case 12:
        if constexpr (MAXN >= 12) return launch_line_n<T, 12, NC>(geo, aff, b, s);
        return hipErrorInvalidValue;
      default: return hipErrorInvalidValue;
    }
  });
}

// The FP32 launch from the arguments that the force kernels share.
inline LineArgs<float> line_args(const ForceArgs& a) {
  return LineArgs<float>{a.ibool, a.aff,  a.gam_pt, a.gam_el, a.tri,   a.xi,    a.mat,     a.u,
                         a.dtab,  a.part, a.pos0,   a.count,  a.nspec, a.nglob, a.nmodels, a.aux};
}

template <int NC>
hipError_t launch_line_f32(int n, int geo, int64_t naff, const ForceArgs& a, hipStream_t s) {
  if (a.list) return hipErrorInvalidValue;
  return launch_line_any<float, NC, kLineMaxN>(n, geo, naff, line_args(a), s);
}

}  // namespace
}  // namespace semx

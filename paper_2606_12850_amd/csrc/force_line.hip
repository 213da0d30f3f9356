// The elastic operator on the line kernel.
#include "force_line.hpp"

namespace semx {
namespace {

// Memory skeleton of force_line_kernel<float, NG, 3>: the same groups, loads and
// stores, no contractions, no pointwise arithmetic and no LDS.
template <int NG, int GEO, bool AFF>
__global__ __launch_bounds__((LineShape<float, NG>::BLK)) void force_line_skeleton_kernel(LineArgs<float> a) {
  using S = LineShape<float, NG>;
  constexpr int N2 = S::N2, N3 = S::N3, EPW = S::EPW;
  const int ngrp = ((int)a.count + EPW - 1) / EPW;
  const int grp = xcd_group(ngrp);
  if (grp >= ngrp) return;  // uniform over the block
  const int e = (int)threadIdx.x / N2, c = (int)threadIdx.x - e * N2;
  const int el = grp * EPW + e;
  if ((int)threadIdx.x >= EPW * N2 || el >= (int)a.count) return;
  const int i = c % NG, j = c / NG, pos = (int)a.pos0 + el, model = blockIdx.y;
  const float* __restrict__ u = a.u + (size_t)model * a.nglob * 3;
  const float* __restrict__ mat = a.mat + ((size_t)model * a.nspec + pos) * 2 * N3 + c;
  float uc[3][NG], m[NG];
  if constexpr (AFF) {
    const int4 r = *reinterpret_cast<const int4*>(a.aff + (size_t)pos * 4);
    const float* p = u + (int64_t)(r.x + i * r.y + j * r.z) * 3;
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q) uc[q][k] = p[(int64_t)k * r.w * 3 + q];
  } else {
    const int32_t* ib = a.ibool + (size_t)pos * N3 + c;
    int node[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) node[k] = ldnt(ib + k * N2);
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q) uc[q][k] = u[(int64_t)node[k] * 3 + q];
  }
  LineGeom<float, GEO> geo;
  geo.load(a, pos, GEO == kTrilinear ? a.xi[i] : 0.0f, GEO == kTrilinear ? a.xi[j] : 0.0f);
  float g = 0.0f;
  if constexpr (GEO != kStored)
    for (float x : geo.g) g += x;
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    m[k] = g + ldnt(mat + k * N2) + ldnt(mat + N3 + k * N2);
    if constexpr (GEO == kStored) {
#pragma unroll
      for (int d = 0; d < 9; ++d) m[k] += ldnt(a.gam_pt + ((size_t)pos * 9 + d) * N3 + c + k * N2);
    }
  }
  float* out = a.part + (((size_t)model * a.nspec + pos) * N3 + c) * 3;
#pragma unroll
  for (int k = 0; k < NG; ++k)
#pragma unroll
    for (int q = 0; q < 3; ++q) out[k * N2 * 3 + q] = m[k] * uc[q][k];
}

template <int NG, int GEO>
hipError_t launch_skeleton(bool aff, const LineArgs<float>& a, hipStream_t s) {
  using S = LineShape<float, NG>;
  const int64_t ngrp = (a.count + S::EPW - 1) / S::EPW;
  const dim3 grid((unsigned)((ngrp + kNumXcd - 1) / kNumXcd * kNumXcd), (unsigned)a.nmodels);
  if (aff) force_line_skeleton_kernel<NG, GEO, true><<<grid, S::BLK, 0, s>>>(a);
  else force_line_skeleton_kernel<NG, GEO, false><<<grid, S::BLK, 0, s>>>(a);
  return hipGetLastError();
}

template <int NG>
hipError_t launch_skeleton_n(int geo, bool aff, const LineArgs<float>& a, hipStream_t s) {
  switch (geo) {
    case kRegular: return launch_skeleton<NG, kRegular>(aff, a, s);
    case kStored: return launch_skeleton<NG, kStored>(aff, a, s);
    case kTrilinear: return launch_skeleton<NG, kTrilinear>(aff, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_force_line(int n, int geo, int64_t naff, const ForceArgs& a, hipStream_t s) {
  return launch_line_f32<3>(n, geo, naff, a, s);
}

hipError_t launch_force_line_skeleton(int n, int geo, int64_t naff, const ForceArgs& a, hipStream_t s) {
  if (a.list || !a.part) return hipErrorInvalidValue;
  return split_affine(naff, line_args(a), [&](const LineArgs<float>& b, bool aff) -> hipError_t {
    switch (n) {
      case 2: return launch_skeleton_n<2>(geo, aff, b, s);
      case 3: return launch_skeleton_n<3>(geo, aff, b, s);
      case 4: return launch_skeleton_n<4>(geo, aff, b, s);
      case 5: return launch_skeleton_n<5>(geo, aff, b, s);
      case 6: return launch_skeleton_n<6>(geo, aff, b, s);
      case 7: return launch_skeleton_n<7>(geo, aff, b, s);
      case 8: return launch_skeleton_n<8>(geo, aff, b, s);
      case 9: return launch_skeleton_n<9>(geo, aff, b, s);
      case 10: return launch_skeleton_n<10>(geo, aff, b, s);
      case 11: return launch_skeleton_n<11>(geo, aff, b, s);
      case 12: return launch_skeleton_n<12>(geo, aff, b, s);
      default: return hipErrorInvalidValue;
    }
  });
}

}  // namespace semx

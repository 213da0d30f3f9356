// FP64 storage path: the same discrete operator and time loop as the FP32
// path, with every field, coefficient and sum in double.
//
//   f = -K u   (Sec. II-B weak form, GLL quadrature, lumped mass):
//     du_c/dxi_d at every GLL point by the 1-D derivative matrix,
//     grad u = du/dxi Gamma, sigma = lambda tr(grad u) I + mu (grad u + grad u^T),
//     Phi_cd = W sum_b sigma_cb Gamma_db, F_c = -sum_d D^T_d Phi_cd, scatter-add;
//   explicit Newmark, beta = 0, gamma = 1/2 (Sec. V-C), point sources, receivers.
//
// It serves runs that must agree with an FP64 reference to FP64 rounding and
// finite-difference checks that need FP64 forward solves.  Large passes take
// the line kernel (force_line.hpp); the kernels here are plain: one workgroup
// per element and model, one GLL point per lane, LDS holding one component's
// three cubes at a time (3 n^3 doubles, 24 KB at NGLL 10).  Assembly is coloured (plain read-modify-write: no two elements
// of a colour share a node, so it is deterministic) or atomic (hardware FP64
// atomic adds).
#include <hip/hip_runtime.h>

#include "newmark.hpp"
#include "semx_internal.hpp"

namespace semx {
namespace {

constexpr int kT = 256;
template <int NG, class X>
__global__ void force64_kernel(int64_t pos0, const int32_t* __restrict__ list, int64_t nspec, int64_t nglob, int atomic,
                               const int32_t* __restrict__ ibool, const double* __restrict__ gam,
                               const double* __restrict__ mat, const double* __restrict__ Dg,
                               const double* __restrict__ u, double* __restrict__ f, double* __restrict__ part,
                               X aux) {
  if (run_aux(aux)) return;  // uniform over the block
  constexpr int n3 = NG * NG * NG;
  __shared__ double D[NG * NG];  // D[a * NG + b] = l'_b(xi_a)
  __shared__ double s[3][n3];
  const int64_t slot = pos0 + ((int)blockIdx.x - aux_lead(aux));
  const int64_t pos = list ? list[slot] : slot;
  const int64_t model = blockIdx.y;
  const int q = threadIdx.x;
  for (int t = q; t < NG * NG; t += blockDim.x) D[t] = Dg[t];
  const bool live = q < n3;
  const int i = q % NG, j = (q / NG) % NG, k = q / (NG * NG);
  int64_t g = 0;
  if (live) {
    g = ibool[pos * n3 + q];
    const double* um = u + (model * nglob + g) * 3;
    s[0][q] = um[0];
    s[1][q] = um[1];
    s[2][q] = um[2];
  }
  __syncthreads();
  double phi[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  if (live) {
    double du[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // du[c][d] = d u_c / d xi_d
#pragma unroll
    for (int a = 0; a < NG; ++a) {
      const double d0 = D[i * NG + a], d1 = D[j * NG + a], d2 = D[k * NG + a];
      const int q0 = a + NG * (j + NG * k), q1 = i + NG * (a + NG * k), q2 = i + NG * (j + NG * a);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        du[c][0] += d0 * s[c][q0];
        du[c][1] += d1 * s[c][q1];
        du[c][2] += d2 * s[c][q2];
      }
    }
    const double* G = gam + pos * 9 * n3 + q;  // Gamma_db = d xi_d / d x_b at [(3 d + b) n3]
    double Gm[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int b = 0; b < 3; ++b) Gm[d][b] = G[(3 * d + b) * n3];
    double gr[3][3];  // gr[c][b] = d u_c / d x_b
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int b = 0; b < 3; ++b) gr[c][b] = du[c][0] * Gm[0][b] + du[c][1] * Gm[1][b] + du[c][2] * Gm[2][b];
    const double* mp = mat + (model * nspec + pos) * 2 * n3;
    const double lw = mp[q], mw = mp[n3 + q];  // lambda W, mu W
    const double ltr = lw * (gr[0][0] + gr[1][1] + gr[2][2]);
    double sig[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int b = 0; b < 3; ++b) sig[c][b] = mw * (gr[c][b] + gr[b][c]) + (c == b ? ltr : 0.0);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d) phi[c][d] = sig[c][0] * Gm[d][0] + sig[c][1] * Gm[d][1] + sig[c][2] * Gm[d][2];
  }
  double F[3] = {0, 0, 0};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    __syncthreads();
    if (live) {
      s[0][q] = phi[c][0];
      s[1][q] = phi[c][1];
      s[2][q] = phi[c][2];
    }
    __syncthreads();
    if (live) {
      double acc = 0.0;
#pragma unroll
      for (int a = 0; a < NG; ++a)
        acc += D[a * NG + i] * s[0][a + NG * (j + NG * k)] + D[a * NG + j] * s[1][i + NG * (a + NG * k)] +
               D[a * NG + k] * s[2][i + NG * (j + NG * a)];
      F[c] = -acc;
    }
  }
  if (live) {
    double* fm = part ? part + ((model * nspec + pos) * n3 + q) * 3 : f + (model * nglob + g) * 3;
    if (part) {
      fm[0] = F[0];
      fm[1] = F[1];
      fm[2] = F[2];
    } else if (atomic) {
      atomicAdd(fm + 0, F[0]);
      atomicAdd(fm + 1, F[1]);
      atomicAdd(fm + 2, F[2]);
    } else {
      fm[0] += F[0];
      fm[1] += F[1];
      fm[2] += F[2];
    }
  }
}

__global__ void fill64_kernel(double* __restrict__ p, int64_t n, double v) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    p[t] = v;
}

// lambda W and mu W in FP64 at launch position pos (user element order[pos]).
__global__ void material64_kernel(int n3, int64_t nspec, int nmodels, const int32_t* __restrict__ order,
                                  const double* __restrict__ lam, const double* __restrict__ mu,
                                  const double* __restrict__ wdet, double* __restrict__ mat) {
  const int64_t total = (int64_t)nmodels * nspec * n3;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t mp = t / n3;
    const int q = (int)(t - mp * n3);
    const int64_t model = mp / nspec, pos = mp - model * nspec;
    const int64_t src = (model * nspec + order[pos]) * n3 + q;
    const double W = wdet[pos * n3 + q];
    mat[mp * 2 * n3 + q] = lam[src] * W;
    mat[mp * 2 * n3 + n3 + q] = mu[src] * W;
  }
}

// Gamma of the first point of each element, and whether it holds for all points
// of the regular elements (the first nreg positions): their Gamma may differ by
// what the rounding of the vertex coordinates (half an ulp each) does to it.
__global__ void gam_el64_kernel(int n3, int64_t nspec, int64_t nreg, const double* __restrict__ vert,
                                const int32_t* __restrict__ ev, const int32_t* __restrict__ order,
                                const double* __restrict__ gam, double* __restrict__ gam_el, int* __restrict__ bad) {
  for (int64_t pos = blockIdx.x * (int64_t)(blockDim.x / 64) + threadIdx.x / 64; pos < nspec;
       pos += (int64_t)gridDim.x * (blockDim.x / 64)) {
    const int lane = threadIdx.x & 63;
    const double* G = gam + pos * 9 * n3;
    if (lane < 9) gam_el[pos * 9 + lane] = G[(int64_t)lane * n3];
    if (pos >= nreg) continue;
    double x = 0.0, g = 0.0, dev = 0.0;
    for (int v = 0; v < 8; ++v)
      for (int b = 0; b < 3; ++b) x = fmax(x, fabs(vert[3 * (int64_t)ev[8 * (int64_t)order[pos] + v] + b]));
    for (int d = 0; d < 9; ++d) {
      const double g0 = G[(int64_t)d * n3];
      g = fmax(g, fabs(g0));
      for (int q = lane; q < n3; q += 64) dev = fmax(dev, fabs(G[(int64_t)d * n3 + q] - g0));
    }
    if (!(dev <= 4 * 2.220446049250313e-16 * g * (1.0 + g * x))) atomicOr(bad, 1);
  }
}

__global__ void minv64_kernel(int64_t n, const double* __restrict__ mass, double* __restrict__ minv) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    minv[t] = mass[t] > 0.0 ? 1.0 / mass[t] : 0.0;  // a node no element reaches stays at rest
}

// Newmark update, one lane per degree of freedom; kCorrect: acc = M^{-1} f,
// v += dt/2 acc (acc stored to a with kStoreA); kPredict: u += dt v + dt^2/2
// acc, v += dt/2 acc, f = 0 for the coming force pass unless kKeepF.
template <int MODE>
__global__ void newmark64_kernel(int64_t nnodes, double dt, const double* __restrict__ minv, double* __restrict__ u,
                                 double* __restrict__ v, double* __restrict__ a, double* __restrict__ f) {
  const double hdt = 0.5 * dt, hdt2 = 0.5 * dt * dt;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < 3 * nnodes;
       t += (int64_t)gridDim.x * blockDim.x) {
    double acc, vv = v[t];
    if constexpr ((MODE & kCorrect) != 0) {
      acc = minv[t / 3] * f[t];
      vv += hdt * acc;
      if constexpr ((MODE & kStoreA) != 0) a[t] = acc;
    } else {
      acc = a[t];
    }
    if constexpr ((MODE & kPredict) != 0) {
      u[t] += dt * vv + hdt2 * acc;
      vv += hdt * acc;
      if constexpr ((MODE & kKeepF) == 0) f[t] = 0.0;
    }
    v[t] = vv;
  }
}

__global__ void accel64_kernel(int64_t nnodes, const double* __restrict__ minv, const double* __restrict__ f,
                               double* __restrict__ a) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < 3 * nnodes;
       t += (int64_t)gridDim.x * blockDim.x)
    a[t] = minv[t / 3] * f[t];
}

__global__ void source64_kernel(int nsrc, int n3, int64_t nstf, int64_t m, int nmodels, int64_t nglob,
                                const int32_t* __restrict__ nodes, const double* __restrict__ wdir,
                                const double* __restrict__ stf, double* __restrict__ f) {
  const int64_t total = (int64_t)nmodels * nsrc * n3;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t sq = t % ((int64_t)nsrc * n3);
    const int64_t model = t / ((int64_t)nsrc * n3);
    const int s = (int)(sq / n3);
    const double amp = (m >= 0 && m < nstf) ? stf[(int64_t)s * nstf + m] : 0.0;
    if (amp == 0.0) continue;
    double* fg = f + (model * nglob + nodes[sq]) * 3;
    atomicAdd(fg + 0, amp * wdir[3 * sq + 0]);
    atomicAdd(fg + 1, amp * wdir[3 * sq + 1]);
    atomicAdd(fg + 2, amp * wdir[3 * sq + 2]);
  }
}

// one block of kT lanes per (receiver, model)
__global__ void receiver64_kernel(int nrec, int n3, int64_t nglob, int64_t nt_max, int64_t it,
                                  const int32_t* __restrict__ nodes, const double* __restrict__ wts,
                                  const double* __restrict__ u, double* __restrict__ seis) {
  __shared__ double red[3][kT];
  const int r = blockIdx.x;
  const int64_t model = blockIdx.y;
  const double* um = u + model * nglob * 3;
  double s0 = 0, s1 = 0, s2 = 0;
  for (int q = threadIdx.x; q < n3; q += blockDim.x) {
    const double wq = wts[(int64_t)r * n3 + q];
    const int64_t g = nodes[(int64_t)r * n3 + q];
    s0 += wq * um[3 * g + 0];
    s1 += wq * um[3 * g + 1];
    s2 += wq * um[3 * g + 2];
  }
  red[0][threadIdx.x] = s0;
  red[1][threadIdx.x] = s1;
  red[2][threadIdx.x] = s2;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int c = 0; c < 3; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 3) seis[((model * nrec + r) * 3 + threadIdx.x) * nt_max + it] = red[threadIdx.x][0];
}

__device__ inline void block_sum64(double v, double* out) {
  __shared__ double red[kT];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(out, red[0]);
}

// out += sum_g mass_g |x_g|^2 over one model
__global__ void mnorm64_kernel(int64_t nglob, const double* __restrict__ mass, const double* __restrict__ x,
                               double* __restrict__ out) {
  double s = 0.0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < 3 * nglob; t += (int64_t)gridDim.x * blockDim.x)
    s += mass[t / 3] * x[t] * x[t];
  block_sum64(s, out);
}

__global__ void dot64_kernel(int64_t n, const double* __restrict__ x, const double* __restrict__ y,
                             double* __restrict__ out) {
  double s = 0.0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    s += x[t] * y[t];
  block_sum64(s, out);
}

__global__ void finite64_kernel(int64_t n, const double* __restrict__ x, int* __restrict__ flag) {
  bool bad = false;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    bad |= !isfinite(x[t]);
  if (bad) atomicOr(flag, 1);
}

// Line kernel (force_line.hpp) instead of one lane per point: where a launch
// fills the chip.  Per-point Gamma: at NGLL 2-5 the line kernel has fewer of
// its 72 bytes a point in flight.  Force applies of a box, lane per point / line:
//   one Gamma per element  NGLL 5, 1000000 points 33.9 / 25.5 us, 216000 12.8 / 11.6, 42875 8.8 / 8.4;
//                          NGLL 9, 729000 44.9 / 24.8;  NGLL 10, 125000 15.7 / 16.3
//   Gamma at each point    NGLL 5, 1000000 points 33.9 / 38.2;  NGLL 7, 753571 38.5 / 31.0, 175616 13.5 / 12.5
bool use_line64(const semx_ctx* c, bool parts, int geo) {
  const int64_t points = (int64_t)c->nmodels * c->nspec * c->n3;
  if (!parts) return false;
  return geo == kRegular ? points >= (1 << 17) : c->n >= 6 && points >= (1 << 18);
}

LineArgs<double> line_args64(const semx_ctx* c, const double* u) {
  LineArgs<double> a{};
  a.ibool = c->d_ibool.as<int32_t>();
  a.aff = c->d_aff.as<int32_t>();
  a.gam_pt = c->d_gam64.as<double>();
  a.gam_el = c->d_gam64_el.as<double>();
  a.mat = c->d_mat64.as<double>();
  a.u = u;
  a.dtab = c->d_dtab64.as<double>();
  a.part = c->d_part.as<double>();
  a.nspec = c->nspec;
  a.nglob = c->nglob;
  a.nmodels = c->nmodels;
  return a;
}

template <int NG>
hipError_t launch_force64_n(const semx_ctx* c, const double* u, double* f, const AuxArgs<double>* aux) {
  constexpr int n3 = NG * NG * NG;
  const unsigned threads = (unsigned)((n3 + 63) / 64 * 64);
  const bool atomic = c->assembly == SEMX_ASM_ATOMIC;
  const bool parts = parts_active(c), colored = !atomic && !parts;
  for (const auto& L : colored ? c->colored_launches : c->kind_launches) {
    if (L.count <= 0) continue;
    const int geo = !L.irregular && c->affine64 ? kRegular : kStored;
    if (use_line64(c, parts, geo)) {
      LineArgs<double> a = line_args64(c, u);
      a.pos0 = L.pos0;
      a.count = L.count;
      a.aux = aux;
      aux = nullptr;  // rides in the first launch
      const hipError_t e = launch_force_line64(NG, geo, L.naff, a, c->stream);
      if (e != hipSuccess) return e;
      continue;
    }
    const int32_t* list = colored ? colour_list(c) : atomic ? c->d_alist.as<int32_t>() : nullptr;
    with_aux(aux, (int)threads, kNumXcd, [&](auto x, unsigned lead) {
      force64_kernel<NG><<<dim3((unsigned)L.count + lead, (unsigned)c->nmodels), threads, 0, c->stream>>>(
          L.pos0, list, c->nspec, c->nglob, atomic ? 1 : 0, c->d_ibool.as<int32_t>(), c->d_gam64.as<double>(),
          c->d_mat64.as<double>(), c->d_D64.as<double>(), u, f, parts ? c->d_part.as<double>() : nullptr, x);
    });
    aux = nullptr;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// aux: bookkeeping waves of the step that ride in the pass (element-local forces only)
hipError_t launch_force64(const semx_ctx* c, const double* u, double* f, const AuxArgs<double>* aux = nullptr) {
  switch (c->n) {
    case 2: return launch_force64_n<2>(c, u, f, aux);
    case 3: return launch_force64_n<3>(c, u, f, aux);
    case 4: return launch_force64_n<4>(c, u, f, aux);
    case 5: return launch_force64_n<5>(c, u, f, aux);
    case 6: return launch_force64_n<6>(c, u, f, aux);
    case 7: return launch_force64_n<7>(c, u, f, aux);
    case 8: return launch_force64_n<8>(c, u, f, aux);
    case 9: return launch_force64_n<9>(c, u, f, aux);
    case 10: return launch_force64_n<10>(c, u, f, aux);
    default: return hipErrorInvalidValue;
  }
}

int zero64(semx_ctx* c, double* p, int64_t n) {
  fill64_kernel<<<grid_1d(n), kT, 0, c->stream>>>(p, n, 0.0);
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

int64_t len64(const semx_ctx* c) { return (int64_t)c->nmodels * c->nglob * 3; }

int inject64(semx_ctx* c, int64_t m, double* f) {
  if (c->src.nsrc == 0) return SEMX_OK;
  const int64_t total = (int64_t)c->nmodels * c->src.nsrc * c->n3;
  source64_kernel<<<grid_1d(total), kT, 0, c->stream>>>(c->src.nsrc, c->n3, c->src.nstf, m, c->nmodels, c->nglob,
                                                         c->src.nodes.as<int32_t>(), c->src.wdir64.as<double>(),
                                                         c->src.stf64.as<double>(), f);
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

int record64(semx_ctx* c, int64_t idx) {
  if (c->rec.nrec == 0 || idx < 0 || idx >= c->rec.nt_max) return SEMX_OK;
  dim3 grid(c->rec.nrec, c->nmodels);
  receiver64_kernel<<<grid, kT, 0, c->stream>>>(c->rec.nrec, c->n3, c->nglob, c->rec.nt_max, idx,
                                                c->rec.nodes.as<int32_t>(), c->rec.wts64.as<double>(),
                                                c->d_u.as<double>(), c->rec.seis64.as<double>());
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

}  // namespace

int f64_model_setup(semx_ctx* c, const double* lam_dev, const double* mu_dev) {
  const int64_t npt = (int64_t)c->nmodels * c->nspec * c->n3;
  int rc = dev_alloc(c, c->d_mat64, sizeof(double) * 2 * npt);
  if (!rc) rc = dev_alloc(c, c->d_minv64, sizeof(double) * c->nmodels * c->nglob);
  if (!rc && c->d_D64.bytes != sizeof(double) * c->n * c->n) rc = dev_alloc(c, c->d_D64, sizeof(double) * c->n * c->n);
  std::vector<double> tab;
  line_table(c->n, c->D, tab);
  if (!rc) rc = dev_alloc(c, c->d_dtab64, sizeof(double) * tab.size());
  if (!rc) rc = dev_alloc(c, c->d_gam64_el, sizeof(double) * 9 * c->nspec);
  if (rc) return rc;
  SEMX_HIP(c, hipMemcpy(c->d_dtab64.p, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice));
  int* flag = scratch_flags(c);
  SEMX_HIP(c, hipMemsetAsync(flag, 0, sizeof(int), c->stream));
  gam_el64_kernel<<<grid_1d(c->nspec * 64, 4096), kT, 0, c->stream>>>(
      c->n3, c->nspec, c->nregular, c->d_vert.as<double>(), c->d_elem_vert.as<int32_t>(), c->d_order.as<int32_t>(),
      c->d_gam64.as<double>(), c->d_gam64_el.as<double>(), flag);
  SEMX_HIP(c, hipGetLastError());
  int uneven = 0;
  SEMX_HIP(c, hipMemcpyAsync(&uneven, flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  SEMX_HIP(c, hipStreamSynchronize(c->stream));
  c->affine64 = uneven == 0;
  SEMX_HIP(c, hipMemcpyAsync(c->d_D64.p, c->D.data(), sizeof(double) * c->n * c->n, hipMemcpyHostToDevice, c->stream));
  material64_kernel<<<grid_1d(npt, 8192), kT, 0, c->stream>>>(c->n3, c->nspec, c->nmodels, c->d_order.as<int32_t>(),
                                                               lam_dev, mu_dev, c->d_wdet.as<double>(),
                                                               c->d_mat64.as<double>());
  minv64_kernel<<<grid_1d((int64_t)c->nmodels * c->nglob), kT, 0, c->stream>>>(
      (int64_t)c->nmodels * c->nglob, c->d_mass64.as<double>(), c->d_minv64.as<double>());
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

int f64_force_into(semx_ctx* c, const double* u, double* f, bool f_zeroed) {
  if (parts_active(c)) {
    hipError_t e = launch_force64(c, u, f);
    if (e == hipSuccess) e = launch_gather64(c, f, nullptr, c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "FP64 force kernel launch");
    return SEMX_OK;
  }
  if (c->assembly != SEMX_ASM_ATOMIC) {
    int rc = build_colored(c);
    if (rc) return rc;
  }
  if (!f_zeroed) {
    int rc = zero64(c, f, len64(c));
    if (rc) return rc;
  }
  hipError_t e = launch_force64(c, u, f);
  if (e != hipSuccess) return hip_fail(c, e, "FP64 force kernel launch");
  return SEMX_OK;
}

int f64_finalize(semx_ctx* c) {
  if (!c->pending_correct) return SEMX_OK;
  int rc = settle_force(c);
  if (rc) return rc;
  const int64_t nn = (int64_t)c->nmodels * c->nglob;
  newmark64_kernel<kCorrect | kStoreA><<<grid_1d(3 * nn), kT, 0, c->stream>>>(
      nn, c->dt, c->d_minv64.as<double>(), c->d_u.as<double>(), c->d_v.as<double>(), c->d_a.as<double>(),
      c->d_f.as<double>());
  SEMX_HIP(c, hipGetLastError());
  c->pending_correct = false;
  return SEMX_OK;
}

int f64_reset(semx_ctx* c) {
  const int64_t len = len64(c);
  for (auto* b : {&c->d_u, &c->d_v, &c->d_a, &c->d_f}) {
    int rc = zero64(c, b->as<double>(), len);
    if (rc) return rc;
  }
  c->it = 0;
  c->pending_correct = false;
  if (c->rec.nrec > 0 && c->rec.seis64.p) {
    int rc = zero64(c, c->rec.seis64.as<double>(), c->rec.seis64.bytes / sizeof(double));
    if (rc) return rc;
  }
  if (c->src.nsrc > 0) {
    int rc = inject64(c, 0, c->d_f.as<double>());
    if (rc) return rc;
    const int64_t nn = (int64_t)c->nmodels * c->nglob;
    accel64_kernel<<<grid_1d(3 * nn), kT, 0, c->stream>>>(nn, c->d_minv64.as<double>(), c->d_f.as<double>(),
                                                           c->d_a.as<double>());
    SEMX_HIP(c, hipGetLastError());
    rc = zero64(c, c->d_f.as<double>(), len);
    if (rc) return rc;
  }
  return energy_reset(c);
}

int f64_step_once(semx_ctx* c, bool record) {
  const int64_t nn = (int64_t)c->nmodels * c->nglob;
  double *u = c->d_u.as<double>(), *v = c->d_v.as<double>(), *a = c->d_a.as<double>(), *f = c->d_f.as<double>();
  const double* minv = c->d_minv64.as<double>();
  const bool track = c->track_energy;
  const bool keep = track || parts_active(c);  // the gather overwrites f
  c->track_energy = false;
  // a tracked step keeps f^n through the Newmark pass for the potential
  // term, or computes -K u^n into the work vector when no force is pending
  const double* f_pe = f;
  if (track && !c->pending_correct) {
    int rc = f64_force_into(c, u, c->d_work.as<double>(), false);
    if (rc) return rc;
    f_pe = c->d_work.as<double>();
  }
  const bool parts = parts_active(c);
  if (track || !parts) {  // the energy pass reads f^n; other passes need f summed or cleared
    int rc = settle_force(c);
    if (rc) return rc;
  }
  if (c->f_in_part) {
    c->f_in_part = false;
    const hipError_t e = launch_newmark_parts64(c, c->part_src ? c->d_srcbits.as<uint32_t>() : nullptr, c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "Newmark pass launch");
  } else if (c->pending_correct) {
    if (keep) newmark64_kernel<kCorrect | kPredict | kKeepF><<<grid_1d(3 * nn), kT, 0, c->stream>>>(nn, c->dt, minv, u, v, a, f);
    else newmark64_kernel<kCorrect | kPredict><<<grid_1d(3 * nn), kT, 0, c->stream>>>(nn, c->dt, minv, u, v, a, f);
  } else {
    if (keep) newmark64_kernel<kPredict | kKeepF><<<grid_1d(3 * nn), kT, 0, c->stream>>>(nn, c->dt, minv, u, v, a, f);
    else newmark64_kernel<kPredict><<<grid_1d(3 * nn), kT, 0, c->stream>>>(nn, c->dt, minv, u, v, a, f);
  }
  SEMX_HIP(c, hipGetLastError());
  const bool src_in_f = c->pending_correct;
  if (track) {
    int rc = energy_track(c, f_pe, src_in_f);
    if (rc) return rc;
  }
  int rc = SEMX_OK;
  if (parts) {
    // receivers, source work and the coming source force ride in the force launch,
    // or go before it
    const bool pre = prestores(c);
    if (pre) rc = build_first_tl(c);
    const bool ride = aux_fits(c);
    const AuxArgs<double> aux = ride ? aux_args64(c, c->it, track && src_in_f, record, pre) : AuxArgs<double>{};
    if (!rc && !ride) rc = step_aux64(c, c->it, track && src_in_f, record, pre);
    if (rc) return rc;
    const hipError_t e = launch_force64(c, u, f, &aux);
    if (e != hipSuccess) return hip_fail(c, e, "FP64 force kernel launch");
    c->f_in_part = true;
    c->part_src = pre;
  } else {
    rc = step_aux64(c, c->it, track && src_in_f, false, false);
    if (!rc) rc = f64_force_into(c, u, f, !track);
    if (!rc) rc = inject64(c, c->it + 1, f);
    if (!rc && record) rc = record64(c, c->it);
    if (rc) return rc;
  }
  c->it++;
  c->pending_correct = true;
  if (track) c->energy_it = c->it;
  return SEMX_OK;
}

int f64_check_finite(semx_ctx* c, bool* ok) {
  int* flag = scratch_flags(c);
  SEMX_HIP(c, hipMemsetAsync(flag, 0, sizeof(int), c->stream));
  const int64_t len = len64(c);
  finite64_kernel<<<grid_1d(len, 4096), kT, 0, c->stream>>>(len, c->d_u.as<double>(), flag);
  finite64_kernel<<<grid_1d(len, 4096), kT, 0, c->stream>>>(len, c->d_v.as<double>(), flag);
  SEMX_HIP(c, hipGetLastError());
  int h = 0;
  SEMX_HIP(c, hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  SEMX_HIP(c, hipStreamSynchronize(c->stream));
  *ok = (h == 0);
  return SEMX_OK;
}

}  // namespace semx

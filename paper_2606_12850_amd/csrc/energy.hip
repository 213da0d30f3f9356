// Discrete energy of the explicit Newmark scheme and the work of the point
// sources (Sec. II-B weak form with the diagonal GLL mass; Sec. V-C
// second-order Newmark).  With K, M symmetric, the central-difference form of
// the scheme conserves
//   E^{n+1/2} = 1/2 (v^{n+1/2})^T M v^{n+1/2} + 1/2 (u^{n+1})^T K u^n,
// v^{n+1/2} = (u^{n+1} - u^n) / dt (the scheme's half-step velocity), up to the
// work of the sources: E^{n+1/2} - E^{n-1/2} = 1/2 (u^{n+1} - u^{n-1})^T f_src^n.
//
// Bookkeeping on the time loop, model 0 of the batch, FP64 sums:
//  * energy_track(): after the Newmark pass of step n (u holds u^{n+1}, v the
//    half-step velocity, f_pe the force f^n = -K u^n + f_src^n), one pass
//    sums v^T M v and u^{n+1} . f_pe in fixed-size blocks, reduced in a fixed
//    order (deterministic);
//  * every step, one wave of the force launch (aux.hpp), or one block of
//    step_aux_kernel where the force pass carries no such waves, goes over the
//    source points: it adds 1/2 (u^{n+1} - u^{n-1}) . f_src^n to the running
//    source work and, on tracked steps, sums u^{n+1} . f_src^n (the source part
//    of f^n, which the potential term must not see); it keeps u at the source
//    points of the last two steps.
// acc (double[8]): 0 sum M v^2, 1 sum u . f_pe, 2 sum u . f_src, 3 running
// source work.  The caller's state and kernels are not touched.
#include <algorithm>

#include "semx_internal.hpp"

namespace semx {
namespace {

constexpr int kEnergyBlocks = 1024;
constexpr int kT = 256;

__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// part[b][0] = sum M v^2, part[b][1] = sum u . f over the entries of block b
// (grid-stride over nc * nglob entries of model 0).
template <class T>
__global__ __launch_bounds__(kT) void energy_pass_kernel(int64_t nglob, int nc, const double* __restrict__ mass,
                                                         const T* __restrict__ v, const T* __restrict__ u,
                                                         const T* __restrict__ f, double* __restrict__ part) {
  __shared__ double red[kT];
  double kin = 0.0, pot = 0.0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nc * nglob;
       t += (int64_t)gridDim.x * blockDim.x) {
    const double vv = v[t];
    kin += mass[t / nc] * vv * vv;
    pot += (double)u[t] * (double)f[t];
  }
  kin = block_sum(kin, red);
  pot = block_sum(pot, red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = kin;
    part[2 * blockIdx.x + 1] = pot;
  }
}

// acc[0], acc[1] = sums of the block partials, in block order.
__global__ void energy_reduce_kernel(int nblk, const double* __restrict__ part, double* __restrict__ acc) {
  __shared__ double red[kT];
  double kin = 0.0, pot = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    kin += part[2 * b];
    pot += part[2 * b + 1];
  }
  kin = block_sum(kin, red);
  pot = block_sum(pot, red);
  if (threadIdx.x == 0) {
    acc[0] = kin;
    acc[1] = pot;
  }
}

// The bookkeeping of a step in a launch of its own: a block per receiver and one
// for the source work, whose 256 lanes take what a single wave of aux.hpp takes
// in four parts (the same sums in the same order).  At NGLL 16 (4096 points) the
// waves' launch took 25 us more than this one.
template <class T>
__global__ __launch_bounds__(kT) void step_aux_kernel(AuxArgs<T> A) {
  __shared__ double red[2][kT];
  __shared__ T rred[3][kT];
  const int unit = blockIdx.x, model = blockIdx.y, lane = threadIdx.x;
  if (unit < A.nrec) {  // uniform over the block, as are all branches here
    const int64_t it = A.step ? *A.step : A.it;
    if (it < 0 || it >= A.nt_max) return;
    const T* um = A.u + (int64_t)model * A.nglob * A.nc;
    const int32_t* nodes = A.rnodes + (int64_t)unit * A.n3;
    const T* wts = A.rwts + (int64_t)unit * A.n3;
    T s[3] = {0, 0, 0};
#pragma unroll 4
    for (int q = lane; q < A.n3; q += kT) {
      const T w = wts[q];
      const int64_t g = nodes[q];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c < A.nc) s[c] += w * um[A.nc * g + c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) rred[c][lane] = s[c];
    __syncthreads();
    if (lane >= 64) return;
    for (int c = 0; c < A.nc; ++c) {
      const T v = tree_sum(rred[c][lane], rred[c][lane + 64], rred[c][lane + 128], rred[c][lane + 192]);
      if (lane == 0) A.seis[(((int64_t)model * A.nrec + unit) * A.nc + c) * A.nt_max + it] = v;
    }
    return;
  }
  if (model != 0) return;
  const int rest = unit - A.nrec;
  if (!A.energy || rest > 0) {
    aux_source(A, (int64_t)(rest - A.energy) * kT + lane);
    return;
  }
  const int64_t n = A.step ? *A.step : A.it;
  T* slot = A.hist + (size_t)((n + 1) & 1) * A.per;
  const bool live = n >= 0 && n < A.nstf;
  double work = 0.0, corr = 0.0;
  // four points a lane at a time, their loads in one round trip each (a step of
  // 16^3 elements of NGLL 5 with 1024 sources, 128000 points, took 728 us one at
  // a time, now 622; with 32 sources 36, now 30)
  constexpr int kPts = 4;
  for (int k0 = lane; k0 < A.npt; k0 += kPts * kT) {
    int p[kPts], g[kPts];
    T amp[kPts], un[kPts][3], old[kPts][3], wd[kPts][3];
#pragma unroll
    for (int j = 0; j < kPts; ++j) p[j] = A.pts[min(k0 + j * kT, A.npt - 1)];
#pragma unroll
    for (int j = 0; j < kPts; ++j) {
      g[j] = A.snodes[p[j]] * A.nc;
      amp[j] = live ? A.stf[(int64_t)(p[j] / A.n3) * A.nstf + n] : (T)0;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c < A.nc) {
          wd[j][c] = A.wdir[(int64_t)A.nc * p[j] + c];
          old[j][c] = slot[(int64_t)A.nc * min(k0 + j * kT, A.npt - 1) + c];
        }
    }
#pragma unroll
    for (int j = 0; j < kPts; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c < A.nc) un[j][c] = A.u[g[j] + c];
#pragma unroll
    for (int j = 0; j < kPts; ++j) {
      if (k0 + j * kT >= A.npt) break;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c < A.nc) {
          const double fs = (double)amp[j] * (double)wd[j][c];
          work += 0.5 * ((double)un[j][c] - (double)old[j][c]) * fs;
          corr += (double)un[j][c] * fs;
          slot[(int64_t)A.nc * (k0 + j * kT) + c] = un[j][c];
        }
    }
  }
  red[0][lane] = work;
  red[1][lane] = corr;
  __syncthreads();
  if (lane >= 64) return;
  work = tree_sum(red[0][lane], red[0][lane + 64], red[0][lane + 128], red[0][lane + 192]);
  corr = tree_sum(red[1][lane], red[1][lane + 64], red[1][lane + 128], red[1][lane + 192]);
  if (lane == 0) {
    if (n > A.it0) A.acc[3] += work;
    if (A.with_corr) A.acc[2] = corr;
  }
}

// u at the source points (model 0) into hist (at a reset or a new state).
template <class T>
__global__ void source_gather_kernel(int npt, int nc, const int32_t* __restrict__ pts,
                                     const int32_t* __restrict__ nodes, const T* __restrict__ u,
                                     T* __restrict__ hist) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < npt; k += gridDim.x * blockDim.x)
    for (int c = 0; c < nc; ++c) hist[(int64_t)nc * k + c] = u[(int64_t)nc * nodes[pts[k]] + c];
}

__global__ void zero_doubles_kernel(double* __restrict__ p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0;
}

}  // namespace

int energy_reset(semx_ctx* c) {
  int rc = SEMX_OK;
  if (!c->d_eacc.p) rc = dev_alloc(c, c->d_eacc, sizeof(double) * 8);
  if (!rc && !c->d_epart.p) rc = dev_alloc(c, c->d_epart, sizeof(double) * 2 * kEnergyBlocks);
  if (rc) return rc;
  zero_doubles_kernel<<<1, 64, 0, c->stream>>>(c->d_eacc.as<double>(), 8);
  SEMX_HIP(c, hipGetLastError());
  c->energy_it = -1;
  c->energy_it0 = c->it;
  const int npt = c->src.nsrc > 0 ? c->src.npts : 0;
  if (npt == 0) return SEMX_OK;
  const size_t tsz = c->storage == SEMX_F64 ? sizeof(double) : sizeof(float);
  const size_t bytes = 2 * (size_t)npt * c->ncomp * tsz;
  if (c->d_ehist.bytes != bytes) {
    rc = dev_alloc(c, c->d_ehist, bytes);
    if (rc) return rc;
  }
  SEMX_HIP(c, hipMemsetAsync(c->d_ehist.p, 0, bytes, c->stream));
  const size_t per = (size_t)npt * c->ncomp;
  const unsigned nb = (unsigned)std::min(1024, (npt + kT - 1) / kT);
  const size_t slot = (size_t)(c->it & 1) * per;
  if (c->storage == SEMX_F64)
    source_gather_kernel<double><<<nb, kT, 0, c->stream>>>(npt, c->ncomp, c->src.pts.as<int32_t>(),
                                                           c->src.nodes.as<int32_t>(),
                                                           c->d_u.as<double>(), c->d_ehist.as<double>() + slot);
  else
    source_gather_kernel<float><<<nb, kT, 0, c->stream>>>(npt, c->ncomp, c->src.pts.as<int32_t>(),
                                                          c->src.nodes.as<int32_t>(),
                                                          c->d_u.as<float>(), c->d_ehist.as<float>() + slot);
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

namespace {

template <class T>
AuxArgs<T> aux_args_t(semx_ctx* c, int64_t n, bool with_corr, bool record, const int64_t* dstep, bool prestore,
                      const T* rwts, T* seis, const T* wdir, const T* stf) {
  AuxArgs<T> A{};
  const bool src = c->src.nsrc > 0 && c->d_ehist.p != nullptr;
  const bool rec = record && c->rec.nrec > 0 && (dstep || (n >= 0 && n < c->rec.nt_max));
  const bool pre = prestore && c->src.nsrc > 0 && c->src.nsn > 0;
  A.nrec = rec ? c->rec.nrec : 0;
  A.energy = src ? 1 : 0;
  A.nsn = pre ? c->src.nsn : 0;
  A.units = A.nrec + A.energy + (int)(((int64_t)c->nmodels * A.nsn * c->ncomp + 63) / 64);
  A.npt = c->src.npts;
  A.n3 = c->n3;
  A.nc = c->ncomp;
  A.nmodels = c->nmodels;
  A.with_corr = with_corr ? 1 : 0;
  A.nglob = c->nglob;
  A.nt_max = c->rec.nt_max;
  A.it = n;
  A.nstf = c->src.nstf;
  A.it0 = c->energy_it0;
  A.step = dstep;
  A.rnodes = c->rec.nodes.as<int32_t>();
  A.rwts = rwts;
  A.seis = seis;
  A.pts = c->src.pts.as<int32_t>();
  A.snodes = c->src.nodes.as<int32_t>();
  A.wdir = wdir;
  A.stf = stf;
  A.hist = c->d_ehist.as<T>();
  A.per = (int64_t)c->src.npts * c->ncomp;
  A.acc = c->d_eacc.as<double>();
  A.u = c->d_u.as<T>();
  A.snode = c->src.snode.as<int32_t>();
  A.sptr = c->src.sptr.as<int32_t>();
  A.sidx = c->src.sidx.as<int32_t>();
  A.f = c->d_f.as<T>();
  return A;
}

template <class T>
int launch_aux(semx_ctx* c, AuxArgs<T> A) {
  if (A.units == 0) return SEMX_OK;
  A.blocks = A.nrec + A.energy + (int)(((int64_t)c->nmodels * A.nsn * c->ncomp + kT - 1) / kT);
  step_aux_kernel<T><<<dim3((unsigned)A.blocks, A.nrec > 0 ? (unsigned)c->nmodels : 1u), kT, 0, c->stream>>>(A);
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

}  // namespace

AuxArgs<float> aux_args(semx_ctx* c, int64_t n, bool with_corr, bool record, const int64_t* dstep, bool prestore) {
  return aux_args_t<float>(c, n, with_corr, record, dstep, prestore, c->rec.wts.as<float>(), c->rec.seis.as<float>(),
                           c->src.wdir.as<float>(), c->src.stf.as<float>());
}

AuxArgs<double> aux_args64(semx_ctx* c, int64_t n, bool with_corr, bool record, bool prestore) {
  return aux_args_t<double>(c, n, with_corr, record, nullptr, prestore, c->rec.wts64.as<double>(),
                            c->rec.seis64.as<double>(), c->src.wdir64.as<double>(), c->src.stf64.as<double>());
}

int step_aux(semx_ctx* c, int64_t n, bool with_corr, bool record, const int64_t* dstep, bool prestore) {
  return launch_aux(c, aux_args(c, n, with_corr, record, dstep, prestore));
}

int step_aux64(semx_ctx* c, int64_t n, bool with_corr, bool record, bool prestore) {
  return launch_aux(c, aux_args64(c, n, with_corr, record, prestore));
}

// One wave sums the source work in the force launch, 256 lanes in a launch of
// its own: some 10 and 5 us per 1000 source points, the launch itself 5.  Up to
// 1024 points, or what the mesh's force takes as long for, the wave ends with the
// elements (us per step, in the force launch / before it: NGLL 5, 16^3, 32
// sources of 125 points 54 / 30, 1024 of them 1660 / 622; 48^3, 32 sources
// 238 / 215; with 8 sources 20 and 186 in the force launch).
bool aux_fits(const semx_ctx* c) {
  const int64_t points = (int64_t)c->nmodels * c->nspec * c->n3;
  return c->src.nsrc == 0 || c->src.npts <= std::max<int64_t>(1024, points / 4096);
}

int energy_track(semx_ctx* c, const void* f_pe, bool source_in_f) {
  if (!c->d_eacc.p) return fail(c, SEMX_ESTATE, "energy: the run was not reset");
  double* part = c->d_epart.as<double>();
  if (c->storage == SEMX_F64)
    energy_pass_kernel<double><<<kEnergyBlocks, kT, 0, c->stream>>>(
        c->nglob, c->ncomp, c->d_mass64.as<double>(), c->d_v.as<double>(), c->d_u.as<double>(),
        static_cast<const double*>(f_pe), part);
  else
    energy_pass_kernel<float><<<kEnergyBlocks, kT, 0, c->stream>>>(c->nglob, c->ncomp, c->d_mass64.as<double>(),
                                                                  c->d_v.as<float>(), c->d_u.as<float>(),
                                                                  static_cast<const float*>(f_pe), part);
  SEMX_HIP(c, hipGetLastError());
  energy_reduce_kernel<<<1, kT, 0, c->stream>>>(kEnergyBlocks, part, c->d_eacc.as<double>());
  SEMX_HIP(c, hipGetLastError());
  if (!source_in_f) zero_doubles_kernel<<<1, 64, 0, c->stream>>>(c->d_eacc.as<double>() + 2, 1);
  SEMX_HIP(c, hipGetLastError());
  return SEMX_OK;
}

int energy_read(semx_ctx* c, double* kin, double* pot, double* work) {
  if (c->energy_it != c->it || !c->d_eacc.p)
    return fail(c, SEMX_ESTATE,
                "energy: no half step tracked at the current time index (call semx_step after a reset or a new state)");
  double h[4] = {0, 0, 0, 0};
  SEMX_HIP(c, hipMemcpyAsync(h, c->d_eacc.p, sizeof(h), hipMemcpyDeviceToHost, c->stream));
  SEMX_HIP(c, hipStreamSynchronize(c->stream));
  *kin = 0.5 * h[0];
  *pot = -0.5 * (h[1] - h[2]);
  if (work) *work = h[3];
  return SEMX_OK;
}

}  // namespace semx

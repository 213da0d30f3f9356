// The time loop's bookkeeping of one step, wave by wave: receivers, source
// work and the coming source force.  All of it reads u^{n+1}, which the force
// pass leaves alone, and with element-local forces the force pass does not
// touch f, so these waves ride in the force launch as a few more blocks (a
// launch of their own took 4.7 us a step, as long as the force pass of a mesh
// of some hundred elements, and as long again to submit).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace semx {

template <class T>
struct AuxArgs {
  int units;   // waves of row 0 of the grid (0: nothing to do)
  int blocks;  // leading blocks of the launch that hold them (set at the launch)
  int nrec;    // receivers to record (0: none); row y of the grid is model y
  int energy;  // source work (model 0)
  int npt;
  int n3, nc, nmodels;
  int with_corr;
  int64_t nglob, nt_max, it, nstf, it0;
  const int64_t* step;  // device step counter of graph-captured steps, or null
  const int32_t* rnodes;
  const T* rwts;
  T* seis;
  const int32_t* pts;
  const int32_t* snodes;
  const T* wdir;
  const T* stf;
  T* hist;
  int64_t per;
  double* acc;
  const T* u;
  // the source force of sample it + 1, stored at the nsn source nodes (0: none)
  int nsn;
  const int32_t* snode;
  const int32_t* sptr;
  const int32_t* sidx;
  T* f;
};

// A launch that carries none of these waves: its kernel has neither their code
// nor their arguments (with both in every kernel an apply of one element took
// 0.1-0.5 us more, and each launch of a pass colour by colour as much).
struct NoAux {};

// Leading blocks of a launch with `threads` lanes a block; a multiple of the
// XCD count, so that the blocks after them keep their XCDs.
template <class T>
inline unsigned aux_blocks(const AuxArgs<T>& A, int threads, int xcds) {
  if (A.units <= 0) return 0;
  const int per = threads / 64;
  return (unsigned)(((A.units + per - 1) / per + xcds - 1) / xcds * xcds);
}

// Sum over 256 virtual lanes (lane + 64 w, w = 0..3), in the order of a
// halving tree over 256 entries.
template <class V>
__device__ __forceinline__ V tree_sum(V s0, V s1, V s2, V s3) {
  V v = (s0 + s2) + (s1 + s3);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  return v;
}

// Receiver r of model `model`: sum_q l_q(x_r) u[node_q] per component, sample
// `it` of seis [nmodels][nrec][nc][nt_max].
template <class T>
__device__ __forceinline__ void aux_receiver(const AuxArgs<T>& A, int r, int model, int lane) {
  const int64_t it = A.step ? *A.step : A.it;
  if (it < 0 || it >= A.nt_max) return;
  const T* um = A.u + (int64_t)model * A.nglob * A.nc;
  const int32_t* nodes = A.rnodes + (int64_t)r * A.n3;
  const T* wts = A.rwts + (int64_t)r * A.n3;
  T s[4][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  for (int q0 = lane; q0 < A.n3; q0 += 256) {
    int64_t g[4];
    T w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int q = q0 + 64 * k;
      g[k] = q < A.n3 ? nodes[q] : -1;
      w[k] = q < A.n3 ? wts[q] : (T)0;
    }
    if (A.nc == 3) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (g[k] >= 0) {
#pragma unroll
          for (int c = 0; c < 3; ++c) s[k][c] += w[k] * um[3 * g[k] + c];
        }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (g[k] >= 0) s[k][0] += w[k] * um[g[k]];
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T v = tree_sum(s[0][c], s[1][c], s[2][c], s[3][c]);
    if (lane == 0 && c < A.nc) A.seis[(((int64_t)model * A.nrec + r) * A.nc + c) * A.nt_max + it] = v;
  }
}

// The source points with a nonzero weight (model 0): pts[k] = s n3 + q,
// f_src^n at that point, component c = stf[s][n] * wdir[(s n3 + q) nc + c];
// hist is indexed by k.  acc[3] += 1/2 sum (u^{n+1} - u^{n-1}) . f_src^n from
// the second step on; corr: acc[2] = sum u^{n+1} . f_src^n; the history slot of
// u^{n-1} (written two steps ago) is overwritten with u^{n+1}.
template <class T>
__device__ __forceinline__ void aux_energy(const AuxArgs<T>& A, int lane) {
  const int64_t n = A.step ? *A.step : A.it;
  T* slot = A.hist + (size_t)((n + 1) & 1) * A.per;
  const bool with_work = n > A.it0;
  const bool live = n >= 0 && n < A.nstf;
  // two points a lane at a time: their indices, then their values, in one
  // round trip each (one at a time the force launch of 270 acoustic elements of
  // NGLL 8 took 7.1 instead of 5.9 us, this wave its last; more points a lane
  // cost the kernel that carries the wave its occupancy)
  auto pass = [&](int first, double& work0, double& work1, double& corr0, double& corr1) {
    for (int k0 = lane + first; k0 < A.npt; k0 += 256) {
      const bool two = k0 + 64 < A.npt;
      const int k1 = two ? k0 + 64 : k0;
      const int p0 = A.pts[k0], p1 = A.pts[k1];
      const int g0 = A.snodes[p0] * A.nc, g1 = A.snodes[p1] * A.nc;
      const T amp0 = live ? A.stf[(int64_t)(p0 / A.n3) * A.nstf + n] : (T)0;
      const T amp1 = live ? A.stf[(int64_t)(p1 / A.n3) * A.nstf + n] : (T)0;
#pragma unroll 1
      for (int c = 0; c < A.nc; ++c) {
        const T u0 = A.u[g0 + c], u1 = A.u[g1 + c];
        const double fs0 = (double)amp0 * (double)A.wdir[A.nc * p0 + c];
        const double fs1 = (double)amp1 * (double)A.wdir[A.nc * p1 + c];
        const T old0 = slot[A.nc * k0 + c], old1 = slot[A.nc * k1 + c];
        work0 += 0.5 * ((double)u0 - (double)old0) * fs0;
        corr0 += (double)u0 * fs0;
        slot[A.nc * k0 + c] = u0;
        if (two) {
          work1 += 0.5 * ((double)u1 - (double)old1) * fs1;
          corr1 += (double)u1 * fs1;
          slot[A.nc * k1 + c] = u1;
        }
      }
    }
  };
  double w0 = 0, w1 = 0, w2 = 0, w3 = 0, c0 = 0, c1 = 0, c2 = 0, c3 = 0;
  pass(0, w0, w1, c0, c1);
  pass(128, w2, w3, c2, c3);
  const double ws = tree_sum(w0, w1, w2, w3), cs = tree_sum(c0, c1, c2, c3);
  if (lane == 0) {
    if (with_work) A.acc[3] += ws;
    if (A.with_corr) A.acc[2] = cs;
  }
}

// Source force of the coming sample: one lane per (model, source node,
// component) sums the (source, point) pairs that reach the node in a fixed
// order.  The stores touch only source nodes, which nothing else reads here.
template <class T>
__device__ __forceinline__ void aux_source(const AuxArgs<T>& A, int64_t t) {
  const int64_t m = (A.step ? *A.step : A.it) + 1, per_m = (int64_t)A.nsn * A.nc;
  if (t >= A.nmodels * per_m) return;
  const int64_t r = t % per_m;
  const int i = (int)(r / A.nc), c = (int)(r % A.nc);
  T sum = 0;
  for (int k = A.sptr[i]; k < A.sptr[i + 1]; ++k) {
    const int p = A.sidx[k];
    const T amp = (m >= 0 && m < A.nstf) ? A.stf[(int64_t)(p / A.n3) * A.nstf + m] : (T)0;
    sum += amp * A.wdir[(int64_t)A.nc * p + c];
  }
  A.f[((t / per_m) * A.nglob + A.snode[i]) * A.nc + c] = sum;
}

// True for the leading blocks of a launch (which then return).
template <class T>
__device__ __forceinline__ bool run_aux(const AuxArgs<T>& A) {
  if ((int)blockIdx.x >= A.blocks) return false;  // uniform over the block
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int unit = (int)blockIdx.x * (int)(blockDim.x >> 6) + wave, model = blockIdx.y;
  if (unit < A.nrec) {
    aux_receiver(A, unit, model, lane);
  } else if (model == 0 && unit < A.units) {
    const int rest = unit - A.nrec;
    if (A.energy && rest == 0) aux_energy(A, lane);
    else aux_source(A, (int64_t)(rest - A.energy) * 64 + lane);
  }
  return true;
}
__device__ __forceinline__ bool run_aux(const NoAux&) { return false; }

// Blocks that come before the launch's own.
template <class T>
__device__ __forceinline__ int aux_lead(const AuxArgs<T>& A) {
  return A.blocks;
}
__device__ __forceinline__ int aux_lead(const NoAux&) { return 0; }

// Calls launch(aux, lead): the waves `p` of a launch with `threads` lanes a block
// and their leading blocks, or NoAux and 0.
template <class T, class F>
inline void with_aux(const AuxArgs<T>* p, int threads, int xcds, F launch) {
  if (p && p->units > 0) {
    AuxArgs<T> A = *p;
    A.blocks = (int)aux_blocks(A, threads, xcds);
    launch(A, (unsigned)A.blocks);
  } else {
    launch(NoAux{}, 0u);
  }
}

}  // namespace semx

// The explicit Newmark (beta = 0, gamma = 1/2) update of one entry (node,
// component), shared by the passes that apply it.
#pragma once
#include <hip/hip_runtime.h>

namespace semx {

// mode bit 1 (kCorrect): acc = M^{-1} f, v += dt/2 acc, and acc is stored to
// a if kStoreA; without it acc is read from a.  Bit 2 (kPredict): u += dt v +
// dt^2/2 acc, v += dt/2 acc, f = 0 unless kKeepF (the coming force pass
// overwrites every node).  A step is "correct then predict" in one pass, so a
// never has to be written.  kSeg (the adjoint's forward recomputation): also
// store acc to seg_a and the predicted u to seg_u, the segment buffers.
constexpr int kCorrect = 1, kPredict = 2, kStoreA = 4, kKeepF = 8, kSeg = 16;

// m = M^{-1} at the node, ff and aa its f and a; uu and vv are updated in
// place, the acceleration used is returned.
template <int MODE, class T>
__device__ __forceinline__ T newmark_entry(T m, T ff, T aa, T dt, T hdt, T hdt2, T& uu, T& vv) {
  T acc;
  if constexpr ((MODE & kCorrect) != 0) {
    acc = m * ff;
    vv = vv + hdt * acc;
  } else {
    acc = aa;
  }
  if constexpr ((MODE & kPredict) != 0) {
    uu = uu + dt * vv + hdt2 * acc;
    vv = vv + hdt * acc;
  }
  return acc;
}

}  // namespace semx

// The scalar (acoustic) operator on the line kernel.
#include "force_line.hpp"

namespace semx {

hipError_t launch_force_line_acoustic(int n, int geo, int64_t naff, const ForceArgs& a, hipStream_t s) {
  return launch_line_f32<1>(n, geo, naff, a, s);
}

}  // namespace semx

// The elastic operator on the line kernel.
#include "force_line.hpp"

namespace semx {

hipError_t launch_force_line(int n, int geo, int64_t naff, const ForceArgs& a, hipStream_t s) {
  return launch_line_f32<3>(n, geo, naff, a, s);
}

}  // namespace semx

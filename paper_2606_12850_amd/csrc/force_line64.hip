// The elastic operator in double on the line kernel.
#include "force_line.hpp"

namespace semx {

hipError_t launch_force_line64(int n, int geo, int64_t naff, const LineArgs<double>& a, hipStream_t s) {
  return launch_line_any<double, 3, 10>(n, geo, naff, a, s);
}

}  // namespace semx

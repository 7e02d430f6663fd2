// The line pass along columns (see line_launch.hpp).
#include "line_launch.hpp"

namespace sgpe {

hipError_t launch_line_col(const LineArgs& a, const LineArgs* tab, int count, int n, int n_lines, bool full, bool nln,
                           int points, hipStream_t s) {
  return line_dispatch<true>(a, tab, count, n, n_lines, full, nln, points, s);
}

hipError_t launch_line_col(const LineArgsT<double>& a, int n, int n_lines, bool full, int points, hipStream_t s) {
  return line_dispatch_c128<true>(a, n, n_lines, full, points, s);
}

}  // namespace sgpe

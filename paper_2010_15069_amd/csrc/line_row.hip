// The line pass along rows, and the entry points of both axes (see line_launch.hpp).
#include "line_launch.hpp"

namespace sgpe {

hipError_t launch_line_col(const LineArgs& a, const LineArgs* tab, int count, int n, int n_lines, bool full, bool nln,
                           int points, hipStream_t s);
hipError_t launch_line_col(const LineArgsT<double>& a, int n, int n_lines, bool full, int points, hipStream_t s);

hipError_t launch_line(const LineArgs& a, int n, int n_lines, bool col, bool full, bool nln, int points,
                       hipStream_t s) {
  if (col) return launch_line_col(a, nullptr, 1, n, n_lines, full, nln, points, s);
  return line_dispatch<false>(a, nullptr, 1, n, n_lines, full, nln, points, s);
}

hipError_t launch_line(const LineArgsT<double>& a, int n, int n_lines, bool col, bool full, int points,
                       hipStream_t s) {
  if (col) return launch_line_col(a, n, n_lines, full, points, s);
  return line_dispatch_c128<false>(a, n, n_lines, full, points, s);
}

hipError_t launch_line_batch(const LineArgs& shape, const LineArgs* tab, int count, int n, int n_lines, bool col,
                             bool full, int points, hipStream_t s) {
  if (!tab) return hipErrorInvalidValue;
  if (col) return launch_line_col(shape, tab, count, n, n_lines, full, false, points, s);
  return line_dispatch<false>(shape, tab, count, n, n_lines, full, false, points, s);
}

}  // namespace sgpe

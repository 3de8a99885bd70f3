// Launch arithmetic of the increment builder.  Plain C++ (constexpr functions are device functions, too), so that
// it can be checked on the host at sizes that no test runs.
#pragma once

namespace evk {

// Words that a launch of gx x gy workgroups of nt threads clears: thread t of workgroup (bx, by) takes first, first +
// step, ..  (A tall input's launch has more than 2^31 threads.)
struct ClearShare { long long first, step; };
constexpr ClearShare clear_share(unsigned gx, unsigned gy, unsigned nt, unsigned bx, unsigned by, unsigned t) {
  return ClearShare{((long long)by * gx + bx) * nt + t, (long long)gx * gy * nt};
}

}  // namespace evk

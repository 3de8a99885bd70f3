// Launch arithmetic of the increment builder.  Plain C++ (constexpr functions are device functions, too), so that
// it can be checked on the host at sizes that no test runs.
#pragma once

namespace evk {

// Wide inputs: a workgroup is 64 sites, 2^ls columns x 64 / 2^ls rows (all inside one row of tiles), of a block of
// channels.  Rows of 64 columns, or of the next power of two over a narrow image's width: at least half of a
// narrow image's lanes have a site, and the workgroups of every input with fewer than 2^31 elements, 9 channels or more,
// that takes fewer than 2^23 8 x 8 tiles fit a launch of fewer than 2^32 threads along x.
constexpr int builder_wide_ls(int w) { return w > 32 ? 6 : w > 16 ? 5 : w > 8 ? 4 : 3; }
constexpr long long builder_wide_groups(int h, int w) {
  const int ls = builder_wide_ls(w);
  return (((long long)h + 7) / 8 << (ls - 3)) * (((long long)w + (1 << ls) - 1) >> ls);
}

// Words that a launch of gx x gy workgroups of nt threads clears: thread t of workgroup (bx, by) takes first, first +
// step, ..  (A tall input's launch has more than 2^31 threads.)
struct ClearShare { long long first, step; };
constexpr ClearShare clear_share(unsigned gx, unsigned gy, unsigned nt, unsigned bx, unsigned by, unsigned t) {
  return ClearShare{((long long)by * gx + bx) * nt + t, (long long)gx * gy * nt};
}

}  // namespace evk

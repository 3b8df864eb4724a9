// surf_hj.hip -- launchers of the whole-box redistancing, compiled once per
// precision (SURF_REAL).
#include "surf_launch.hpp"

namespace surf {

template <typename R>
void launch_pin(hipStream_t st, dim3 grid, const Grid& g, const Par<R>& p, const R* vof, R* g0,
                R* chi, const R* side) {
  auto k = g.dim == 3 ? k_pin<R, 3> : k_pin<R, 2>;
  hipLaunchKernelGGL(k, grid, dim3(PIN_TX * PIN_TY), 0, st, g, p, vof, g0, chi, side);
}

// n workgroups
static dim3 hj_grid(int n) {
  return n <= HJ_GRID_X ? dim3(n) : dim3(HJ_GRID_X, (n + HJ_GRID_X - 1) / HJ_GRID_X);
}

template <typename R>
void launch_hj2(hipStream_t st, bool many, const HjArgs<R>& a) {
  const dim3 grid = hj_grid(8 * a.per_xcd), block(256);
  // lane offsets within a row: 32 bits reach 4 GiB
  using W = unsigned long long;
  const bool wide = (W)a.g.n[0] * sizeof(R) > 0xffffffffull;
  auto k = many ? (wide ? k_hj2<R, 4, W> : k_hj2<R, 4, unsigned>)
                : (wide ? k_hj2<R, 1, W> : k_hj2<R, 1, unsigned>);
  hipLaunchKernelGGL(k, grid, block, 0, st, a);
}

template <typename R>
void launch_hj3(hipStream_t st, bool many, bool first, const HjArgs<R>& a) {
  const dim3 grid = hj_grid(8 * a.per_xcd), block(256);
  constexpr bool F32 = sizeof(R) == 4;
  const bool off32 = F32 && (unsigned long long)a.g.n[0] * a.g.n[1] * sizeof(R) <= 0xffffffffull;
  auto k = many ? (first ? (off32 ? k_hj3<R, 2, true, F32> : k_hj3<R, 2, true, false>)
                         : (off32 ? k_hj3<R, 2, false, F32> : k_hj3<R, 2, false, false>))
                : (first ? (off32 ? k_hj3<R, 1, true, F32> : k_hj3<R, 1, true, false>)
                         : (off32 ? k_hj3<R, 1, false, F32> : k_hj3<R, 1, false, false>));
  hipLaunchKernelGGL(k, grid, block, 0, st, a);
}

template void launch_pin<SURF_REAL>(hipStream_t, dim3, const Grid&, const Par<SURF_REAL>&,
                                    const SURF_REAL*, SURF_REAL*, SURF_REAL*, const SURF_REAL*);
template void launch_hj2<SURF_REAL>(hipStream_t, bool, const HjArgs<SURF_REAL>&);
template void launch_hj3<SURF_REAL>(hipStream_t, bool, bool, const HjArgs<SURF_REAL>&);

}  // namespace surf

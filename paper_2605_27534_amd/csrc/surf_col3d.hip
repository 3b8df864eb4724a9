// surf_col3d.hip -- launcher of the 3D plane-marching transport, compiled
// once per precision (SURF_REAL).
#include "surf_launch.hpp"

namespace surf {

template <typename R>
void launch_col3d(hipStream_t st, const Col3Args<R>& a, bool has_u, bool bulk) {
  const dim3 grid(8 * a.per_xcd), block(64 * C3Shape<R>::WAVES);
#define SURF_LAUNCH(...) hipLaunchKernelGGL((k_col3d<R, __VA_ARGS__>), grid, block, 0, st, a)
  if (a.Pst) {  // the instance that also stores the advected state
    if (has_u && bulk) SURF_LAUNCH(true, true, true);
    else if (has_u) SURF_LAUNCH(true, false, true);
    else if (bulk) SURF_LAUNCH(false, true, true);
    else SURF_LAUNCH(false, false, true);
    return;
  }
  if (has_u && bulk) SURF_LAUNCH(true, true, false);
  else if (has_u) SURF_LAUNCH(true, false, false);
  else if (bulk) SURF_LAUNCH(false, true, false);
  else SURF_LAUNCH(false, false, false);
#undef SURF_LAUNCH
}

template void launch_col3d<SURF_REAL>(hipStream_t, const Col3Args<SURF_REAL>&, bool, bool);

}  // namespace surf

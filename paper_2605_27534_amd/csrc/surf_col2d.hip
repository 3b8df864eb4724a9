// surf_col2d.hip -- launcher of the 2D column-streaming transport, compiled
// once per precision (SURF_REAL) and number of rows per wave (SURF_ROWS).
#include "surf_launch.hpp"

namespace surf {

template <typename R, int TY>
void launch_col2d(hipStream_t st, bool axisym, int variant, const ColArgs<R>& a, bool has_u,
                  bool bulk) {
  const dim3 grid(8 * a.per_xcd), block(64 * COL_WAVES);
#define SURF_LAUNCH(...) hipLaunchKernelGGL((k_col2d<R, TY, __VA_ARGS__>), grid, block, 0, st, a)
  if (axisym) {
    if (has_u && variant) {
      // substep-1 variants on the rings: Cartesian face values, ring weights
      if (bulk) {
        if (variant == 1) SURF_LAUNCH(true, true, true, 1, false);
        else if (variant == 2) SURF_LAUNCH(true, true, true, 0, true);
        else SURF_LAUNCH(true, true, true, 1, true);
      } else {
        if (variant == 1) SURF_LAUNCH(true, false, true, 1, false);
        else if (variant == 2) SURF_LAUNCH(true, false, true, 0, true);
        else SURF_LAUNCH(true, false, true, 1, true);
      }
      return;
    }
    if (has_u && bulk) SURF_LAUNCH(true, true, true);
    else if (has_u) SURF_LAUNCH(true, false, true);
    else if (bulk) SURF_LAUNCH(false, true, true);
    else SURF_LAUNCH(false, false, true);
    return;
  }
  if (has_u && variant) {  // the scheme only matters with a flow
    if (bulk) {
      if (variant == 1) SURF_LAUNCH(true, true, false, 1, false);
      else if (variant == 2) SURF_LAUNCH(true, true, false, 0, true);
      else SURF_LAUNCH(true, true, false, 1, true);
    } else {
      if (variant == 1) SURF_LAUNCH(true, false, false, 1, false);
      else if (variant == 2) SURF_LAUNCH(true, false, false, 0, true);
      else SURF_LAUNCH(true, false, false, 1, true);
    }
    return;
  }
  if (has_u && bulk) SURF_LAUNCH(true, true);
  else if (has_u) SURF_LAUNCH(true, false);
  else if (bulk) SURF_LAUNCH(false, true);
  else SURF_LAUNCH(false, false);
#undef SURF_LAUNCH
}

template void launch_col2d<SURF_REAL, SURF_ROWS>(hipStream_t, bool, int, const ColArgs<SURF_REAL>&,
                                                 bool, bool);

}  // namespace surf

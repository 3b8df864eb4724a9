// surf_batch_col2d.hip -- launcher of the batched column-streaming transport,
// compiled once per precision (SURF_REAL).
#include "surf_launch.hpp"

namespace surf {

template <typename R>
void launch_batch_col2d(hipStream_t st, int ty, bool rings, int grid, const ColArgs<R>* inst,
                        const int2* queue, int nqueue, const int* first, int parity,
                        double* part) {
  const dim3 gr(grid), bl(64 * COL_WAVES);
#define SURF_LAUNCH(...)                                                                       \
  hipLaunchKernelGGL((k_batch_col2d<R, __VA_ARGS__>), gr, bl, 0, st, inst, queue, nqueue, first, \
                     parity, part)
  if (rings) {
    if (ty == 16) SURF_LAUNCH(16, true);
    else SURF_LAUNCH(8, true);
  } else if (ty == 16) {
    SURF_LAUNCH(16);
  } else {
    SURF_LAUNCH(8);
  }
#undef SURF_LAUNCH
}

template void launch_batch_col2d<SURF_REAL>(hipStream_t, int, bool, int,
                                            const ColArgs<SURF_REAL>*, const int2*, int,
                                            const int*, int, double*);

}  // namespace surf

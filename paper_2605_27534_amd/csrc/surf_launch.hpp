// surf_launch.hpp -- launchers of the kernel families that are compiled in
// translation units of their own (one per family and precision, so that the
// library builds in parallel); each is defined for float and double.
#pragma once
#include "surf_col2d.hpp"
#include "surf_col3d.hpp"
#include "surf_hj.hpp"

namespace surf {

// k_col2d with TY rows per wave (2, 4 or 8); variant: bit 0 the MC limiter,
// bit 1 the transverse term of substep 1
template <typename R, int TY>
void launch_col2d(hipStream_t st, bool axisym, int variant, const ColArgs<R>& a, bool has_u,
                  bool bulk);
template <typename R>
void launch_batch_col2d(hipStream_t st, int ty, bool rings, int grid, const ColArgs<R>* inst,
                        const int2* queue, int nqueue, const int* first, int parity, double* part);
// the advected state is stored too where a.Pst is set
template <typename R>
void launch_col3d(hipStream_t st, const Col3Args<R>& a, bool has_u, bool bulk);
template <typename R>
void launch_pin(hipStream_t st, dim3 grid, const Grid& g, const Par<R>& p, const R* vof, R* g0,
                R* chi, const R* side);
// many: four (2D) or two (3D) sweeps, else one
template <typename R>
void launch_hj2(hipStream_t st, bool many, const HjArgs<R>& a);
template <typename R>
void launch_hj3(hipStream_t st, bool many, bool first, const HjArgs<R>& a);

}  // namespace surf

// surf_hj.hpp -- the level set of a whole box from a VoF field (section 2.5):
// pin data, then Godunov Jacobi sweeps over every cell.
//
//   k_pin    pin data g0 (and, for a full build, chi0): one cell per thread
//   k_hj2    S sweeps of a 2D box in one launch
//   k_hj3    S sweeps of a 3D box in one launch
//
// The sweeps run on w = s chi, s the sign of the cell's own chi0 (the sign
// bit of its pin datum).  A cell that is not pinned has six (four)
// neighbours of its own sign, or it would be cut, so with w the Godunov
// Hamiltonian has one form for both sides: per axis max(w - w_-, w - w_+, 0),
// no branch on the sign.  A cell whose fraction is NaN is not cut and cuts none
// of its neighbours; a warm start takes it for the side its level set lies on,
// since on the other side its neighbours' w would see an interface there.
#pragma once
#include "surf_common.hpp"
#include "surf_col2d.hpp"

namespace surf {

template <typename R> struct HjBits;
template <> struct HjBits<float> {
  static __device__ __forceinline__ float fold(float v, float g) {
    return __uint_as_float(__float_as_uint(v) ^ (__float_as_uint(g) & 0x80000000u));
  }
};
template <> struct HjBits<double> {
  static __device__ __forceinline__ double fold(double v, double g) {
    return __longlong_as_double(__double_as_longlong(v) ^
                                (__double_as_longlong(g) & (long long)0x8000000000000000ull));
  }
};

// Pin data: cells whose face neighbour has chi0 = (f - 1/2) h of the opposite
// (or zero) sign are pinned to the subcell distance h chi0 / Delta
// (Russo-Smereka); the others carry only the sign of chi0, stored as
// +-infinity.  chi (a full build) receives chi0; side (a warm start) is the
// level set, which stands in for a chi0 that is NaN.  Workgroups of 64 x 4 cells
// of one plane on a (nx/64, ny/4, nz) grid, looping where that exceeds the
// grid limit: coordinates without divisions (one thread per linear index,
// which divided twice in 64 bits, took 47 us at 192^3 FP32 beside a separate
// 13 us launch for chi0; this takes 28 us for both).
constexpr int PIN_TX = 64, PIN_TY = 4;
template <typename R, int DIM>
__global__ void __launch_bounds__(PIN_TX * PIN_TY) k_pin(Grid g, Par<R> p,
                                                        const R* __restrict__ vof,
                                                        R* __restrict__ g0, R* __restrict__ chi,
                                                        const R* __restrict__ side) {
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int i = blockIdx.x * PIN_TX + threadIdx.x % PIN_TX;
  if (i >= nx) return;
  const int im = map_axis(i - 1, nx, g.bc[0][0], g.bc[0][1]);
  const int ip = map_axis(i + 1, nx, g.bc[0][0], g.bc[0][1]);
  for (int k = blockIdx.z; k < nz; k += gridDim.z)
    for (int j = blockIdx.y * PIN_TY + threadIdx.x / PIN_TX; j < ny; j += gridDim.y * PIN_TY) {
      const long long row = (long long)nx * (j + (long long)ny * k);
      const int jm = map_axis(j - 1, ny, g.bc[1][0], g.bc[1][1]);
      const int jp = map_axis(j + 1, ny, g.bc[1][0], g.bc[1][1]);
      long long at[2 * DIM];
      at[0] = row + im;
      at[1] = row + ip;
      at[2] = (long long)nx * (jm + (long long)ny * k) + i;
      at[3] = (long long)nx * (jp + (long long)ny * k) + i;
      if constexpr (DIM == 3) {
        const int km = map_axis(k - 1, nz, g.bc[2][0], g.bc[2][1]);
        const int kp = map_axis(k + 1, nz, g.bc[2][0], g.bc[2][1]);
        at[4] = (long long)nx * (j + (long long)ny * km) + i;
        at[5] = (long long)nx * (j + (long long)ny * kp) + i;
      }
      R nb[2 * DIM], x0 = (vof[row + i] - R(0.5)) * p.h;
#pragma unroll
      for (int d = 0; d < 2 * DIM; ++d) nb[d] = (vof[at[d]] - R(0.5)) * p.h;
      if (side) {  // uniform
        if (isnan(x0)) x0 = side[row + i];
#pragma unroll
        for (int d = 0; d < 2 * DIM; ++d)
          if (isnan(nb[d])) nb[d] = side[at[d]];
      }
      bool cut = false;
      R jump = R(0), grad2 = R(0);
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const R xm = nb[2 * d], xp = nb[2 * d + 1];
        cut = cut || (x0 * xm <= R(0)) || (x0 * xp <= R(0));
        jump = fmax(jump, fmax(fabs(xm - x0), fabs(xp - x0)));
        const R cd = R(0.5) * (xp - xm);
        grad2 += cd * cd;
      }
      R v = x0 > R(0) ? R(INFINITY) : R(-INFINITY);
      if (cut) {
        const R Delta = fmax(fmax(rsqrt_<R>(grad2), jump), R(1e-30) * p.h);
        v = p.h * x0 / Delta;
      }
      g0[row + i] = v;
      if (chi) chi[row + i] = x0;
    }
}

// One Godunov update of w = s chi from the differences to the neighbours:
// w - dtau (|grad| - 1), the pinned value where pin is finite, clamped
// (comparisons, so that a NaN passes).  G2 is the sum of the squared one-sided
// differences (not yet divided by h).
template <typename R>
__device__ __forceinline__ R hj_finish(const Par<R>& p, R dtau, R w, R pin, R G2) {
  const R e = rsqrt_<R>(G2) * p.inv_h - R(1);
  R v = w - dtau * e;
  v = pin < R(INFINITY) ? pin : v;
  v = v > p.chimax ? p.chimax : v;
  return v < -p.chimax ? -p.chimax : v;
}
template <typename R>
__device__ __forceinline__ R hj_axis(R w, R lo, R hi) {
  const R m = fmax(fmax(w - lo, w - hi), R(0));
  return m * m;
}

template <typename R>
struct HjArgs {
  Grid g;
  Par<R> p;
  const R* src;
  const R* g0;
  R* dst;
  R dtau;
  int strips, yblocks, zblocks;  // block counts (2D: yblocks row chunks)
  int nwg, per_xcd;
  // 3D: per block two numbers, the value that every cell of the block holds in
  // src or in dst (NaN: not one value, not known, or a pinned cell or both
  // signs in the block) and the sign of its pin data (0: pinned or both)
  const R* fl_in;
  R* fl_out;
  R* fl_init;  // first launch: src's flags, reset to "not known"
  int skip;    // uniform blocks may take the shortcut
};

// Workgroups along x of a grid that needs more: an axis holds fewer than 2^32
// threads, which boxes of 4 by 10^9 (2D) and 4 x 4 by 10^8 cells (3D) exceed.
// A multiple of 8, so that the order over the XCDs stays.
constexpr int HJ_GRID_X = 1 << 20;

// ---- 2D.  Work unit: one wave, 64 columns and HJ2_TY rows, marching along y.
// Level l of the sweeps runs l rows behind the loads, on the rows of level
// l - 1 kept in registers; the x neighbours come from the lanes beside it, so
// each level costs one column on each side (64 - 2 S columns come out) and
// one row at each end.  With S = 4 a full build (72 sweeps) takes 184 us at
// 1024^2 FP32 and 141 us at 128^2, against 716 and 271 us for one sweep per
// launch with each linear index divided into coordinates (FP64: 348 against
// 747 us, 222 against 273).
// O: the lanes' byte offsets in a row, 32 bits where they reach its end.
constexpr int HJ2_TY = 16, HJ_LOOKAHEAD = 4;
template <typename R, int S, typename O>
__global__ void __launch_bounds__(256) k_hj2(HjArgs<R> a) {
  constexpr int OUT = 64 - 2 * S, NY = HJ2_TY + 2 * S;
  const int b = blockIdx.x + HJ_GRID_X * blockIdx.y;
  const int wg = (b & 7) * a.per_xcd + (b >> 3);
  if ((b >> 3) >= a.per_xcd || wg >= a.nwg) return;
  const Grid& g = a.g;
  const Par<R>& p = a.p;
  const int nx = g.n[0], ny = g.n[1];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sx = wg % a.strips, x0 = sx * OUT, y0 = ((wg / a.strips) * 4 + wv) * HJ2_TY;
  if (y0 >= ny) return;
  const int xs = x0 - S + lane;
  const int mx = map_axis(xs, nx, g.bc[0][0], g.bc[0][1]);
  const bool out_lane = lane >= S && lane < 64 - S && xs < nx;
  const O vmx = (O)mx * (O)sizeof(R), vxs = (O)xs * (O)sizeof(R);  // vxs: output lanes only
  R A[S + 1][NY], gv[NY];
  auto load = [&](const int k) {
    const long long row = (long long)nx * map_axis(y0 - S + k, ny, g.bc[1][0], g.bc[1][1]);
    gv[k] = lane_ld<R, O>(a.g0 + row, vmx);
    A[0][k] = lane_ld<R, O>(a.src + row, vmx);
  };
#pragma unroll
  for (int k = 0; k < HJ_LOOKAHEAD; ++k) load(k);
#pragma unroll
  for (int i = 0; i < NY; ++i) {
    if (i + HJ_LOOKAHEAD < NY) load(i + HJ_LOOKAHEAD);
    __builtin_amdgcn_sched_barrier(0);
    A[0][i] = HjBits<R>::fold(A[0][i], gv[i]);
#pragma unroll
    for (int l = 1; l <= S; ++l) {
      const int r = i - l;  // the row this level updates
      if (r < l || r >= NY - l) continue;
      const R w = A[l - 1][r];
      const R G2 = hj_axis<R>(w, from_left(w), from_right(w)) +
                   hj_axis<R>(w, A[l - 1][r - 1], A[l - 1][r + 1]);
      A[l][r] = hj_finish<R>(p, a.dtau, w, fabs(gv[r]), G2);
    }
    const int o = i - S;
    if (o >= S && o < NY - S) {
      const int y = y0 - S + o;
      if (out_lane && y < ny)
        lane_st<R, O>(HjBits<R>::fold(A[S][o], gv[o]), a.dst + (long long)nx * y, vxs);
    }
  }
}

// ---- 3D.  Work unit: one wave, a block of 60 x 4 x 4 cells, marching along
// z with the block's rows and S halo rows on each side in registers (S = 1
// or 2 sweeps, level l one plane behind level l - 1).  No LDS, no barrier.
// A block whose cells all hold one value, with 26 neighbours that hold the
// same value and no pinned cell or other sign among them, is only filled with
// the value its cells take, and not even that where dst holds it already:
// away from the interface a full build is uniform until the front reaches a
// block and at the clamp after it has passed.  Bound: the vector
// instructions of the other blocks (49 per cell and sweep, the halo's among
// them).  192^3 FP32, ball of radius 42 cells: 19.8 us per launch of two sweeps
// and 1.11 ms per full build, against 49 us per one-sweep launch and 5.40 ms
// before (that kernel divided each linear index into coordinates, and its
// vector units never idled).  Blocks of 8 planes took 1.21 ms (longer chains on
// fewer waves), of 6 planes 1.12 ms; consecutive blocks on different XCDs,
// instead of slabs of one XCD, 1.37 against 1.21 ms.
constexpr int HJ3_X = 60, HJ3_Y = 4, HJ3_Z = 4, HJ3_HALO = 2;
template <typename R, int S, bool FIRST, bool OFF32>
__global__ void __launch_bounds__(256) k_hj3(HjArgs<R> a) {
  constexpr int NR = HJ3_Y + 2 * S, NZ = HJ3_Z + 2 * S, LA = sizeof(R) == 4 ? 4 : 2, ES = (int)sizeof(R);
  // XCD x (workgroups b with b % 8 == x) takes the z blocks x, x + 8, ...:
  // the blocks of a slab share halo rows in its L2, and the slabs that still
  // change, which lie around the interface, spread over all XCDs
  const int b = blockIdx.x + HJ_GRID_X * blockIdx.y;
  const int ygroups = (a.yblocks + 3) / 4, slab = a.strips * ygroups;
  const int bz = (b >> 3) / slab * 8 + (b & 7), wg = (b >> 3) % slab;
  if (bz >= a.zblocks) return;
  const Grid& g = a.g;
  const Par<R>& p = a.p;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bx = wg % a.strips, by = wg / a.strips * 4 + wv;
  if (by >= a.yblocks) return;
  const int blk = bx + a.strips * (by + a.yblocks * bz);
  const int x0 = bx * HJ3_X, y0 = by * HJ3_Y, z0 = bz * HJ3_Z;
  const int xs = x0 - HJ3_HALO + lane;
  const bool out_lane = lane >= HJ3_HALO && lane < HJ3_HALO + HJ3_X && xs < nx;
  if (!FIRST && a.skip) {
    const int nb[3] = {a.strips, a.yblocks, a.zblocks};
    int q[3] = {bx + lane % 3 - 1, by + (lane / 3) % 3 - 1, bz + (lane / 9) % 3 - 1};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const bool per = g.bc[d][0] == BC_PERIODIC;  // past another side: this block's image
      q[d] = q[d] < 0 ? (per ? nb[d] - 1 : 0) : (q[d] >= nb[d] ? (per ? 0 : nb[d] - 1) : q[d]);
    }
    const int o = q[0] + nb[0] * (q[1] + nb[1] * q[2]);
    const R v = a.fl_in[2 * o], s = a.fl_in[2 * o + 1];
    const R mine = a.fl_in[2 * blk], ms = a.fl_in[2 * blk + 1], held = a.fl_out[2 * blk];
    if (__all(s == ms && v == mine)) {  // a NaN is never equal
      R w = ms > R(0) ? mine : -mine;
#pragma unroll
      for (int l = 0; l < S; ++l) w = hj_finish<R>(p, a.dtau, w, R(INFINITY), R(0));
      const R r = ms > R(0) ? w : -w;
      if (held == r) return;  // dst holds it already
      if (out_lane)
        for (int z = z0; z < z0 + HJ3_Z && z < nz; ++z)
#pragma unroll
          for (int y = y0; y < y0 + HJ3_Y; ++y)
            if (y < ny)
              lane_st<R, unsigned>(r, a.dst + (long long)nx * (y + (long long)ny * z), xs * ES);
      if (lane == 0) {
        a.fl_out[2 * blk] = r;
        a.fl_out[2 * blk + 1] = ms;
      }
      return;
    }
  }
  const int mx = map_axis(xs, nx, g.bc[0][0], g.bc[0][1]);
  // nx < 2^28 (at least 16 rows among 4e9 cells)
  const unsigned vmx = mx * ES, vxs = xs * ES;
  // OFF32 (FP32, planes of at most 4 GiB): rows take 32-bit byte offsets from the
  // plane; else a pointer each
  unsigned ro[NR], vo[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    ro[r] = (unsigned)nx * (unsigned)map_axis(y0 - S + r, ny, g.bc[1][0], g.bc[1][1]);
    vo[r] = (ro[r] + (unsigned)mx) * ES;
  }
  const long long area = (long long)nx * ny;
  R A[S + 1][NZ][NR], gv[NZ][NR];
  auto load = [&](const int k) {
    const long long pl = area * map_axis(z0 - S + k, nz, g.bc[2][0], g.bc[2][1]);
    const R* const gp = a.g0 + pl;
    const R* const sp = a.src + pl;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      gv[k][r] = OFF32 ? lane_ld<R>(gp, vo[r]) : lane_ld<R>(gp + ro[r], vmx);
      A[0][k][r] = OFF32 ? lane_ld<R>(sp, vo[r]) : lane_ld<R>(sp + ro[r], vmx);
    }
  };
#pragma unroll
  for (int k = 0; k < LA; ++k) load(k);
  bool same = true, allp = true, alln = true;
  R ref = R(0);
#pragma unroll
  for (int i = 0; i < NZ; ++i) {
    if (i + LA < NZ) load(i + LA);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < NR; ++r) A[0][i][r] = HjBits<R>::fold(A[0][i][r], gv[i][r]);
#pragma unroll
    for (int l = 1; l <= S; ++l) {
      const int k = i - l;  // the plane this level updates
      if (k < l || k >= NZ - l) continue;
#pragma unroll
      for (int r = l; r < NR - l; ++r) {
        const R w = A[l - 1][k][r];
        const R G2 = hj_axis<R>(w, from_left(w), from_right(w)) +
                     hj_axis<R>(w, A[l - 1][k][r - 1], A[l - 1][k][r + 1]) +
                     hj_axis<R>(w, A[l - 1][k - 1][r], A[l - 1][k + 1][r]);
        A[l][k][r] = hj_finish<R>(p, a.dtau, w, fabs(gv[k][r]), G2);
      }
    }
    const int o = i - S;
    if (o >= S && o < NZ - S) {
      const int z = z0 - S + o;
      R* const dp = a.dst + area * z;
#pragma unroll
      for (int r = S; r < NR - S; ++r) {
        const int y = y0 - S + r;
        const R v = HjBits<R>::fold(A[S][o][r], gv[o][r]);
        if (o == S && r == S)  // the block's first cell
          ref = sizeof(R) == 4 ? (R)__int_as_float(__builtin_amdgcn_readlane(
                                     __float_as_int((float)v), HJ3_HALO))
                               : (R)readlane_d((double)v, HJ3_HALO);
        A[S][o][r] = v;
        if (y < ny && z < nz) {  // uniform
          // lanes that store nothing vote with any value of the block
          same = same && (!out_lane || v == ref);
          if (FIRST) {
            allp = allp && (!out_lane || gv[o][r] == R(INFINITY));
            alln = alln && (!out_lane || gv[o][r] == R(-INFINITY));
          }
        }
      }
      if (out_lane && z < nz) {
#pragma unroll
        for (int r = S; r < NR - S; ++r) {
          if (y0 - S + r >= ny) break;  // uniform
          // an output lane's column is its own: vo is its offset
          if (OFF32) lane_st<R>(A[S][o][r], dp, vo[r]);
          else lane_st<R>(A[S][o][r], dp + ro[r], vxs);
        }
      }
    }
  }
  const bool one = __all(same);
  R s = R(0);
  if (FIRST) {
    const bool ap = __all(allp), an = __all(alln);
    s = ap ? R(1) : (an ? R(-1) : R(0));
    if (lane == 0) {
      a.fl_init[2 * blk] = R(NAN);
      a.fl_init[2 * blk + 1] = s;
    }
  } else {
    s = a.fl_in[2 * blk + 1];
  }
  if (lane == 0) {
    a.fl_out[2 * blk] = one && s != R(0) ? ref : R(NAN);
    a.fl_out[2 * blk + 1] = s;
  }
}

}  // namespace surf

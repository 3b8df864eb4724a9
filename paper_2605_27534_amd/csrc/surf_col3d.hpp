// surf_col3d.hpp -- the 3D transport step (substeps 1 and 2, the source,
// the equation of state and the reduction record) for the weighted flux
// form, as plane-marching workgroups.
//
// Work unit: a workgroup owns a strip of 64 columns along x (lane L holds
// column x0 - 3 + L, lanes 3 .. 60 produce output), the 16 rows y0 - 1 ..
// y0 + 14 (rows 1 .. 14 produce output) and a chunk of tz planes.  A thread
// holds C3Shape::RPT adjacent rows of its column (wave w the rows y0 - 1 + w
// RPT ..), so that the face between two of them is computed once and most y
// neighbours are registers.  It marches along z:
//   plane s:   the advected state of its rows (x-face fluxes through wave-wide
//              DPP shifts, y-face fluxes from the thread's rows and the two
//              rows beyond each end, loaded for plane s alone, z-face fluxes
//              from registers), then phi, delta, c* and Gamma* (sections 3.1,
//              2.6);
//   plane s-1: the z-face weighted fluxes, the update with the source,
//              sigma(Gamma) and the reduction terms (sections 2.3, 2.6);
//   plane s:   the weighted fluxes of the x and y faces (section 3.2,
//              Appendix A); phi, delta, c*, Gamma* of the neighbour waves' rows
//              come from LDS (two buffers, one barrier per plane).
// The plane loop is a loop, not unrolled: the body fits the instruction cache,
// and the loads of plane s + 1 are issued while plane s is computed.
//
// Boundaries as in the 2D kernel: walls and open sides mirror ghost values,
// periodic sides wrap; advective flux zero through walls, the interior value
// through open sides (accounted in the outflow budget): with mirrored ghosts
// the upwind cell holds the interior value and its minmod slope is 0, so the
// general expression gives just that.  Diffusive and confinement fluxes are
// zero through both.  Ghost cells carry finite values that reach no output.
// Strips that touch an x side run a variant with the lane selects; rows and
// planes are uniform over the wave, and their sides cost scalar branches.
//
// Bound: vector instructions, about 260 per row of 64 lanes and plane (HBM's
// floor is 121 us at 256^3 FP32 for the 36 bytes per cell, at the rate a large
// copy reaches).  FP32: 355 -> 218 us at 256^3, 62 -> 46 us at 128^3; FP64,
// 101x77x90: 134 -> 52 us.  Before, a thread held one row of sixteen waves, the
// plane loop was unrolled (58 KB of code a variant), side workgroups spilled
// scalars, and two barriers a plane ordered exchanges through LDS.  Two planes
// a turn (no register moves) spill a few vector registers, and one reload a
// plane, which waits for every load in flight, costs more than the moves:
// 370 us.
#pragma once
#include "surf_col2d.hpp"

namespace surf {

constexpr int C3_ROWS = 16, C3_OUT_ROWS = 14;  // rows and output rows per workgroup

// Rows per thread and waves per workgroup, and the waves per SIMD the
// registers leave room for: in FP32 two workgroups to a CU, so that one
// computes while the other waits at its barrier.
template <typename R>
struct C3Shape {
  static constexpr int RPT = sizeof(R) == 4 ? 4 : 2, WAVES = 16 / RPT, OCC = 2;
};

template <typename R>
struct Col3Lds {
  // phi, delta, c*, Gamma* of each wave's first and last row, plane s in
  // buffer s & 1
  R q[2][C3Shape<R>::WAVES][2][4][64];
};

template <typename R>
struct Col3Args {
  Grid g;
  Par<R> p;
  const R* chi;
  const R* u[3];
  const R* F;
  const R* psi;
  R* Fo;
  R* Po;
  R* sig;
  double* part;
  const double* state;  // running state: the time keys the FP32 stochastic rounding
  R dt;
  R area_dt;   // h^2 dt
  int strips;  // ceil(nx / 58)
  int yblocks; // ceil(ny / 14)
  int zchunks; // ceil(nz / tz)
  int tz;      // planes per chunk
  int nwg;
  int per_xcd;
  // optional: the advected state xi* (F*, psi*) of every cell, the input of
  // the adjoint step's substep-2 and advection transposes
  R* Fst = nullptr;
  R* Pst = nullptr;
};

// Buffer access: the array's resource in scalar registers, a lane byte offset
// that is the same for every access of an array, and a scalar byte offset
// (rows and planes): no vector address arithmetic.  Fields are under 2 GiB.
using BufRsrc = __amdgpu_buffer_rsrc_t;
template <typename R>
__device__ __forceinline__ BufRsrc buf_of(const R* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ float buf_ld(float, BufRsrc r, int v, int s) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
}
__device__ __forceinline__ double buf_ld(double, BufRsrc r, int v, int s) {
  const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0);
  return __longlong_as_double(((long long)x[1] << 32) | (unsigned)x[0]);
}
__device__ __forceinline__ void buf_st(float x, BufRsrc r, int v, int s) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, v, s, 0);
}
__device__ __forceinline__ void buf_st(double x, BufRsrc r, int v, int s) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const long long b = __double_as_longlong(x);
  u2 w;
  w[0] = (unsigned)b;
  w[1] = (unsigned)(b >> 32);
  __builtin_amdgcn_raw_buffer_store_b64(w, r, v, s, 0);
}

// Face and level-set data of one plane (Uz: the z face above it), and what a
// plane leaves for the next one.
template <typename R>
struct Col3In {
  R C[C3Shape<R>::RPT], Ux[C3Shape<R>::RPT], Uy[C3Shape<R>::RPT + 1], Uz[C3Shape<R>::RPT];
};
template <typename R>
struct Col3Carry {
  static constexpr int N = C3Shape<R>::RPT;
  R D[2][N];             // z difference below plane s
  R gz[2][N];            // advective flux through z face s
  R X[2][N], A[2][N];    // state and advective increment of plane s - 1 (FP64: X = xi*)
  R c[N], G[N], ph[N], de[N], iP[N];
  R div[2][N];           // weighted divergence of plane s - 1 but for its z face s
  R Uz[N];               // velocity of z face s
};

// a b + c in one rounding; the functions below contract nothing by themselves,
// so that every instance rounds alike and both cells of a face see one flux
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The kernel's arguments, read again through a pointer the compiler cannot see
// through: scalar loads of a plane's constants and resources, which would
// otherwise outnumber the scalar registers and be spilled to vector lanes.
using Col3Kernarg = const __attribute__((address_space(4))) int*;
template <typename R>
__device__ __forceinline__ Col3Args<R> col3_args(Col3Kernarg ka) {
  asm volatile("" : "+s"(ka));
  struct Words {
    int w[sizeof(Col3Args<R>) / 4];
  } v;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(Col3Args<R>) / 4); ++i) v.w[i] = ka[i];
  return __builtin_bit_cast(Col3Args<R>, v);
}

// One workgroup: strip x0, rows y0 - 1 .. y0 + 14, planes z0 .. z0 + tz - 1.
// IX: every column the strip reads lies inside the box away from the x sides.
template <typename R, bool HU, bool BULK, bool IX, bool ST>
struct Col3Wg {
  static constexpr bool SRND = sizeof(R) == 4;  // FP32: stochastically rounded state
  static constexpr int RPT = C3Shape<R>::RPT, WAVES = C3Shape<R>::WAVES;
  static constexpr int NX = RPT + 4;  // rows of the y stencil: rows -2 .. RPT + 1
  static constexpr int ES = (int)sizeof(R);
  Col3Kernarg ka;
  Col3Lds<R>& L;
  int x0, y0, z0, lane, wv, ys;
  unsigned tkey;
  bool out_lane, x_side, x_wall, x_lo_open, x_hi_open;
  // row and face masks of the wave's rows ys .. ys + RPT - 1 and the faces
  // below each (face RPT lies above the last row)
  unsigned omask, yside, ywall, yopen;
  int ro[NX], rux[RPT], ruy[RPT + 1];  // lane byte offsets of the rows in a plane
  ColAcc<R>& acc;

  __device__ __forceinline__ void setup(const Col3Args<R>& a) {
    const Grid& g = a.g;
    const int nx = g.n[0], ny = g.n[1];
    const bool px = !IX && g.bc[0][0] == BC_PERIODIC, py = g.bc[1][0] == BC_PERIODIC;
    const int xs = x0 - 3 + lane;
    int mx = xs, fxm = xs + 1;
    x_side = x_wall = x_lo_open = x_hi_open = false;
    if constexpr (!IX) {
      mx = map_axis(xs, nx, g.bc[0][0], g.bc[0][1]);
      const int fx = xs + 1;  // the lane's right face
      const bool out = !px && (fx < 0 || fx > nx);
      fxm = px ? ((fx % nx) + nx) % nx : (out ? 0 : fx);
      x_side = !px && (fx == 0 || fx == nx);
      x_wall = !px && ((fx == 0 && g.bc[0][0] == BC_WALL) || (fx == nx && g.bc[0][1] == BC_WALL));
      x_lo_open = !px && xs == 0 && g.bc[0][0] == BC_OPEN;
      x_hi_open = !px && xs == nx - 1 && g.bc[0][1] == BC_OPEN;
    }
    out_lane = lane >= 3 && lane < 3 + COL_OUT && (IX || xs < nx);
    ys = y0 - 1 + wv * RPT;
    omask = yside = ywall = yopen = 0;
#pragma unroll
    for (int r = 0; r < NX; ++r)
      ro[r] = (nx * map_axis(ys - 2 + r, ny, g.bc[1][0], g.bc[1][1]) + mx) * ES;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int y = ys + r, b = wv * RPT + r;
      rux[r] = ((nx + 1) * map_axis(y, ny, g.bc[1][0], g.bc[1][1]) + fxm) * ES;
      if (b >= 1 && b <= C3_OUT_ROWS && y < ny) omask |= 1u << r;
    }
#pragma unroll
    for (int r = 0; r <= RPT; ++r) {
      int f = ys + r;
      if (!py && (f == 0 || f == ny)) {
        yside |= 1u << r;
        const int bc = g.bc[1][f == 0 ? 0 : 1];
        if (bc == BC_WALL) ywall |= 1u << r;
        if (bc == BC_OPEN) yopen |= 1u << r;
      }
      if (py) f = f < 0 ? f + ny : (f >= ny ? (f - ny) % ny : f);
      else f = f < 0 ? 0 : (f > ny ? ny : f);
      ruy[r] = (nx * f + mx) * ES;
    }
    omask = __builtin_amdgcn_readfirstlane(omask);
    yside = __builtin_amdgcn_readfirstlane(yside);
    ywall = __builtin_amdgcn_readfirstlane(ywall);
    yopen = __builtin_amdgcn_readfirstlane(yopen);
  }

  static __device__ __forceinline__ int mapz(const Grid& g, int q) {
    return map_axis_sel3(q, g.n[2], g.bc[2][0] == BC_PERIODIC);
  }
  static __device__ __forceinline__ int map_axis_sel3(int q, int n, bool per) {
    const int lo = per ? q + n : -1 - q, hi = per ? q - n : 2 * n - 1 - q;
    q = q < 0 ? lo : (q >= n ? hi : q);
    q = q < 0 ? 0 : q;
    return q >= n ? n - 1 : q;
  }
  __device__ __forceinline__ void load_state(const Col3Args<R>& a, int z, R (&f)[RPT],
                                             R (&q)[RPT]) const {
    const int o = a.g.n[0] * a.g.n[1] * ES * mapz(a.g, z);
    const BufRsrc bF = buf_of<R>(a.F), bP = buf_of<R>(a.psi);
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      f[r] = BULK ? buf_ld(R(0), bF, ro[2 + r], o) : R(0);
      q[r] = buf_ld(R(0), bP, ro[2 + r], o);
    }
  }
  // z face j (below plane j)
  __device__ __forceinline__ void load_face_z(const Col3Args<R>& a, int j, R (&u)[RPT]) const {
    if constexpr (HU) {
      const int nz = a.g.n[2];
      const bool pz = a.g.bc[2][0] == BC_PERIODIC;
      const int k = pz ? (j < 0 ? j + nz : (j >= nz ? j - nz : j))
                       : (j < 0 ? 0 : (j > nz ? nz : j));
      const int o = a.g.n[0] * a.g.n[1] * ES * k;
      const BufRsrc b = buf_of<R>(a.u[2]);
#pragma unroll
      for (int r = 0; r < RPT; ++r) u[r] = buf_ld(R(0), b, ro[2 + r], o);
    } else {
#pragma unroll
      for (int r = 0; r < RPT; ++r) u[r] = R(0);
    }
  }
  __device__ __forceinline__ void load_plane(const Col3Args<R>& a, int z, Col3In<R>& n) const {
    const int nx = a.g.n[0], ny = a.g.n[1];
    const int k = mapz(a.g, z), o = nx * ny * ES * k;
    if constexpr (HU) {
      const int ox = (nx + 1) * ny * ES * k, oy = nx * (ny + 1) * ES * k;
      const BufRsrc bUx = buf_of<R>(a.u[0]), bUy = buf_of<R>(a.u[1]);
#pragma unroll
      for (int r = 0; r < RPT; ++r) n.Ux[r] = buf_ld(R(0), bUx, rux[r], ox);
#pragma unroll
      for (int r = 0; r <= RPT; ++r) n.Uy[r] = buf_ld(R(0), bUy, ruy[r], oy);
    }
    const BufRsrc bC = buf_of<R>(a.chi);
#pragma unroll
    for (int r = 0; r < RPT; ++r) n.C[r] = buf_ld(R(0), bC, ro[2 + r], o);
    load_face_z(a, z + 1, n.Uz);
  }

  // state of plane z on the two rows below and the two above the thread's
  __device__ __forceinline__ void load_rows(const Col3Args<R>& a, int z, R (&H)[2][4]) const {
    const int o = a.g.n[0] * a.g.n[1] * ES * mapz(a.g, z);
    const BufRsrc bF = buf_of<R>(a.F), bP = buf_of<R>(a.psi);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = ro[r < 2 ? r : RPT + r];
      H[0][r] = BULK ? buf_ld(R(0), bF, q, o) : R(0);
      H[1][r] = buf_ld(R(0), bP, q, o);
    }
  }

  // update, source, sigma and reduction terms of the output rows of plane o
  __device__ __forceinline__ void update(const Col3Args<R>& a, const int o, const Col3Carry<R>& c,
                                         const R (&w)[2][RPT], const unsigned omask) {
#pragma clang fp contract(off)
    const Par<R>& p = a.p;
    const int nx = a.g.n[0], ny = a.g.n[1];
    const R dcoef = p.Db * R(0.5) * p.inv_h * p.inv_h, scoef = p.Ds * R(0.5) * p.inv_h * p.inv_h;
    const R kl = p.kin == KIN_LANGMUIR ? R(1) : R(0);
    R Fn[RPT], Pn[RPT], sg[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const R divF = dcoef * (c.div[0][r] + w[0][r]);
      const R divP = scoef * (c.div[1][r] + w[1][r]);
      const R ps = SRND ? c.X[1][r] + c.A[1][r] : c.X[1][r];
      const R q = BULK ? fma_(-p.kd, ps, p.ka * c.c[r] * fma_(-kl, ps, p.ginf * c.de[r])) : R(0);
      if constexpr (SRND) {
        // one random word per cell and step: 16 bits for each field
        const unsigned rk = fmix32((unsigned)(nx * (ny * o + ys + r) + x0 - 3 + lane) ^ tkey);
        Fn[r] = BULK ? upd<R>(c.X[0][r], fma_(a.dt, divF - q, c.A[0][r]), rk) : R(0);
        Pn[r] = upd<R>(c.X[1][r], fma_(a.dt, divP + q, c.A[1][r]), rk >> 16);
      } else {
        Fn[r] = BULK ? fma_(a.dt, divF - q, c.X[0][r]) : R(0);
        Pn[r] = fma_(a.dt, divP + q, ps);
      }
      sg[r] = quot<R>(Pn[r], c.de[r] + p.eta_eps, c.iP[r]);
    }
    // the equation of state: one uniform switch for all rows
    Par<R> pe = p;
    if (p.eos == EOS_LIN) {
      pe.eos = EOS_LIN;
#pragma unroll
      for (int r = 0; r < RPT; ++r) sg[r] = eos<R>(sg[r], pe);
    } else if (p.eos == EOS_LANG) {
      pe.eos = EOS_LANG;
#pragma unroll
      for (int r = 0; r < RPT; ++r) sg[r] = eos<R>(sg[r], pe);
    } else {
      pe.eos = EOS_TANH;
#pragma unroll
      for (int r = 0; r < RPT; ++r) sg[r] = eos<R>(sg[r], pe);
    }
    const BufRsrc bFo = buf_of<R>(a.Fo), bPo = buf_of<R>(a.Po), bS = buf_of<R>(a.sig);
    const int oz = __builtin_amdgcn_readfirstlane(nx * ny * ES * o);
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      if (!(omask >> r & 1)) continue;  // uniform
      // an output lane's column is its own
      if (BULK) buf_st(Fn[r], bFo, ro[2 + r], oz);
      buf_st(Pn[r], bPo, ro[2 + r], oz);
      if (a.sig) buf_st(sg[r], bS, ro[2 + r], oz);
      acc.sF += (double)Fn[r];
      acc.sP += (double)Pn[r];
      acc.sD += (double)c.de[r];
      acc.sSD += (double)(sg[r] * c.de[r]);
      if (BULK) {
        acc.mxC = fmax(acc.mxC, rdiv<R>(Fn[r], c.ph[r] + p.eta));
        acc.mnF = fmin(acc.mnF, Fn[r]);
      }
      acc.mnP = fmin(acc.mnP, Pn[r]);
      acc.nbad += isfinite(Pn[r] + sg[r] + Fn[r]) ? 0 : 1;
    }
  }

  // advective flux through z face s + 1, and the z differences moved on
  __device__ __forceinline__ void flux_z(const Col3Args<R>& a, const int s,
                                         const R (&X)[2][3][RPT], const R (&Uz)[RPT],
                                         const Col3Carry<R>& c, Col3Carry<R>& n) const {
    const R hcfl = R(0.5) * (a.dt * a.p.inv_h);
    const int nz = a.g.n[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const R d = X[q][1][r] - X[q][0][r];
        n.gz[q][r] = (HU && (q || BULK)) ? bcg_face<R>(Uz[r], X[q][0][r], X[q][1][r], c.D[q][r], d,
                                                       X[q][2][r] - X[q][1][r], hcfl)
                                         : R(0);
        n.D[q][r] = d;
      }
    if (HU && a.g.bc[2][0] != BC_PERIODIC &&
        ((s + 1 == 0 && a.g.bc[2][0] == BC_WALL) || (s + 1 == nz && a.g.bc[2][1] == BC_WALL))) {
#pragma unroll
      for (int r = 0; r < RPT; ++r) n.gz[0][r] = n.gz[1][r] = R(0);
    }
  }

  // Plane s: X holds the state of the thread's rows on planes s, s + 1, s + 2
  // and leaves it moved by one; `in`, H and `c` are of plane s and leave as
  // those of plane s + 1 (`c` as `n`).
  __device__ __forceinline__ void plane(const int s_, R (&X)[2][3][RPT], R (&H)[2][4],
                                        Col3In<R>& in, const Col3Carry<R>& c, Col3Carry<R>& n) {
#pragma clang fp contract(off)
    const Col3Args<R> a = col3_args<R>(ka);
    const int s = __builtin_amdgcn_readfirstlane(s_);  // uniform: keep it scalar
    const Grid& g = a.g;
    const Par<R> p = a.p;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int pz = g.bc[2][0] == BC_PERIODIC;
    const R cfl = a.dt * p.inv_h, hcfl = R(0.5) * cfl;
    // the row masks stay bits of a register: tested ahead of the loop, each
    // would hold a 64-bit scalar mask of its own
    unsigned omask = this->omask, yside = this->yside, ywall = this->ywall, yopen = this->yopen;
    asm volatile("" : "+s"(omask), "+s"(yside), "+s"(ywall), "+s"(yopen));
    // ---- the next plane's loads
    R nX[2][RPT];
    load_state(a, s + 3, nX[0], nX[1]);
    __builtin_amdgcn_sched_barrier(0);
    // ---- advective flux through z face s + 1 (planes s, s + 1)
    flux_z(a, s, X, in.Uz, c, n);
    R (&fz)[2][RPT] = n.gz;
#pragma unroll
    for (int r = 0; r < RPT; ++r) n.Uz[r] = in.Uz[r];
    {
      // ---- y faces of plane s: face r between rows r - 1 and r
      R fy[2][RPT + 1];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        R v[NX];
        v[0] = H[q][0];
        v[1] = H[q][1];
        v[RPT + 2] = H[q][2];
        v[RPT + 3] = H[q][3];
#pragma unroll
        for (int r = 0; r < RPT; ++r) v[2 + r] = X[q][0][r];
#pragma unroll
        for (int r = 0; r <= RPT; ++r)
          fy[q][r] = (HU && (q || BULK))
                         ? bcg_face<R>(in.Uy[r], v[r + 1], v[r + 2], v[r + 1] - v[r],
                                       v[r + 2] - v[r + 1], v[r + 3] - v[r + 2], hcfl)
                         : R(0);
      }
      if (HU) load_rows(a, s + 1, H);
      if (HU && ywall) {  // uniform
#pragma unroll
        for (int r = 0; r <= RPT; ++r)
          if (ywall >> r & 1) fy[0][r] = fy[1][r] = R(0);
      }
      const int out_plane = s >= z0 && s < nz && s < z0 + a.tz;
      R ax[2][RPT], fx[2][RPT], fl[2][RPT];
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        // ---- advected state, phase field, c*, Gamma* of row r
        R sq[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const R x = X[q][0][r];
          sq[q] = x;
          n.X[q][r] = x;
          n.A[q][r] = R(0);
          fx[q][r] = fl[q][r] = R(0);
          if constexpr (HU) {
            if (q || BULK) {
              // the right face of this lane's cell; the left one is the lane
              // to the left's
              const R xr = from_right(x), e = xr - x;
              R f = bcg_face<R>(in.Ux[r], x, xr, from_left(e), e, from_right(e), hcfl);
              if constexpr (!IX) f = x_wall ? R(0) : f;
              fx[q][r] = f;
              fl[q][r] = from_left(f);
              const R div = ((f - fl[q][r]) + (fy[q][r + 1] - fy[q][r])) + (fz[q][r] - c.gz[q][r]);
              if constexpr (SRND) n.A[q][r] = -cfl * div;
              sq[q] = SRND ? x + n.A[q][r] : fma_(-cfl, div, x);
            }
          }
          if (!SRND) n.X[q][r] = sq[q];
        }
        if (!BULK) sq[0] = R(0);
        if (HU) {
          // twice the cell-mean speeds of the output cells (on a periodic axis
          // the upper face of the last cell is face 0, as in the fluxes)
          const R us = fabs(from_left(in.Ux[r]) + in.Ux[r]) + fabs(in.Uy[r] + in.Uy[r + 1]) +
                       fabs(c.Uz[r] + in.Uz[r]);
          const bool ok = out_lane && (out_plane & (int)(omask >> r));
          acc.usum = fmax(acc.usum, ok ? us : R(0));
        }
        if (ST && out_lane && (out_plane & (int)(omask >> r))) {
          const int o = nx * ny * ES * s;
          if (BULK) buf_st(sq[0], buf_of<R>(a.Fst), ro[2 + r], o);
          buf_st(sq[1], buf_of<R>(a.Pst), ro[2 + r], o);
        }
        R om;
        phase<R>(in.C[r], p, n.ph[r], om, n.de[r]);
        const R dnF = n.ph[r] + p.eta, dnP = n.de[r] + p.eta_eps;
        n.iP[r] = rrcp<R>(dnP);
        n.c[r] = quot<R>(sq[0], dnF, rrcp<R>(dnF));
        n.G[r] = quot<R>(sq[1], dnP, n.iP[r]);
        // ---- weighted x fluxes (right face by DPP)
        R wF = (n.ph[r] + from_right(n.ph[r])) * (from_right(n.c[r]) - n.c[r]);
        R wP = (n.de[r] + from_right(n.de[r])) * (from_right(n.G[r]) - n.G[r]);
        if constexpr (!IX) {
          wF = x_side ? R(0) : wF;
          wP = x_side ? R(0) : wP;
        }
        ax[0][r] = wF - from_left(wF);
        ax[1][r] = wP - from_left(wP);
      }
      // ---- open-side budget of the output cells' faces
      const int zlo = !pz && s == 0 && g.bc[2][0] == BC_OPEN;
      const int zhi = !pz && s == nz - 1 && g.bc[2][1] == BC_OPEN;
      if (HU && out_plane && (!IX || yopen || zlo || zhi)) {
        if (out_lane) {
#pragma unroll
          for (int r = 0; r < RPT; ++r) {
            if (!(omask >> r & 1)) continue;
            if (!IX && x_lo_open) acc.out -= (double)(a.area_dt * (fl[0][r] + fl[1][r]));
            if (!IX && x_hi_open) acc.out += (double)(a.area_dt * (fx[0][r] + fx[1][r]));
            if ((yopen >> r & 1) && ys + r == 0)
              acc.out -= (double)(a.area_dt * (fy[0][r] + fy[1][r]));
            if ((yopen >> (r + 1) & 1) && ys + r + 1 == ny)
              acc.out += (double)(a.area_dt * (fy[0][r + 1] + fy[1][r + 1]));
            if (zlo) acc.out -= (double)(a.area_dt * (c.gz[0][r] + c.gz[1][r]));
            if (zhi) acc.out += (double)(a.area_dt * (fz[0][r] + fz[1][r]));
          }
        }
      }
      // ---- the next plane's level set and velocities, into the registers this
      // plane is done with
      load_plane(a, s + 1, in);
      __builtin_amdgcn_sched_barrier(0);
      // ---- the wave's end rows for its neighbours
      R (&sq)[WAVES][2][4][64] = L.q[s & 1];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = e ? RPT - 1 : 0;
        sq[wv][e][0][lane] = n.ph[r];
        sq[wv][e][1][lane] = n.de[r];
        sq[wv][e][2][lane] = n.c[r];
        sq[wv][e][3][lane] = n.G[r];
      }
      // ---- weighted flux through z face s, then plane s - 1
      R w[2][RPT];
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        w[0][r] = (c.ph[r] + n.ph[r]) * (n.c[r] - c.c[r]);
        w[1][r] = (c.de[r] + n.de[r]) * (n.G[r] - c.G[r]);
      }
      if (!pz && (s == 0 || s == nz)) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) w[0][r] = w[1][r] = R(0);
      }
      if (s > z0 && out_lane) {
        update(a, s - 1, c, w, omask);
      }
      __syncthreads();
      // ---- weighted y fluxes of plane s: face r between rows r - 1 and r
      R t[RPT + 2][4];
      const int up = wv > 0 ? wv - 1 : 0, dn = wv < WAVES - 1 ? wv + 1 : wv;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        t[0][k] = sq[up][1][k][lane];
        t[RPT + 1][k] = sq[dn][0][k][lane];
      }
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        t[r + 1][0] = n.ph[r];
        t[r + 1][1] = n.de[r];
        t[r + 1][2] = n.c[r];
        t[r + 1][3] = n.G[r];
      }
      R wy[2][RPT + 1];
#pragma unroll
      for (int r = 0; r <= RPT; ++r) {
        wy[0][r] = (t[r][0] + t[r + 1][0]) * (t[r + 1][2] - t[r][2]);
        wy[1][r] = (t[r][1] + t[r + 1][1]) * (t[r + 1][3] - t[r][3]);
      }
      if (yside) {  // uniform
#pragma unroll
        for (int r = 0; r <= RPT; ++r)
          if (yside >> r & 1) wy[0][r] = wy[1][r] = R(0);
      }
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        n.div[0][r] = (ax[0][r] + (wy[0][r + 1] - wy[0][r])) - w[0][r];
        n.div[1][r] = (ax[1][r] + (wy[1][r + 1] - wy[1][r])) - w[1][r];
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        X[q][0][r] = X[q][1][r];
        X[q][1][r] = X[q][2][r];
        X[q][2][r] = nX[q][r];
      }
  }

  __device__ __forceinline__ void run() {
    const Col3Args<R> a = col3_args<R>(ka);
    setup(a);
    const int nz = a.g.n[2];
    const int s_end = z0 + a.tz < nz ? z0 + a.tz : nz;  // last plane advected
    R X[2][3][RPT], H[2][4] = {};
    Col3In<R> in{};
    Col3Carry<R> c{}, n{};
    // face z0 - 1, then on to plane z0 - 1
    load_state(a, z0 - 3, n.D[0], n.D[1]);
    load_state(a, z0 - 2, X[0][0], X[1][0]);
    load_state(a, z0 - 1, X[0][1], X[1][1]);
    load_state(a, z0, X[0][2], X[1][2]);
    load_face_z(a, z0 - 1, c.Uz);
    R N[2][RPT];
    load_state(a, z0 + 1, N[0], N[1]);
    load_plane(a, z0 - 1, in);
    if (HU) load_rows(a, z0 - 1, H);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        c.D[q][r] = X[q][0][r] - n.D[q][r];
      }
    flux_z(a, z0 - 2, X, c.Uz, c, n);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        c.gz[q][r] = n.gz[q][r];
        c.D[q][r] = n.D[q][r];
        X[q][0][r] = X[q][1][r];
        X[q][1][r] = X[q][2][r];
        X[q][2][r] = N[q][r];
      }
#pragma unroll 1
    for (int s = z0 - 1; s <= s_end; ++s) {
      plane(s, X, H, in, c, n);
      c = n;
    }
    acc.usum *= R(0.5);
  }
};

template <typename R, bool HU, bool BULK, bool ST>
__global__ void __launch_bounds__(64 * C3Shape<R>::WAVES, C3Shape<R>::OCC) k_col3d(Col3Args<R> a) {
  __shared__ Col3Lds<R> L;
  const int b = blockIdx.x;
  const int wg = (b & 7) * a.per_xcd + (b >> 3);  // banded over the XCDs
  if (wg >= a.nwg) return;  // uniform per workgroup: no barrier is skipped by part of it
  const int nx = a.g.n[0];
  // the wave index is uniform over the wave: say so
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sx = wg % a.strips, rest = wg / a.strips;
  const int yb = rest % a.yblocks, zc = rest / a.yblocks;
  const int x0 = sx * COL_OUT, y0 = yb * C3_OUT_ROWS, z0 = zc * a.tz;
  ColAcc<R> acc{0.0, 0.0, 0.0, 0.0, 0.0, R(0), R(-INFINITY), R(INFINITY), R(INFINITY), 0};
  const bool ix = x0 >= 3 && x0 + 62 <= nx;
  const unsigned tk = sizeof(R) == 4 ? step_key(a.state[S_TIME]) : 0u;
  const Col3Kernarg ka = (Col3Kernarg)__builtin_amdgcn_kernarg_segment_ptr();
  if (ix) {
    Col3Wg<R, HU, BULK, true, ST> w{ka, L, x0, y0, z0, lane, wv, 0, tk, false, false, false,
                                    false, false, 0, 0, 0, 0, {}, {}, {}, acc};
    w.run();
  } else {
    Col3Wg<R, HU, BULK, false, ST> w{ka, L, x0, y0, z0, lane, wv, 0, tk, false, false, false,
                                     false, false, 0, 0, 0, 0, {}, {}, {}, acc};
    w.run();
  }
  double v[NPART];
  v[P_SUM_F] = acc.sF;
  v[P_SUM_PSI] = acc.sP;
  v[P_SUM_DELTA] = acc.sD;
  v[P_SUM_SIGDELTA] = acc.sSD;
  v[P_OUTFLOW] = acc.out;
  v[P_MAX_USUM] = (double)acc.usum;
  v[P_MAX_C] = (double)acc.mxC;
  v[P_MIN_F] = (double)acc.mnF;
  v[P_MIN_PSI] = (double)acc.mnP;
  v[P_NBAD] = (double)acc.nbad;
  block_partials<R, 64 * C3Shape<R>::WAVES>(v, a.part + (long long)wg * NPART);
}

}  // namespace surf

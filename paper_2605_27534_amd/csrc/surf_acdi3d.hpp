// surf_acdi3d.hpp -- the ACDI step of a 3D box (surf_acdi.hpp has the
// equations), minmod limiter without the transverse term: k_acdi3_adv and
// k_acdi3_reg, the same two substeps as k_acdi_adv and k_acdi_reg.
//
// Work unit of both: one wave, a strip of 64 columns (the outer ones halo, x
// neighbours by wave-wide DPP shifts) and RPT rows, marching along z through a
// chunk of tz planes.  Own rows' planes stay in registers, so that a plane
// costs its own loads and the halo rows'; every load of the next plane is
// issued before the arithmetic of this one.  Each face's flux is computed
// once: through x faces by the lane on the low side and handed on by a shift,
// through y faces by the wave (those at a block's ends by both blocks, from
// the same values in the same order), through z faces carried to the next
// plane (at a chunk's ends by both chunks).  No LDS, no barrier.
// Bound: the traffic, 24 and 16 bytes a cell in FP32 (670 MB at 256^3: 135 us at
// the rate a large copy reaches) with the halo rows and planes on top, which
// come from the caches.  One ACDI step of a 256^3 box (FP32) takes 188 us, of a
// 160^3 box in FP64 127 us; one cell per thread, every face's flux and every
// difference formed by both its cells, took 365 and 282 us.  Two or eight
// rows per wave (FP32) took 195 and 211 us.
#pragma once
#include "surf_acdi.hpp"

namespace surf {

template <typename R> struct A3Shape { static constexpr int RPT = sizeof(R) == 4 ? 4 : 2; };
constexpr int A3_ADV_HALO = 2, A3_REG_HALO = 1;  // halo columns on each side
constexpr int A3_WAVES = 4;                      // per workgroup: consecutive row blocks

template <typename R>
struct Acdi3Args {
  AcdiArgs<R> a;
  const R* phi;   // adv: phi; reg: phi*
  const R* s;     // reg: s(phi*)
  const R* u[3];  // adv: face velocities or null
  R* out0;        // adv: phi*; reg: phi
  R* out1;        // adv: s(phi*); reg: the level set
  int strips, ygroups, zchunks, tz, nwg, per_xcd;
};

// 1 / max(sqrt(g2), 1/2)
__device__ __forceinline__ float a3_rnorm(float g2) {
  return fmin(__builtin_amdgcn_rsqf(g2), 2.0f);
}
__device__ __forceinline__ double a3_rnorm(double g2) { return 1.0 / fmax(sqrt(g2), 0.5); }

// the wave's strip, first row and planes; false when it has none
template <typename R, int HALO>
__device__ __forceinline__ bool a3_unit(const Acdi3Args<R>& q, int& x0, int& y0, int& z0, int& z1) {
  const int b = blockIdx.x, wg = (b & 7) * q.per_xcd + (b >> 3);
  if (wg >= q.nwg) return false;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  x0 = wg % q.strips * (64 - 2 * HALO);
  const int r = wg / q.strips;
  y0 = (r % q.ygroups * A3_WAVES + wv) * A3Shape<R>::RPT;
  z0 = r / q.ygroups * q.tz;
  z1 = min(z0 + q.tz, q.a.g.n[2]);
  return y0 < q.a.g.n[1];
}

template <typename R, typename O, bool HU>
__global__ void __launch_bounds__(64 * A3_WAVES) k_acdi3_adv(Acdi3Args<R> q) {
  constexpr int N = A3Shape<R>::RPT;
  constexpr O ES = sizeof(R);
  const AcdiArgs<R>& a = q.a;
  const Grid& g = a.g;
  int x0, y0, z0, z1;
  if (!a3_unit<R, A3_ADV_HALO>(q, x0, y0, z0, z1)) return;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lane = threadIdx.x & 63, xs = x0 - A3_ADV_HALO + (int)lane;
  const bool out_lane = lane >= A3_ADV_HALO && lane < 64 - A3_ADV_HALO && xs < nx;
  const bool perx = g.bc[0][0] == BC_PERIODIC, pery = g.bc[1][0] == BC_PERIODIC,
             perz = g.bc[2][0] == BC_PERIODIC;
  const O mx = (O)map_axis_sel(xs, nx, g.bc[0][0], g.bc[0][1]);
  int xf = xs + 1;  // the face on this lane's high side
  const bool bxlo = !perx && xf == 0, bxhi = !perx && xf == nx;
  xf = perx && xf == nx ? 0 : (xf < 0 ? 0 : (xf > nx ? nx : xf));
  const bool sides = !perx && (x0 - A3_ADV_HALO < 0 || x0 + 64 - A3_ADV_HALO > nx);  // uniform
  // lane offsets within a plane: rows y0 - 2 .. y0 + N + 1 of cells, the x and
  // y faces (the z faces' rows are the cells')
  O ro[N + 4], xo[N], yo[N + 1];
#pragma unroll
  for (int r = 0; r < N + 4; ++r)
    ro[r] = ((O)nx * (O)map_axis(y0 + r - 2, ny, g.bc[1][0], g.bc[1][1]) + mx) * ES;
#pragma unroll
  for (int r = 0; r < N; ++r) xo[r] = ((O)(nx + 1) * (O)min(y0 + r, ny - 1) + (O)xf) * ES;
#pragma unroll
  for (int r = 0; r <= N; ++r)
    yo[r] = ((O)nx * (O)(pery && y0 + r == ny ? 0 : min(y0 + r, ny)) + mx) * ES;
  const long long area = (long long)nx * ny;
  auto plane = [&](int z) { return q.phi + area * map_axis(z, nz, g.bc[2][0], g.bc[2][1]); };
  const R half = R(0.5) * a.cfl;
  // own rows of the planes z - 1 .. z + 2; W: halo rows of plane z
  R A[N], B[N], C[N], D[N], W[4], Ux[N], Uy[N + 1], Uz[N], Fz[N];
  auto own = [&](R* v, int z) {
    const R* const p = plane(z);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = lane_ld<R, O>(p, ro[r + 2]);
  };
  auto rest = [&](R* w, R* ux, R* uy, R* uz, int z) {
    const R* const p = plane(z);
    w[0] = lane_ld<R, O>(p, ro[0]);
    w[1] = lane_ld<R, O>(p, ro[1]);
    w[2] = lane_ld<R, O>(p, ro[N + 2]);
    w[3] = lane_ld<R, O>(p, ro[N + 3]);
    const int zf = perz && z + 1 == nz ? 0 : min(z + 1, nz);  // the face above plane z
    const int zc = min(z, nz - 1);
    const R* const px = q.u[0] + (long long)(nx + 1) * ny * zc;
    const R* const py = q.u[1] + (long long)nx * (ny + 1) * zc;
    const R* const pz = q.u[2] + area * zf;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      ux[r] = lane_ld<R, O>(px, xo[r]);
      uz[r] = lane_ld<R, O>(pz, ro[r + 2]);
    }
#pragma unroll
    for (int r = 0; r <= N; ++r) uy[r] = lane_ld<R, O>(py, yo[r]);
  };
  // the flux through the z face between planes z and z + 1 (values v0 .. v3 of
  // the planes z - 1 .. z + 2)
  auto zflux = [&](int z, R uf, R v0, R v1, R v2, R v3) {
    R f = bcg_face<R>(uf, v1, v2, v1 - v0, v2 - v1, v3 - v2, half);
    if (!perz && z + 1 == 0) f = g.bc[2][0] == BC_OPEN ? uf * v2 : R(0);
    if (!perz && z + 1 == nz) f = g.bc[2][1] == BC_OPEN ? uf * v1 : R(0);
    return f;
  };
  own(B, z0);
  if constexpr (HU) {
    R P[N], U0[N];
    own(P, z0 - 2);
    own(A, z0 - 1);
    own(C, z0 + 1);
    own(D, z0 + 2);
#pragma unroll
    for (int r = 0; r < N; ++r)  // the face below the chunk
      U0[r] = lane_ld<R, O>(q.u[2] + area * z0, ro[r + 2]);
    rest(W, Ux, Uy, Uz, z0);
#pragma unroll
    for (int r = 0; r < N; ++r) Fz[r] = zflux(z0 - 1, U0[r], P[r], A[r], B[r], C[r]);
  }
  for (int z = z0; z < z1; ++z) {
    R E[N], Wn[4], Uxn[N], Uyn[N + 1], Uzn[N];
    if (z + 1 < z1) {
      if constexpr (HU) {
        own(E, z + 3);
        rest(Wn, Uxn, Uyn, Uzn, z + 1);
      } else {
        own(E, z + 1);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    R st[N];
    if constexpr (HU) {
      R Y[N + 4], Fy[N + 1];
      Y[0] = W[0];
      Y[1] = W[1];
      Y[N + 2] = W[2];
      Y[N + 3] = W[3];
#pragma unroll
      for (int r = 0; r < N; ++r) Y[r + 2] = B[r];
#pragma unroll
      for (int r = 0; r <= N; ++r) {  // the face below row y0 + r
        Fy[r] = bcg_face<R>(Uy[r], Y[r + 1], Y[r + 2], Y[r + 1] - Y[r], Y[r + 2] - Y[r + 1],
                            Y[r + 3] - Y[r + 2], half);
        if (!pery && y0 + r == 0) Fy[r] = g.bc[1][0] == BC_OPEN ? Uy[r] * Y[r + 2] : R(0);
        if (!pery && y0 + r == ny) Fy[r] = g.bc[1][1] == BC_OPEN ? Uy[r] * Y[r + 1] : R(0);
      }
#pragma unroll
      for (int r = 0; r < N; ++r) {
        const R xr = from_right(B[r]), d = xr - B[r];
        R Fx = bcg_face<R>(Ux[r], B[r], xr, from_left(d), d, from_right(d), half);
        if (sides) {
          if (bxlo) Fx = g.bc[0][0] == BC_OPEN ? Ux[r] * xr : R(0);
          if (bxhi) Fx = g.bc[0][1] == BC_OPEN ? Ux[r] * B[r] : R(0);
        }
        const R Fn = zflux(z, Uz[r], A[r], B[r], C[r], D[r]);
        R div = Fx - from_left(Fx);
        div = div - Fy[r] + Fy[r + 1];
        div = div - Fz[r] + Fn;
        Fz[r] = Fn;
        st[r] = B[r] - a.cfl * div;
      }
    } else {
#pragma unroll
      for (int r = 0; r < N; ++r) st[r] = B[r];
    }
    R* const o0 = q.out0 + area * z;
    R* const o1 = q.out1 + area * z;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const R sv = acdi_s<R>(st[r], a.p.eps, a.ve);
      if (out_lane && y0 + r < ny) {
        lane_st<R, O>(st[r], o0, ro[r + 2]);  // an output lane's row is its own
        lane_st<R, O>(sv, o1, ro[r + 2]);
      }
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
      if constexpr (HU) {
        A[r] = B[r];
        B[r] = C[r];
        C[r] = D[r];
        D[r] = E[r];
        Ux[r] = Uxn[r];
        Uz[r] = Uzn[r];
      } else {
        B[r] = E[r];
      }
    }
    if constexpr (HU) {
#pragma unroll
      for (int r = 0; r <= N; ++r) Uy[r] = Uyn[r];
#pragma unroll
      for (int k = 0; k < 4; ++k) W[k] = Wn[k];
    }
  }
}

// The regularization.  The transverse derivatives of a face are means of two
// cells' centred differences; each cell's three differences are formed once.
// With e = exp(-|s_f| / eps), 1 - tanh^2(s_f / (2 eps)) = 4 e / (1 + e)^2.
template <typename R, typename O>
__global__ void __launch_bounds__(64 * A3_WAVES) k_acdi3_reg(Acdi3Args<R> q) {
  constexpr int N = A3Shape<R>::RPT;
  constexpr O ES = sizeof(R);
  const AcdiArgs<R>& a = q.a;
  const Par<R>& p = a.p;
  const Grid& g = a.g;
  int x0, y0, z0, z1;
  if (!a3_unit<R, A3_REG_HALO>(q, x0, y0, z0, z1)) return;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lane = threadIdx.x & 63, xs = x0 - A3_REG_HALO + (int)lane;
  const bool out_lane = lane >= A3_REG_HALO && lane < 64 - A3_REG_HALO && xs < nx;
  const bool perx = g.bc[0][0] == BC_PERIODIC, pery = g.bc[1][0] == BC_PERIODIC,
             perz = g.bc[2][0] == BC_PERIODIC;
  const O mx = (O)map_axis_sel(xs, nx, g.bc[0][0], g.bc[0][1]);
  const bool noflux = !perx && (xs + 1 == 0 || xs + 1 == nx);  // the face on the high side
  const bool sides = !perx && (x0 - A3_REG_HALO < 0 || x0 + 64 - A3_REG_HALO > nx);  // uniform
  O ro[N + 2];  // lane offsets of the rows y0 - 1 .. y0 + N within a plane
#pragma unroll
  for (int r = 0; r < N + 2; ++r)
    ro[r] = ((O)nx * (O)map_axis(y0 + r - 1, ny, g.bc[1][0], g.bc[1][1]) + mx) * ES;
  const long long area = (long long)nx * ny;
  auto at = [&](int z) { return area * map_axis(z, nz, g.bc[2][0], g.bc[2][1]); };
  const R qh = R(0.25) * p.inv_h, ce = a.zeta * (p.eps * p.inv_h), cx = R(-0.5) * p.inv_eps;
  auto flux = [&](R sL, R sR, R pL, R pR, R t0, R t1) {
    const R gn = (sR - sL) * p.inv_h, ta = t0 * qh, tb = t1 * qh;
    const R nd = gn * a3_rnorm(gn * gn + ta * ta + tb * tb);
    const R e = rexp<R>(fabs(sL + sR) * cx), w = rrcp<R>(R(1) + e);
    return ce * (pR - pL) - a.zeta * (e * w * w * nd);
  };
  auto rows = [&](R* v, const R* f, int z) {  // all rows of a plane
    const R* const b = f + at(z);
#pragma unroll
    for (int r = 0; r < N + 2; ++r) v[r] = lane_ld<R, O>(b, ro[r]);
  };
  auto xdiff = [&](R* v, const R* s) {
#pragma unroll
    for (int r = 0; r < N + 2; ++r) v[r] = from_right(s[r]) - from_left(s[r]);
  };
  // s on the planes z - 1, z, z + 1 and phi* on z, z + 1; the centred x
  // differences of planes z and z + 1
  R S0[N + 2], S1[N + 2], S2[N + 2], P1[N + 2], P2[N + 2], X1[N + 2], X2[N + 2], Gz[N];
  {
    R P0[N + 2], X0[N + 2];
    rows(S0, q.s, z0 - 1);
    rows(S1, q.s, z0);
    rows(P0, q.phi, z0 - 1);
    rows(P1, q.phi, z0);
    rows(S2, q.s, z0 + 1);
    rows(P2, q.phi, z0 + 1);
    xdiff(X0, S0);
    xdiff(X1, S1);
    const bool has = perz || z0 > 0;
#pragma unroll
    for (int r = 1; r <= N; ++r)
      Gz[r - 1] = has ? flux(S0[r], S1[r], P0[r], P1[r], X0[r] + X1[r],
                             (S0[r + 1] - S0[r - 1]) + (S1[r + 1] - S1[r - 1]))
                      : R(0);
  }
  for (int z = z0; z < z1; ++z) {
    R Sn[N + 2], Pn[N + 2];
    if (z + 1 < z1) {
      rows(Sn, q.s, z + 2);
      rows(Pn, q.phi, z + 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    xdiff(X2, S2);
    R Z[N + 2], Gy[N + 1];
#pragma unroll
    for (int r = 0; r < N + 2; ++r) Z[r] = S2[r] - S0[r];
#pragma unroll
    for (int r = 0; r <= N; ++r) {  // the face below row y0 + r
      Gy[r] = flux(S1[r], S1[r + 1], P1[r], P1[r + 1], X1[r] + X1[r + 1], Z[r] + Z[r + 1]);
      if (!pery && (y0 + r == 0 || y0 + r == ny)) Gy[r] = R(0);
    }
    const bool hasz = perz || z + 1 < nz;
    R* const o0 = q.out0 + area * z;
    R* const o1 = q.out1 + area * z;
#pragma unroll
    for (int r = 1; r <= N; ++r) {
      const R dy = S1[r + 1] - S1[r - 1];
      R Gx = flux(S1[r], from_right(S1[r]), P1[r], from_right(P1[r]), dy + from_right(dy),
                  Z[r] + from_right(Z[r]));
      if (sides) Gx = noflux ? R(0) : Gx;
      R Gn = flux(S1[r], S2[r], P1[r], P2[r], X1[r] + X2[r], dy + (S2[r + 1] - S2[r - 1]));
      if (!hasz) Gn = R(0);
      R acc = Gx - from_left(Gx);
      acc += Gy[r] - Gy[r - 1];
      acc += Gn - Gz[r - 1];
      Gz[r - 1] = Gn;
      const R phn = P1[r] + a.cfl * acc;
      const R chi = -acdi_s<R>(phn, p.eps, a.ve);
      if (out_lane && y0 + r - 1 < ny) {
        lane_st<R, O>(phn, o0, ro[r]);
        lane_st<R, O>(fmin(fmax(chi, -p.chimax), p.chimax), o1, ro[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < N + 2; ++r) {
      S0[r] = S1[r];
      S1[r] = S2[r];
      S2[r] = Sn[r];
      P1[r] = P2[r];
      P2[r] = Pn[r];
      X1[r] = X2[r];
    }
  }
}

}  // namespace surf

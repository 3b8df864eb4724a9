// surf_adjoint.hpp -- discrete adjoint of one step (weighted flux form) for
// gfx950, in gather form (no atomics): each cell collects the transposed
// contributions of the faces whose stencils reach it.
//
//   k_adv_star   recompute the advected state xi* = A(xi^n) (section 3.1)
//   k_adj_src, k_adj3_src (2D, 3D)
//                nu = J_R^T mu: transpose of substep 2 (confinement +
//                diffusion, sections 2.6, 3.2) and of the exchange source
//                (Appendix C), plus per-workgroup partials of dL/dtheta
//   k_adj_adv    lambda^n = J_A^T nu (+ the loss term of t^n): transpose of
//                the advection with the minmod branches frozen at xi^n
//   k_loss_seed  lambda^N from the loss term of the last step
//   k_loss_w     loss weights w_n and the loss from the forward totals
//   k_adj_c0     dL/dc0 = lambda_F^0 phi
#pragma once
#include "surf_col2d.hpp"  // mm()
#include "surf_kernels.hpp"

namespace surf {

constexpr int NADJ = 4;  // dL/d(k_a, k_d, D_b, D_s)

template <typename R>
struct AdjArgs {
  Grid g;
  Par<R> p;
  const R* chi;
  const R* u[3];
  const R* F;     // state at t^n
  const R* psi;
  const R* Fs;    // advected state xi*
  const R* Ps;
  const R* mF;    // lambda^{n+1}
  const R* mP;
  R* nF;          // nu = J_R^T lambda^{n+1}
  R* nP;
  R* lF;          // lambda^n
  R* lP;
  const double* w;  // loss weight of t^n or nullptr
  double* part;     // [nblk][NADJ]
  R dt;
  int has_u;
  long long ncell;
};

// Launch shape of the per-cell adjoint kernels: 32 x 8 cells of one
// plane per 256-thread workgroup (a wave holds two rows of 32), grid
// (ceil(nx/32), ceil(ny/8), nz), so that a cell's coordinates come from the
// workgroup and thread indices (no integer division); cell indices are
// 32-bit (grids under 2^31 cells).
constexpr int ADJ_TX = 32, ADJ_TY = 8;

__device__ __forceinline__ bool adj_cell(const Grid& g, int* x) {
  x[0] = blockIdx.x * ADJ_TX + (int)(threadIdx.x % ADJ_TX);
  x[1] = blockIdx.y * ADJ_TY + (int)(threadIdx.x / ADJ_TX);
  x[2] = blockIdx.z;
  return x[0] < g.n[0] && x[1] < g.n[1];
}

// stride of axis d in the cell layout
__device__ __forceinline__ int axis_stride(const Grid& g, int d) {
  return d == 0 ? 1 : (d == 1 ? g.n[0] : g.n[0] * g.n[1]);
}

// 32-bit face index along d (the d coordinate runs 0..n_d)
__device__ __forceinline__ int face_index32(const Grid& g, int d, const int* y) {
  const int mx = g.n[0] + (d == 0), my = g.n[1] + (d == 1);
  return y[0] + mx * (y[1] + my * y[2]);
}

// the advected state xi* = xi - dt/h sum_d (flux_hi - flux_lo), fluxes as in
// the forward step (BCG-minmod face values); per axis the five cells c-2 ..
// c+2 (mapped) are loaded once and serve both faces
template <typename R, int DIM, bool BULK>
__device__ __forceinline__ void adv_star_cell(const AdjArgs<R>& a, const int* x) {
  const Grid& g = a.g;
  const Par<R>& p = a.p;
  const int c = x[0] + g.n[0] * (x[1] + g.n[1] * x[2]);
  const R cfl = a.dt * p.inv_h;
  R divF = R(0), divP = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const bool per = g.bc[d][0] == BC_PERIODIC;
    const int nd = g.n[d], st = axis_stride(g, d);
    // inside along d (2 <= x_d <= n_d - 3) the stencil needs no mapping and
    // neither face lies on a side
    const bool in = x[d] >= 2 && x[d] <= nd - 3;
    int idx[5];
    int ylo[3] = {x[0], x[1], x[2]};
    const int flo_i = face_index32(g, d, ylo);
    int fhi_i = flo_i + st;
    if (in) {
#pragma unroll
      for (int o = -2; o <= 2; ++o) idx[o + 2] = c + o * st;
    } else {
#pragma unroll
      for (int o = -2; o <= 2; ++o)
        idx[o + 2] = c + (map_axis(x[d] + o, nd, g.bc[d][0], g.bc[d][1]) - x[d]) * st;
      int yhi[3] = {x[0], x[1], x[2]};
      yhi[d] = (per && x[d] + 1 == nd) ? 0 : x[d] + 1;
      fhi_i = face_index32(g, d, yhi);
    }
    const R ulo = a.u[d][flo_i], uhi = a.u[d][fhi_i];
    const bool blo = !per && x[d] == 0, bhi = !per && x[d] == nd - 1;
#pragma unroll
    for (int f = BULK ? 0 : 1; f < 2; ++f) {
      const R* xi = f == 0 ? a.F : a.psi;
      const R v0 = xi[idx[0]], v1 = xi[idx[1]], v2 = xi[idx[2]], v3 = xi[idx[3]],
              v4 = xi[idx[4]];
      const R flo = blo ? (g.bc[d][0] == BC_OPEN ? ulo * v2 : R(0))
                        : adv_flux<R>(ulo, v0, v1, v2, v3, cfl);
      const R fhi = bhi ? (g.bc[d][1] == BC_OPEN ? uhi * v2 : R(0))
                        : adv_flux<R>(uhi, v1, v2, v3, v4, cfl);
      if (f == 0) {
        divF += -flo;
        divF += fhi;
      } else {
        divP += -flo;
        divP += fhi;
      }
    }
  }
  if (BULK) ((R*)a.Fs)[c] = a.F[c] - cfl * divF;
  ((R*)a.Ps)[c] = a.psi[c] - cfl * divP;
}

template <typename R, int DIM, bool BULK>
__global__ void __launch_bounds__(ADJ_TX * ADJ_TY) k_adv_star(AdjArgs<R> a) {
  int x[3];
  if (adj_cell(a.g, x)) adv_star_cell<R, DIM, BULK>(a, x);
}

template <int NT>
__device__ __forceinline__ void block_sum4(double* v, double* out) {
  __shared__ double red[NT / 64][NADJ];
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int s = 0; s < NADJ; ++s) {
    double x = wave_sum(v[s]);
    if (lane == 0) red[w][s] = x;
  }
  __syncthreads();
  if (threadIdx.x < NADJ) {
    double x = red[0][threadIdx.x];
    for (int q = 1; q < NT / 64; ++q) x += red[q][threadIdx.x];
    out[threadIdx.x] = x;
  }
}

// nu = mu + dt (L^T mu + dq/dxi* (mu_psi - mu_F)); the weighted operator is
// D M diag(1/w) with M the symmetric face-weighted graph Laplacian, so
// (L^T mu)_i = D sum_f wbar_f (mu_nb - mu_i) / (w_i h^2).  The divisions by
// the weights are multiplications by their reciprocals, as in the forward
// step.  2D (3D: k_adj3_src).
template <typename R, bool BULK>
__device__ __forceinline__ void adj_src_cell(const AdjArgs<R>& a, const int* x, double* acc) {
  {
    const Grid& g = a.g;
    const Par<R>& p = a.p;
    const int c = x[0] + g.n[0] * (x[1] + g.n[1] * x[2]);
    R ph, om, de;
    phase<R>(a.chi[c], p, ph, om, de);
    const R wF = ph + p.eta, wP = de + p.eta_eps;
    const R iwF = rrcp<R>(wF), iwP = rrcp<R>(wP);
    const R muF = a.mF[c], muP = a.mP[c];
    const R cF = BULK ? a.Fs[c] * iwF : R(0), cP = a.Ps[c] * iwP;
    R LtF = R(0), LtP = R(0), SF = R(0), SP = R(0);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int st = axis_stride(g, d);
#pragma unroll
      for (int s = -1; s <= 1; s += 2) {
        bool bnd = (s < 0 && x[d] == 0 && g.bc[d][0] != BC_PERIODIC) ||
                   (s > 0 && x[d] == g.n[d] - 1 && g.bc[d][1] != BC_PERIODIC);
        if (bnd) continue;
        const int o = c + (map_axis(x[d] + s, g.n[d], g.bc[d][0], g.bc[d][1]) - x[d]) * st;
        R pho, omo, deo;
        phase<R>(a.chi[o], p, pho, omo, deo);
        R fbar = R(0.5) * (ph + pho), dbar = R(0.5) * (de + deo);
        if (BULK) {
          LtF += fbar * (a.mF[o] - muF);
          SF += fbar * (a.Fs[o] * rrcp<R>(pho + p.eta) - cF);
        }
        LtP += dbar * (a.mP[o] - muP);
        SP += dbar * (a.Ps[o] * rrcp<R>(deo + p.eta_eps) - cP);
      }
    }
    const R ih2 = p.inv_h * p.inv_h;
    LtF *= p.Db * ih2 * iwF;
    LtP *= p.Ds * ih2 * iwP;
    SF *= ih2;
    SP *= ih2;
    const R diff = muP - muF;
    R nuF = muF, nuP = muP + a.dt * LtP;
    if (BULK) {
      const R Psv = a.Ps[c];
      R dqdF, dqdP, dqdka;
      if (p.kin == KIN_LANGMUIR) {
        dqdF = p.ka * (p.ginf * de - Psv) * iwF;
        dqdP = -p.ka * cF - p.kd;
        dqdka = cF * (p.ginf * de - Psv);
      } else {
        dqdF = p.ka * p.ginf * de * iwF;
        dqdP = -p.kd;
        dqdka = cF * p.ginf * de;
      }
      nuF = muF + a.dt * (LtF + dqdF * diff);
      nuP += a.dt * dqdP * diff;
      acc[0] += (double)(a.dt * dqdka * diff);
      acc[1] += (double)(a.dt * (-Psv) * diff);
      acc[2] += (double)(a.dt * SF * muF);
    }
    acc[3] += (double)(a.dt * SP * muP);
    a.nF[c] = nuF;
    a.nP[c] = nuP;
  }
}

template <typename R, bool BULK>
__global__ void __launch_bounds__(ADJ_TX * ADJ_TY) k_adj_src(AdjArgs<R> a) {
  double acc[NADJ] = {0.0, 0.0, 0.0, 0.0};
  int x[3];
  if (adj_cell(a.g, x)) adj_src_cell<R, BULK>(a, x, acc);
  const int blk = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  block_sum4<ADJ_TX * ADJ_TY>(acc, a.part + (long long)blk * NADJ);
}

// The same in 3D as marching waves: 64 columns (the outer ones halo) and N
// rows along z through a chunk of tz planes.  The phase, the weights'
// reciprocals and the concentrations of a cell are formed once per plane and
// wave (the halo rows' by two waves), each face's terms once (through x faces
// by the lane on the low side, carried to the next plane through z faces), and
// the sums of dL/dtheta are reduced once per workgroup.  Bound: the vector
// instructions.  128^3 FP32: 21 us, against 30 with one cell per thread (455
// instructions each: seven phases, 35 gathers, a reduction per 64 cells).
template <typename R> struct Adj3Shape { static constexpr int N = sizeof(R) == 4 ? 4 : 2; };
constexpr int ADJ3_X = 62, ADJ3_WAVES = 4;  // output columns; waves (row blocks) per workgroup
template <typename R>
struct Adj3Args {
  AdjArgs<R> a;
  int strips, ygroups, tz, nwg, per_xcd;
};

template <typename R, typename O, bool BULK>
__global__ void __launch_bounds__(64 * ADJ3_WAVES) k_adj3_src(Adj3Args<R> q) {
  constexpr int N = Adj3Shape<R>::N;
  constexpr O ES = sizeof(R);
  const int b = blockIdx.x, wg = (b & 7) * q.per_xcd + (b >> 3);
  if (wg >= q.nwg) return;
  const AdjArgs<R>& a = q.a;
  const Grid& g = a.g;
  const Par<R>& p = a.p;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x0 = wg % q.strips * ADJ3_X, r0 = wg / q.strips;
  const int y0 = (r0 % q.ygroups * ADJ3_WAVES + wv) * N;
  const int z0 = r0 / q.ygroups * q.tz, z1 = min(z0 + q.tz, nz);
  double acc[NADJ] = {0.0, 0.0, 0.0, 0.0};
  if (y0 < ny) {  // uniform
    const int xs = x0 - 1 + lane;
    const bool out_lane = lane >= 1 && lane <= ADJ3_X && xs < nx;
    const bool perx = g.bc[0][0] == BC_PERIODIC, pery = g.bc[1][0] == BC_PERIODIC,
               perz = g.bc[2][0] == BC_PERIODIC;
    const bool noflux = !perx && (xs + 1 == 0 || xs + 1 == nx);  // the face on the high side
    const bool sides = !perx && (x0 == 0 || x0 + ADJ3_X >= nx);  // uniform
    const O mx = (O)map_axis_sel(xs, nx, g.bc[0][0], g.bc[0][1]);
    O ro[N + 2];  // lane offsets of the rows y0 - 1 .. y0 + N within a plane
#pragma unroll
    for (int r = 0; r < N + 2; ++r)
      ro[r] = ((O)nx * (O)map_axis(y0 + r - 1, ny, g.bc[1][0], g.bc[1][1]) + mx) * ES;
    const long long area = (long long)nx * ny;
    const R ih2 = p.inv_h * p.inv_h;
    struct Raw {
      R chi[N + 2], f[N + 2], s[N + 2], mf[N + 2], mp[N + 2];
    };
    struct Plane {  // phase, delta, concentrations, lambda; reciprocal weights and psi* of own rows
      R ph[N + 2], de[N + 2], cf[N + 2], cp[N + 2], mf[N + 2], mp[N + 2], iwf[N], iwp[N], ps[N];
    };
    auto load = [&](Raw& w, int z) {
      const long long o = area * map_axis(z, nz, g.bc[2][0], g.bc[2][1]);
#pragma unroll
      for (int r = 0; r < N + 2; ++r) {
        w.chi[r] = lane_ld<R, O>(a.chi + o, ro[r]);
        w.s[r] = lane_ld<R, O>(a.Ps + o, ro[r]);
        w.mp[r] = lane_ld<R, O>(a.mP + o, ro[r]);
        if (BULK) w.f[r] = lane_ld<R, O>(a.Fs + o, ro[r]);
        if (BULK) w.mf[r] = lane_ld<R, O>(a.mF + o, ro[r]);
      }
    };
    auto derive = [&](Plane& d, const Raw& w) {
#pragma unroll
      for (int r = 0; r < N + 2; ++r) {
        R om;
        phase<R>(w.chi[r], p, d.ph[r], om, d.de[r]);
        const R iwf = rrcp<R>(d.ph[r] + p.eta), iwp = rrcp<R>(d.de[r] + p.eta_eps);
        d.cf[r] = BULK ? w.f[r] * iwf : R(0);
        d.cp[r] = w.s[r] * iwp;
        d.mf[r] = BULK ? w.mf[r] : R(0);
        d.mp[r] = w.mp[r];
        if (r >= 1 && r <= N) {
          d.iwf[r - 1] = iwf;
          d.iwp[r - 1] = iwp;
          d.ps[r - 1] = w.s[r];
        }
      }
    };
    struct Face {  // through a face, towards its low side: the four operators' terms
      R lf, lp, sf, sp;
    };
    auto face = [&](R ph0, R ph1, R de0, R de1, R mf0, R mf1, R mp0, R mp1, R cf0, R cf1, R cp0,
                    R cp1) {
      const R fbar = R(0.5) * (ph0 + ph1), dbar = R(0.5) * (de0 + de1);
      Face f;
      f.lf = BULK ? fbar * (mf1 - mf0) : R(0);
      f.sf = BULK ? fbar * (cf1 - cf0) : R(0);
      f.lp = dbar * (mp1 - mp0);
      f.sp = dbar * (cp1 - cp0);
      return f;
    };
    auto rows = [&](const Plane& u, int i, const Plane& v, int j) {
      return face(u.ph[i], v.ph[j], u.de[i], v.de[j], u.mf[i], v.mf[j], u.mp[i], v.mp[j], u.cf[i],
                  v.cf[j], u.cp[i], v.cp[j]);
    };
    Raw w;
    Plane c, n;
    Face fz[N];  // the faces below the plane
    load(w, z0 - 1);
    derive(n, w);
    load(w, z0);
    derive(c, w);
    load(w, z0 + 1);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      fz[r] = rows(n, r + 1, c, r + 1);
      if (!perz && z0 == 0) fz[r] = Face{R(0), R(0), R(0), R(0)};
    }
    for (int z = z0; z < z1; ++z) {
      derive(n, w);
      if (z + 1 < z1) load(w, z + 2);
      __builtin_amdgcn_sched_barrier(0);
      Face fy = rows(c, 0, c, 1);  // the face below the row
      if (!pery && y0 == 0) fy = Face{R(0), R(0), R(0), R(0)};
      R* const oF = a.nF + area * z;
      R* const oP = a.nP + area * z;
#pragma unroll
      for (int r = 1; r <= N; ++r) {
        Face hy = rows(c, r, c, r + 1), hz = rows(c, r, n, r);
        if (!pery && y0 + r == ny) hy = Face{R(0), R(0), R(0), R(0)};
        if (!perz && z + 1 == nz) hz = Face{R(0), R(0), R(0), R(0)};
        Face hx = face(c.ph[r], from_right(c.ph[r]), c.de[r], from_right(c.de[r]), c.mf[r],
                       BULK ? from_right(c.mf[r]) : R(0), c.mp[r], from_right(c.mp[r]), c.cf[r],
                       BULK ? from_right(c.cf[r]) : R(0), c.cp[r], from_right(c.cp[r]));
        if (sides) {
          hx.lf = noflux ? R(0) : hx.lf;
          hx.lp = noflux ? R(0) : hx.lp;
          hx.sf = noflux ? R(0) : hx.sf;
          hx.sp = noflux ? R(0) : hx.sp;
        }
        auto sum = [&](R lx, R xh, R ly, R yh, R lz, R zh) { return ((xh - lx) + (yh - ly)) + (zh - lz); };
        R LtP = sum(from_left(hx.lp), hx.lp, fy.lp, hy.lp, fz[r - 1].lp, hz.lp);
        R SP = sum(from_left(hx.sp), hx.sp, fy.sp, hy.sp, fz[r - 1].sp, hz.sp);
        const R iwF = c.iwf[r - 1], Psv = c.ps[r - 1], de = c.de[r], muF = c.mf[r], muP = c.mp[r];
        LtP *= p.Ds * ih2 * c.iwp[r - 1];
        SP *= ih2;
        R nuF = muF, nuP = muP + a.dt * LtP;
        const bool out = out_lane && y0 + r - 1 < ny;
        if (BULK) {
          R LtF = sum(from_left(hx.lf), hx.lf, fy.lf, hy.lf, fz[r - 1].lf, hz.lf);
          R SF = sum(from_left(hx.sf), hx.sf, fy.sf, hy.sf, fz[r - 1].sf, hz.sf);
          LtF *= p.Db * ih2 * iwF;
          SF *= ih2;
          const R diff = muP - muF, cF = c.cf[r];
          R dqdF, dqdP, dqdka;
          if (p.kin == KIN_LANGMUIR) {
            dqdF = p.ka * (p.ginf * de - Psv) * iwF;
            dqdP = -p.ka * cF - p.kd;
            dqdka = cF * (p.ginf * de - Psv);
          } else {
            dqdF = p.ka * p.ginf * de * iwF;
            dqdP = -p.kd;
            dqdka = cF * p.ginf * de;
          }
          nuF = muF + a.dt * (LtF + dqdF * diff);
          nuP += a.dt * dqdP * diff;
          if (out) {
            acc[0] += (double)(a.dt * dqdka * diff);
            acc[1] += (double)(a.dt * (-Psv) * diff);
            acc[2] += (double)(a.dt * SF * muF);
          }
        }
        if (out) {
          acc[3] += (double)(a.dt * SP * muP);
          if (BULK) lane_st<R, O>(nuF, oF, ro[r]);
          lane_st<R, O>(nuP, oP, ro[r]);
        }
        fy = hy;
        fz[r - 1] = hz;
      }
      c = n;
    }
  }
  block_sum4<64 * ADJ3_WAVES>(acc, a.part + (long long)wg * NADJ);
}

// derivative of the equation of state
template <typename R>
__device__ __forceinline__ R eos_prime(R G, const Par<R>& p) {
  R x = G * p.inv_ginf;
  if (p.eos == EOS_LIN) return -p.sigma0 * p.E * p.inv_ginf;
  if (p.eos == EOS_LANG) {
    if (x <= R(0) || x >= R(1) - R(1e-6)) return R(0);
    return -p.sigma0 * p.E * p.inv_ginf / (R(1) - x);
  }
  R t = rtanh<R>(p.E * x);
  return -p.sigma0 * p.E * p.inv_ginf * (R(1) - t * t);
}

// lambda_j = nu_j + (dt/h) sum_f dflux_f/dxi_j (nu_R(f) - nu_L(f)), over the
// faces f whose (mirrored or wrapped) stencil holds j: along each axis the
// faces j-1/2 .. j+5/2 (face k lies between cells j+k-1 and j+k).
//
// The flux of a face is u (xi_b + kk minmod(s1, s2)), b the upwind cell, s1 =
// xi_b - xi_{b-1}, s2 = xi_{b+1} - xi_b, kk = (1 - |u| dt/h)/2 with u's sign.
// With c = u dt/h and h = |c| (1 - |c|) / 2, which is kk c for either sign, its
// derivatives times dt/h are
//   at b - 1   -h where minmod takes s1,
//   at b       c + h where it takes s1, c - h where it takes s2, else c,
//   at b + 1   h where it takes s2.
//
// which argument minmod takes; ties go to s2, none for opposite signs or zero
template <typename R>
__device__ __forceinline__ void adj_select(R s1, R s2, bool& t1, bool& t2) {
  const R m = mm<R>(s1, s2);
  const bool any = m != R(0);
  t2 = any && m == s2;
  t1 = any && m != s2;
}

// The cell j is the cell above of face -1 (u < 0); the cell above (u > 0) or
// the upwind cell of face 0; the upwind cell or the cell below of face 1; and
// the cell below of face 2 (u > 0).  So only the choices that minmod makes
// about the cells j - 1, j and j + 1 enter, from xi at j - 2 .. j + 2 (mirrored
// or wrapped); c and h serve both fields.  Beside a wall or an open side a
// stencil that reaches one cell past it reaches the side's cell a second time
// (the cell below of face 1 at the low side, the cell above of face 0 at the
// high one), but there the mirrored difference is 0 and minmod takes neither
// argument; the side's own face carries u xi of that cell (open) or nothing,
// and the faces beyond do not exist.
template <typename R, typename O, bool BULK>
struct AdjAxis {
  R u[4], v[2][5], w[2][5];
  bool side;            // uniform: some lane's stencils leave the box or touch a side
  bool lo, hi;          // this lane's cell lies at a wall or open side
  bool none0, none3;    // faces -1 and 2 are not there for it
  bool openlo, openhi;
  // o: the cell's byte offset in its plane x[2] (uniform)
  __device__ __forceinline__ void load(const AdjArgs<R>& a, O o, int d, const int* x) {
    constexpr O ES = sizeof(R);
    const Grid& g = a.g;
    const int nx = g.n[0], ny = g.n[1], nd = g.n[d], X = x[d];
    const long long area = (long long)nx * ny;
    side = !__all(X >= 2 && X <= nd - 3);
    const bool per = g.bc[d][0] == BC_PERIODIC;
    int m[5], f[4];  // the cells' and faces' coordinates along d
#pragma unroll
    for (int k = 0; k < 5; ++k) m[k] = X + k - 2;
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = X + k - 1;
    if (side) {
#pragma unroll
      for (int k = 0; k < 5; ++k) m[k] = map_axis_sel(m[k], nd, g.bc[d][0], g.bc[d][1]);
#pragma unroll
      for (int k = 0; k < 4; ++k)  // on a periodic axis face nd is face 0
        f[k] = f[k] < 0 ? (per ? f[k] + nd : 0) : (f[k] >= nd ? (per ? f[k] - nd : nd) : f[k]);
      lo = !per && X == 0;
      hi = !per && X == nd - 1;
      none0 = !per && X <= 1;
      none3 = !per && X >= nd - 2;
      openlo = g.bc[d][0] == BC_OPEN;
      openhi = g.bc[d][1] == BC_OPEN;
    }
    // scalar plane pointer and lane offset of the cell at m
    auto cell = [&](const R* p, int k) {
      if (d == 2) return lane_ld<R, O>(p + area * m[k], o);
      const O off = side ? o + (O)(m[k] - X) * (d == 0 ? ES : (O)nx * ES)
                         : o + (O)(k - 2) * (d == 0 ? ES : (O)nx * ES);
      return lane_ld<R, O>(p + area * x[2], off);
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const R* const p = a.u[d];
      if (d == 0)
        u[k] = lane_ld<R, O>(p + (long long)(nx + 1) * ny * x[2], ((O)(nx + 1) * (O)x[1] + (O)f[k]) * ES);
      else if (d == 1)
        u[k] = lane_ld<R, O>(p + (long long)nx * (ny + 1) * x[2], ((O)nx * (O)f[k] + (O)x[0]) * ES);
      else
        u[k] = lane_ld<R, O>(p + area * f[k], o);
    }
#pragma unroll
    for (int q = BULK ? 0 : 1; q < 2; ++q) {
      const R* xi = q == 0 ? a.F : a.psi;
      const R* nu = q == 0 ? a.nF : a.nP;
#pragma unroll
      for (int k = 0; k < 5; ++k) v[q][k] = cell(xi, k);
#pragma unroll
      for (int k = 0; k < 5; ++k) w[q][k] = cell(nu, k);
    }
  }
  // SIDE: with the corrections at the sides (a branch of its own: as selects
  // they would run in every wave)
  template <bool SIDE>
  __device__ __forceinline__ void add(R cfl, R& lamF, R& lamP) const {
    auto pick = [](bool b, R h) { return b ? h : R(0); };
    R cf[4], hf[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cf[k] = u[k] * cfl;
      hf[k] = R(0.5) * fabs(cf[k]) * (R(1) - fabs(cf[k]));
    }
    const bool p1 = cf[1] > R(0), p2 = cf[2] > R(0);
    R h0 = pick(!(cf[0] > R(0)), hf[0]), h3 = pick(cf[3] > R(0), hf[3]);
    if (SIDE) {
      h0 = pick(!none0, h0);
      h3 = pick(!none3, h3);
    }
#pragma unroll
    for (int f = BULK ? 0 : 1; f < 2; ++f) {
      const R* const x = v[f];
      const R* const n = w[f];
      // minmod's choices about j - 1, j and j + 1
      const R d0 = x[1] - x[0], d1 = x[2] - x[1], d2 = x[3] - x[2], d3 = x[4] - x[3];
      bool m1, m2, c1, c2, q1, q2;
      adj_select<R>(d0, d1, m1, m2);
      adj_select<R>(d1, d2, c1, c2);
      adj_select<R>(d2, d3, q1, q2);
      auto up = [&](R cc, R h) { return cc + (pick(c1, h) - pick(c2, h)); };
      const R w0 = pick(m2, h0), w3 = -pick(q1, h3);
      const R w1 = p1 ? pick(m2, hf[1]) : up(cf[1], hf[1]);
      const R w2 = p2 ? up(cf[2], hf[2]) : -pick(q1, hf[2]);
      R t1 = w1 * (n[2] - n[1]), t2 = w2 * (n[3] - n[2]);
      if (SIDE) {
        t1 = lo ? pick(openlo, cf[1] * n[2]) : t1;
        t2 = hi ? pick(openhi, -(cf[2] * n[2])) : t2;
      }
      R& lam = f == 0 ? lamF : lamP;
      lam += w0 * (n[1] - n[0]);
      lam += t1;
      lam += t2;
      lam += w3 * (n[4] - n[3]);
    }
  }
};

// Every axis's values are loaded, at scalar plane pointers and lane offsets,
// before any is used.  Bound: instruction issue and the L1's throughput on the
// 64 gathers a cell.  128^3 FP32: 35 us, against 61 when every face's weights
// were formed from seven cells for each of its roles and the columns at the x
// sides went through workgroups of their own, which took most of the
// instructions.
template <typename R, typename O, int DIM, bool BULK, bool HU>
__device__ __forceinline__ void adj_adv_cell(const AdjArgs<R>& a, const int* x) {
  const Grid& g = a.g;
  const Par<R>& p = a.p;
  const int c = x[0] + g.n[0] * (x[1] + g.n[1] * x[2]);
  R lamF = a.nF[c], lamP = a.nP[c];
  if (HU) {
    const R cfl = a.dt * p.inv_h;
    const O o = ((O)g.n[0] * (O)x[1] + (O)x[0]) * (O)sizeof(R);
    AdjAxis<R, O, BULK> ax[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) ax[d].load(a, o, d, x);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      if (ax[d].side) ax[d].template add<true>(cfl, lamF, lamP);
      else ax[d].template add<false>(cfl, lamF, lamP);
    }
  }
  if (a.w) {
    R ph, om, de;
    phase<R>(a.chi[c], p, ph, om, de);
    R e = de + p.eta_eps;
    lamP += (R)(*a.w) * eos_prime<R>(a.psi[c] / e, p) * de / e;
  }
  a.lF[c] = BULK ? lamF : a.mF[c];
  a.lP[c] = lamP;
}

template <typename R, typename O, int DIM, bool BULK, bool HU>
__global__ void __launch_bounds__(ADJ_TX * ADJ_TY) k_adj_adv(AdjArgs<R> a) {
  int x[3];
  if (adj_cell(a.g, x)) adj_adv_cell<R, O, DIM, BULK, HU>(a, x);
}

template <typename R>
__global__ void __launch_bounds__(BLOCK) k_loss_seed(Grid g, Par<R> p, const R* __restrict__ chi,
                                                     const R* __restrict__ psi,
                                                     const double* __restrict__ w, R* lF, R* lP,
                                                     long long ncell) {
  long long c = (long long)blockIdx.x * BLOCK + threadIdx.x;
  if (c >= ncell) return;
  R ph, om, de;
  phase<R>(chi[c], p, ph, om, de);
  R e = de + p.eta_eps;
  if (lF) lF[c] = R(0);
  lP[c] = (R)(*w) * eos_prime<R>(psi[c] / e, p) * de / e;
}

// w_n = (2/N)(<sigma>^n - target^n) vol / sum(delta vol) for n = 1..N (row
// n-1 of the forward totals) and L = mean (<sigma>^n - target^n)^2
__global__ void k_loss_w(const double* __restrict__ tot, long long stride,
                         const double* __restrict__ target, int N, double vol,
                         double* __restrict__ w, double* __restrict__ loss) {
  __shared__ double part[BLOCK];
  double s = 0.0;
  for (int n = threadIdx.x; n < N; n += BLOCK) {
    const double* t = tot + (long long)n * stride;
    double r = t[13] - target[n];
    w[n] = 2.0 / N * r * vol / t[4];
    s += r * r;
  }
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int i = 0; i < BLOCK; ++i) acc += part[i];
    if (loss) *loss = acc / N;
  }
}

__global__ void k_adj_final(const double* __restrict__ part, int nblk, double* __restrict__ dtheta) {
  double v[NADJ] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int b = threadIdx.x; b < nblk; b += FIN_BLOCK)
    for (int s = 0; s < NADJ; ++s) v[s] += part[(long long)b * NADJ + s];
  __shared__ double tot[NADJ];
  block_sum4<FIN_BLOCK>(v, tot);
  __syncthreads();
  if (threadIdx.x < NADJ) dtheta[threadIdx.x] += tot[threadIdx.x];
}

template <typename R>
__global__ void __launch_bounds__(BLOCK) k_adj_c0(Grid g, Par<R> p, const R* __restrict__ chi,
                                                  const R* __restrict__ lF, R* __restrict__ gc0,
                                                  long long ncell) {
  long long c = (long long)blockIdx.x * BLOCK + threadIdx.x;
  if (c >= ncell) return;
  R ph, om, de;
  phase<R>(chi[c], p, ph, om, de);
  gc0[c] = lF[c] * ph;
}

}  // namespace surf

// surf_geo3d.hpp -- the moving-interface geometry in 3D (section 2.5):
// warm-start Jacobi sweeps restricted to the tiles near the interface.
//
// The box is cut into 16^3 tiles with one flag each (quiescent at +clamp,
// quiescent at -clamp, live).  A tile whose VoF is uniform and whose 3x3x3
// tile neighbourhood was quiescent with the same sign after the previous
// step keeps the clamp value: every cell it can reach in K <= 16 sweeps is at
// the clamp, where a Godunov sweep changes nothing.  The other tiles are
// rebuilt by K sweeps over the live tiles only.  The level set stays in one
// buffer (R); the other (S) is the sweeps' ping-pong partner.  Both hold the
// clamp on every quiescent tile, each with a flag array saying so, so that a
// sweep reads its neighbours from one buffer without looking at flags.  A
// geometry prepared while a transport still reads R sweeps between S and a
// third buffer T instead (R -> S -> T -> S ... -> T), which then becomes R:
// classify gives T the clamp on quiescent tiles too, and the last sweep
// writes T's flags.
//   k_geo3_classify  one workgroup per tile: the decision; a quiescent tile
//                    writes the clamp into S only if S's flag says S does not
//                    hold it yet; a live tile with cut cells its pin data
//                    (Russo-Smereka distance of cut cells, signed infinity
//                    elsewhere), any other live tile only its side, as its
//                    flag; the decision goes to S's flags (G3_CUT, G3_PLUS or
//                    G3_MINUS for live tiles);
//   k_geo3_list      one workgroup: the live tiles in tile order;
//   k_geo3_sweep     one Jacobi sweep over the listed tiles, R -> S or
//                    S -> R (K even, so the result ends in R); the last one
//                    writes R's flags.
#pragma once
#include "surf_common.hpp"
#include "surf_hj.hpp"
#include "surf_step2d.hpp"

namespace surf {

constexpr int G3 = 16;                    // tile edge
constexpr int G3_THREADS = 256;

// live tiles in S's flags: with a cut cell, or all on one side
enum { G3_CUT = Q_TODO, G3_PLUS = Q_TODO + 1, G3_MINUS = Q_TODO + 2 };

struct Geo3Args {
  Grid g;
  int tiles[3];
  int ntiles;
  int per_xcd;  // ceil(ntiles / 8): tiles per XCD band of the classify grid
};

// ---- access within 16-lane rows: lanes 16 r .. 16 r + 15 hold one row of a
// tile.  edge holds, in the row's first and last lane, the value beyond that
// end of the row.
constexpr int DPP_ROW_SL1 = 0x101, DPP_ROW_SR1 = 0x111;
template <int CTRL>
__device__ __forceinline__ float row_shift(float edge, float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double row_shift(double edge, double v) {
  const long long e = __double_as_longlong(edge), b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)(e & 0xffffffffll), (int)(b & 0xffffffffll), CTRL,
                                             0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Bound: one read of the VoF and the waves' latency; 36 us at 256^3 FP32 (a
// third of the tiles live) against 42 with a ghost lookup and a vector address
// for each load and the pin data of every live tile written.
template <typename R, typename O>
__global__ void __launch_bounds__(G3_THREADS) k_geo3_classify(Geo3Args ga, Par<R> p,
                                                              const R* __restrict__ vof,
                                                              R* __restrict__ chiS,
                                                              R* __restrict__ g0,
                                                              const uint8_t* __restrict__ q_in,
                                                              uint8_t* __restrict__ q_out,
                                                              R* __restrict__ chiT,
                                                              uint8_t* __restrict__ qT,
                                                              double* __restrict__ state) {
  __shared__ uint8_t sQ[27];
  __shared__ int sVote[G3_THREADS / 64];
  // consecutive tiles (x neighbours, sharing cache lines) on one XCD
  const int b = blockIdx.x;
  const int t = (b & 7) * ga.per_xcd + (b >> 3);
  if (t >= ga.ntiles) return;
  const Grid& g = ga.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int tid = threadIdx.x;
  const int tx = t % ga.tiles[0], ty = (t / ga.tiles[0]) % ga.tiles[1],
            tz = t / (ga.tiles[0] * ga.tiles[1]);
  const int x0 = tx * G3, y0 = ty * G3, z0 = tz * G3;
  // this thread's cells: x = tid % 16, y = tid / 16, z = 0 .. 15.  The
  // loads go to mapped (always valid) cells and are all issued before any
  // is used; only the cells inside the box take part in the vote.  Columns
  // past the box edge hold a ghost and store nothing.
  const int lx = tid % G3, ly = tid / G3;
  const int gx = x0 + lx, gy = y0 + ly;
  const bool colin = gx < nx && gy < ny;
  const int cx = map_axis_sel(gx, nx, g.bc[0][0], g.bc[0][1]);
  const long long pl = (long long)nx * ny;
  const O row = (O)nx * (O)map_axis_sel(gy, ny, g.bc[1][0], g.bc[1][1]);
  const O co = (row + (O)cx) * (O)sizeof(R);
  const uint8_t qs_old = q_out[t];  // read before thread 0 rewrites it
  const uint8_t qt_old = qT ? qT[t] : (uint8_t)0;
  // the plane z0 + k (scalar); past the box the ghost plane
  const R* const vz = vof + pl * z0;
  const R* const vg = vof + pl * map_axis(nz, nz, g.bc[2][0], g.bc[2][1]);
  auto plane = [&](int k) { return z0 + k < nz ? vz + pl * k : vg; };
  bool one = true, zero = true;
  R f[G3];
#pragma unroll
  for (int k = 0; k < G3; ++k) f[k] = lane_ld<R, O>(plane(k), co);
#pragma unroll
  for (int k = 0; k < G3; ++k) {
    const bool out = !colin | (z0 + k >= nz);
    one = one & (out | (f[k] == R(1)));
    zero = zero & (out | (f[k] == R(0)));
  }
  if (tid < 27) {
    int u[3] = {tx + tid % 3 - 1, ty + (tid / 3) % 3 - 1, tz + tid / 9 - 1};
    bool ok = true;
    for (int d = 0; d < 3; ++d) {
      if (u[d] < 0 || u[d] >= ga.tiles[d]) {
        if (g.bc[d][u[d] < 0 ? 0 : 1] == BC_PERIODIC) u[d] = (u[d] + ga.tiles[d]) % ga.tiles[d];
        else ok = false;
      }
    }
    sQ[tid] = ok ? q_in[u[0] + ga.tiles[0] * (u[1] + ga.tiles[1] * u[2])] : (uint8_t)255;
  }
  const bool w1 = __all(one), w0 = __all(zero);
  if ((tid & 63) == 0) sVote[tid >> 6] = (w1 ? 1 : 0) | (w0 ? 2 : 0);
  __syncthreads();
  int m = 3;
#pragma unroll
  for (int w = 0; w < G3_THREADS / 64; ++w) m &= sVote[w];
  const int want = (m & 1) ? Q_POS : ((m & 2) ? Q_NEG : -1);
  bool quiet = true, nb_quiet = true;
  for (int i = 0; i < 27; ++i) {
    const uint8_t q = sQ[i];
    if (q == 255) continue;
    if ((int)q != want) quiet = false;
    if (q == Q_LIVE) nb_quiet = false;
  }
  if (quiet) {  // R already holds the clamp here; S (and T) get it unless they have it
    const R v = want == Q_POS ? p.chimax : -p.chimax;
    if ((int)qs_old != want) {
#pragma unroll
      for (int k = 0; k < G3; ++k) {
        const int gz = z0 + k;
        if (colin && gz < nz) chiS[(long long)gx + (long long)nx * (gy + (long long)ny * gz)] = v;
      }
    }
    if (qT && (int)qt_old != want) {
#pragma unroll
      for (int k = 0; k < G3; ++k) {
        const int gz = z0 + k;
        if (colin && gz < nz) chiT[(long long)gx + (long long)nx * (gy + (long long)ny * gz)] = v;
      }
    }
    if (tid == 0) {
      q_out[t] = (uint8_t)want;
      if (qT) qT[t] = (uint8_t)want;
    }
    return;
  }
  if (tid == 0) {
    // the VoF changed under a tile whose whole neighbourhood was quiescent
    if (nb_quiet) atomicOr((unsigned*)(state + S_FLAGS), (unsigned)STATUS_GEOM_JUMP);
  }
  // live: pin data of the tile's cells, in two halves of 8 planes; the
  // neighbour rows of each half and the values beyond the tile in x are loaded
  // before any is used, the x neighbours come from the lanes beside it
  const int ex = lx == 0 ? map_axis_sel(x0 - 1, nx, g.bc[0][0], g.bc[0][1])
                         : (lx == G3 - 1 ? map_axis_sel(x0 + G3, nx, g.bc[0][0], g.bc[0][1]) : cx);
  const O eo = (row + (O)ex) * (O)sizeof(R);
  const O mo = ((O)nx * (O)map_axis_sel(gy - 1, ny, g.bc[1][0], g.bc[1][1]) + (O)cx) * (O)sizeof(R);
  const O po = ((O)nx * (O)map_axis_sel(gy + 1, ny, g.bc[1][0], g.bc[1][1]) + (O)cx) * (O)sizeof(R);
  R zlo = lane_ld<R, O>(vof + pl * map_axis(z0 - 1, nz, g.bc[2][0], g.bc[2][1]), co);
  R zhi = lane_ld<R, O>(vof + pl * map_axis(z0 + G3, nz, g.bc[2][0], g.bc[2][1]), co);
  auto x_of = [&](R v) { return (v - R(0.5)) * p.h; };
  zlo = x_of(zlo);
  zhi = x_of(zhi);
#pragma unroll
  for (int k = 0; k < G3; ++k) f[k] = x_of(f[k]);
  bool anycut = false;
  R pin[G3];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    R ne[G3 / 2], nym[G3 / 2], nyp[G3 / 2];
#pragma unroll
    for (int j = 0; j < G3 / 2; ++j) {
      const R* const pz = plane(half * (G3 / 2) + j);
      ne[j] = lane_ld<R, O>(pz, eo);
      nym[j] = lane_ld<R, O>(pz, mo);
      nyp[j] = lane_ld<R, O>(pz, po);
    }
#pragma unroll
    for (int j = 0; j < G3 / 2; ++j) {
      const int k = half * (G3 / 2) + j;
      const R x0v = f[k], xe = x_of(ne[j]);
      const R nb[6] = {row_shift<DPP_ROW_SR1>(xe, x0v), row_shift<DPP_ROW_SL1>(xe, x0v),
                       x_of(nym[j]), x_of(nyp[j]),
                       k > 0 ? f[k - 1] : zlo, k < G3 - 1 ? f[k + 1] : zhi};
      bool cut = false;
      R jump = R(0), grad2 = R(0);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const R xm = nb[2 * d], xp = nb[2 * d + 1];
        cut = cut | (x0v * xm <= R(0)) | (x0v * xp <= R(0));
        jump = fmax(jump, fmax(fabs(xm - x0v), fabs(xp - x0v)));
        const R cd = R(0.5) * (xp - xm);
        grad2 += cd * cd;
      }
      const R Delta = fmax(fmax(rsqrt_<R>(grad2), jump), R(1e-30) * p.h);
      pin[k] = cut ? p.h * x0v / Delta : (x0v > R(0) ? R(INFINITY) : R(-INFINITY));
      anycut = anycut | (cut & colin & (z0 + k < nz));
    }
  }
  // without a cut cell the tile lies on one side, that of any of its cells but
  // those whose fraction is NaN
  const bool wc = __any(anycut), wp = __any(colin & (f[0] > R(0)));
  __syncthreads();  // the first vote has been read
  if ((tid & 63) == 0) sVote[tid >> 6] = (wc ? 1 : 0) | (wp ? 2 : 0);
  __syncthreads();
  int votes = 0;
#pragma unroll
  for (int w = 0; w < G3_THREADS / 64; ++w) votes |= sVote[w];
  const bool cuts = votes & 1;
  if (tid == 0) q_out[t] = (uint8_t)(cuts ? G3_CUT : ((votes & 2) ? G3_PLUS : G3_MINUS));
  if (!cuts) return;  // the code says what every pin datum of the tile is
  R* const gz0 = g0 + pl * z0;
#pragma unroll
  for (int k = 0; k < G3; ++k)
    if (colin & (z0 + k < nz)) lane_st<R, O>(pin[k], gz0 + pl * k, co);
}

// live[0] = count, live[1 + r] = the r-th live tile in tile order
constexpr int G3_LIST_THREADS = 1024;
__global__ void __launch_bounds__(G3_LIST_THREADS) k_geo3_list(const uint8_t* __restrict__ q,
                                                               int ntiles, int* __restrict__ live) {
  __shared__ int sWave[G3_LIST_THREADS / 64];
  __shared__ int sBase;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) sBase = 0;
  __syncthreads();
  for (int base = 0; base < ntiles; base += G3_LIST_THREADS) {
    const int t = base + tid;
    const bool todo = t < ntiles && q[t] >= G3_CUT;
    const unsigned long long mk = __ballot(todo);
    const int below = __popcll(mk & ((1ull << lane) - 1ull));
    if (lane == 0) sWave[wv] = __popcll(mk);
    __syncthreads();
    int off = sBase;
    for (int w = 0; w < wv; ++w) off += sWave[w];
    if (todo) live[1 + off + below] = t;
    __syncthreads();
    if (tid == 0) {
      int tot = 0;
      for (int w = 0; w < G3_LIST_THREADS / 64; ++w) tot += sWave[w];
      sBase += tot;
    }
    __syncthreads();
  }
  if (tid == 0) live[0] = sBase;
}

// One Jacobi sweep (Godunov, pinned cut cells, clamp) over the listed tiles.
// A workgroup takes a tile, each of its four waves G3_SZ = 4 planes of it, and
// lane (x, q) the four rows 4 q .. 4 q + 3 of column x on those planes: 32
// values, one row beyond each end included, 16 values beyond the tile in x
// and, only in a tile with cut cells, 16 pin data, all loaded before any is
// used; the x neighbours come from the lanes beside it.  Loads take a scalar
// plane pointer and a lane offset that no plane changes (O: 32 bits, or 64
// where a plane is larger than 4 GiB), so that they cost no vector
// instruction.  The update is the one of the whole-box sweeps on w = s chi, s
// the sign of the cell's pin datum.  Neighbours come from src everywhere:
// quiescent tiles hold the clamp in every buffer a sweep reads.  Persistent
// grid (a multiple of 8 workgroups).  The last sweep also writes each tile's
// new flag.  Bound: the latency of one round (all waves of the band are in
// flight at once: tile, flag, loads, store) and the traffic, 8 bytes a cell and
// the halo's, which comes from the memory-side cache; 46 vector instructions a
// cell take 6 of the 15 us of a sweep over the 1300 live tiles of a 256^3 box
// (FP32, sphere of radius 77).  Before, with seven loads a cell, 64-bit
// addresses for each and pin data read everywhere: 104 instructions, 21.5 us.
// Two sweeps in one launch, the tile and its halo in LDS, took 44 us for the
// two: three barriers and five code paths in a row leave too few waves to hide
// them.
constexpr int G3_SZ = 4, G3_ROWS = 4;
constexpr int G3_SWEEP_THREADS = 64 * (G3 / G3_SZ), G3_SWEEP_GRID = 2048;
template <typename R, typename O, bool LAST>
__global__ void __launch_bounds__(G3_SWEEP_THREADS) k_geo3_sweep(Geo3Args ga, Par<R> p, R dtau,
                                                                 const R* __restrict__ src,
                                                                 R* __restrict__ dst,
                                                                 const R* __restrict__ g0,
                                                                 const uint8_t* __restrict__ qs,
                                                                 uint8_t* __restrict__ qr,
                                                                 const int* __restrict__ live) {
  __shared__ int sVote[G3_SWEEP_THREADS / 64];
  const Grid& g = ga.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const long long pl = (long long)nx * ny;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lx = lane & 15, lr = (lane >> 4) * G3_ROWS;
  // XCD k (workgroups b with b % 8 == k) takes the k-th eighth of the list,
  // so that neighbouring tiles, which share cache lines, meet in one L2
  const int n = live[0];
  const int per = (n + 7) / 8, xcd = blockIdx.x & 7, slots = gridDim.x >> 3;
  const int lo = xcd * per, hi = min(n, lo + per);
  for (int it = lo + (blockIdx.x >> 3); it < hi; it += slots) {
    const int t = live[1 + it];
    const int x0 = (t % ga.tiles[0]) * G3, y0 = ((t / ga.tiles[0]) % ga.tiles[1]) * G3,
              z0 = (t / (ga.tiles[0] * ga.tiles[1])) * G3 + wv * G3_SZ;  // this wave's first plane
    const int code = qs[t];
    bool allpos = true, allneg = true;
    if (z0 < nz) {
      const int gx = x0 + lx, gy = y0 + lr;
      // columns and rows past the box hold its ghosts and store nothing
      const int cx = map_axis_sel(gx, nx, g.bc[0][0], g.bc[0][1]);
      const int ex = lx == 0 ? map_axis_sel(x0 - 1, nx, g.bc[0][0], g.bc[0][1])
                             : (lx == G3 - 1 ? map_axis_sel(x0 + G3, nx, g.bc[0][0], g.bc[0][1]) : cx);
      O ro[G3_ROWS + 2], eo[G3_ROWS];
#pragma unroll
      for (int r = -1; r <= G3_ROWS; ++r) {
        const O row = (O)nx * (O)map_axis_sel(gy + r, ny, g.bc[1][0], g.bc[1][1]);
        ro[r + 1] = (row + (O)cx) * (O)sizeof(R);
        if (r >= 0 && r < G3_ROWS) eo[r] = (row + (O)ex) * (O)sizeof(R);
      }
      // what g0 holds where the tile has no cut cell
      const R side = code == G3_PLUS ? R(INFINITY) : R(-INFINITY);
      R c[G3_SZ + 2][G3_ROWS + 2], e[G3_SZ][G3_ROWS], gv[G3_SZ][G3_ROWS];
#pragma unroll
      for (int k = -1; k <= G3_SZ; ++k) {
        const long long pz = pl * map_axis(z0 + k, nz, g.bc[2][0], g.bc[2][1]);
        const R* const sp = src + pz;
        const R* const gp = g0 + pz;
        const bool own = k >= 0 && k < G3_SZ;
#pragma unroll
        for (int r = own ? -1 : 0; r < G3_ROWS + (own ? 1 : 0); ++r) {
          c[k + 1][r + 1] = lane_ld<R, O>(sp, ro[r + 1]);
          if (own && r >= 0 && r < G3_ROWS) {
            e[k][r] = lane_ld<R, O>(sp, eo[r]);
            gv[k][r] = code == G3_CUT ? lane_ld<R, O>(gp, ro[r + 1]) : side;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < G3_SZ; ++k) {
        if (z0 + k >= nz) break;  // uniform
        R* const dp = dst + pl * (z0 + k);
#pragma unroll
        for (int r = 0; r < G3_ROWS; ++r) {
          const R v = c[k + 1][r + 1], s = gv[k][r];
          auto fold = [&](R a) { return HjBits<R>::fold(a, s); };
          const R w = fold(v);
          const R G2 = hj_axis<R>(w, fold(row_shift<DPP_ROW_SR1>(e[k][r], v)),
                                  fold(row_shift<DPP_ROW_SL1>(e[k][r], v))) +
                       hj_axis<R>(w, fold(c[k + 1][r]), fold(c[k + 1][r + 2])) +
                       hj_axis<R>(w, fold(c[k][r + 1]), fold(c[k + 2][r + 1]));
          const R nv = fold(hj_finish<R>(p, dtau, w, fabs(s), G2));
          if (gx < nx && gy + r < ny) {
            lane_st<R, O>(nv, dp, ro[r + 1]);
            if (LAST) {
              allpos = allpos && nv == p.chimax;
              allneg = allneg && nv == -p.chimax;
            }
          }
        }
      }
    }
    if (LAST) {
      const bool wp = __all(allpos), wn = __all(allneg);
      if (lane == 0) sVote[wv] = (wp ? 1 : 0) | (wn ? 2 : 0);
      __syncthreads();
      if (threadIdx.x == 0) {
        int m = 3;
        for (int w = 0; w < G3_SWEEP_THREADS / 64; ++w) m &= sVote[w];
        qr[t] = (m & 1) ? Q_POS : ((m & 2) ? Q_NEG : Q_LIVE);
      }
      __syncthreads();
    }
  }
}

}  // namespace surf

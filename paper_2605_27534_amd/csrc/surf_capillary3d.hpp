// surf_capillary3d.hpp -- the interfacial forces for the coupling to a flow
// solver (section 2.4) in 3D: the capillary force sigma kappa delta_s n and
// the Marangoni force delta_m grad_s sigma with delta_m = A_f / V_c, on the
// faces of the velocity grid.  The rules are those of the 2D kernel
// (surf_capillary.hpp), carried to 3D:
//   * a cell is interfacial when 1e-6 < c < 1 - 1e-6;
//   * the Youngs normal m = -grad c from the 3x3x3 stencil (along each axis
//     the difference of the two neighbouring planes, each summed over its
//     3x3 cells with the weights (1, 2, 1) x (1, 2, 1));
//   * kappa by height functions (Cummins, Francois and Kothe 2005): along an
//     axis a, the fluid-1 heights H(p, q) of the nine columns of nine cells
//     through the cell and its neighbours in the other two axes b < c, and
//     kappa = (H_bb (1 + H_c^2) + H_cc (1 + H_b^2) - 2 H_bc H_b H_c)
//             / (1 + H_b^2 + H_c^2)^(3/2)
//     (centred differences; H_bb, H_cc over h, H_bc over 4h).  The axes are
//     tried in the order of m's components, largest first (ties to the
//     higher axis), zero ones skipped; the first whose columns all close
//     (end cells full on the fluid-1 side and empty on the other) gives
//     kappa.  Where none closes the cell takes the mean of the height
//     curvatures of the interfacial cells of its 3x3x3 block (in the order
//     dz, dy, dx from -1 to 1), or where there is none the level set's
//     curvature moved to the interface, kappa / (1 - chi kappa / 2);
//   * delta_m = A_f / h: the plane m.x = alpha leaving the fraction c of the
//     unit cube on its side m.x <= alpha, A_f its area inside the cube.  With
//     the axes reflected so that n = |m| / |m|_1 >= 0 and k the axis of n's
//     largest component, the plane is z_k = (alpha - L)/n_k over the unit
//     square of the other two axes, L = n_i x_i + n_j x_j.  With G(t) the
//     area of {L <= t} in the square (piecewise quadratic in t) and I(t) its
//     integral from 0 (piecewise cubic), the volume below the plane is
//     (I(alpha) - I(alpha - n_k)) / n_k and A_f = (G(alpha) - G(alpha - n_k))
//     |n| / n_k: no division by a small component (n_k >= 1/3, and the
//     pieces of G and I that divide by n_i or n_j are taken only on their
//     own intervals).  alpha by Newton's method on that volume inside a
//     shrinking bracket, bisecting when a step leaves it.
// On a face kappa is the mean over its interfacial cells, delta_m and sigma
// the means of both; grad_s sigma is the face gradient of sigma (compact
// normal difference, the two cells' centred transverse differences averaged)
// minus its part along the same face gradient of chi.  Faces on walls and
// open sides carry no force; on a periodic axis the last face repeats the
// first.  The geometry runs in FP64 in both precisions.
//
// Four launches.  k_iface3_begin clears the tile counter.  k_iface3_scan
// streams: some workgroups zero the face arrays, the others read the fractions
// and list the 8^3 tiles that hold interfacial cells.  k_iface3_cells takes
// the listed tiles, two waves each (a sphere's surface leaves some tens of
// interfacial cells to a tile, one per lane; one wave takes the heights, the
// other the areas), and writes each interfacial
// cell's height curvature (NaN where no axis closes) and delta_m into two
// scratch cell arrays, and nothing for the other cells.  k_iface3_faces takes
// the listed tiles, lists the faces of their interfacial cells (the low ones,
// and a high one when the cell beyond is not interfacial, so that no face is
// computed twice) and computes those, reading the scratch arrays only at
// interfacial cells and filling in the curvature of a cell without heights
// from the first array, which no thread writes.
// At 256^3 FP32 (a sphere of radius 0.3: some 4600 tiles hold 110000
// interfacial cells) the four take 200 us against 440 for six fills and two
// passes over all 16^3 tiles, which read the fractions twice and left most
// lanes of a cut tile's waves idle:
//   scan 93 us, the zero fill and the one read of the fractions (470 MB: 95 us
//     at the rate a large copy reaches), so at its bound;
//   cells 64 us (123 with the fractions read from memory and one wave doing
//     both parts in turn), bound by the instructions of the 81 LDS reads and
//     of Newton's method;
//   faces 38 us (73 with the tile's cells as tasks and branches in every ghost
//     lookup), bound by the latency of its dependent gathers.
#pragma once
#include "surf_capillary.hpp"

namespace surf {

constexpr int IF3_HL = 4;  // height columns reach IF3_HL cells each side

template <typename R>
struct Iface3Args {
  Grid g;
  const R* vof;
  const R* chi;
  const R* sig;
  R* kh;     // height curvature per cell
  R* dm;     // delta_m per cell
  R* fc[3];  // capillary force per face set (or null)
  R* fm[3];  // Marangoni force per face set (or null)
  double h;
  int* list;  // [0] the number of listed tiles, then the tiles
};

__device__ __forceinline__ bool if3_cut(double c) { return c > IFACE_CUT && c < 1.0 - IFACE_CUT; }

// the cell index of (x, y, z) mapped into the box (mirrored or wrapped
// ghosts); IN: the caller's tile is far enough from every side
template <bool IN = false>
__device__ __forceinline__ long long if3_index(const Grid& g, int x, int y, int z) {
  if constexpr (IN) return cell_index(g, x, y, z);
  const int i = map_axis_sel(x, g.n[0], g.bc[0][0], g.bc[0][1]);
  const int j = map_axis_sel(y, g.n[1], g.bc[1][0], g.bc[1][1]);
  const int k = map_axis_sel(z, g.n[2], g.bc[2][0], g.bc[2][1]);
  return cell_index(g, i, j, k);
}

template <bool IN = false, typename R>
__device__ __forceinline__ double if3_at(const R* a, const Grid& g, int x, int y, int z) {
  return (double)a[if3_index<IN>(g, x, y, z)];
}

// ---- PLIC area in the unit cube
// G(t) = area of {a x + b y <= t} in the unit square and I(t) = its integral
// over [0, t], for 0 <= a <= b: with s = a + b, G is t^2 / (2ab) on [0, a],
// (t - a/2) / b on [a, b] and symmetric about (s/2, 1/2) (the square's
// centre), so I(t) = t - s/2 + I(s - t) past s/2.
// The divisors are taken once (Newton's method evaluates each piece some
// dozens of times, and an FP64 division is a dozen instructions); 1/(ab) is
// infinite for a = 0, where its piece is empty.
struct Plic {
  double a, b, s, r2ab, r6ab, rb, r2b, ca;
  __device__ __forceinline__ Plic(double a_, double b_) : a(a_), b(b_), s(a_ + b_) {
    rb = 1.0 / b;
    r2b = 0.5 * rb;
    r2ab = 1.0 / (2.0 * a * b);
    r6ab = r2ab * (1.0 / 3.0);
    ca = a * a * rb * (1.0 / 6.0);
  }
  __device__ __forceinline__ double G(double t) const {
    const bool flip = t > 0.5 * s;
    const double u = flip ? s - t : t;  // up to s/2, so u <= b
    double g = u <= a ? u * u * r2ab : (u - 0.5 * a) * rb;
    g = u <= 0.0 ? 0.0 : g;
    return flip ? 1.0 - g : g;
  }
  __device__ __forceinline__ double I(double t) const {
    const bool flip = t > 0.5 * s;
    const double u = flip ? s - t : t;
    double v = u <= a ? u * u * u * r6ab : ca + (u * u - a * u) * r2b;
    v = u <= 0.0 ? 0.0 : v;
    return flip ? t - 0.5 * s + v : v;
  }
};

__device__ __forceinline__ double plic_area3(double m0, double m1, double m2, double c) {
  if (!if3_cut(c)) return 0.0;
  double n0 = fabs(m0), n1 = fabs(m1), n2 = fabs(m2);
  const double s = n0 + n1 + n2;
  if (!(s > 0.0)) return 0.0;
  const double rs = 1.0 / s;
  n0 *= rs;
  n1 *= rs;
  n2 *= rs;
  const double nk = fmax(fmax(n0, n1), n2), a = fmin(fmin(n0, n1), n2);
  const double b = fmax(fmin(n0, n1), fmin(fmax(n0, n1), n2));  // the median
  const double rk = 1.0 / nk;
  const Plic q(a, b);
  // the plane leaves the same area cutting off 1 - c from the opposite
  // corner: solve for the smaller volume, where V and G carry no cancellation
  if (c > 0.5) c = 1.0 - c;
  // V(alpha) = (I(alpha) - I(alpha - nk)) / nk rises from 0 to 1 on [0, 1]:
  // alpha^3 / (6 a b nk) up to a, (alpha^2 - a alpha + a^2/3) / (2 b nk) up to b,
  // (alpha - (a + b)/2) / nk between a + b and nk.  Newton starts from the
  // inverse of the piece c falls into (the linear one also stands in for the
  // cubic around b), so that a few steps suffice
  const double v1 = q.ca * rk, v2 = (b * b - a * b + a * a * (1.0 / 3.0)) * q.r2b * rk;
  double lo = 0.0, hi = 1.0, al;
  if (c < v1) al = cbrt(6.0 * a * b * nk * c);
  else if (c < v2) al = 0.5 * (a + sqrt(fmax(8.0 * b * nk * c - a * a * (1.0 / 3.0), 0.0)));
  else al = nk * c + 0.5 * (a + b);
  al = fmin(fmax(al, 1e-300), 1.0);
  for (int it = 0; it < 200; ++it) {
    const double f = (q.I(al) - q.I(al - nk)) * rk - c;
    if (f == 0.0) break;
    if (f < 0.0) lo = al;
    else hi = al;
    const double dv = (q.G(al) - q.G(al - nk)) * rk;
    double nx = dv > 0.0 ? al - f / dv : 0.5 * (lo + hi);
    if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
    const double step = fabs(nx - al);
    al = nx;
    if (step <= 1e-15 * al) break;  // rounding: the bracket would only wander
  }
  const double band = q.G(al) - q.G(al - nk);
  return band * sqrt(nk * nk + a * a + b * b) * rk;
}

// ---- the cells pass
// fv(x, y, z): the fraction of cell (x, y, z), ghosts mapped
template <typename FV>
__device__ __forceinline__ void if3_youngs(const FV& fv, int x, int y, int z, double* m) {
  const double w[3] = {1.0, 2.0, 1.0};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int b = d == 0 ? 1 : 0, cc = d == 2 ? 1 : 2;
    double s = 0.0;
#pragma unroll
    for (int p = -1; p <= 1; ++p)
#pragma unroll
      for (int r = -1; r <= 1; ++r) {
        int o[3] = {0, 0, 0};
        o[b] = p;
        o[cc] = r;
        o[d] = 1;
        const double hi = fv(x + o[0], y + o[1], z + o[2]);
        o[d] = -1;
        const double lo = fv(x + o[0], y + o[1], z + o[2]);
        s += w[p + 1] * w[r + 1] * (hi - lo);
      }
    m[d] = -s;
  }
}

// kappa by height functions; false when no axis closes
template <typename FV>
__device__ __forceinline__ bool if3_heights(const FV& fv, double h, int x, int y, int z,
                                            const double* m, double& kappa) {
  // axes by |m| descending, ties to the higher axis (scalars, not an indexed
  // array, which would live in memory)
  const double f0 = fabs(m[0]), f1 = fabs(m[1]), f2 = fabs(m[2]);
  const int first = f2 >= f1 && f2 >= f0 ? 2 : (f1 >= f0 ? 1 : 0);
  const int hi_ = first == 2 ? 1 : 2, lo_ = first == 0 ? 1 : 0;  // the other two
  const double fh = hi_ == 2 ? f2 : f1, fl = lo_ == 0 ? f0 : f1;
  const int second = fh >= fl ? hi_ : lo_, third = fh >= fl ? lo_ : hi_;
  for (int q = 0; q < 3; ++q) {
    const int ax = q == 0 ? first : (q == 1 ? second : third);
    const double ma = ax == 0 ? m[0] : (ax == 1 ? m[1] : m[2]);
    if (ma == 0.0) continue;
    const int b = ax == 0 ? 1 : 0;
    // the offset along axis e of cell l of column (p, r): l along ax, p along
    // b, r along the third axis (no indexed arrays, so that the 81 loads are
    // issued together)
    auto off = [&](int e, int p, int r, int l) { return e == ax ? l : (e == b ? p : r); };
    double H[9];
    bool ok = true;
#pragma unroll
    for (int pr = 0; pr < 9; ++pr) {  // column (p, r) = (pr / 3 - 1, pr % 3 - 1)
      const int p = pr / 3 - 1, r = pr % 3 - 1;
      double col[2 * IF3_HL + 1];  // the column's nine values gathered together
#pragma unroll
      for (int l = -IF3_HL; l <= IF3_HL; ++l)
        col[l + IF3_HL] = fv(x + off(0, p, r, l), y + off(1, p, r, l), z + off(2, p, r, l));
      double sum = 0.0;
#pragma unroll
      for (int l = 0; l <= 2 * IF3_HL; ++l) sum += col[l];
      const double lo = col[0], hi = col[2 * IF3_HL];
      const double full = ma > 0.0 ? lo : hi, empty = ma > 0.0 ? hi : lo;
      if (!(full >= 1.0 - IFACE_CUT && empty <= IFACE_CUT)) ok = false;
      H[pr] = sum;
    }
    if (!ok) continue;
    // H[3 (p + 1) + (r + 1)]
    const double Hb = 0.5 * (H[7] - H[1]);
    const double Hc = 0.5 * (H[5] - H[3]);
    const double Hbb = (H[7] - 2.0 * H[4] + H[1]) / h;
    const double Hcc = (H[5] - 2.0 * H[4] + H[3]) / h;
    const double Hbc = (H[8] - H[6] - H[2] + H[0]) / (4.0 * h);
    const double qq = 1.0 + Hb * Hb + Hc * Hc;
    kappa = (Hbb * (1.0 + Hc * Hc) + Hcc * (1.0 + Hb * Hb) - 2.0 * Hbc * Hb * Hc) / (qq * sqrt(qq));
    return true;
  }
  return false;
}

constexpr int IF3_T = 8;                   // 8^3 tiles
constexpr int IF3_S = IF3_T + 2 * IF3_HL;  // the staged region's edge
constexpr int IF3_SX = 64;                 // cells along x per scanning workgroup (8 tiles)
constexpr int IF3_FILL = 1 << 14;          // values zeroed per filling workgroup
constexpr int IF3_GRID = 1024;             // persistent workgroups over the listed tiles

__global__ void k_iface3_begin(int* list) {
  if (threadIdx.x == 0) list[0] = 0;
}

// The first nfill workgroups zero the face arrays, fill_wgs[d] workgroups for
// each array of the face set d; the others scan 64 x 8 x 8 cells each and
// append their tiles that hold interfacial cells to the list.
template <typename R>
__global__ void __launch_bounds__(256) k_iface3_scan(Iface3Args<R> a, int fill0, int fill1,
                                                     int fill2, int nfill, int regions_x,
                                                     int regions_y) {
  const Grid& g = a.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int t = threadIdx.x;
  int b = blockIdx.x;
  if (b < nfill) {
    const int per[3] = {fill0, fill1, fill2};
    for (int set = 0; set < 2; ++set)
      for (int d = 0; d < 3; ++d) {
        R* f = set ? a.fm[d] : a.fc[d];
        if (!f) continue;
        if (b >= per[d]) {
          b -= per[d];
          continue;
        }
        const long long n = (long long)(nx + (d == 0)) * (ny + (d == 1)) * (nz + (d == 2));
        const long long lo = (long long)b * IF3_FILL, hi = lo + IF3_FILL < n ? lo + IF3_FILL : n;
        constexpr int V = 16 / (int)sizeof(R);
        if ((((size_t)f) & 15) == 0) {
          const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
          for (long long q = lo + (long long)t * V; q + V <= hi; q += 256 * V) *(float4*)(f + q) = z;
          const long long tail = lo + (hi - lo) / V * V;
          if (tail + t < hi) f[tail + t] = R(0);
        } else {
          for (long long q = lo + t; q < hi; q += 256) f[q] = R(0);
        }
        return;
      }
    return;
  }
  b -= nfill;
  __shared__ unsigned sBits[4];
  const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rx = b % regions_x, r = b / regions_x, ry = r % regions_y, rz = r / regions_y;
  const int x = rx * IF3_SX + lane, y0 = ry * IF3_T + 2 * wv, z0 = rz * IF3_T;
  const int xc = x < nx ? x : nx - 1;
  R v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int y = min(y0 + (k & 1), ny - 1), z = min(z0 + (k >> 1), nz - 1);
    v[k] = a.vof[(long long)xc + (long long)nx * (y + (long long)ny * z)];
  }
  // cells past the box repeat its last row or plane, which belongs to the same
  // tile or to one listed anyway; lanes past it vote for nothing
  bool cut = false;
#pragma unroll
  for (int k = 0; k < 16; ++k) cut = cut || if3_cut((double)v[k]);
  const unsigned long long m = __ballot(cut && x < nx);
  unsigned bits = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) bits |= ((m >> (8 * q)) & 0xffull) ? (1u << q) : 0u;
  if (lane == 0) sBits[wv] = bits;
  __syncthreads();
  if (t == 0) {
    unsigned all = sBits[0] | sBits[1] | sBits[2] | sBits[3];
    if (all) {
      int at = 1 + atomicAdd(a.list, __popc(all));
      const int tx = (nx + IF3_T - 1) / IF3_T, ty = (ny + IF3_T - 1) / IF3_T;
      for (; all; all &= all - 1u)
        a.list[at++] = rx * (IF3_SX / IF3_T) + __ffs(all) - 1 + tx * (ry + ty * rz);
    }
  }
}

// the face index of cell (x, y, z) with coordinate d replaced by f
__device__ __forceinline__ long long if3_face_index(const Grid& g, int d, int x, int y, int z,
                                                    int f) {
  return face_index(g, d, d == 0 ? f : x, d == 1 ? f : y, d == 2 ? f : z);
}

template <typename R>
__global__ void __launch_bounds__(128) k_iface3_cells(Iface3Args<R> a) {
  __shared__ unsigned short sList[IF3_T * IF3_T * IF3_T];
  __shared__ float sV[IF3_S][IF3_S][IF3_S];  // FP32 fractions of the tile and its halo
  const Grid& g = a.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tx = (nx + IF3_T - 1) / IF3_T, ty = (ny + IF3_T - 1) / IF3_T;
  const int count = a.list[0];
  for (int i = blockIdx.x; i < count; i += gridDim.x) {
    const int tile = a.list[1 + i];
    const int x0 = (tile % tx) * IF3_T, y0 = (tile / tx % ty) * IF3_T, z0 = tile / (tx * ty) * IF3_T;
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    if constexpr (sizeof(R) == 4) {
      // FP32: the tile and IF3_HL cells around it (mapped) staged in LDS
      __syncthreads();  // the last tile's reads are done
#pragma unroll
      for (int h = 0; h < IF3_S * IF3_S / 128; ++h) {  // a z-column of the region each
        const int q = (int)threadIdx.x + 128 * h, sx = q % IF3_S, sy = q / IF3_S;
        R v[IF3_S];
#pragma unroll
        for (int k = 0; k < IF3_S; ++k)
          v[k] = a.vof[if3_index(g, x0 - IF3_HL + sx, y0 - IF3_HL + sy, z0 - IF3_HL + k)];
#pragma unroll
        for (int k = 0; k < IF3_S; ++k) sV[k][sy][sx] = v[k];
      }
    }
    __syncthreads();
    // the tile's interfacial cells in the order of planes and lanes (both waves
    // write the same list)
    int total = 0;
#pragma unroll
    for (int k = 0; k < IF3_T; ++k) {
      const bool in = x < nx && y < ny && z0 + k < nz;
      double c = 0.0;
      if constexpr (sizeof(R) == 4)
        c = (double)sV[k + IF3_HL][(lane >> 3) + IF3_HL][(lane & 7) + IF3_HL];
      else if (in)
        c = (double)a.vof[cell_index(g, x, y, z0 + k)];
      const bool cut = in && if3_cut(c);
      const unsigned long long m = __ballot(cut);
      if (cut) sList[total + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)((k << 6) | lane);
      total += __popcll(m);
    }
    __syncthreads();
    auto cell = [&](const auto& fv) {
      for (int q = lane; q < total; q += 64) {
        const int e = sList[q];
        const int cx = x0 + (e & 7), cy = y0 + ((e >> 3) & 7), cz = z0 + (e >> 6);
        const long long cl = cell_index(g, cx, cy, cz);
        const double c = (double)fv(cx, cy, cz);
        double m3[3], kap = 0.0;
        if3_youngs(fv, cx, cy, cz, m3);
        if (wv == 0) {  // uniform
          if (!if3_heights(fv, a.h, cx, cy, cz, m3, kap)) kap = (double)NAN;
          a.kh[cl] = (R)kap;
        } else {
          a.dm[cl] = (R)(plic_area3(m3[0], m3[1], m3[2], c) / a.h);
        }
      }
    };
    if constexpr (sizeof(R) == 4)
      cell([&](int X, int Y, int Z) {
        return (double)sV[Z - z0 + IF3_HL][Y - y0 + IF3_HL][X - x0 + IF3_HL];
      });
    else
      cell([&](int X, int Y, int Z) { return if3_at(a.vof, g, X, Y, Z); });
  }
}

// ---- the faces pass
// the level set's curvature at cell (x, y, z), moved to the interface
template <bool IN, typename R>
__device__ __forceinline__ double if3_levelset_kappa(const Iface3Args<R>& a, int x, int y, int z) {
  const double h = a.h;
  auto C = [&](int dx, int dy, int dz) { return if3_at<IN>(a.chi, a.g, x + dx, y + dy, z + dz); };
  const double c0 = C(0, 0, 0);
  const double gx = (C(1, 0, 0) - C(-1, 0, 0)) / (2.0 * h);
  const double gy = (C(0, 1, 0) - C(0, -1, 0)) / (2.0 * h);
  const double gz = (C(0, 0, 1) - C(0, 0, -1)) / (2.0 * h);
  const double hxx = (C(1, 0, 0) - 2.0 * c0 + C(-1, 0, 0)) / (h * h);
  const double hyy = (C(0, 1, 0) - 2.0 * c0 + C(0, -1, 0)) / (h * h);
  const double hzz = (C(0, 0, 1) - 2.0 * c0 + C(0, 0, -1)) / (h * h);
  const double hxy = (C(1, 1, 0) - C(1, -1, 0) - C(-1, 1, 0) + C(-1, -1, 0)) / (4.0 * h * h);
  const double hxz = (C(1, 0, 1) - C(1, 0, -1) - C(-1, 0, 1) + C(-1, 0, -1)) / (4.0 * h * h);
  const double hyz = (C(0, 1, 1) - C(0, 1, -1) - C(0, -1, 1) + C(0, -1, -1)) / (4.0 * h * h);
  const double gm = fmax(sqrt(gx * gx + gy * gy + gz * gz), 1e-6);
  const double num = hxx * (gy * gy + gz * gz) + hyy * (gx * gx + gz * gz) +
                     hzz * (gx * gx + gy * gy) -
                     2.0 * (gx * gy * hxy + gx * gz * hxz + gy * gz * hyz);
  const double kc = num / (gm * gm * gm);
  return kc / (1.0 - c0 * kc / 2.0);
}

// kappa of an interfacial cell (mapped coordinates)
template <bool IN, typename R>
__device__ __forceinline__ double if3_kappa(const Iface3Args<R>& a, int x, int y, int z) {
  const double kh = (double)a.kh[cell_index(a.g, x, y, z)];
  if (!isnan(kh)) return kh;
  // every neighbour's fraction and scratch curvature loaded first (the
  // curvature is used only where the neighbour is interfacial)
  R fv[27], kv[27];
#pragma unroll
  for (int q = 0; q < 27; ++q) {
    const long long i = if3_index<IN>(a.g, x + q % 3 - 1, y + (q / 3) % 3 - 1, z + q / 9 - 1);
    fv[q] = a.vof[i];
    kv[q] = a.kh[i];
  }
  double s = 0.0;
  int cnt = 0;
#pragma unroll
  for (int q = 0; q < 27; ++q) {  // dz, dy, dx from -1 to 1
    if (q == 13 || !if3_cut((double)fv[q])) continue;
    const double v = (double)kv[q];
    if (!isnan(v)) {
      s += v;
      ++cnt;
    }
  }
  return cnt ? s / cnt : if3_levelset_kappa<IN>(a, x, y, z);
}

// the face gradient of a cell field across the face between cells L and R
// (R = L + e_d, both mapped into the box)
template <bool IN, typename R>
__device__ __forceinline__ void if3_face_grad(const Iface3Args<R>& a, const R* f, int d,
                                              const int* L, const int* Rc, double* gr) {
  const double ih = 1.0 / a.h, iq = 0.25 * ih;
  const double nrm =
      (if3_at<IN>(f, a.g, Rc[0], Rc[1], Rc[2]) - if3_at<IN>(f, a.g, L[0], L[1], L[2])) * ih;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    double s = 0.0;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const int* X = side == 0 ? L : Rc;
      const int px = X[0] + (t == 0), py = X[1] + (t == 1), pz = X[2] + (t == 2);
      const int qx = X[0] - (t == 0), qy = X[1] - (t == 1), qz = X[2] - (t == 2);
      s += (if3_at<IN>(f, a.g, px, py, pz) - if3_at<IN>(f, a.g, qx, qy, qz)) * iq;
    }
    gr[t] = t == d ? nrm : s;
  }
}

// the two forces on the face along d between cells L and R
template <bool IN, typename R>
__device__ __forceinline__ void if3_face(const Iface3Args<R>& a, int d, const int* L,
                                         const int* Rc, double& cap, double& ma) {
  const long long iL = cell_index(a.g, L[0], L[1], L[2]), iR = cell_index(a.g, Rc[0], Rc[1], Rc[2]);
  const double cL = (double)a.vof[iL], cR = (double)a.vof[iR];
  const bool cutL = if3_cut(cL), cutR = if3_cut(cR);
  cap = ma = 0.0;
  // every load that needs no decision comes first, the gradients' among them
  double gs[3], gc[3];
  if3_face_grad<IN>(a, a.sig, d, L, Rc, gs);
  if3_face_grad<IN>(a, a.chi, d, L, Rc, gc);
  const double dL = (double)a.dm[iL], dR = (double)a.dm[iR];
  const double kL = cutL ? if3_kappa<IN>(a, L[0], L[1], L[2]) : 0.0;
  const double kR = cutR ? if3_kappa<IN>(a, Rc[0], Rc[1], Rc[2]) : 0.0;
  const double kf = cutL && cutR ? 0.5 * (kL + kR) : (cutL ? kL : (cutR ? kR : 0.0));
  const double sf = 0.5 * ((double)a.sig[iL] + (double)a.sig[iR]);
  cap = -sf * kf * (cR - cL) / a.h;
  const double rn = 1.0 / fmax(sqrt(gc[0] * gc[0] + gc[1] * gc[1] + gc[2] * gc[2]), 1e-6);
  const double n0 = gc[0] * rn, n1 = gc[1] * rn, n2 = gc[2] * rn;
  const double nd = d == 0 ? n0 : (d == 1 ? n1 : n2);
  const double ndot = n0 * gs[0] + n1 * gs[1] + n2 * gs[2];
  const double dmf = 0.5 * ((cutL ? dL : 0.0) + (cutR ? dR : 0.0));
  const double gsd = d == 0 ? gs[0] : (d == 1 ? gs[1] : gs[2]);
  ma = dmf * (gsd - nd * ndot);
}

// The faces of the listed tiles' interfacial cells: the low face of each along
// every axis, and its high face when the cell beyond is not interfacial (that
// cell's low face otherwise); on a periodic axis face n is face 0, written by
// whoever computes face 0.  Faces on other sides keep the zero.
constexpr int IF3_FT = 256;  // threads
template <typename R>
__global__ void __launch_bounds__(IF3_FT) k_iface3_faces(Iface3Args<R> a) {
  __shared__ unsigned short sList[6 * IF3_T * IF3_T * IF3_T];
  __shared__ int sCount;
  const Grid& g = a.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int t = threadIdx.x;
  const int tx = (nx + IF3_T - 1) / IF3_T, ty = (ny + IF3_T - 1) / IF3_T;
  const int count = a.list[0];
  for (int i = blockIdx.x; i < count; i += gridDim.x) {
    const int tile = a.list[1 + i];
    const int x0 = (tile % tx) * IF3_T, y0 = (tile / tx % ty) * IF3_T, z0 = tile / (tx * ty) * IF3_T;
    // a tile's faces read up to two cells beyond it: where those lie in the box
    // no ghost lookup is needed (faces 64 -> 38 us at 256^3, most of it address
    // arithmetic)
    const bool in = x0 >= 2 && y0 >= 2 && z0 >= 2 && x0 + IF3_T + 2 <= nx &&
                    y0 + IF3_T + 2 <= ny && z0 + IF3_T + 2 <= nz;
    __syncthreads();  // the last tile's list is done with
    if (t == 0) sCount = 0;
    __syncthreads();
    constexpr int CPT = IF3_T * IF3_T * IF3_T / IF3_FT;  // cells per thread
    R v[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = t + IF3_FT * k;
      const int x = x0 + (c & 7), y = y0 + ((c >> 3) & 7), z = z0 + (c >> 6);
      v[k] = x < nx && y < ny && z < nz ? a.vof[cell_index(g, x, y, z)] : R(0);
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (!if3_cut((double)v[k])) continue;
      const int c = t + IF3_FT * k;
      const int X[3] = {x0 + (c & 7), y0 + ((c >> 3) & 7), z0 + (c >> 6)};
      unsigned tasks = 0;  // bit d: low face, bit 3 + d: high face
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const bool per = g.bc[d][0] == BC_PERIODIC;
        if (X[d] > 0 || per) tasks |= 1u << d;
        if (X[d] < g.n[d] - 1 || per) {
          const int q = X[d] == g.n[d] - 1 ? 0 : X[d] + 1;
          const R nb = a.vof[cell_index(g, d == 0 ? q : X[0], d == 1 ? q : X[1], d == 2 ? q : X[2])];
          if (!if3_cut((double)nb)) tasks |= 8u << d;
        }
      }
      int at = atomicAdd(&sCount, __popc(tasks));
      for (; tasks; tasks &= tasks - 1u)
        sList[at++] = (unsigned short)(((__ffs(tasks) - 1) << 9) | c);
    }
    __syncthreads();
    const int n = sCount;
    for (int q = t; q < n; q += IF3_FT) {
      const int e = sList[q], c = e & 511, k = e >> 9, d = k % 3;
      const int X[3] = {x0 + (c & 7), y0 + ((c >> 3) & 7), z0 + (c >> 6)};
      const int nd = g.n[d], xd = d == 0 ? X[0] : (d == 1 ? X[1] : X[2]);
      int f = xd + (k >= 3 ? 1 : 0);
      if (f == nd) f = 0;  // periodic
      const int ld = f == 0 ? nd - 1 : f - 1;
      const int Rc[3] = {d == 0 ? f : X[0], d == 1 ? f : X[1], d == 2 ? f : X[2]};
      const int L[3] = {d == 0 ? ld : X[0], d == 1 ? ld : X[1], d == 2 ? ld : X[2]};
      double fc = 0.0, fm = 0.0;
      if (in) if3_face<true>(a, d, L, Rc, fc, fm);
      else if3_face<false>(a, d, L, Rc, fc, fm);
      R* cap = d == 0 ? a.fc[0] : (d == 1 ? a.fc[1] : a.fc[2]);
      R* ma = d == 0 ? a.fm[0] : (d == 1 ? a.fm[1] : a.fm[2]);
      const long long fi = if3_face_index(g, d, X[0], X[1], X[2], f);
      if (cap) cap[fi] = (R)fc;
      if (ma) ma[fi] = (R)fm;
      if (f == 0) {  // only a periodic axis has tasks on face 0
        const long long fn = if3_face_index(g, d, X[0], X[1], X[2], nd);
        if (cap) cap[fn] = (R)fc;
        if (ma) ma[fn] = (R)fm;
      }
    }
  }
}

}  // namespace surf

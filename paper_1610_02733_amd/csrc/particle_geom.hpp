// Device helpers shared by the particle kernels and their adjoints: periodic
// wrap with image counting, the cube of lattice sites around a particle and
// the trilinear weights of its corners (Eq. 5).
#pragma once

#include "lbmd_internal.hpp"

namespace lbmd_impl {
using namespace lbmd_dev;

// Periodic wrap into [0, L) with image counting for any displacement
// (x -= k L, k = floor(x / L)); a value that rounds to exactly L after the
// shift moves to 0 in the next image.
__device__ __forceinline__ void wrap_coord(double& x, int32_t& im, double L) {
  if (x >= 0.0 && x < L) return;
  double k = floor(x / L);
  if (fabs(k) > 1e9) k = copysign(1e9, k);  // keep the image count in range
  x -= k * L;
  im += (int32_t)k;
  if (x >= L) {
    x -= L;
    im += 1;
  } else if (x < 0.0) {
    x += L;
    im -= 1;
  }
}

// Integer cube corner from a coordinate, kept inside [0, n) whatever the
// input (the coupling always addresses valid sites).
__device__ __forceinline__ int cell_of(int c, int n) {
  c %= n;
  return c < 0 ? c + n : c;
}

// Element i of an array of less than 4 GB: one 32-bit offset on a scalar base.
template <typename U>
__device__ __forceinline__ U& el(U* base, uint32_t i) {
  return *reinterpret_cast<U*>(reinterpret_cast<char*>(base) + i * (uint32_t)sizeof(U));
}
template <typename U>
__device__ __forceinline__ const U& el(const U* base, uint32_t i) {
  return *reinterpret_cast<const U*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(U));
}

// v plus the value of another lane of its row of 16, by a DPP control word.
template <int Ctrl>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), Ctrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), Ctrl, 0xF, 0xF, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over groups of L <= 16 neighbouring lanes, on every lane: lanes 1 and 2
// apart by quad permutations, then the mirrored half row and row, which hold
// the other groups' sums.
template <int L>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(L == 2 || L == 4 || L == 8 || L == 16, "groups of a row of 16 lanes");
  v = dpp_add<0xB1>(v);                    // quad_perm [1, 0, 3, 2]
  if (L > 2) v = dpp_add<0x4E>(v);         // quad_perm [2, 3, 0, 1]
  if (L > 4) v = dpp_add<0x141>(v);        // row_half_mirror
  return L > 8 ? dpp_add<0x140>(v) : v;    // row_mirror
}

// Force cell of a position on its replica's cell grid (clamped to the grid).
__device__ __forceinline__ void local_cell_coords(const double X[3], const RepMD& m, int c[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    int q = (int)floor(X[d] * m.inv_edge[d]);
    q = q < 0 ? 0 : (q >= m.nb[d] ? m.nb[d] - 1 : q);
    c[d] = q;
  }
}
__device__ __forceinline__ int local_cell(const double X[3], const RepMD& m) {
  int c[3];
  local_cell_coords(X, m, c);
  return c[0] + m.nb[0] * (c[1] + m.nb[1] * c[2]);
}

// D3Q19 velocities in the library's order (opposite pairs adjacent).
static __device__ const int8_t kVel[19][3] = {
    {0, 0, 0},  {1, 0, 0},  {-1, 0, 0}, {0, 1, 0},  {0, -1, 0}, {0, 0, 1},  {0, 0, -1},
    {1, 1, 0},  {-1, -1, 0}, {1, -1, 0}, {-1, 1, 0}, {1, 0, 1},  {-1, 0, -1}, {1, 0, -1},
    {-1, 0, 1}, {0, 1, 1},  {0, -1, -1}, {0, 1, -1}, {0, -1, 1}};

struct Cube {
  int base[3];
  double s[3];
};

__device__ __forceinline__ void cube_of(const double X[3], const Geom& g, Cube& q) {
  const int n3[3] = {g.nx, g.ny, g.nz};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double fl = floor(X[d]);
    q.s[d] = X[d] - fl;
    q.base[d] = cell_of((int)fl, n3[d]);
  }
}

// Site (replica-local) and trilinear weight (Eq. 5) of corner k of the cube.
__device__ __forceinline__ void corner_of(const Cube& q, const Geom& g, int k, int& cx, int& cy,
                                          int& cz, int& site, double& w) {
  cx = q.base[0] + (k & 1);
  cy = q.base[1] + ((k >> 1) & 1);
  cz = q.base[2] + ((k >> 2) & 1);
  cx = cx == g.nx ? 0 : cx;
  cy = cy == g.ny ? 0 : cy;
  cz = cz == g.nz ? 0 : cz;
  site = cx + g.nx * (cy + g.ny * cz);
  w = ((k & 1) ? q.s[0] : 1.0 - q.s[0]) * ((k & 2) ? q.s[1] : 1.0 - q.s[1]) *
      ((k & 4) ? q.s[2] : 1.0 - q.s[2]);
}

// Particle noise amplitude for the stencil weights' squared sum S: the
// random force balances the dissipation of the explicit MD step (Eq. 4, 6).
// The step damps the relative velocity w of the particle and the fluid at its
// stencil (the fluid takes -dP there at once: an effective mass rho0 / S) as
// w <- (1 - a) w + (1/m + S/rho0) dP_rand, a = gamma tau (1/m + S/rho0),
// whose equilibrium variance is kT (1/m + S/rho0) when <dP_rand^2> =
// 2 gamma kT tau (1 - a/2): F_rand = sqrt(2 gamma kT / tau) sqrt(1 - a/2) xi.
// Zero for a >= 2 (beyond the explicit step's stability bound).
// (bal0, bal1: the two constants of the balance 1 - a/2, linear in S.)
__device__ __forceinline__ double noise_balance(const RepMD& m, double S) {
  return m.bal0 - m.bal1 * S;
}
__device__ __forceinline__ double noise_amplitude(const RepMD& m, double S) {
  const double bal = noise_balance(m, S);
  return bal > 0.0 ? m.amp * sqrt(bal) : 0.0;
}

// Kernels that give a particle one lane per corner of its cube (8 | kBlock,
// so the lanes of a particle are always active together).
constexpr int kCornerLanes = 8;

// ---------------------------------------------------------------------------
// Interpolation / spreading stencils (Eq. 5 and Eq. 7 use the same one).
// A particle's stencil is described by a Cube: the lowest site index per
// axis (wrapped) and the offset s of the particle from a reference site.
//   ST = 0, trilinear: the 8 corners of the cube with lower corner floor(X),
//     s = X - floor(X).
//   ST = 1, three-point kernel per axis (Roma, Peskin and Berger 1999; the
//     higher-order scheme the paper mentions, Sec. 4): the 3 sites nearest
//     along each axis, c - 1, c, c + 1 with c = floor(X + 1/2), s = X - c;
//     the axis weight of a site at distance r from the particle is
//       (1 + sqrt(1 - 3 r^2)) / 3                for |r| <= 1/2,
//       (5 - 3|r| - sqrt(1 - 3 (1 - |r|)^2)) / 6 for 1/2 <= |r| <= 3/2;
//     27 sites.
// Along an axis both square roots of the three-point kernel are one and the
// same: with the site at r = s - o, |r| = 1 -+ s for o = +-1, so 1 - |r| = +-s
// and the weights are (2 -+ 3s - q)/6 and (1 + q)/3, q = sqrt(1 - 3 s^2).
// kLanes is the lane count per particle of the kernels that gather a
// stencil's sites one lane each (refill, re-gather after a cube change):
// 8, or 32 with lanes 27-31 idle.
// ---------------------------------------------------------------------------
template <int ST>
struct Stencil;

template <>
struct Stencil<0> {
  static constexpr int kSites = 8, kLanes = 8;
  static constexpr int W = 2;  // sites per axis
  __device__ static __forceinline__ int base_of(double x, int, double& s) {
    const double fl = floor(x);
    s = x - fl;
    return (int)fl;
  }
  __device__ static __forceinline__ void axis_weights(double s, double w[W]) {
    w[0] = 1.0 - s;
    w[1] = s;
  }
  __device__ static __forceinline__ void offsets(int k, int& ox, int& oy, int& oz) {
    ox = k & 1;
    oy = (k >> 1) & 1;
    oz = (k >> 2) & 1;
  }
};

template <>
struct Stencil<1> {
  static constexpr int kSites = 27, kLanes = 32;
  static constexpr int W = 3;
  __device__ static __forceinline__ int base_of(double x, int n, double& s) {
    const double c = floor(x + 0.5);
    s = x - c;
    const int b = (int)c - 1;
    return b < 0 ? b + n : b;  // (c = 0: the site below is the last one)
  }
  __device__ static __forceinline__ void axis_weights(double s, double w[W]) {
    const double q = sqrt(1.0 - 3.0 * s * s), a = 2.0 - q;
    w[0] = (a - 3.0 * s) * (1.0 / 6.0);
    w[1] = (1.0 + q) * (1.0 / 3.0);
    w[2] = (a + 3.0 * s) * (1.0 / 6.0);
  }
  __device__ static __forceinline__ void offsets(int k, int& ox, int& oy, int& oz) {
    ox = k % 3;
    oy = (k / 3) % 3;
    oz = k / 9;
  }
};

template <int ST>
__device__ __forceinline__ void locate(const double X[3], const Geom& g, Cube& q) {
  const int n3[3] = {g.nx, g.ny, g.nz};
  bool in = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    q.base[d] = Stencil<ST>::base_of(X[d], n3[d], q.s[d]);
    in = in & ((unsigned)q.base[d] < (unsigned)n3[d]);
  }
  if (!in) {  // (positions are wrapped: only at bound ones outside the box)
#pragma unroll
    for (int d = 0; d < 3; ++d) q.base[d] = cell_of(q.base[d], n3[d]);
  }
}

// Site k of the stencil with lowest site q.base.
template <int ST>
__device__ __forceinline__ void stencil_site(const Cube& q, const Geom& g, int k, int& cx, int& cy,
                                             int& cz, int& site) {
  int ox, oy, oz;
  Stencil<ST>::offsets(k, ox, oy, oz);
  cx = q.base[0] + ox;
  cy = q.base[1] + oy;
  cz = q.base[2] + oz;
  cx = cx >= g.nx ? cx - g.nx : cx;
  cy = cy >= g.ny ? cy - g.ny : cy;
  cz = cz >= g.nz ? cz - g.nz : cz;
  site = cx + g.nx * (cy + g.ny * cz);
}

// The sites of a stencil axis by axis: off[d][o] is what site o of axis d
// adds to the site index (x, nx y, nx ny z) and w[d][o] its weight, so that a
// site costs two additions and two products.
template <int ST>
struct StencilAxes {
  int off[3][Stencil<ST>::W];
  double w[3][Stencil<ST>::W];
};

template <int ST>
__device__ __forceinline__ void stencil_axes(const Cube& q, const Geom& g, StencilAxes<ST>& ax) {
  constexpr int W = Stencil<ST>::W;
  const int n3[3] = {g.nx, g.ny, g.nz}, unit[3] = {1, g.nx, g.A};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    Stencil<ST>::axis_weights(q.s[d], ax.w[d]);
    const int first = q.base[d] * unit[d], period = n3[d] * unit[d];
#pragma unroll
    for (int o = 0; o < W; ++o) {
      const int f = first + o * unit[d];
      ax.off[d][o] = f >= period ? f - period : f;
    }
  }
}

// v[o] by selects (an index known only at run time would put v in scratch).
template <typename U>
__device__ __forceinline__ U pick(const U (&v)[2], int o) {
  const U a = v[0], b = v[1];
  return o == 0 ? a : b;
}
template <typename U>
__device__ __forceinline__ U pick(const U (&v)[3], int o) {
  const U a = v[0], b = v[1], c = v[2];
  const U ab = o == 0 ? a : b;
  return o == 2 ? c : ab;
}

// The weights' squared sum over the stencil: the product of the axes' sums.
template <int ST>
__device__ __forceinline__ double squared_weights(const StencilAxes<ST>& ax) {
  double S = 1.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double a = 0.0;
#pragma unroll
    for (int o = 0; o < Stencil<ST>::W; ++o) a += ax.w[d][o] * ax.w[d][o];
    S *= a;
  }
  return S;
}

}  // namespace lbmd_impl

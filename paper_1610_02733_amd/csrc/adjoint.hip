// Reverse-mode kernels of one coupled cycle (n MD steps, then one LB step;
// Eq. 3-8): the adjoint of the collide-and-stream step and of one MD step of
// the particle coupling.  The forward state they linearise about comes from
// a recorded re-run of the cycle (populations read by the cycle, the transfer
// field and mark words of its LB step, per-MD-step particle records); the
// noise is regenerated from the same counters as in the forward kernels.
//
// Adjoint variables, all with respect to the forward quantity of the same
// name at the matching point of the sweep:
//   pbar  stored (post-collision) populations, pull storage, two buffers
//   jbar  transfer field J (force density of the LB step)
//   abar  (j, rho) of the post-stream state at a site, as read by the MD steps
//   xbar, vbar  particle position and velocity
// Single system (one replica); conservative force constant in time.
#include <algorithm>

#include "particle_geom.hpp"

namespace lbmd_impl {
using namespace lbmd_dev;

template <typename T>
struct AdjLBArgs {
  const T* __restrict__ src;                  // populations the cycle read (slot)
  const T* __restrict__ pin;                  // adjoint of the cycle's output
  T* __restrict__ pout;                       // adjoint of the cycle's input
  const Vec4<T>* jrec;                        // J at the LB step (marked sites)
  const unsigned long long* __restrict__ mrec;
  Vec4<T>* jbar;
  Vec4<T>* clear;                             // set to zero where J was recorded, or null (may be jrec)
  const RepLB<T>* __restrict__ rep;
  double* __restrict__ nuacc;                 // [gridDim][4]
  long long t_lb;
};

// ---------------------------------------------------------------------------
// Adjoint of the fused collide-and-stream step, one thread per site r.
//
// Forward: out_i(r) = C_i(f(r), F(r)) with f_i(r) = src_i(r - c_i) (pull) and
// F = g + J(r).  Reverse: the collision adjoint at r turns out-bar(r) into
// f-bar(r) and F-bar(r); the transpose of the pull sends f-bar_i(r) back to
// the stored entry it came from, src-bar_i(r - c_i), written exactly once
// per entry (a push, no atomics).  F-bar is kept where a transfer was
// recorded (the sites the MD steps touched).  The derivatives of the result
// with respect to the relaxation factors are summed per block.
// ---------------------------------------------------------------------------
//
// Off: the type of the entries' offsets, 32 bits where the lattice allows (half
// the registers); the pull and the push each compute theirs.  FP32 is held to
// 4 waves per SIMD, which is one round of the chip at 64^3.  The pushed runs
// are shifted, so two wavefronts share their end lines: plain stores, which
// the caches merge (16.1 us at 64^3 streamed, 17.7 plain, but then 12.4 against
// 9.1 us for the fold that follows; ten cycles of 160 x 144 x 128 with two MD
// steps 5.80 against 5.42 ms).
template <typename T, typename Off>
__device__ __forceinline__ void adjoint_offsets(const Geom& g, int x, int y, int z, Off off[19]) {
  const int xm = x == 0 ? g.nx - 1 : x - 1, xp = x == g.nx - 1 ? 0 : x + 1;
  const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y == g.ny - 1 ? 0 : y + 1;
  const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z == g.nz - 1 ? 0 : z + 1;
  const int X[3] = {xm, x, xp}, Y[3] = {ym * g.nx, y * g.nx, yp * g.nx};
  const Off A = (Off)g.A, Z[3] = {(Off)zm * 19 * A, (Off)z * 19 * A, (Off)zp * 19 * A};
  // (the source is r - c: the lower neighbour for c = +1)
  constexpr int8_t c[19][3] = {{0, 0, 0},   {1, 0, 0},   {-1, 0, 0}, {0, 1, 0},  {0, -1, 0},
                               {0, 0, 1},   {0, 0, -1},  {1, 1, 0},  {-1, -1, 0}, {1, -1, 0},
                               {-1, 1, 0},  {1, 0, 1},   {-1, 0, -1}, {1, 0, -1}, {-1, 0, 1},
                               {0, 1, 1},   {0, -1, -1}, {0, 1, -1}, {0, -1, 1}};
#pragma unroll
  for (int i = 0; i < 19; ++i)
    off[i] = Z[1 - c[i][2]] + (Off)(Y[1 - c[i][1]] + X[1 - c[i][0]]);
}

template <typename T, typename Off>
__global__ __launch_bounds__(kBlock, sizeof(T) == 4 ? 4 : 1) void k_collide_stream_adjoint(
    AdjLBArgs<T> a) {
  const RepLB<T>& q = a.rep[0];
  const uint32_t step_lo = (uint32_t)((unsigned long long)a.t_lb & 0xFFFFFFFFull);
  const uint32_t step_hi = (uint32_t)((unsigned long long)a.t_lb >> 32);
  double acc[3] = {0.0, 0.0, 0.0};
  for (int r = blockIdx.x * kBlock + threadIdx.x; r < q.g.S; r += gridDim.x * kBlock) {
    int x, y, z;
    site_coords(q.g, r, x, y, z);
    Off off[19];
    adjoint_offsets<T>(q.g, x, y, z, off);
    const Off own = (Off)z * 19 * (Off)q.g.A + (Off)(y * q.g.nx + x);
    T d[19], dbo[19], dbi[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      d[i] = __builtin_nontemporal_load(a.src + (size_t)i * q.g.A + off[i]);
      dbo[i] = __builtin_nontemporal_load(a.pin + (size_t)i * q.g.A + own);
    }
    const bool marked = (a.mrec[r >> 6] >> (r & 63)) & 1ull;
    T Fx = q.k.g[0], Fy = q.k.g[1], Fz = q.k.g[2];
    if (marked) {
      const Vec4<T> jv = a.jrec[r];
      Fx += jv.x;
      Fy += jv.y;
      Fz += jv.z;
    }
    uint32_t hw[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (q.k.noise) {
      const Words4 o0 = philox10(Words4{(uint32_t)r, step_lo, q.tag0, step_hi}, q.key0, q.key1);
      const Words4 o1 = philox10(Words4{(uint32_t)r, step_lo, q.tag1, step_hi}, q.key0, q.key1);
      hw[0] = o0.w0; hw[1] = o0.w1; hw[2] = o0.w2; hw[3] = o0.w3;
      hw[4] = o1.w0; hw[5] = o1.w1; hw[6] = o1.w2; hw[7] = o1.w3;
    }
    T Fbx, Fby, Fbz, gb[3];
    collide_deviation_adjoint<T>(d, Fx, Fy, Fz, hw, q.k, dbo, dbi, Fbx, Fby, Fbz, gb);
    asm("" : "+v"(x), "+v"(y), "+v"(z));  // (the offsets are not kept through the collision)
    adjoint_offsets<T>(q.g, x, y, z, off);
#pragma unroll
    for (int i = 0; i < 19; ++i) a.pout[(size_t)i * q.g.A + off[i]] = dbi[i];
    if (marked) {
      a.jbar[r] = Vec4<T>{Fbx, Fby, Fbz, T(0)};
      if (a.clear) a.clear[r] = Vec4<T>{T(0), T(0), T(0), T(0)};
    }
    acc[0] += (double)gb[0];
    acc[1] += (double)gb[1];
    acc[2] += (double)gb[2];
  }
  // block sums, accumulated into this block's own slot (deterministic)
  __shared__ double sh[kBlock / 64][3];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double s = acc[k];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) sh[wv][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += sh[w][threadIdx.x];
    a.nuacc[(size_t)blockIdx.x * 4 + threadIdx.x] += s;
  }
}

// Fold of the MD steps' reads into the population adjoint: the MD steps of a
// cycle read rho(r) = sum_i f_i(r) and j(r) = sum_i c_i f_i(r) of the
// post-stream state, so f-bar_i(r) gains rho-bar(r) + c_i . j-bar(r), which
// the pull transpose sends to src-bar_i(r - c_i).  Only marked sites can
// carry a read; abar is cleared for the next cycle.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_adjoint_fold(const RepLB<T>* __restrict__ rep,
                                                         const unsigned long long* __restrict__ mrec,
                                                         Vec4<T>* __restrict__ abar,
                                                         T* __restrict__ pout) {
  const Geom& g = rep[0].g;
  for (int r = blockIdx.x * kBlock + threadIdx.x; r < g.S; r += gridDim.x * kBlock) {
    if (!((mrec[r >> 6] >> (r & 63)) & 1ull)) continue;
    const Vec4<T> ab = abar[r];
    abar[r] = Vec4<T>{T(0), T(0), T(0), T(0)};
    int x, y, z;
    size_t off[19];
    site_coords(g, r, x, y, z);
    pull_offsets(g, x, y, z, off);
#pragma unroll
    for (int i = 0; i < 19; ++i)
      pout[off[i]] +=
          ab.w + (T)kVel[i][0] * ab.x + (T)kVel[i][1] * ab.y + (T)kVel[i][2] * ab.z;
  }
}

struct AdjMDArgs {
  double* rec;                     // [kAdjRec][N] record of this MD step
  const double* prev;              // that of the step reversed before it in this cycle, or null
  bool more;                       // another MD step of this cycle follows
  const double* __restrict__ fcons;
  double* __restrict__ xbar;
  double* __restrict__ vbar;
  double* __restrict__ pacc;       // [4][N]
  const RepMD* __restrict__ md;
  const int32_t* __restrict__ pid;  // particle identity of each slot (noise counter)
  int64_t N;
  long long t_md;                  // MD step being reversed
};

// Adds of four components a lane, `site` per lane (negative: none).  The four
// lanes of a quad take each other's sites in turn, a component each, so that
// one instruction adds 16 whole sites (one request each) instead of one
// component of 64.
template <int Ctrl>
__device__ __forceinline__ int quad_of(int v) {
  return __builtin_amdgcn_update_dpp(0, v, Ctrl, 0xF, 0xF, false);
}
template <int Ctrl>
__device__ __forceinline__ float quad_of(float v) {
  return __int_as_float(quad_of<Ctrl>(__float_as_int(v)));
}
template <int Ctrl>
__device__ __forceinline__ double quad_of(double v) {
  return __hiloint2double(quad_of<Ctrl>(__double2hiint(v)), quad_of<Ctrl>(__double2loint(v)));
}
template <typename T, int From>
__device__ __forceinline__ void quad_add(Vec4<T>* field, int site, const T add[4], int comps) {
  constexpr int ctrl = From * 0x55;  // quad_perm: every lane takes lane From
  const int c = threadIdx.x & 3;
  const T v0 = quad_of<ctrl>(add[0]), v1 = quad_of<ctrl>(add[1]), v2 = quad_of<ctrl>(add[2]),
          v3 = quad_of<ctrl>(add[3]);
  const int at = quad_of<ctrl>(site);
  const T v = c < 2 ? (c == 0 ? v0 : v1) : (c == 2 ? v2 : v3);
  if (at >= 0 && c < comps) atomicAdd((T*)(field + at) + c, v);
}
template <typename T>
__device__ __forceinline__ void quad_adds(Vec4<T>* field, int site, const double add[4],
                                          int comps) {
  const T t[4] = {(T)add[0], (T)add[1], (T)add[2], (T)add[3]};
  quad_add<T, 0>(field, site, t, comps);
  quad_add<T, 1>(field, site, t, comps);
  quad_add<T, 2>(field, site, t, comps);
  quad_add<T, 3>(field, site, t, comps);
}

// ---------------------------------------------------------------------------
// Adjoint of one MD step (Eq. 4-8 with velocity Verlet), eight lanes per
// particle, one per corner k of its cube.  Forward, with s = X - floor(X)
// and w_k(s) the corner weights:
//   u   = sum_k w_k U_k / rho_k          (U_k = j_k [+ J_k in variant 2])
//   Fc  = -gamma (V - u) + A xi,         A = c sqrt(gamma B), c = sqrt(2 kT / tau),
//                                         B = 1 - gamma tau (1/m + S/rho0) / 2,
//                                         S = sum_k w_k^2 (noise_amplitude)
//   J_k += -w_k tau Fc                   (transfer, Eq. 7-8)
//   V1  = V + h (f + Fc);  X' = X + tau V1;  V' = V1 + h (f + Fc)
// Reverse: from X'-bar, V'-bar and J-bar at the corners, the adjoints of X,
// V, Fc, u, gamma and f.  Sums over corners are DPP sums over the lanes; the weights are piecewise linear in X, so their slopes enter
// through both the interpolation and the transfer.  The reads of the
// interpolation then have adjoints
//   j-bar_k += w_k / rho_k u-bar,   rho-bar_k -= w_k / rho_k^2 (U_k . u-bar),
// which are added right here, four components to a request (quad_adds).
// In variant 2 the read includes J, so J-bar gains the same j-bar once every
// particle of the step has read it: J-bar is the LB step's plus what abar has
// gained.  The steps alternate between two such sums: a step reads `gin` and
// adds to `abar`, which misses what the step before gave (to `gin`), so that
// is added again along with it, one add where the corner is the same; the last
// step's is the cycle's abar.  (rho-bar, which no step reads, goes to the
// cycle's, `rbar`, at once.)  What a lane gave is kept in its own entries of
// the step's record, which nothing reads any more: the U rows, and the site in
// the 1/rho row.
// Bound by a chain of loads and some 200 dependent FP64 instructions, then by
// the requests of the adds, so four components go to a request (quad_adds).
// One wavefront a block, as 1000 particles fill only half the CUs.  1000
// particles in variant 2, us a step: 9.1 with J-bar itself kept up to date, by
// a kernel of its own; 6.5 so (a sweep of 50 cycles of five steps 3430 and
// 2900).  J-bar in two whole buffers took 6.2, but rounded more: the derivatives
// with respect to V were off by 5.8e-8, against 5.5e-8 before and 5.3e-8 so.
// ---------------------------------------------------------------------------
constexpr int kAdjCouple = 64;  // one wavefront
template <typename T, bool Reread>
__global__ __launch_bounds__(kAdjCouple) void k_couple_adjoint(AdjMDArgs a,
                                                               const Vec4<T>* __restrict__ jbar,
                                                               const Vec4<T>* __restrict__ gin,
                                                               Vec4<T>* abar, Vec4<T>* rbar) {
  const RepMD m = scalar_copy(a.md);
  const int64_t N = a.N;
  const unsigned long long t_md = (unsigned long long)a.t_md;
  const uint32_t step_lo = (uint32_t)(t_md & 0xFFFFFFFFull), step_hi = (uint32_t)(t_md >> 32);
  for (int64_t t = (int64_t)blockIdx.x * kAdjCouple + threadIdx.x; t < N * kCornerLanes;
       t += (int64_t)gridDim.x * kAdjCouple) {
    const int64_t p = t / kCornerLanes;
    const int k = (int)(t & (kCornerLanes - 1));
    double* r = a.rec;
    double X[3], V[3], gave[4] = {0.0, 0.0, 0.0, 0.0};
    int gave_at = -1;
    if (Reread && a.prev) {
#pragma unroll
      for (int d = 0; d < 3; ++d) gave[d] = a.prev[(6 + 3 * k + d) * N + p];
      gave_at = (int)a.prev[(30 + k) * N + p];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      X[d] = r[d * N + p];
      V[d] = r[(3 + d) * N + p];
    }
    if (!isfinite(X[0])) {  // skipped by the forward step (all 8 lanes)
      if (Reread) {
        quad_adds(abar, gave_at, gave, 3);
        if (a.more) r[(30 + k) * N + p] = -1.0;
      }
      continue;
    }
    Cube q;
    locate<0>(X, m.g, q);
    int cx, cy, cz, site;
    stencil_site<0>(q, m.g, k, cx, cy, cz, site);
    // w_k and d w_k / d s_e
    const double a0 = (k & 1) ? q.s[0] : 1.0 - q.s[0], e0 = (k & 1) ? 1.0 : -1.0;
    const double a1 = (k & 2) ? q.s[1] : 1.0 - q.s[1], e1 = (k & 2) ? 1.0 : -1.0;
    const double a2 = (k & 4) ? q.s[2] : 1.0 - q.s[2], e2 = (k & 4) ? 1.0 : -1.0;
    const double w = a0 * a1 * a2;
    const double dw[3] = {e0 * a1 * a2, a0 * e1 * a2, a0 * a1 * e2};
    const double ir = r[(30 + k) * N + p];
    const double U[3] = {r[(6 + 3 * k) * N + p], r[(7 + 3 * k) * N + p], r[(8 + 3 * k) * N + p]};
    const Vec4<T> jb = jbar[site];
    double jbv[3] = {(double)jb.x, (double)jb.y, (double)jb.z};
    if (Reread && a.prev) {
      const Vec4<T> gn = gin[site];
      jbv[0] += (double)gn.x;
      jbv[1] += (double)gn.y;
      jbv[2] += (double)gn.z;
    }
    double u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = group_sum<8>(w * ir * U[d]);
    // noise amplitude A(gamma, S) and its derivatives (zero where A = 0:
    // gamma = 0, or the balance factor clamped)
    // (S is the product of the axes' squared sums (1 - s)^2 + s^2)
    double sq[3], ds[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      sq[d] = (1.0 - q.s[d]) * (1.0 - q.s[d]) + q.s[d] * q.s[d];
      ds[d] = 4.0 * q.s[d] - 2.0;
    }
    const double S = sq[0] * sq[1] * sq[2];
    const double dS[3] = {ds[0] * sq[1] * sq[2], sq[0] * ds[1] * sq[2], sq[0] * sq[1] * ds[2]};
    const double A = m.noise ? noise_amplitude(m, S) : 0.0;
    const double c2 = m.gamma > 0.0 ? m.amp * m.amp / m.gamma : 0.0;  // 2 kT / tau
    const double a_damp = 2.0 * (1.0 - noise_balance(m, S));
    const double dA_dg = A > 0.0 ? c2 * (1.0 - a_damp) / (2.0 * A) : 0.0;
    const double dA_dS = A > 0.0 ? -c2 * m.gamma * m.gamma * m.tau / (4.0 * m.rho0 * A) : 0.0;
    double xi[3] = {0.0, 0.0, 0.0};
    if (m.noise) {
      const Words4 o = philox10(Words4{(uint32_t)a.pid[p], step_lo, m.tag, step_hi}, m.key0,
                                m.key1);
      const uint32_t ws[3] = {o.w0, o.w1, o.w2};
#pragma unroll
      for (int d = 0; d < 3; ++d)
        xi[d] = 3.4641016151377546 * (((double)(ws[d] >> 8) + 0.5) * 5.9604644775390625e-08 - 0.5);
    }
    double Fc[3], xb[3], vb[3], Fcb[3], fb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      Fc[d] = -m.gamma * (V[d] - u[d]) + A * xi[d];
      xb[d] = a.xbar[d * N + p];
      vb[d] = a.vbar[d * N + p];
      const double v1b = vb[d] + m.tau * xb[d];
      Fcb[d] = m.h * (vb[d] + v1b);
      fb[d] = Fcb[d];  // f enters exactly where Fc does
      vb[d] = v1b;
    }
    // transfer J_k += -w_k tau Fc
    const double gk = jbv[0] * Fc[0] + jbv[1] * Fc[1] + jbv[2] * Fc[2];
    double xs[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      Fcb[d] += group_sum<8>(-m.tau * w * jbv[d]);
      xs[d] = -m.tau * gk * dw[d];
    }
    // friction and noise
    double ub[3], gbar = 0.0, nb = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      vb[d] -= m.gamma * Fcb[d];
      ub[d] = m.gamma * Fcb[d];
      gbar += Fcb[d] * (-(V[d] - u[d]) + dA_dg * xi[d]);
      nb += Fcb[d] * xi[d];
    }
    // interpolation weights (through u, the transfer and the noise amplitude)
    const double uk = ir * (U[0] * ub[0] + U[1] * ub[1] + U[2] * ub[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) xs[d] = group_sum<8>(xs[d] + uk * dw[d]) + nb * dA_dS * dS[d];
    if (k == 0) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        a.xbar[d * N + p] = xb[d] + xs[d];
        a.vbar[d * N + p] = vb[d];
        a.pacc[(1 + d) * N + p] += fb[d];
      }
      a.pacc[p] += gbar;
    }
    double give[4];
#pragma unroll
    for (int d = 0; d < 3; ++d) give[d] = w * ir * ub[d];
    give[3] = -w * ir * uk;
    if (Reread) {
      if (a.more) {
#pragma unroll
        for (int d = 0; d < 3; ++d) r[(6 + 3 * k + d) * N + p] = give[d];
        r[(30 + k) * N + p] = (double)site;
      }
      const int other = gave_at == site ? -1 : gave_at;
      if (__any(other >= 0)) quad_adds(abar, other, gave, 3);
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (gave_at == site) give[d] += gave[d];
    }
    if (Reread && abar != rbar) {
      quad_adds(abar, site, give, 3);
      atomicAdd((T*)(rbar + site) + 3, (T)give[3]);
    } else {
      quad_adds(abar, site, give, 4);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Whether the MD steps of a cycle change the J-bar that the next one reads,
// and the sum they then use in turn with abar: the J recorded for the cycle's
// LB step, which only the reverse LB step at the same site reads.
static bool rereads(const Context* c) {
  return c->p[0].variant == 2 && c->plan.Ntot > 0 && c->plan.n_sub > 1;
}
template <typename T>
static Vec4<T>* other_abar(const Context* c) {
  const AdjState& s = c->adj;
  return (Vec4<T>*)(s.ws + s.lay.jrec) + (size_t)s.slot * (size_t)c->plan.Stot;
}

template <typename T>
static hipError_t lb_adjoint_t(Context* c) {
  const AdjState& s = c->adj;
  const AdjLayout& L = s.lay;
  const size_t S = (size_t)c->plan.Stot;
  const int j = s.slot;
  AdjLBArgs<T> a;
  a.src = (const T*)s.src[j];
  a.pin = (const T*)(s.ws + L.pbar[s.pbar_cur]);
  a.pout = (T*)(s.ws + L.pbar[1 - s.pbar_cur]);
  a.jrec = (const Vec4<T>*)(s.ws + L.jrec) + (size_t)j * S;
  a.mrec = (const unsigned long long*)(s.ws + L.mrec) + (size_t)j * (S / 64);
  a.jbar = (Vec4<T>*)(s.ws + L.jbar);
  a.clear = rereads(c) ? other_abar<T>(c) : nullptr;
  a.rep = (const RepLB<T>*)at(c, c->plan.lay.rep_lb);
  a.nuacc = (double*)(s.ws + L.nuacc);
  a.t_lb = (long long)s.t_lb[j];
  const int blocks = (int)std::min<int64_t>(kAdjBlocks, (c->plan.Stot + kBlock - 1) / kBlock);
  if (19ull * (unsigned long long)c->plan.Stot < (1ull << 32))
    hipLaunchKernelGGL((k_collide_stream_adjoint<T, uint32_t>), dim3(blocks), dim3(kBlock), 0,
                       c->stream, a);
  else
    hipLaunchKernelGGL((k_collide_stream_adjoint<T, size_t>), dim3(blocks), dim3(kBlock), 0,
                       c->stream, a);
  return hipGetLastError();
}

hipError_t launch_collide_stream_adjoint(Context* c) {
  return c->plan.prec == 32 ? lb_adjoint_t<float>(c) : lb_adjoint_t<double>(c);
}

static AdjMDArgs md_adjoint_args(Context* c) {
  const AdjState& s = c->adj;
  const AdjLayout& L = s.lay;
  const size_t N = (size_t)c->plan.Ntot;
  AdjMDArgs a;
  a.rec = (double*)(s.ws + L.prec) +
          ((size_t)s.slot * c->plan.n_sub + (size_t)s.sub) * kAdjRec * N;
  a.prev = s.sub + 1 < c->plan.n_sub ? a.rec + kAdjRec * N : nullptr;
  a.more = s.sub > 0;
  a.fcons = (const double*)at(c, c->plan.lay.fcons);
  a.xbar = (double*)(s.ws + L.xbar);
  a.vbar = (double*)(s.ws + L.vbar);
  a.pacc = (double*)(s.ws + L.pacc);
  a.md = (const RepMD*)at(c, c->plan.lay.rep_md);
  a.pid = (const int32_t*)at(c, c->plan.lay.pid);
  a.N = c->plan.Ntot;
  a.t_md = (long long)(s.t_md[s.slot] + s.sub);
  return a;
}

template <typename T>
static hipError_t couple_adjoint_t(Context* c) {
  const AdjMDArgs a = md_adjoint_args(c);
  Vec4<T>* jbar = (Vec4<T>*)(c->adj.ws + c->adj.lay.jbar);
  Vec4<T>* abar = (Vec4<T>*)(c->adj.ws + c->adj.lay.abar);
  const dim3 grid((unsigned)((a.N * kCornerLanes + kAdjCouple - 1) / kAdjCouple));
  if (rereads(c)) {
    // (step 0, the last one reversed, adds to abar)
    Vec4<T>* sum[2] = {abar, other_abar<T>(c)};
    const int out = c->adj.sub & 1;
    hipLaunchKernelGGL((k_couple_adjoint<T, true>), grid, dim3(kAdjCouple), 0, c->stream, a,
                       (const Vec4<T>*)jbar, (const Vec4<T>*)sum[1 - out], sum[out], abar);
  } else {
    hipLaunchKernelGGL((k_couple_adjoint<T, false>), grid, dim3(kAdjCouple), 0, c->stream, a,
                       (const Vec4<T>*)jbar, (const Vec4<T>*)nullptr, abar, abar);
  }
  return hipGetLastError();
}

hipError_t launch_couple_adjoint(Context* c) {
  if (c->plan.Ntot == 0) return hipSuccess;
  return c->plan.prec == 32 ? couple_adjoint_t<float>(c) : couple_adjoint_t<double>(c);
}

template <typename T>
static hipError_t fold_t(Context* c) {
  const AdjState& s = c->adj;
  const size_t S = (size_t)c->plan.Stot;
  const int blocks = (int)std::min<int64_t>(kAdjBlocks, (c->plan.Stot + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_adjoint_fold<T>, dim3(blocks), dim3(kBlock), 0, c->stream,
                     (const RepLB<T>*)at(c, c->plan.lay.rep_lb),
                     (const unsigned long long*)(s.ws + s.lay.mrec) + (size_t)s.slot * (S / 64),
                     (Vec4<T>*)(s.ws + s.lay.abar), (T*)(s.ws + s.lay.pbar[1 - s.pbar_cur]));
  return hipGetLastError();
}

// After the MD steps of a cycle were reversed: their reads into the adjoint
// of the cycle's input populations.
hipError_t launch_adjoint_fold(Context* c) {
  if (c->plan.Ntot == 0) return hipSuccess;
  return c->plan.prec == 32 ? fold_t<float>(c) : fold_t<double>(c);
}

// Sums of the swept cycles' derivatives: out[0..3] over the particles (pacc),
// out[4], out[5] over the blocks of the reverse LB step (nuacc, bulk and
// shear).  One block, a fixed order.
__global__ __launch_bounds__(kBlock) void k_adjoint_totals(const double* __restrict__ pacc,
                                                           int64_t N,
                                                           const double* __restrict__ nuacc,
                                                           double* __restrict__ out) {
  __shared__ double sh[kBlock / 64][6];
  double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t p = threadIdx.x; p < N; p += kBlock)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += pacc[k * N + p];
  for (int b = threadIdx.x; b < kAdjBlocks; b += kBlock)
#pragma unroll
    for (int k = 0; k < 2; ++k) acc[4 + k] += nuacc[(size_t)b * 4 + k];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double s = acc[k];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) sh[wv][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += sh[w][threadIdx.x];
    out[threadIdx.x] = s;
  }
}

hipError_t launch_adjoint_totals(Context* c, double* d_out) {
  const AdjState& s = c->adj;
  hipLaunchKernelGGL(k_adjoint_totals, dim3(1), dim3(kBlock), 0, c->stream,
                     (const double*)(s.ws + s.lay.pacc), c->plan.Ntot,
                     (const double*)(s.ws + s.lay.nuacc), d_out);
  return hipGetLastError();
}

}  // namespace lbmd_impl

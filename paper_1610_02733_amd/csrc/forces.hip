// Conservative particle forces F_cons (Eq. 4; they act on the particles
// only) for the bead-spring workloads, with pairs found through a cell list:
// model 2, harmonic bonds between consecutive beads of a chain and the purely
// repulsive WCA potential between all pairs; model 3, the paper's
// Kremer-Grest polymer (Sec. 3), FENE bonds and the Lennard-Jones potential
// cut at 2^(7/6) sigma.  Also the binning of particles into cells.
#include <algorithm>
#include <cmath>

#include "couple_state.hpp"

namespace lbmd_impl {

// ---------------------------------------------------------------------------
// Binning: cell = floor(x / edge) per axis on each replica's grid of
// nb[0] x nb[1] x nb[2] cells of edge L / nb >= the pair cut-off (local_cell);
// cells of all replicas share one global index space (offset cell_off).
// Non-finite particles go to no cell (they are left out of the force loop).
// A cell holds up to cell_cap particles in slots of its own, taken in the
// order of an atomic count; the rest go to an overflow list (cell_insert).
// After an MD step the coupling kernel bins the particles (it knows the new
// positions first) and clears the other half of the counts (bin_parity), so
// the force kernel follows it directly.  At bound positions both halves are
// cleared and k_bin_count bins the particles.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_bin_clear(int32_t* __restrict__ count, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) count[i] = 0;
}

__global__ __launch_bounds__(kBlock) void k_bin_count(const double* __restrict__ x, int64_t N,
                                                      const RepMD* __restrict__ md,
                                                      const int32_t* __restrict__ part_rep,
                                                      const Clock* __restrict__ clock,
                                                      int pos_step, int64_t ncells, int cap,
                                                      int32_t* __restrict__ count,
                                                      int32_t* __restrict__ bin,
                                                      int32_t* __restrict__ slot,
                                                      int32_t* __restrict__ ovf) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= N) return;
  const int par = bin_parity(clock, pos_step);
  const double X[3] = {x[p], x[N + p], x[2 * N + p]};
  const RepMD& m = md[part_rep[p]];
  if (m.force_model < 2 || !(isfinite(X[0]) && isfinite(X[1]) && isfinite(X[2]))) {
    bin[p] = -1;
    return;
  }
  const int c = m.cell_off + local_cell(X, m);
  bin[p] = (int32_t)(par * ncells + c);
  cell_insert(count + par * ncells, slot, ovf, count + 2 * ncells + par, cap, c, (int)p);
}

// ---------------------------------------------------------------------------
// Forces: each particle sums its own bond and WCA forces (no atomics; every
// pair is evaluated from both sides, so the pair forces cancel up to
// rounding), with minimum-image separations.  Force models 0 and 1 give zero
// or the constant f_ext.
//
// 32 lanes per particle.  Lanes 0-26 take one neighbouring cell each (offsets
// -1, 0, +1 per axis; on an axis with fewer than 3 cells, cells 0, 1, 2 of
// that axis instead, so every distinct cell is taken once) and put its
// particles into the particle's list in LDS, at the place a prefix sum of the
// cell counts gives; then all 32 lanes share the list evenly.  (One lane per
// cell throughout ran as long as its fullest cell, about twice the even
// share, with the cut-off test and force of two slots per cell evaluated
// whether filled or not.)  Lanes 27 and 28 add the bond to the chain's
// previous and next bead, lane 29 scans the overflow list (empty unless a
// cell holds more than cell_cap particles; a pair closer than the cut-off
// lies in neighbouring cells, so the list's particles need only the distance
// test); the lane sums are a butterfly reduction.  The half of the counts
// comes with the particle's own count entry.  Lanes 0-2 store the force and,
// after an MD step, apply the second half-kick of velocity Verlet (new
// conservative force + the coupling force held over the step).  After an MD
// step the launch also carries the step's after-step work in extra blocks:
// this kernel runs after every particle of the step has read the transfer
// field.
//
// Dense systems are bound by FP64 issue, dilute ones by the chain of three
// dependent loads (cell entry and position, counts and slots, positions).
// The pair arithmetic therefore has no division but one reciprocal: minimum
// images by 1/L, 1/r^2 by two Newton steps on the hardware's estimate.
// Measured with the five divisions and one lane per cell it had before: 13.8,
// 19.0 and 29.4 us per MD step for 128^3 WCA chains, Kremer-Grest chains and
// 5 x 2560 Kremer-Grest beads at 0.32 per site; now 9.5, 10.2 and 16.5 us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double min_image(double d, double L, double inv_L) {
  return d - L * rint(d * inv_L);
}

// 1/a for finite normal a > 0: two Newton steps square the estimate's error
// twice, to the last bit or two.
__device__ __forceinline__ double reciprocal(double a) {
  double y = __builtin_amdgcn_rcp(a);
  y = fma(y, fma(-a, y, 1.0), y);
  return fma(y, fma(-a, y, 1.0), y);
}

constexpr int kForceLanes = 32;

// Sum over the 32 lanes of a particle, on every lane.
__device__ __forceinline__ double lane32_sum(double v) {
  v = group_sum<16>(v);
  return v + __shfl_xor(v, 16, kForceLanes);
}

template <typename T>
struct ForceArgs {
  const double* __restrict__ x;
  double* __restrict__ v;
  double* __restrict__ f;
  const double* __restrict__ fc_held;
  const RepMD* __restrict__ md;
  const int32_t* __restrict__ part_rep;
  const int32_t* __restrict__ count;  // [2][ncells] + [2] overflow lengths (CoupleArgs::bin_count)
  const int32_t* __restrict__ bin;    // [N] count entries (CoupleArgs::bin)
  const int32_t* __restrict__ slot;
  const int32_t* __restrict__ ovf;
  int64_t N;
  int64_t ncells;
  int cap;
};

// Pair force of the WCA or cut Lennard-Jones potential on the particle at X
// from one at Y, added to F when `use` and Y lies within the cut-off.
__device__ __forceinline__ void add_pair_force(const double X[3], const double Y[3], bool use,
                                               const RepMD& m, double F[3]) {
  double dx[3], r2 = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    dx[d] = min_image(X[d] - Y[d], m.L[d], m.inv_L[d]);
    r2 += dx[d] * dx[d];
  }
  if (!use || !(r2 < m.pair_rc2)) return;
  const double ir2 = r2 > 0.0 ? reciprocal(r2) : __builtin_inf();
  const double sr2 = m.pair_sig2 * ir2;
  const double sr6 = sr2 * sr2 * sr2;
  const double fm = m.pair_eps24 * (2.0 * sr6 * sr6 - sr6) * ir2;
#pragma unroll
  for (int d = 0; d < 3; ++d) F[d] += fm * dx[d];
}

// Candidates of one particle at a time in LDS (a longer list is taken in
// windows): 8 KB a block, which leaves the waves per CU to the registers.
constexpr int kPairList = 256;

// Forces of the particle the 32 lanes share: replica constants m, its slot p.
template <typename T, bool Kick>
__device__ __forceinline__ void force_particle(const ForceArgs<T>& a, const RepMD& m, int64_t p,
                                               int lane, int32_t* __restrict__ list) {
  const int64_t N = a.N;
  double F[3] = {0.0, 0.0, 0.0};
  // (the cells are written for every particle when a replica has them)
  const bool pairs = m.force_model >= 2;
  const int g = pairs ? a.bin[p] : -1;
  const double X[3] = {a.x[p], a.x[N + p], a.x[2 * N + p]};
  // lanes 0-2 finish the particle, one component each
  const bool kick = Kick && lane < 3 && m.split_kick;
  double vv = 0.0, fh = 0.0;
  if (kick) {
    vv = a.v[lane * N + p];
    fh = a.fc_held[lane * N + p];
  }
  // the bond partner of lanes 27 and 28
  bool bond = false;
  int64_t qb = p;
  if (pairs && (lane == 27 || lane == 28)) {
    int pos;
    div_fast((int)(p - m.part_off), m.chain_len, m.inv_chain, pos);
    bond = lane == 27 ? pos > 0 : pos < m.chain_len - 1;
    if (bond) qb = lane == 27 ? p - 1 : p + 1;
  }
  const double B[3] = {a.x[qb], a.x[N + qb], a.x[2 * N + qb]};
  if (g >= 0) {
    const int half = g >= a.ncells ? 1 : 0;
    // this lane's cell: its count and first eight slots at once (cap >= 8; a
    // slot past the count holds a stale index and is not used)
    int n = 0;
    const int32_t* __restrict__ sl = a.slot;
    int4 s0 = make_int4(0, 0, 0, 0), s1 = s0;
    {
      const int o[3] = {lane % 3, (lane / 3) % 3, lane / 9};
      int cc[3], q3[3];
      local_cell_coords(X, m, cc);
      bool use = lane < 27;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (m.nb[d] < 3) {
          q3[d] = o[d];
          use = use && o[d] < m.nb[d];
        } else {
          const int qq = cc[d] + o[d] - 1;
          q3[d] = qq < 0 ? qq + m.nb[d] : (qq >= m.nb[d] ? qq - m.nb[d] : qq);
        }
      }
      if (use) {
        const int cell = m.cell_off + q3[0] + m.nb[0] * (q3[1] + m.nb[1] * q3[2]);
        sl += (int64_t)cell * a.cap;
        n = min(a.count[half * a.ncells + cell], a.cap);
        s0 = reinterpret_cast<const int4*>(sl)[0];
        s1 = reinterpret_cast<const int4*>(sl)[1];
      }
    }
    const int no = lane == 29 ? a.count[2 * a.ncells + half] : 0;
    if (bond) {
      // (while the counts and slots are on their way) harmonic (model 2) or
      // FENE (model 3, no finite force at r >= R0)
      double dx[3], r2 = 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        dx[d] = min_image(X[d] - B[d], m.L[d], m.inv_L[d]);
        r2 += dx[d] * dx[d];
      }
      double fm;
      if (m.force_model == 2) {
        const double r = sqrt(r2);
        fm = -m.k_bond * (r - m.r0_bond) / r;
      } else {
        const double x2 = r2 / (m.r0_bond * m.r0_bond);
        fm = x2 < 1.0 ? -m.k_bond / (1.0 - x2) : __builtin_nan("");
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) F[d] += fm * dx[d];
    }
    // place of the cell's particles in the list, and the list's length: the
    // sum over the lanes up to this one, inside a row of 16 by DPP shifts,
    // the lower row's total into the upper one by a row broadcast
    int pre = n;
    pre += __builtin_amdgcn_update_dpp(0, pre, 0x111, 0xF, 0xF, true);
    pre += __builtin_amdgcn_update_dpp(0, pre, 0x112, 0xF, 0xF, true);
    pre += __builtin_amdgcn_update_dpp(0, pre, 0x114, 0xF, 0xF, true);
    pre += __builtin_amdgcn_update_dpp(0, pre, 0x118, 0xF, 0xF, true);
    pre += __builtin_amdgcn_update_dpp(0, pre, 0x142, 0xA, 0xF, false);
    const int total = __shfl(pre, kForceLanes - 1, kForceLanes);
    pre -= n;
    for (int w = 0; w < total; w += kPairList) {
      const int at = pre - w;
      const int s8[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j < n && (unsigned)(at + j) < (unsigned)kPairList) list[at + j] = s8[j];
      for (int j = 8; j < n; ++j)
        if ((unsigned)(at + j) < (unsigned)kPairList) list[at + j] = sl[j];
      // the 32 lanes belong to one wavefront, whose LDS accesses are in order
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int len = min(total - w, kPairList);
      for (int i = lane; i < len; i += kForceLanes) {
        const int q = list[i];
        const double Y[3] = {a.x[q], a.x[N + q], a.x[2 * N + q]};
        add_pair_force(X, Y, q != p, m, F);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (no > 0) {
      const int rep = a.part_rep[p];
      for (int e = 0; e < no; ++e) {
        const int q = a.ovf[e];
        const double Y[3] = {a.x[q], a.x[N + q], a.x[2 * N + q]};
        add_pair_force(X, Y, q != p && a.part_rep[q] == rep, m, F);
      }
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) F[d] = lane32_sum(F[d]);
  if (m.force_model == 1) {
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d] = m.f_ext[d];
  }
  if (lane < 3) {
    const double f = lane == 0 ? F[0] : (lane == 1 ? F[1] : F[2]);
    a.f[lane * N + p] = f;
    if (kick && isfinite(vv)) a.v[lane * N + p] = vv + m.h * (f + fh);
  }
}

// Blocks [0, nfb) compute the forces; with AfterST >= 0 (after an MD step,
// not recording) blocks [nfb, nfb + 2 nseg) do the after-step work
// of the MD step just taken (after_step_item), which is independent of the
// forces: it touches J, the claims and the corner cache only.
// The replica's constants are in scalar registers: read once with a single
// replica (One); otherwise per wavefront, whose two particles nearly always
// belong to one replica (and are taken one after the other where they do
// not).
// Held to 7 waves per SIMD: the latency of a particle's loads is hidden by the
// other waves, and 1e4 particles with their after-step blocks then run in one
// round (5 waves as the registers would have it: 883 against 821 us for three
// cycles of the 128^3 polymer, 1549 against 1430 us for five of 5 x 2560
// dense beads; 6: 821 and 1520; 8, with spills: 843 and 1515).
template <typename T, bool Kick, int AfterST, bool One>
__global__ __launch_bounds__(kBlock, 7) void k_forces(ForceArgs<T> a, CoupleArgs<T> ca, int64_t nseg,
                                                   int per, int L, int64_t nfb) {
  if constexpr (AfterST >= 0) {
    if (blockIdx.x >= nfb) {
      after_step_item<T, AfterST, false, false>(ca, (int64_t)blockIdx.x - nfb, nseg, per, L);
      return;
    }
  }
  __shared__ int32_t lists[kBlock / kForceLanes][kPairList];
  const int64_t N = a.N;
  RepMD m1;
  if constexpr (One) m1 = scalar_copy(a.md);
  const int lane = threadIdx.x & (kForceLanes - 1);
  int32_t* list = lists[threadIdx.x / kForceLanes];
  // lanes come in whole particles (32 | kBlock), as the shuffles require
  for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < N * kForceLanes;
       t += nfb * kBlock) {
    const int64_t p = t / kForceLanes;
    if constexpr (One) {
      force_particle<T, Kick>(a, m1, p, lane, list);
    } else {
      const int rep = a.part_rep[p];
      // (a loop on the wavefront's own mask, so that the body stays inside it)
      for (unsigned long long todo = __ballot(1); todo != 0;) {
        const bool mine = rep == __builtin_amdgcn_readlane(rep, __ffsll(todo) - 1);
        if (mine) {
          // (read again from the lanes taken: the compiler would put `rep`, a
          // vector register, in place of a value known to equal it)
          const RepMD mr = scalar_copy(a.md + __builtin_amdgcn_readfirstlane(rep));
          force_particle<T, Kick>(a, mr, p, lane, list);
        }
        todo &= ~__ballot(mine);
      }
    }
  }
}

// Force cells per axis: edge just above the pair cut-off (2^(1/6) sigma for
// WCA, 2^(7/6) sigma for the Kremer-Grest model), so the 27 neighbouring
// cells hold every interacting pair.  Larger cells (about one
// particle per cell on average) were measured slower on chains: a chain's
// beads then crowd a few cells and the per-lane cell loops serialise.
int cells_per_axis(const lbmd_params* p, int d) {
  const double rc = std::pow(2.0, p->force_model == 3 ? 7.0 / 6.0 : 1.0 / 6.0) * p->wca_sigma;
  const int L[3] = {p->nx, p->ny, p->nz};
  const int q = (int)std::floor((double)L[d] / rc);
  return q < 1 ? 1 : q;
}

int64_t force_cells(const lbmd_params* p) {
  if (p->force_model < 2) return 0;
  int64_t n = 1;
  for (int d = 0; d < 3; ++d) n *= cells_per_axis(p, d);
  return n;
}

// Particle slots per force cell.  A WCA cell (edge ~1.12 sigma, ~1.4
// sigma^3) holds about one bead even at melt density; a Kremer-Grest cell
// (edge ~2.24 sigma, ~11 sigma^3) holds about ten there.  Particles past the
// capacity are still found, through the overflow list, at a cost per pair.
int force_cell_capacity(const lbmd_params* p) {
  if (p->force_model < 2) return 0;
  return p->force_model == 3 ? 32 : 8;
}

template <typename T>
static ForceArgs<T> force_args(Context* c) {
  const Layout& L = c->plan.lay;
  ForceArgs<T> a;
  a.x = (const double*)c->x;
  a.v = (double*)c->v;
  a.f = (double*)at(c, L.fcons);
  a.fc_held = (const double*)at(c, L.fc_held);
  a.md = (const RepMD*)at(c, L.rep_md);
  a.part_rep = (const int32_t*)at(c, L.part_rep);
  a.count = (const int32_t*)at(c, L.bin_count);
  a.bin = (const int32_t*)at(c, L.bin_of);
  a.slot = (const int32_t*)at(c, L.bin_slot);
  a.ovf = (const int32_t*)at(c, L.bin_ovf);
  a.N = c->plan.Ntot;
  a.ncells = c->plan.Ctot;
  a.cap = c->plan.cell_cap;
  return a;
}

// Bin the particles of bead-spring replicas (models 2, 3) at the current
// positions, those of MD step clock->t_md + pos_step, from scratch: both
// halves of the counts are cleared first (a fill kernel, so the sequence
// may be captured in a graph).
static hipError_t launch_binning(Context* c, int pos_step) {
  const int64_t N = c->plan.Ntot, C = c->plan.Ctot;
  const Layout& L = c->plan.lay;
  int32_t* count = (int32_t*)at(c, L.bin_count);
  const int64_t nc = 2 * C + 2;
  hipLaunchKernelGGL(k_bin_clear, dim3((unsigned)((nc + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                     c->stream, count, nc);
  hipLaunchKernelGGL(k_bin_count, dim3((unsigned)((N + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                     c->stream, (const double*)c->x, N, (const RepMD*)at(c, L.rep_md),
                     (const int32_t*)at(c, L.part_rep), (const Clock*)clock_of(c, c->clk), pos_step,
                     C, c->plan.cell_cap, count, (int32_t*)at(c, L.bin_of),
                     (int32_t*)at(c, L.bin_slot), (int32_t*)at(c, L.bin_ovf));
  return hipGetLastError();
}

template <typename T, bool Kick, int AfterST>
static hipError_t forces_t(Context* c, int substep = 0) {
  const ForceArgs<T> a = force_args<T>(c);
  const int64_t nfb = (a.N * kForceLanes + kBlock - 1) / kBlock;
  CoupleArgs<T> ca{};
  int64_t nseg = 0;
  int per = 0, L = 0;
  if (AfterST >= 0) {
    constexpr int ST = AfterST >= 0 ? AfterST : 0;
    ca = couple_args<T>(c, substep);
    // the coupling kernel's lanes per particle (tuned or default)
    L = c->tune.couple_lanes > 0 ? c->tune.couple_lanes : default_lanes<ST>(a.N);
    per = (Stencil<ST>::kSites + L - 1) / L;
    nseg = (a.N * L + kBlock - 1) / kBlock;
  }
  const dim3 grid((unsigned)(nfb + 2 * nseg));
  if (c->plan.R == 1)
    hipLaunchKernelGGL((k_forces<T, Kick, AfterST, true>), grid, dim3(kBlock), 0, c->stream, a,
                       ca, nseg, per, L, nfb);
  else
    hipLaunchKernelGGL((k_forces<T, Kick, AfterST, false>), grid, dim3(kBlock), 0, c->stream, a,
                       ca, nseg, per, L, nfb);
  return hipGetLastError();
}

// Conservative forces at the current positions (all force models).
hipError_t launch_forces(Context* c) {
  if (c->plan.Ntot == 0) return hipSuccess;
  hipError_t e;
  if (c->plan.any_forces2 && (e = launch_binning(c, c->subs)) != hipSuccess) return e;
  return c->plan.prec == 32 ? forces_t<float, false, -1>(c) : forces_t<double, false, -1>(c);
}

// Forces at the bound positions; the corner cache is stale from here on.
hipError_t launch_init_forces(Context* c) {
  hipError_t e = launch_forces(c);
  if (e != hipSuccess) return e;
  return invalidate_corner_cache(c);
}

// After an MD step of replicas with position-dependent forces: forces at
// the new positions (binned by the coupling kernel, or here while
// recording), the second half-kick and the step's after-step work in the
// same launch (so the coupling step launches no after-step kernel of its
// own).
template <typename T>
static hipError_t forces_and_kick_t(Context* c, int substep) {
  if (c->rec_part) return forces_t<T, true, -1>(c, substep);
  return c->p[0].stencil == 1 ? forces_t<T, true, 1>(c, substep)
                              : forces_t<T, true, 0>(c, substep);
}

hipError_t launch_forces_and_kick(Context* c, int substep) {
  if (c->plan.Ntot == 0) return hipSuccess;
  if (c->rec_part) {
    const hipError_t e = launch_binning(c, substep + 1);
    if (e != hipSuccess) return e;
  }
  return c->plan.prec == 32 ? forces_and_kick_t<float>(c, substep)
                            : forces_and_kick_t<double>(c, substep);
}

}  // namespace lbmd_impl

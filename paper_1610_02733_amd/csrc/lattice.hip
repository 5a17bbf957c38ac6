// Lattice kernels: the fused pull collide-and-stream step (Eq. 3 with the
// MRT collision, fluid noise and Guo forcing of Sec. 2-3), the FP64 moment
// reductions (Eq. 1-2) and population / transfer copies.  All kernels cover
// every replica of a context in one launch.
#include <algorithm>
#include <mutex>

#include "forcing.hpp"
#include "lbmd_internal.hpp"

namespace lbmd_impl {
using namespace lbmd_dev;

// Replica of a 256-site work item: binary search over the item offsets
// (uniform across the block).
__device__ __forceinline__ int replica_of_item(const int32_t* __restrict__ item_off, int R,
                                               int item) {
  int lo = 0, hi = R;  // item_off[lo] <= item < item_off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (item_off[mid] <= item)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// ---------------------------------------------------------------------------
// Fused collide-and-stream, one thread per site, pull scheme.
//
// The source buffer holds post-collision deviations at the site that produced
// them; the thread at site r gathers population i from r - c_i (the
// post-stream state), adds the pending momentum transfer J(r) as the force
// density of this LB step, collides and writes its 19 results at r in the
// other buffer (coalesced).  J is only read where the site's bit in `mark` is
// set (the coupling sets it when it transfers momentum there), and is cleared
// with it (the shared-site flag in w too), so the untouched bulk of
// the lattice costs no transfer traffic.
// In variant 3 (VarC) the interval's transfer already belongs to the state:
// the collision adds it as the momentum and stress increments of the paper's
// variant C and relaxes with the body force alone.  A work item is 256
// consecutive sites of one replica; replica offsets are multiples of 64, so
// one wavefront owns exactly one 64-bit mark word.  Persistent grid: blocks
// stride over the items.
//
// Row path (replicas with nx = 64, 128 or 256: a wavefront is 64 sites of
// one x row and an item holds whole rows).  Every thread loads the 19
// entries at its own x in the rows that the y and z shifts select, so each
// wavefront load is an aligned, contiguous 64-value run; the +-x shift of the
// ten populations with c_x != 0 is then done in registers: a DPP rotation by
// one lane inside the wavefront, and for the two end lanes of a wavefront the
// value of the neighbouring wavefront of the same row (periodic) through LDS.
// Gathering the shifted entries straight from memory instead makes each
// wavefront touch a partial cache line on either side, which a neighbouring
// wavefront fetches again (measured 1.06x the algorithmic traffic).
// ---------------------------------------------------------------------------
template <typename T>
struct StreamArgs {
  T* pop[2];
  Vec4<T>* __restrict__ J;
  unsigned long long* __restrict__ mark;
  const RepLB<T>* __restrict__ rep;
  const int32_t* __restrict__ item_off;
  const Clock* __restrict__ clock;
  Clock* __restrict__ next;  // the step's advanced clock goes here (null: nowhere)
  int md_steps;              // MD steps of the interval the step ends
  Vec4<T>* __restrict__ jrec;                 // recording: J consumed at marked sites
  unsigned long long* __restrict__ mrec;      // recording: mark words
  int R, nitems;
  int reverse;  // items in reverse order every other step (keep_stores)
  int varc;  // variant 3: J belongs to the fluid state (fields read j + J)
};

// Values of the x neighbours inside a wavefront: lane l receives v of lane
// l - 1 (from_left; lane 0 receives lane 63) or of lane l + 1 (from_right;
// lane 63 receives lane 0).  DPP wave_ror:1 / wave_rol:1.
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x13C, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x134, 0xF, 0xF, false));
}
__device__ __forceinline__ double from_left(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x13C, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x13C, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_right(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x134, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x134, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// End-lane values of each wavefront for the row path, double-buffered by the
// parity of the block's row-path items (one barrier per such item, so a
// wavefront writing one buffer has passed the barrier that follows every read
// of it).
template <typename T>
struct RowEdges {
  T v[2][2][kBlock / 64][5];
};

// The 19 post-stream populations of site (x, y, z) on the row path (all
// threads of the block call it, `act` or not).  Offsets are 32-bit (the row
// path is taken only for replicas of fewer than 2^32 / 19 sites): population
// i of the row (y', z') is at plane(z') + i A + row(y'), with i A folded into
// the scalar base.
template <typename T>
__device__ __forceinline__ void pull_row(const T* __restrict__ sbase, const Geom& g, bool act,
                                         int x, int y, int z, int lane, int wv, RowEdges<T>& edge,
                                         int& par, T d[19]) {
  // populations pulled from x - 1 (c_x = +1) and from x + 1 (c_x = -1)
  constexpr int kFromLeft[5] = {1, 7, 9, 11, 13};
  constexpr int kFromRight[5] = {2, 8, 10, 12, 14};
  const uint32_t A = (uint32_t)g.A;
  const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y == g.ny - 1 ? 0 : y + 1;
  const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z == g.nz - 1 ? 0 : z + 1;
  const uint32_t z0 = (uint32_t)z * 19u * A, zl = (uint32_t)zm * 19u * A,
                 zh = (uint32_t)zp * 19u * A;
  const uint32_t r0 = (uint32_t)(y * g.nx + x), rl = (uint32_t)(ym * g.nx + x),
                 rh = (uint32_t)(yp * g.nx + x);
  // (plane, row) of each population's source: z - c_z, y - c_y
  const uint32_t o00 = z0 + r0, o0l = z0 + rl, o0h = z0 + rh;
  const uint32_t ol0 = zl + r0, olh = zl + rh, oll = zl + rl;
  const uint32_t oh0 = zh + r0, ohl = zh + rl, ohh = zh + rh;
  const uint32_t off[19] = {o00, o00, o00, o0l, o0h, ol0, oh0, o0l, o0h, o0h,
                            o0l, ol0, oh0, oh0, ol0, oll, ohh, ohl, olh};
  // every population is read once: non-temporal loads keep the stream from
  // evicting the transfer field and the mark words
#pragma unroll
  for (int i = 0; i < 19; ++i)
    d[i] = act ? __builtin_nontemporal_load(sbase + (size_t)i * A + off[i]) : T(0);
  // the x shift: rotate by one lane; the end lanes take the neighbouring
  // wavefront's end value (periodic inside the row of nx/64 wavefronts)
  if (lane == 63) {
#pragma unroll
    for (int j = 0; j < 5; ++j) edge.v[par][0][wv][j] = d[kFromLeft[j]];
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 5; ++j) edge.v[par][1][wv][j] = d[kFromRight[j]];
  }
  __syncthreads();
  const int wpr = g.nx >> 6;  // wavefronts per row: 1, 2 or 4
  const int wl = wv & (wpr - 1), rb = wv - wl;
  const int wleft = rb + ((wl + wpr - 1) & (wpr - 1));
  const int wright = rb + ((wl + 1) & (wpr - 1));
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const T l = from_left(d[kFromLeft[j]]);
    const T r = from_right(d[kFromRight[j]]);
    d[kFromLeft[j]] = lane == 0 ? edge.v[par][0][wleft][j] : l;
    d[kFromRight[j]] = lane == 63 ? edge.v[par][1][wright][j] : r;
  }
  par ^= 1;
}

// The same on the general path with 32-bit offsets inside population i's
// slab, i A folded into the scalar base (the replica's 19 S entries fit 32
// bits).
template <typename T>
__device__ __forceinline__ void pull_off32(const T* __restrict__ sbase, const Geom& g, int x,
                                           int y, int z, T d[19]) {
  const uint32_t A = (uint32_t)g.A;
  const int xm = x == 0 ? g.nx - 1 : x - 1, xp = x == g.nx - 1 ? 0 : x + 1;
  const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y == g.ny - 1 ? 0 : y + 1;
  const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z == g.nz - 1 ? 0 : z + 1;
  const uint32_t z0 = (uint32_t)z * 19u * A, zl = (uint32_t)zm * 19u * A,
                 zh = (uint32_t)zp * 19u * A;
  const uint32_t r0 = (uint32_t)(y * g.nx), rl = (uint32_t)(ym * g.nx),
                 rh = (uint32_t)(yp * g.nx);
  const uint32_t X0 = (uint32_t)x, Xl = (uint32_t)xm, Xh = (uint32_t)xp;
  // source (plane, row, column) of each population: z - c_z, y - c_y, x - c_x
  const uint32_t off[19] = {z0 + r0 + X0, z0 + r0 + Xl, z0 + r0 + Xh, z0 + rl + X0,
                            z0 + rh + X0, zl + r0 + X0, zh + r0 + X0, z0 + rl + Xl,
                            z0 + rh + Xh, z0 + rh + Xl, z0 + rl + Xh, zl + r0 + Xl,
                            zh + r0 + Xh, zh + r0 + Xl, zl + r0 + Xh, zl + rl + X0,
                            zh + rh + X0, zh + rl + X0, zl + rh + X0};
  // (plain loads: a shifted run straddles cache lines that the neighbouring
  // wavefront reads too, so the lines should stay in L2)
#pragma unroll
  for (int i = 0; i < 19; ++i) d[i] = sbase[(size_t)i * A + off[i]];
}

// Whether the replica's population entries have 32-bit offsets.
__device__ __forceinline__ bool fits_off32(const Geom& g) {
  return 19ull * (unsigned long long)g.S < (1ull << 32);
}

// Item of a block: workgroups go to the 8 XCDs in turn and each XCD has its
// own L2, so on the general path XCD x takes the x-th contiguous range of
// the work; the lines that the shifted runs of neighbouring items share are
// then fetched once.
__device__ __forceinline__ int xcd_first_item() {
  const int G = gridDim.x, q8 = G / 8, r8 = G % 8, xcd = blockIdx.x % 8;
  return xcd * q8 + (xcd < r8 ? xcd : r8) + blockIdx.x / 8;
}

// Stores 19 values, plane i at o + i A: through the caches, or streamed past
// them (keep_stores; a template argument, since a branch's two sides differ in
// nothing but the hint, which the compiler then drops).
template <bool Cached, typename T>
__device__ __forceinline__ void store_planes(T* __restrict__ o, size_t A, const T d[19]) {
  if constexpr (Cached) {
#pragma unroll
    for (int i = 0; i < 19; ++i) o[(size_t)i * A] = d[i];
  } else {
#pragma unroll
    for (int i = 0; i < 19; ++i) __builtin_nontemporal_store(d[i], o + (size_t)i * A);
  }
}

// With Rec, the transfer field and the mark words the step consumes are also
// copied out for the reverse sweep (the adjoint needs the force density of
// the step and the set of sites the MD steps touched).
// Mode: 0 every replica takes the general path, 1 every replica the row
// path, 2 per replica (a batch mixing both).
template <typename T, bool Rec, bool VarC, int Mode, bool Cached>
__global__ __launch_bounds__(kBlock) void k_collide_stream(StreamArgs<T> a) {
  __shared__ RowEdges<T> edge;
  const int cur = a.clock->cur;
  const long long t = a.clock->t_lb;
  const T* __restrict__ src = a.pop[cur];
  T* __restrict__ dst = a.pop[1 - cur];
  const uint32_t step_lo = (uint32_t)((unsigned long long)t & 0xFFFFFFFFull);
  const uint32_t step_hi = (uint32_t)((unsigned long long)t >> 32);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int par = 0;
  // general path: XCD-contiguous items (measured on 512 replicas of 24-48
  // sites per edge: reads 1.20x -> 1.03x the algorithmic bytes).  The row path
  // reads aligned runs and keeps the plain order.
  const int item0 = Mode == 0 ? xcd_first_item() : (int)blockIdx.x;
  for (int it = item0; it < a.nitems; it += gridDim.x) {
    const int item = a.reverse && cur ? a.nitems - 1 - it : it;
    // the replica is uniform across the block: keep its constants in scalar
    // registers
    const int rr = __builtin_amdgcn_readfirstlane(
        a.R == 1 ? 0 : replica_of_item(a.item_off, a.R, item));
    const RepLB<T> q = scalar_copy(a.rep + rr);
    const int local = (item - q.item_off) * kBlock + threadIdx.x;
    const bool act = local < q.g.S;
    const T* __restrict__ sbase = src + 19 * (size_t)q.site_off;
    int x, y, z;
    site_coords(q.g, act ? local : 0, x, y, z);
    T d[19];
    const bool rows = Mode == 2 ? q.rows != 0 : Mode == 1;
    // general path: 32-bit offsets where the replica's entries allow (uniform)
    const bool off32 = !rows && fits_off32(q.g);
    if (rows) {
      pull_row<T>(sbase, q.g, act, x, y, z, lane, wv, edge, par, d);
    } else if (act && off32) {
      pull_off32<T>(sbase, q.g, x, y, z, d);
    } else if (act) {
      size_t off[19];
      pull_offsets(q.g, x, y, z, off);
#pragma unroll
      for (int i = 0; i < 19; ++i) d[i] = __builtin_nontemporal_load(sbase + off[i]);
    }
    if (act) {
      const int gsite = q.site_off + local;
      const unsigned long long word = a.mark[gsite >> 6];
      T Fx = q.k.g[0], Fy = q.k.g[1], Fz = q.k.g[2];
      T Jx = T(0), Jy = T(0), Jz = T(0);
      if ((word >> (gsite & 63)) & 1ull) {
        const Vec4<T> jv = a.J[gsite];
        if (VarC) {
          Jx = jv.x;
          Jy = jv.y;
          Jz = jv.z;
        } else {
          Fx += jv.x;
          Fy += jv.y;
          Fz += jv.z;
        }
        a.J[gsite] = Vec4<T>{T(0), T(0), T(0), T(0)};
        if (Rec) a.jrec[gsite] = jv;
      }
      if (Rec && (gsite & 63) == 0) a.mrec[gsite >> 6] = word;
      uint32_t hw[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (q.k.noise) {
        const Words4 o0 = philox10(Words4{(uint32_t)local, step_lo, q.tag0, step_hi}, q.key0, q.key1);
        const Words4 o1 = philox10(Words4{(uint32_t)local, step_lo, q.tag1, step_hi}, q.key0, q.key1);
        hw[0] = o0.w0; hw[1] = o0.w1; hw[2] = o0.w2; hw[3] = o0.w3;
        hw[4] = o1.w0; hw[5] = o1.w1; hw[6] = o1.w2; hw[7] = o1.w3;
      }
      collide_deviation<T, VarC>(d, Fx, Fy, Fz, hw, q.k, Jx, Jy, Jz);
      T* __restrict__ o = dst + 19 * (size_t)q.site_off;
      if (rows || off32)
        store_planes<Cached>(
            o + (((uint32_t)z * 19u) * (uint32_t)q.g.A + (uint32_t)(y * q.g.nx + x)),
            (size_t)q.g.A, d);
      else
        store_planes<Cached>(o + pop_offset(q.g, 0, x, y, z), (size_t)q.g.A, d);
      if ((gsite & 63) == 0 && word) a.mark[gsite >> 6] = 0ull;
    }
  }
  if (a.next && blockIdx.x == 0 && threadIdx.x == 0)
    *a.next = Clock{t + 1, a.clock->t_md + a.md_steps, 1 - cur, 0};
}

// Cache hints of the population stores, by the size of a population buffer
// against the 256 MB memory-side cache (and the 32 MB of L2 below it).  A
// lattice that is far larger streams past the caches (non-temporal stores).
// One whose step fits in them keeps what it writes, which the next step reads;
// with aligned rows and up to twice that size, every other step also takes its
// items in reverse, so that it starts with the part written last.  Measured,
// streamed against kept, us a step: general path 60^3 (16 MB) 7.2/7.8, 66^3
// (22 MB) 12.3/9.7, 96^3 (67 MB) 28.0/21.4, 121 x 120 x 119 (131 MB) 56.0/39.1,
// 126^3 (152 MB) 64.8/61.4, 132^3 (175 MB) 67.8/71.7, 144^3 (227 MB) 82.9/84.8;
// row path 64 x 64 x 128 (40 MB) 15.6/16.1, 128 x 128 x 64 (80 MB) 29.2/27.3,
// 128^3 (159 MB) 54.0/50.4, 256 x 128 x 128 (319 MB) 103.8/96.5 (109.8 without
// the reversal), 256 x 256 x 96 (478 MB) 155/150, 256 x 256 x 128 (637 MB)
// 204.6/207.7, 256^3 406.8/419.5.  With particles, whose kernels run between
// the steps, the row path gains nothing from keeping its stores (128^3 polymer,
// three cycles and a copy, 794/799).
static bool keep_stores(const Plan& pl) {
  const double mb = 19.0 * (double)pl.P * (pl.prec == 32 ? 4.0 : 8.0) / 1e6;
  if (pl.row_replicas == pl.R) return pl.Ntot == 0 && mb > 60.0 && mb < 520.0;
  return pl.row_replicas == 0 && mb > 20.0 && mb < 160.0;
}

template <typename T>
static StreamArgs<T> stream_args(Context* c) {
  StreamArgs<T> a;
  a.pop[0] = (T*)c->popv[0];
  a.pop[1] = (T*)c->popv[1];
  a.J = (Vec4<T>*)at(c, c->plan.lay.transfer);
  a.jrec = (Vec4<T>*)c->rec_J;
  a.mrec = c->rec_mark;
  a.mark = (unsigned long long*)at(c, c->plan.lay.mark);
  a.rep = (const RepLB<T>*)at(c, c->plan.lay.rep_lb);
  a.item_off = (const int32_t*)at(c, c->plan.lay.item_rep);
  a.clock = clock_of(c, c->clk);
  a.next = nullptr;
  a.md_steps = 0;
  a.R = c->plan.R;
  a.nitems = c->plan.nitems;
  a.varc = c->p[0].variant == 3 ? 1 : 0;
  a.reverse = c->plan.row_replicas == c->plan.R && keep_stores(c->plan) ? 1 : 0;
  return a;
}

template <typename T, int Mode, bool Cached>
static void collide_stream_mode(Context* c, const StreamArgs<T>& a, int blocks) {
  const dim3 grid(blocks), block(kBlock);
  if (c->p[0].variant == 3)  // no adjoint for variant 3: never recording
    hipLaunchKernelGGL((k_collide_stream<T, false, true, Mode, Cached>), grid, block, 0, c->stream,
                       a);
  else if (a.jrec)
    hipLaunchKernelGGL((k_collide_stream<T, true, false, Mode, Cached>), grid, block, 0, c->stream,
                       a);
  else
    hipLaunchKernelGGL((k_collide_stream<T, false, false, Mode, Cached>), grid, block, 0,
                       c->stream, a);
}

template <typename T>
static hipError_t collide_stream_t(Context* c, Clock* next, int md_steps) {
  StreamArgs<T> a = stream_args<T>(c);
  a.next = next;
  a.md_steps = md_steps;
  const int blocks = c->tune.lb_blocks > 0 ? std::min(c->tune.lb_blocks, a.nitems) : a.nitems;
  // the row path's kernel is instantiated on its own when no replica needs
  // the general one (fewer registers, more waves in flight)
  const bool rows = c->plan.row_replicas == c->plan.R, keep = keep_stores(c->plan);
  if (rows && keep)
    collide_stream_mode<T, 1, true>(c, a, blocks);
  else if (rows)
    collide_stream_mode<T, 1, false>(c, a, blocks);
  else if (keep)
    collide_stream_mode<T, 0, true>(c, a, blocks);
  else if (c->plan.row_replicas == 0)
    collide_stream_mode<T, 0, false>(c, a, blocks);
  else
    collide_stream_mode<T, 2, false>(c, a, blocks);
  return hipGetLastError();
}

hipError_t launch_collide_stream(Context* c, Clock* next, int md_steps) {
  return c->plan.prec == 32 ? collide_stream_t<float>(c, next, md_steps)
                            : collide_stream_t<double>(c, next, md_steps);
}

// The clock advanced in place, after an LB step that did not write the other
// entry: a caller captures the step in a graph of its own, which then replays
// from whatever step the entry holds.
__global__ void k_clock_advance(Clock* __restrict__ clk, int md_steps) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    clk->t_lb += 1;
    clk->t_md += md_steps;
    clk->cur = 1 - clk->cur;
  }
}

hipError_t launch_clock_advance(Context* c, int md_steps) {
  hipLaunchKernelGGL(k_clock_advance, dim3(1), dim3(64), 0, c->stream, clock_of(c, c->clk),
                     md_steps);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Block reduction of W <= kRedWidth doubles per thread into out[0..W).
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void block_reduce_store(const double acc[W], double* out) {
  __shared__ double sh[kBlock / 64][W];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    double s = acc[q];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) sh[wv][q] = s;
  }
  __syncthreads();
  if (threadIdx.x < W) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += sh[w][threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Moment sums and fields.  Columns of a partial row: 0 sum drho, 1-3 sum j,
// 4-6 sum J, 7 sum |j/rho|^2.  Fields (density, velocity) of replica
// `field_rep`.
//
// Bound by the 76 (FP32) bytes a site's populations take, so the pass does
// little else: populations pulled as in the collide-stream kernel, J read
// only at marked sites (it is zero elsewhere), and one block reduction per
// chunk of consecutive items instead of one per 256 sites (a reduction of 16
// columns costs more than the loads of an item).  A chunk's sums go to one
// row, numbered by the chunk for a single replica, else by the last item the
// chunk holds of a replica (chunk_row), since a chunk may span several.
// 512 replicas of 24-48 sites per edge (29.2 M sites, 2.2 GB): 457 us = 4.9
// TB/s, against 1000 us with one reduction per item, 64-bit gathers and J
// read at every site; 50 x 41 x 37: 7.0 against 9.1 us.
// ---------------------------------------------------------------------------
constexpr int kMomentCols = 8;

__device__ __forceinline__ int chunk_row(int chunk, int per, int end) {
  const int e = (chunk + 1) * per;
  return (e < end ? e : end) - 1;
}

template <typename T, int Mode>
__global__ __launch_bounds__(kBlock) void k_moments(StreamArgs<T> a, int per, int field_rep,
                                                    T* __restrict__ rho_out,
                                                    T* __restrict__ u_out,
                                                    double* __restrict__ partials) {
  __shared__ RowEdges<T> edge;
  const T* __restrict__ src = a.pop[a.clock->cur];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int chunk = Mode == 0 ? xcd_first_item() : (int)blockIdx.x;
  const int end = min((chunk + 1) * per, a.nitems);
  int par = 0;
  double acc[kMomentCols];
#pragma unroll
  for (int k = 0; k < kMomentCols; ++k) acc[k] = 0.0;
  for (int item = chunk * per; item < end; ++item) {
    const int rr = __builtin_amdgcn_readfirstlane(
        a.R == 1 ? 0 : replica_of_item(a.item_off, a.R, item));
    const RepLB<T> q = scalar_copy(a.rep + rr);
    const int local = (item - q.item_off) * kBlock + threadIdx.x;
    const bool act = local < q.g.S;
    const T* __restrict__ sbase = src + 19 * (size_t)q.site_off;
    int x, y, z;
    site_coords(q.g, act ? local : 0, x, y, z);
    T d[19];
    const bool rows = Mode == 2 ? q.rows != 0 : Mode == 1;
    if (rows) {
      pull_row<T>(sbase, q.g, act, x, y, z, lane, wv, edge, par, d);
    } else if (act && fits_off32(q.g)) {
      pull_off32<T>(sbase, q.g, x, y, z, d);
    } else if (act) {
      size_t off[19];
      pull_offsets(q.g, x, y, z, off);
#pragma unroll
      for (int i = 0; i < 19; ++i) d[i] = sbase[off[i]];
    }
    if (act) {
      T drho, jx, jy, jz;
      moments_deviation<T>(d, drho, jx, jy, jz);
      const T rho = q.k.rho0 + drho;
      acc[0] += (double)drho;
      acc[1] += (double)jx;
      acc[2] += (double)jy;
      acc[3] += (double)jz;
      const int gsite = q.site_off + local;
      if ((a.mark[gsite >> 6] >> (gsite & 63)) & 1ull) {
        const Vec4<T> jv = a.J[gsite];
        acc[4] += (double)jv.x;
        acc[5] += (double)jv.y;
        acc[6] += (double)jv.z;
        if (a.varc) {
          jx += jv.x;
          jy += jv.y;
          jz += jv.z;
        }
      }
      if (rr == field_rep) {
        if (rho_out) rho_out[local] = rho;
        if (u_out) {
          const size_t S = (size_t)q.g.S;
          u_out[local] = jx / rho;
          u_out[S + local] = jy / rho;
          u_out[2 * S + local] = jz / rho;
        }
      }
      const double irho = 1.0 / (double)rho;
      const double ux = (double)jx * irho, uy = (double)jy * irho, uz = (double)jz * irho;
      acc[7] += ux * ux + uy * uy + uz * uz;
    }
    // the chunk's last item of this replica: its row
    const bool last = item + 1 == end || (a.R > 1 && a.item_off[rr + 1] == item + 1);
    if (last) {
      block_reduce_store<kMomentCols>(acc, partials + (size_t)(a.R == 1 ? chunk : item) * kRedWidth);
#pragma unroll
      for (int k = 0; k < kMomentCols; ++k) acc[k] = 0.0;
    }
  }
}

// One block per replica: sum its partial rows (for a single replica one per
// chunk; else those of its chunks), then its particles' momentum and kinetic
// energy (columns 8-10 sum v, 11 sum |v|^2); column 12 is the context's
// non-finite flag.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_finalize(StreamArgs<T> a,
                                                     const RepMD* __restrict__ md,
                                                     const double* __restrict__ partials,
                                                     const double* __restrict__ v, int64_t Ntot,
                                                     double* __restrict__ totals, int per,
                                                     const int32_t* __restrict__ flags) {
  const int rr = blockIdx.x;
  const int i0 = a.item_off[rr], i1 = a.item_off[rr + 1];
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  for (int c = i0 / per + threadIdx.x; c <= (i1 - 1) / per; c += kBlock) {
    const int row = a.R == 1 ? c : chunk_row(c, per, i1);
#pragma unroll
    for (int k = 0; k < kMomentCols; ++k) acc[k] += partials[(size_t)row * kRedWidth + k];
  }
  if (v) {
    const int p0 = md[rr].part_off, n = md[rr].N;
    for (int p = p0 + threadIdx.x; p < p0 + n; p += kBlock) {
      const double vx = v[p], vy = v[Ntot + p], vz = v[2 * Ntot + p];
      acc[8] += vx;
      acc[9] += vy;
      acc[10] += vz;
      acc[11] += vx * vx + vy * vy + vz * vz;
    }
  }
  block_reduce_store<12>(acc, totals + (size_t)rr * kRedWidth);
  // the non-finite flag travels with the totals (column 12)
  if (threadIdx.x == 0) totals[(size_t)rr * kRedWidth + 12] = (double)flags[0];
}

// The same sums for a single large system, in two launches: each block of the
// first sums its share of the rows and the particles into a row of its own
// (`Last` false), one block sums those rows.  One block alone is bound by the
// latency of its rounds (172 us of its own at 256^3 with 1e5 particles).  The
// whole call, us, by one block and so: 256^3 with 1e5 particles 372/236, 160^3
// with 6e4 211/88, 200 x 190 x 180 without 141/127, 128^3 with 1e4 77/72; with
// fewer items than fill the chip the rows behind the chunks' are too few, and
// there is little to gain (72^3 with 3e4 79, 96^3 with 500 58).
template <bool Last>
__global__ __launch_bounds__(kBlock) void k_presum(const double* __restrict__ rows, int nrows,
                                                   const double* __restrict__ v, int64_t N,
                                                   double* __restrict__ out,
                                                   const int32_t* __restrict__ flags) {
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  const int stride = gridDim.x * kBlock, t0 = blockIdx.x * kBlock + threadIdx.x;
  for (int r = t0; r < nrows; r += stride)
#pragma unroll
    for (int k = 0; k < (Last ? 12 : kMomentCols); ++k) acc[k] += rows[(size_t)r * kRedWidth + k];
  if (!Last && v)
    for (int64_t p = t0; p < N; p += stride) {
      const double vx = v[p], vy = v[N + p], vz = v[2 * N + p];
      acc[8] += vx;
      acc[9] += vy;
      acc[10] += vz;
      acc[11] += vx * vx + vy * vy + vz * vz;
    }
  block_reduce_store<12>(acc, out + (size_t)blockIdx.x * kRedWidth);
  if (Last && threadIdx.x == 0) out[12] = (double)flags[0];
}
constexpr int kPresumBlocks = 128;
constexpr int64_t kPresumFrom = 4096;  // rows and particles

// Items per chunk: one reduction per 4 items once there are enough chunks to
// fill the chip several times over; at most max_rows chunks.
static int moment_chunk(int nitems, int max_rows) {
  const int per = std::min(4, std::max(1, nitems / 4096));
  return std::max(per, (nitems + max_rows - 1) / max_rows);
}

template <typename T>
static hipError_t moments_launch(Context* c, const StreamArgs<T>& a, int per, int rep, void* d_rho,
                                 void* d_u, double* partials) {
  const dim3 grid((unsigned)((a.nitems + per - 1) / per));
  if (c->plan.row_replicas == c->plan.R)
    hipLaunchKernelGGL((k_moments<T, 1>), grid, dim3(kBlock), 0, c->stream, a, per, rep,
                       (T*)d_rho, (T*)d_u, partials);
  else if (c->plan.row_replicas == 0)
    hipLaunchKernelGGL((k_moments<T, 0>), grid, dim3(kBlock), 0, c->stream, a, per, rep,
                       (T*)d_rho, (T*)d_u, partials);
  else
    hipLaunchKernelGGL((k_moments<T, 2>), grid, dim3(kBlock), 0, c->stream, a, per, rep,
                       (T*)d_rho, (T*)d_u, partials);
  return hipGetLastError();
}

template <typename T>
static hipError_t moments_t(Context* c, int rep, void* d_rho, void* d_u, double* d_totals) {
  StreamArgs<T> a = stream_args<T>(c);
  double* partials = (double*)at(c, c->plan.lay.partials);
  const int per = moment_chunk(a.nitems, a.nitems);
  const hipError_t e = moments_launch<T>(c, a, per, rep, d_rho, d_u, partials);
  if (e != hipSuccess || !d_totals) return e;
  const int rows = (a.nitems + per - 1) / per;
  // (the first launch's rows go behind the chunks', which leave most of the
  // region free once a chunk is several items)
  if (c->plan.R == 1 && rows + c->plan.Ntot >= kPresumFrom && a.nitems - rows >= kPresumBlocks) {
    const double* v = (const double*)(c->bound ? c->v : nullptr);
    const int32_t* flags = (const int32_t*)at(c, c->plan.lay.flags);
    double* sums = partials + (size_t)rows * kRedWidth;
    hipLaunchKernelGGL(k_presum<false>, dim3(kPresumBlocks), dim3(kBlock), 0, c->stream, partials,
                       rows, v, c->plan.Ntot, sums, flags);
    hipLaunchKernelGGL(k_presum<true>, dim3(1), dim3(kBlock), 0, c->stream, sums, kPresumBlocks,
                       (const double*)nullptr, (int64_t)0, d_totals, flags);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_finalize<T>, dim3(c->plan.R), dim3(kBlock), 0, c->stream, a,
                     (const RepMD*)at(c, c->plan.lay.rep_md), partials,
                     (const double*)(c->bound ? c->v : nullptr), c->plan.Ntot, d_totals, per,
                     (const int32_t*)at(c, c->plan.lay.flags));
  return hipGetLastError();
}

hipError_t launch_moments(Context* c, int rep, void* d_rho, void* d_u, double* d_totals) {
  return c->plan.prec == 32 ? moments_t<float>(c, rep, d_rho, d_u, d_totals)
                            : moments_t<double>(c, rep, d_rho, d_u, d_totals);
}

// ---------------------------------------------------------------------------
// Moments without workspace scratch (lb_moments_noalloc): the reduction rows
// live in a fixed device array of this library instead of the context's
// workspace.  At most kScratchRows chunks, each summed into one row, then
// the totals row.  Every call overwrites all the
// rows it reads, so nothing needs clearing; calls that overlap on one GPU
// (two streams) race on the array.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};
}  // namespace

// Device address of this GPU's copy of the array (current device), looked
// up once per device; in host code the array's name is not a device address.
hipError_t moments_scratch(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = (double*)p;
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

template <typename T>
static hipError_t moments_rows_t(Context* c, void* d_rho, void* d_u, double* rows) {
  StreamArgs<T> a = stream_args<T>(c);
  const int per = moment_chunk(a.nitems, kScratchRows);
  const hipError_t e = moments_launch<T>(c, a, per, 0, d_rho, d_u, rows);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_finalize<T>, dim3(1), dim3(kBlock), 0, c->stream, a,
                     (const RepMD*)at(c, c->plan.lay.rep_md), rows,
                     (const double*)(c->bound ? c->v : nullptr), c->plan.Ntot,
                     rows + (size_t)kScratchRows * kRedWidth, per,
                     (const int32_t*)at(c, c->plan.lay.flags));
  return hipGetLastError();
}

hipError_t launch_moments_rows(Context* c, void* d_rho, void* d_u, double* rows) {
  return c->plan.prec == 32 ? moments_rows_t<float>(c, d_rho, d_u, rows)
                            : moments_rows_t<double>(c, d_rho, d_u, rows);
}

// ---------------------------------------------------------------------------
// Copies between pull storage and the plain post-stream layout of one
// replica ([19][S] and [3][S] arrays in the run precision).
// ---------------------------------------------------------------------------
// Copy out: the populations pulled as in the collide-stream kernel (aligned
// rows or 32-bit offsets) and stored under the same cache hints, one 256-site
// item per block.  Bound by memory, with the 19 separate output arrays as its limit:
// 435 us at 256^3 in FP32 (5.9 TB/s; the collide-stream kernel, which writes
// interleaved planes, 6.3), against 449 us with 64-bit gathers and cached
// stores.
// Variant 3 (pend != nullptr): a copy out adds the increments of the
// transfer the site has received in the current interval (J at marked
// sites), so that it shows the populations as the paper's variant C holds
// them after each MD step.
template <typename T, int Mode, bool Cached>
__global__ __launch_bounds__(kBlock) void k_get_pop(const T* __restrict__ pop,
                                                    T* __restrict__ plain,
                                                    const Vec4<T>* __restrict__ pend,
                                                    const unsigned long long* __restrict__ mark,
                                                    const RepLB<T>* __restrict__ rep, int rr) {
  __shared__ RowEdges<T> edge;
  const RepLB<T> q = scalar_copy(rep + rr);
  const int item = Mode == 0 ? xcd_first_item() : (int)blockIdx.x;
  const int r = item * kBlock + threadIdx.x;
  const bool act = r < q.g.S;
  const T* __restrict__ sbase = pop + 19 * (size_t)q.site_off;
  int x, y, z, par = 0;
  site_coords(q.g, act ? r : 0, x, y, z);
  T d[19];
  if (Mode == 1)
    pull_row<T>(sbase, q.g, act, x, y, z, threadIdx.x & 63, threadIdx.x >> 6, edge, par, d);
  if (!act) return;
  if (Mode == 0) {
    if (fits_off32(q.g)) {
      pull_off32<T>(sbase, q.g, x, y, z, d);
    } else {
      size_t off[19];
      pull_offsets(q.g, x, y, z, off);
#pragma unroll
      for (int i = 0; i < 19; ++i) d[i] = sbase[off[i]];
    }
  }
  const int gs = q.site_off + r;
  if (pend && ((mark[gs >> 6] >> (gs & 63)) & 1ull)) {
    const Vec4<T> jv = pend[gs];
    T drho, jx, jy, jz, sm[6], dd[19];
    moments_deviation<T>(d, drho, jx, jy, jz);
    varc_stress<T>(jx, jy, jz, T(1) / (q.k.rho0 + drho), jv.x, jv.y, jv.z, q.k.hb, q.k.hs, sm);
    mode_increments_to_pops<T>(jv.x, jv.y, jv.z, sm, dd);
#pragma unroll
    for (int i = 0; i < 19; ++i) d[i] += dd[i];
  }
  store_planes<Cached>(plain + r, (size_t)q.g.S, d);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_set_pop(T* __restrict__ pop, int site_off, Geom g,
                                                    const T* __restrict__ plain) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= g.S) return;
  int x, y, z;
  size_t off[19];
  site_coords(g, r, x, y, z);
  pull_offsets(g, x, y, z, off);
  T* __restrict__ base = pop + 19 * (size_t)site_off;
#pragma unroll
  for (int i = 0; i < 19; ++i) base[off[i]] = plain[(size_t)i * g.S + r];
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_get_transfer(const Vec4<T>* __restrict__ J, int site_off,
                                                         int S, T* __restrict__ out) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= S) return;
  const Vec4<T> jv = J[site_off + r];
  out[r] = jv.x;
  out[(size_t)S + r] = jv.y;
  out[2 * (size_t)S + r] = jv.z;
}

template <typename T>
static hipError_t copy_t(Context* c, int rep, void* plain, int what) {
  const lbmd_params& p = c->p[rep];
  Geom g;
  g.nx = p.nx;
  g.ny = p.ny;
  g.nz = p.nz;
  g.S = p.nx * p.ny * p.nz;
  g.A = p.nx * p.ny;
  g.inv_nx = 1.0 / p.nx;
  g.inv_ny = 1.0 / p.ny;
  const int blocks = (g.S + kBlock - 1) / kBlock;
  const int site_off = (int)c->plan.site_off[rep];
  if (what == 2) {
    hipLaunchKernelGGL(k_get_transfer<T>, dim3(blocks), dim3(kBlock), 0, c->stream,
                       (const Vec4<T>*)at(c, c->plan.lay.transfer), site_off, g.S, (T*)plain);
    return hipGetLastError();
  }
  T* pop = (T*)c->popv[c->cur];
  if (what == 1) {
    hipLaunchKernelGGL(k_set_pop<T>, dim3(blocks), dim3(kBlock), 0, c->stream, pop, site_off, g,
                       (const T*)plain);
    return hipGetLastError();
  }
  const Vec4<T>* pend = p.variant == 3 ? (const Vec4<T>*)at(c, c->plan.lay.transfer) : nullptr;
  const unsigned long long* mark = (const unsigned long long*)at(c, c->plan.lay.mark);
  const RepLB<T>* tab = (const RepLB<T>*)at(c, c->plan.lay.rep_lb);
  const bool keep = keep_stores(c->plan);
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, c->stream, (const T*)pop, (T*)plain,
                       pend, mark, tab, rep);
  };
  if (row_path(p))
    keep ? go(k_get_pop<T, 1, true>) : go(k_get_pop<T, 1, false>);
  else
    keep ? go(k_get_pop<T, 0, true>) : go(k_get_pop<T, 0, false>);
  return hipGetLastError();
}

hipError_t launch_get_populations(Context* c, int rep, void* dst) {
  return c->plan.prec == 32 ? copy_t<float>(c, rep, dst, 0) : copy_t<double>(c, rep, dst, 0);
}
hipError_t launch_set_populations(Context* c, int rep, const void* src) {
  return c->plan.prec == 32 ? copy_t<float>(c, rep, (void*)src, 1)
                            : copy_t<double>(c, rep, (void*)src, 1);
}
hipError_t launch_get_transfer(Context* c, int rep, void* dst) {
  return c->plan.prec == 32 ? copy_t<float>(c, rep, dst, 2) : copy_t<double>(c, rep, dst, 2);
}

// ---------------------------------------------------------------------------
// Regions copied and filled one after the other by the whole grid, 16 bytes a
// thread where both ends are aligned (RegionOps).  Bound by memory in the
// large (a state of 256^3 in FP32: saved in 416 us, loaded in 510, against 508
// and 611 with the runtime's copies), by the launch in the small (32^3: 15 and
// 26 us, against 18 and 56).  Past the caches' reach (Big) the copies are
// streamed: kept, 256^3 takes 672 and 807 us.
// ---------------------------------------------------------------------------
typedef uint32_t quad __attribute__((ext_vector_type(4)));

template <bool Big>
__global__ __launch_bounds__(kBlock) void k_region_ops(RegionOps ops) {
  const size_t t0 = (size_t)blockIdx.x * kBlock + threadIdx.x, stride = (size_t)gridDim.x * kBlock;
  long long t_lb = ops.clock_value.t_lb, t_md = ops.clock_value.t_md;
  if (ops.clock_from) {
    long long cnt[2];
    __builtin_memcpy(cnt, ops.clock_from, sizeof(cnt));
    t_lb = cnt[0];
    t_md = cnt[1];
    if (t_lb < 0 || t_md < 0) return;
  }
  for (int k = 0; k < ops.n; ++k) {
    uint32_t* __restrict__ dst = ops.op[k].dst;
    const uint32_t* __restrict__ src = ops.op[k].src;
    const uint32_t f = ops.op[k].fill;
    const size_t words = ops.op[k].words;
    size_t quads = 0;
    if ((((uintptr_t)dst | (uintptr_t)src) & 15) == 0) {
      quads = words / 4;
      quad* __restrict__ d = reinterpret_cast<quad*>(dst);
      const quad* __restrict__ q = reinterpret_cast<const quad*>(src);
      if (!src)
        for (size_t i = t0; i < quads; i += stride) d[i] = quad{f, f, f, f};
      else if (Big)
        for (size_t i = t0; i < quads; i += stride)
          __builtin_nontemporal_store(__builtin_nontemporal_load(q + i), d + i);
      else
        for (size_t i = t0; i < quads; i += stride) d[i] = q[i];
    }
    for (size_t i = 4 * quads + t0; i < words; i += stride) dst[i] = src ? src[i] : f;
  }
  if (t0 == 0 && ops.clock) *ops.clock = Clock{t_lb, t_md, ops.clock_value.cur, 0};
  if (t0 == 0 && ops.counters)
    __builtin_memcpy(ops.counters, ops.counter_value, sizeof(ops.counter_value));
}

hipError_t launch_region_ops(const RegionOps& asked, hipStream_t stream) {
  RegionOps ops = asked;
  ops.n = 0;
  size_t most = 1;
  for (int k = 0; k < asked.n; ++k) {
    const RegionOps::Op& o = asked.op[k];
    if ((((uintptr_t)o.dst | (uintptr_t)o.src) & 3) != 0) {  // (a state at an odd address)
      const hipError_t e =
          hipMemcpyAsync(o.dst, o.src, 4 * o.words, hipMemcpyDeviceToDevice, stream);
      if (e != hipSuccess) return e;
      continue;
    }
    ops.op[ops.n++] = o;
    most = std::max(most, o.words);
  }
  const size_t want = (most / 4 + kBlock - 1) / kBlock;
  const unsigned grid = (unsigned)std::max<size_t>(1, std::min<size_t>(want, 1u << 22));
  if (8 * most > ((size_t)256 << 20))  // source and destination past the memory-side cache
    hipLaunchKernelGGL(k_region_ops<true>, dim3(grid), dim3(kBlock), 0, stream, ops);
  else
    hipLaunchKernelGGL(k_region_ops<false>, dim3(grid), dim3(kBlock), 0, stream, ops);
  return hipGetLastError();
}

// The tables of a single system, carried as launch arguments.
template <typename T>
__global__ void k_tables_one(RepLB<T>* __restrict__ lb, RepLB<T> lb_value, RepMD* __restrict__ md,
                             RepMD md_value, int32_t* __restrict__ item_off, int nitems) {
  if (threadIdx.x == 0) {
    *lb = lb_value;
    *md = md_value;
    item_off[0] = 0;
    item_off[1] = nitems;
  }
}

hipError_t launch_tables_one(Context* c, const RepLB<float>* lb32, const RepLB<double>* lb64,
                             const RepMD& md) {
  const Layout& L = c->plan.lay;
  if (lb32)
    hipLaunchKernelGGL(k_tables_one<float>, dim3(1), dim3(64), 0, c->stream,
                       (RepLB<float>*)at(c, L.rep_lb), *lb32, (RepMD*)at(c, L.rep_md), md,
                       (int32_t*)at(c, L.item_rep), c->plan.nitems);
  else
    hipLaunchKernelGGL(k_tables_one<double>, dim3(1), dim3(64), 0, c->stream,
                       (RepLB<double>*)at(c, L.rep_lb), *lb64, (RepMD*)at(c, L.rep_md), md,
                       (int32_t*)at(c, L.item_rep), c->plan.nitems);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain device copy with 16-byte non-temporal loads and stores: the
// read+write streaming ceiling the roofline of the collide-stream kernel is
// set against (and the known-size dispatch the HBM byte counters are
// calibrated with).
// ---------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_stream_copy(const v4f* __restrict__ src,
                                                        v4f* __restrict__ dst, size_t n4) {
  for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < n4;
       t += (size_t)gridDim.x * kBlock)
    __builtin_nontemporal_store(__builtin_nontemporal_load(src + t), dst + t);
}

// One 16-byte element per thread over the whole range (a persistent grid of
// a few blocks per CU measured 10-20% slower).
hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t stream) {
  const size_t n4 = bytes / 16;
  const size_t want = (n4 + kBlock - 1) / kBlock;
  const unsigned grid = (unsigned)std::max<size_t>(1, std::min<size_t>(want, (size_t)1 << 30));
  hipLaunchKernelGGL(k_stream_copy, dim3(grid), dim3(kBlock), 0, stream, (const v4f*)src,
                     (v4f*)dst, n4);
  return hipGetLastError();
}

}  // namespace lbmd_impl

// sph_kernels.hip -- gfx950 kernels of the WCSPH thermo-fluid hot path
// (arXiv 2512.09904, Section 2).  One advection step is the launch sequence
// clear -> pose -> fold -> scan1..3 -> scatter -> cellsort -> reorder -> build
// -> sumw -> dt -> visc_heat -> half_a -> n_ac x (momentum, continuity) -> end
// -> final.  Every kernel covers all slots of a launch table: block b of the
// grid belongs to the slot whose block range contains b, so one launch
// steps many independent solves (continuous batching) and a solve's result
// does not depend on which other slots share the launch.
//
// No MFMA: the sweeps are sums over neighbour rows, bound by the rows' bytes and
// by vector issue; the build's cutoff test as a matrix product (FP32, exact
// retest near the cutoff) was 5 % faster at 1.9 M particles in one form and 39 %
// slower in another, because placing the hits in order costs as much as the
// test.  Reductions are deterministic (fixed-order wave butterflies and block
// trees, Neumaier-compensated FP64 for the reports); the only atomics are
// integer counters of the cell sort and fault flags.
//
// In FP32 and mixed arithmetic the sweeps take their neighbours from LDS.  A
// block of 256 particles reaches about 2080 others (its cells' stencils), each
// of them about ten times; their records are loaded once per block and the rows
// name them by their number in the block.  Gathered from memory, the same
// records are bound by the rate of scattered lanes.  Kernel times at 1.9 M
// particles, gathered and staged: continuity 431 and 281 us, momentum 484 and
// 343, viscous/heat 781 and 564, kernel sum 450 and 378; at 0.9 M 103 and 69,
// 87 and 64, 406 and 282, 243 and 214.  What is left at 1.9 M (continuity): 0.89
// GB fetched, 0.19 ms at the rate of a large copy, beside 0.2 ms of vector
// instructions; two blocks fit a CU, and they overlap the two in part.
// A block in ten has too many candidates for half a CU's LDS; three of its
// wavefronts are staged then and the fourth gathers.
//
// STAGE = false (FP64 mode; launches without TAB_STAGE): nothing is numbered or
// staged, every row holds sorted indices, and without the staged records' LDS
// three to five waves per SIMD hide the gathers.  The pairs, their order and their
// arithmetic are the same, so both give the same bits.
#include <math.h>

#include <type_traits>

#include "sph_device.h"

namespace sphk {

// Gathered rows (STAGE = false, and the wavefronts whose candidates do not fit) are
// walked ROW_UNROLL entries at a time (SOLID_UNROLL for the wall rows,
// VISC_SOLID_UNROLL for the viscous/heat sweep's wall rows, CONT_UNROLL in the
// continuity sweep of the staged modes, where a block waits for its gathering
// wavefront: with eight it took 287 us at 1.9 M particles, with twelve 281; in
// FP64 twelve spilled, 287 us at 196,000 particles against 116), and the next
// group's indices are loaded before the current group's gathers are
// consumed, so a wavefront keeps two dependent loads in flight.  Entries past
// a row's count are loaded from within the row's capacity (capacities are
// multiples of sixteen, a group beyond the first is loaded only when it
// starts below the count, and the continuity sweep's groups of twelve clamp
// their last loads to the row's last entry) and replaced by a null entry: own
// index, F = 0, which adds exactly zero to every sum.
#define ROW_UNROLL 8
#define SOLID_UNROLL 8
#define VISC_SOLID_UNROLL 4
#define CONT_UNROLL 12

// A block's window of the fluid anchors: the WIN particles around the
// block's own BLOCK (clamped to the array), staged in LDS with coalesced
// loads.  In the Morton order most neighbours of the block's particles fall
// inside it, so their 32-byte gathers become LDS reads; the rest are gathered
// from global memory.  Used by the kernel sums of blocks that are not staged,
// whose anchor gathers (two 16-byte requests per pair) otherwise bound them by
// the vector memory unit's rate of one scattered lane per clock.  512 particles
// (16 KB of LDS per block) rather than 1024: fewer neighbours fall inside, but
// twice as many blocks fit on a CU.
constexpr int WIN = 512;
struct Window {
  uint32_t w0, wn;
};
__device__ __forceinline__ Window window_of(int lb, int nf) {
  Window w;
  w.wn = (uint32_t)min(WIN, nf);
  const int lo = lb * BLOCK - (WIN - BLOCK) / 2;
  w.w0 = (uint32_t)max(0, min(lo, nf - (int)w.wn));
  return w;
}
template <class T>
__device__ __forceinline__ void stage_window(T* lds, const GLB T* g, const Window& w) {
  for (uint32_t q = threadIdx.x; q < w.wn; q += BLOCK) lds[q] = g[w.w0 + q];
}
template <class T>
__device__ __forceinline__ T win_get(const T* lds, const GLB T* g, uint32_t j, const Window& w) {
  const uint32_t d = j - w.w0;
  return d < w.wn ? lds[d] : g[j];
}

// per-thread accumulators for up to NACC (= 2) bodies touched by one fluid
// particle; explicit register arrays (no indexing by a runtime value, so
// nothing goes to scratch)
template <int W>
struct BodyAcc {
  int id0, id1;
  double v0[W], v1[W];
  __device__ void init() {
    id0 = id1 = -1;
#pragma unroll
    for (int k = 0; k < W; ++k) v0[k] = v1[k] = 0.0;
  }
  // Makes b the current body, whose sums are in v0 (a change of body exchanges
  // the two); false when both accumulators hold other bodies.  Nearly every
  // particle touches one body, and a wavefront skips the exchange when no lane
  // needs it.
  __device__ __forceinline__ bool select(int b) {
    if (b != id0) {
      if (id0 >= 0) {
        const int t = id0;
        id0 = id1;
        id1 = t;
#pragma unroll
        for (int k = 0; k < W; ++k) {
          const double u = v0[k];
          v0[k] = v1[k];
          v1[k] = u;
        }
      }
      if (id0 < 0) id0 = b;
      if (id0 != b) return false;
    }
    return true;
  }
  // Bodies of four staged wall entries: those past the row's end take the
  // current body.  True when every lane's four are its current body (the first
  // entry of a row opens it), so that no exchange is needed.
  __device__ __forceinline__ bool current(const float (&w)[4], const bool (&real)[4], int (&b)[4]) {
    if (id0 < 0) id0 = (int)w[0];
    bool odd = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      b[u] = real[u] ? (int)w[u] : id0;
      odd = odd || b[u] != id0;
    }
    return !__any(odd);
  }
  // one wall pair's acceleration f and its moment about the body centre (lever
  // arm l)
  template <class Real, class Real4>
  __device__ __forceinline__ void moment(Real fx, Real fy, Real fz, const Real4 l) {
    const double x = fx, y = fy, z = fz, lx = l.x, ly = l.y, lz = l.z;
    v0[0] += x;
    v0[1] += y;
    v0[2] += z;
    v0[3] = fma(-lz, y, fma(ly, z, v0[3]));
    v0[4] = fma(-lx, z, fma(lz, x, v0[4]));
    v0[5] = fma(-ly, x, fma(lx, y, v0[5]));
  }
  // accelerations to forces of the fluid on the body: components [0, 6) times -m
  __device__ __forceinline__ void to_force(double m) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      v0[k] *= -m;
      v1[k] *= -m;
    }
  }
};

// Deterministic block reduction of per-thread body accumulators: for each
// body and component, the wavefront by DPP lane moves in a fixed order, then
// the four waves in order.  A wavefront skips the bodies none of its lanes
// touches (by LDS permutes over all bodies and components the momentum sweep
// took 411 instead of 396 us at 1.9 M particles).
template <int W>
// out is quantity-major: out[(b * W + k) * nblk + lb]
__device__ __forceinline__ void block_body_reduce(const BodyAcc<W> acc, int nbody, double* out, size_t nblk,
                                                  int lb, bool accumulate, double* lds /* [4][NB][W] */) {
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
  for (int b = 0; b < nbody; ++b) {
    double* o = lds + (wv * NB + b) * W;
    if (!__any(acc.id0 == b || acc.id1 == b)) {
      if (ln < W) o[ln] = 0.0;
      continue;
    }
    double s[W];
#pragma unroll
    for (int k = 0; k < W; ++k)
      s[k] = wave_total((acc.id0 == b ? acc.v0[k] : 0.0) + (acc.id1 == b ? acc.v1[k] : 0.0));
    if (ln == 0) {
#pragma unroll
      for (int k = 0; k < W; ++k) o[k] = s[k];
    }
  }
  __syncthreads();
  if (threadIdx.x < nbody * W) {
    const int b = threadIdx.x / W, k = threadIdx.x % W;
    double s = lds[(0 * NB + b) * W + k];
    s += lds[(1 * NB + b) * W + k];
    s += lds[(2 * NB + b) * W + k];
    s += lds[(3 * NB + b) * W + k];
    double* o = out + (size_t)(b * W + k) * nblk + lb;
    if (accumulate) *o += s;
    else *o = s;
  }
}

// Counter increments of a wavefront whose lanes mostly share counters in
// runs (particles in last step's cell order): each run of consecutive active
// lanes with the same counter index does one atomic add of its length, and
// its lanes take consecutive values.  Inactive lanes form the wave's tail.
// Returns this lane's value of the counter before its own increment.
__device__ __forceinline__ uint32_t run_atomic_inc(uint32_t* cnt, uint32_t r, bool act) {
  const int lane = threadIdx.x & (WAVE - 1);
  const uint32_t prev = (uint32_t)__shfl_up((int)r, 1, WAVE);
  const uint64_t heads = __ballot(act && (lane == 0 || prev != r));
  const int nact = __popcll(__ballot(act));
  const uint64_t below = lane == WAVE - 1 ? ~0ull : ((2ull << lane) - 1);
  const uint64_t upto = heads & below;
  const int h = upto ? 63 - __builtin_clzll(upto) : 0;
  const uint64_t above = heads & ~below;
  const int next = above ? __builtin_ctzll(above) : nact;
  uint32_t old = 0;
  if (act && h == lane) old = atomicAdd(&cnt[r], (uint32_t)(next - lane));
  old = (uint32_t)__shfl((int)old, h, WAVE);
  return old + (uint32_t)(lane - h);
}

// ---------------------------------------------------------------------------
// K: clear per-cell counters
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_clear(const SlotDesc* table, LaunchTab tab) {
  SLOT_PROLOGUE(DOM_CELL);
  const int c = lb * BLOCK + threadIdx.x;
  if (c < S.ncells) {
    S.cnt_f[c] = 0u;
    S.cnt_s[c] = 0u;
  }
}

// ---------------------------------------------------------------------------
// K: prescribed rigid rotation of the bodies at the step's time (Section 4:
// gears turn at fixed speed and temperature).  Angle omega*t from the FP64
// time; Rodrigues rotation about the unit axis.  Also bins the solid particle
// into its cell and stages its arrays for the gather.
// ---------------------------------------------------------------------------
template <class P>
__global__ __launch_bounds__(BLOCK) void k_pose(const SlotDesc* table, LaunchTab tab) {
#pragma clang fp contract(off)
  typedef typename P::Pos Pos;
  typedef typename P::Real Real;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  SLOT_PROLOGUE(DOM_SOLID);
  const int w = lb * BLOCK + threadIdx.x;
  const bool act = w < S.ns;
  uint32_t r = 0;
  if (act) {
  const int b = S.body[w];
  const double th = S.bom[b] * S.ctl->t;
  double sn, cs;
  sincos(th, &sn, &cs);
  const double* a = S.ba[b];
  const double* ctr = S.bc[b];
  const d4 x0 = gpc<d4>(S.x0)[w];
  const d4 n0 = gpc<d4>(S.n0)[w];
  const double u[3] = {x0.x - ctr[0], x0.y - ctr[1], x0.z - ctr[2]};
  const double n[3] = {n0.x, n0.y, n0.z};
  double ru[3], rn[3];
  {
    const double axu[3] = {a[1] * u[2] - a[2] * u[1], a[2] * u[0] - a[0] * u[2], a[0] * u[1] - a[1] * u[0]};
    const double au = a[0] * u[0] + a[1] * u[1] + a[2] * u[2];
    const double axn[3] = {a[1] * n[2] - a[2] * n[1], a[2] * n[0] - a[0] * n[2], a[0] * n[1] - a[1] * n[0]};
    const double an = a[0] * n[0] + a[1] * n[1] + a[2] * n[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ru[k] = u[k] * cs + axu[k] * sn + a[k] * au * (1.0 - cs);
      rn[k] = n[k] * cs + axn[k] * sn + a[k] * an * (1.0 - cs);
    }
  }
  const double om = S.bom[b];
  const double wa[3] = {om * a[0], om * a[1], om * a[2]};
  const double vw[3] = {wa[1] * ru[2] - wa[2] * ru[1], wa[2] * ru[0] - wa[0] * ru[2], wa[0] * ru[1] - wa[1] * ru[0]};
  Pos4 xp;
  xp.x = (Pos)(ctr[0] + ru[0]);
  xp.y = (Pos)(ctr[1] + ru[1]);
  xp.z = (Pos)(ctr[2] + ru[2]);
  xp.w = (Pos)0;
  Real4 nw, vv, lv;
  nw.x = (Real)rn[0]; nw.y = (Real)rn[1]; nw.z = (Real)rn[2]; nw.w = (Real)0;
  vv.x = (Real)vw[0]; vv.y = (Real)vw[1]; vv.z = (Real)vw[2]; vv.w = (Real)0;
  lv.x = (Real)ru[0]; lv.y = (Real)ru[1]; lv.z = (Real)ru[2]; lv.w = (Real)b;
  gp<Pos4>(S.xwb)[w] = xp;
  gp<Real4>(S.nwb)[w] = nw;
  gp<Real4>(S.vwb)[w] = vv;
  gp<Real4>(S.levb)[w] = lv;
  gp<d4>(S.x0b)[w] = x0;
  gp<d4>(S.n0b)[w] = n0;
  S.bodyb[w] = b;
  S.sidb[w] = S.sid[w];
  int c[3];
  if (!cell_coords<Pos>(S, xp.x, xp.y, xp.z, c)) raise_flag(S, F_DOMAIN);
  r = S.rank[cell_linear(S, c[0], c[1], c[2])];
  S.scell[w] = r;
  }
  run_atomic_inc(S.cnt_s, r, act);
}

// ---------------------------------------------------------------------------
// K: fold the drift into the FP64 anchor, stage the fluid arrays for the
// gather, bin into cells, and per-block max |v| for the time step.
// ---------------------------------------------------------------------------
template <class P>
__global__ __launch_bounds__(BLOCK) void k_fold(const SlotDesc* table, LaunchTab tab) {
  typedef typename P::Pos Pos;
  typedef typename P::Real Real;
  typedef typename P::Temp Temp;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  __shared__ double red[BLOCK / WAVE];
  SLOT_PROLOGUE(DOM_FLUID);
  const int i = lb * BLOCK + threadIdx.x;
  double vm = 0.0;
  uint32_t r = 0;
  if (i < S.nf) {
    Pos4 x = gpc<Pos4>(S.xa)[i];
    const Real4 d = gpc<Real4>(S.drift)[i];
    x.x += (Pos)d.x;
    x.y += (Pos)d.y;
    x.z += (Pos)d.z;
    gp<Pos4>(S.xa2)[i] = x;
    gp<Real4>(S.drift)[i] = Real4(0);
    const Real4 v = gpc<Real4>(S.vr)[i];
    gp<Real4>(S.vr2)[i] = v;
    gp<Real>(S.drho2)[i] = gpc<Real>(S.drho)[i];
    const Temp T = gpc<Temp>(S.T)[i];
    gp<Temp>(S.T2)[i] = T;
    S.fid2[i] = S.fid[i];
    if (S.mat) S.mat2[i] = S.mat[i];
    const bool finite = isfinite((double)x.x) && isfinite((double)x.y) && isfinite((double)x.z) &&
                        isfinite((double)v.x) && isfinite((double)v.y) && isfinite((double)v.z) &&
                        isfinite((double)v.w) && isfinite((double)T);
    if (!finite) raise_flag(S, F_NONFINITE);
    // |v| in FP64 from the stored components (eq. 25 takes the max)
    const double v0 = (double)v.x, v1 = (double)v.y, v2 = (double)v.z;
    vm = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
    int c[3];
    if (!cell_coords<Pos>(S, x.x, x.y, x.z, c)) raise_flag(S, F_DOMAIN);
    r = S.rank[cell_linear(S, c[0], c[1], c[2])];
    S.fcell[i] = r;
  }
  run_atomic_inc(S.cnt_f, r, i < S.nf);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vm = fmax(vm, __shfl_xor(vm, o, WAVE));
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = vm;
  __syncthreads();
  if (threadIdx.x == 0)
    S.vmax_part[lb] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// ---------------------------------------------------------------------------
// K: exclusive scan of per-cell counts (three phases: block sums, per-slot scan
// of the block sums, block-local scan plus offset).  Resets counts to serve as
// scatter cursors.
// ---------------------------------------------------------------------------
template <int NW = BLOCK / WAVE>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t& total) {
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    uint32_t y = __shfl_up(x, o, WAVE);
    if (ln >= o) x += y;
  }
  if (ln == WAVE - 1) lds[wv] = x;
  __syncthreads();
  uint32_t off = 0;
  total = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    off += k < wv ? lds[k] : 0u;
    total += lds[k];
  }
  __syncthreads();
  return off + x - v;
}

__global__ __launch_bounds__(BLOCK) void k_scan1(const SlotDesc* table, LaunchTab tab) {
  __shared__ uint32_t red[2][BLOCK / WAVE];
  SLOT_PROLOGUE(DOM_CELL);
  const int c = lb * BLOCK + threadIdx.x;
  uint32_t a = 0, b = 0;
  if (c < S.ncells) {
    a = S.cnt_f[c];
    b = S.cnt_s[c];
  }
  a = wave_sum_u(a);
  b = wave_sum_u(b);
  if (threadIdx.x % WAVE == 0) {
    red[0][threadIdx.x / WAVE] = a;
    red[1][threadIdx.x / WAVE] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    S.bsum_f[lb] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    S.bsum_s[lb] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
  }
}

__global__ __launch_bounds__(BLOCK) void k_scan2(const SlotDesc* table, LaunchTab tab) {
  __shared__ uint32_t lds[BLOCK / WAVE];
  SLOT_PROLOGUE(DOM_SLOT);
  (void)lb;
  const int n = S.nblk[DOM_CELL];
  const int ch = (n + BLOCK - 1) / BLOCK;
  const int b0 = threadIdx.x * ch;
  const int b1 = min(n, b0 + ch);
  for (int set = 0; set < 2; ++set) {
    uint32_t* bs = set ? S.bsum_s : S.bsum_f;
    uint32_t* st = set ? S.start_s : S.start_f;
    uint32_t s = 0;
    for (int k = b0; k < b1; ++k) s += bs[k];
    uint32_t total;
    uint32_t off = block_excl_scan(s, lds, total);
    for (int k = b0; k < b1; ++k) {
      uint32_t t = bs[k];
      bs[k] = off;
      off += t;
    }
    if (threadIdx.x == 0) st[S.ncells] = total;
    __syncthreads();
  }
}

__global__ __launch_bounds__(BLOCK) void k_scan3(const SlotDesc* table, LaunchTab tab) {
  __shared__ uint32_t lds[BLOCK / WAVE];
  SLOT_PROLOGUE(DOM_CELL);
  const int c = lb * BLOCK + threadIdx.x;
  const bool act = c < S.ncells;
  uint32_t a = act ? S.cnt_f[c] : 0u;
  uint32_t b = act ? S.cnt_s[c] : 0u;
  uint32_t ta, tb;
  const uint32_t pa = block_excl_scan(a, lds, ta);
  const uint32_t pb = block_excl_scan(b, lds, tb);
  if (act) {
    S.start_f[c] = S.bsum_f[lb] + pa;
    S.start_s[c] = S.bsum_s[lb] + pb;
    S.cnt_f[c] = 0u;
    S.cnt_s[c] = 0u;
  }
}

// ---------------------------------------------------------------------------
// K: counting-sort scatter; then each cell's run is ordered by original id,
// which makes the order the unique (Morton cell, id) order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_scatter(const SlotDesc* table, LaunchTab tab, int which) {
  SLOT_PROLOGUE(which ? DOM_SOLID : DOM_FLUID);
  const int n = which ? S.ns : S.nf;
  const int i = lb * BLOCK + threadIdx.x;
  const bool act = i < n;
  const uint32_t* cell = which ? S.scell : S.fcell;
  const uint32_t* start = which ? S.start_s : S.start_f;
  const uint32_t* id = which ? S.sidb : S.fid2;
  uint32_t* cnt = which ? S.cnt_s : S.cnt_f;
  uint64_t* key = which ? S.skey : S.fkey;
  const uint32_t r = act ? cell[i] : 0u;
  const uint32_t k = run_atomic_inc(cnt, r, act);
  if (act) key[start[r] + k] = (uint64_t)id[i] << 32 | (uint32_t)i;
}

// Orders each cell's run of keys (original id << 32 | staged index) by id and
// writes the staged indices in that order.  One thread per key position: the
// key's cell comes from its staged index, its rank in the cell is the number
// of the cell's keys below it (ids are unique, so the ranks are a
// permutation of the run), and its staged index goes to that place.  The
// lanes of a wavefront mostly share a cell, so the run's keys are read once
// per wavefront from cache, and the stores of a cell's permutation are
// contiguous.
__global__ __launch_bounds__(BLOCK) void k_cellsort(const SlotDesc* table, LaunchTab tab, int which) {
  SLOT_PROLOGUE(which ? DOM_SOLID : DOM_FLUID);
  const int n = which ? S.ns : S.nf;
  const int p = lb * BLOCK + threadIdx.x;
  if (p >= n) return;
  const uint64_t* key = which ? S.skey : S.fkey;
  const uint32_t* cell = which ? S.scell : S.fcell;
  const uint32_t* start = which ? S.start_s : S.start_f;
  uint32_t* perm = which ? S.sperm : S.fperm;
  const uint64_t kp = key[p];
  const uint32_t r = cell[(uint32_t)kp];
  const uint32_t b = start[r], e = start[r + 1];
  uint32_t rank = 0;
  for (uint32_t q = b; q < e; ++q) rank += key[q] < kp ? 1u : 0u;
  perm[b + rank] = (uint32_t)kp;
}

// A fluid particle's temperature and density rate side by side (16 bytes),
// so the fused first sub-step takes both of a neighbour's in one gather.
template <class P>
struct alignas(16) TempRate {
  typename P::Temp T;
  typename P::Real d;
};

// ---------------------------------------------------------------------------
// K: gather the staged arrays into cell-sorted order (fluid: also the
// (T, Drho) records)
// ---------------------------------------------------------------------------
template <class P>
__global__ __launch_bounds__(BLOCK) void k_reorder(const SlotDesc* table, LaunchTab tab, int which) {
  typedef typename P::Real Real;
  typedef typename P::Temp Temp;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  SLOT_PROLOGUE(which ? DOM_SOLID : DOM_FLUID);
  const int k = lb * BLOCK + threadIdx.x;
  if (!which) {
    if (k >= S.nf) return;
    const uint32_t s = S.fperm[k];
    gp<Pos4>(S.xa)[k] = gpc<Pos4>(S.xa2)[s];
    gp<Real4>(S.vr)[k] = gpc<Real4>(S.vr2)[s];
    const Real dr = gpc<Real>(S.drho2)[s];
    const Temp tk = gpc<Temp>(S.T2)[s];
    gp<Real>(S.drho)[k] = dr;
    gp<Temp>(S.T)[k] = tk;
    GLB TempRate<P>* td = gp<TempRate<P>>(S.td) + k;
    td->T = tk;
    td->d = dr;
    S.fid[k] = S.fid2[s];
    if (S.mat) S.mat[k] = S.mat2[s];
  } else {
    if (k >= S.ns) return;
    const uint32_t s = S.sperm[k];
    gp<d4>(S.x0)[k] = gpc<d4>(S.x0b)[s];
    gp<d4>(S.n0)[k] = gpc<d4>(S.n0b)[s];
    const Pos4 xp = gpc<Pos4>(S.xwb)[s];
    gp<Pos4>(S.xw)[k] = xp;
    int c[3];
    cell_coords<typename P::Pos>(S, xp.x, xp.y, xp.z, c);   // in the grid: checked by the pose
    gp<Real4>(S.so)[k] = cell_offset<P>(S, xp.x, xp.y, xp.z, c);
    Real4 nq = gpc<Real4>(S.nwb)[s];
    const Real4 vq = gpc<Real4>(S.vwb)[s];
    GLB Real* vk = gp<Real>(S.vw) + 4 * (int64_t)k;   // not the kernel sum beside it
    vk[0] = vq.x;
    vk[1] = vq.y;
    vk[2] = vq.z;
    nq.w = -dot_fma(nq.x, nq.y, nq.z, vq.x, vq.y, vq.z);
    gp<Real4>(S.nuw)[k] = nq;
    gp<Real4>(S.lev)[k] = gpc<Real4>(S.levb)[s];
    S.body[k] = S.bodyb[s];
    S.sid[k] = S.sidb[s];
  }
}

// ---------------------------------------------------------------------------
// K: neighbour rows (Section 2.8: neighbour lists and kernel quantities are
// refreshed once per advection step).  The cutoff test d^2 < (2h)^2 is FP64
// with d^2 = (dx dx + dy dy) + dz dz and no contraction.  Every particle also
// stores its cell-relative position, from which the sweeps form r_ij.
//
// Bound by the candidate loop's instructions: 1.9 M particles take 1014 us with
// the vector units 72 % busy at five waves per SIMD; numbering the candidates
// (STAGE) is 70 us of it.
//
// A wavefront holds 64 consecutive particles of the Morton order, i.e. runs
// of particles sharing a cell.  For each run the candidates of its 27-cell
// stencil are spread over the lanes in chunks of CB per lane, each candidate
// loaded once; for each chunk the run's particles are taken one at a time:
// each lane tests its candidates against the particle's position (broadcast
// from its lane into scalar registers), one ballot per candidate slot gives
// the hits, and the hit lanes write their indices to consecutive entries of
// the particle's row (particle-major, so a ballot's stores are contiguous;
// chunks of one run append in candidate order).  Every test is one
// of the particle's own stencil, and no lane waits on another's hits.  A row
// lists the stencil's cells in a fixed order, indices ascending within a
// cell.  At the end each lane moves its particle's row (still in cache) into
// the SELL layout the sweeps read, with stores contiguous across the wave.
// ---------------------------------------------------------------------------
// Wendland C2 weight W = kW (1 - q/2)^4 (1 + 2q), q = |r|/h, from d^2 in FP64.
// |r| comes from the hardware reciprocal square root refined by coupled
// Newton steps for sqrt(x) and 1/(2 sqrt(x)) (Goldschmidt's iteration) and a
// final residual correction, which leaves an error of about one ulp.
__device__ __forceinline__ double kernel_W_d2(double d2, double inv_h, double kW) {
  const double x = d2 > 0.0 ? d2 : 1.0;
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, hh = 0.5 * y;
  const double e = fma(-hh, g, 0.5);
  g = fma(g, e, g);
  hh = fma(hh, e, hh);
  const double res = fma(-g, g, x);
  g = fma(res, hh, g);
  const double q = (d2 > 0.0 ? g : 0.0) * inv_h;
  const double t = 1.0 - 0.5 * q;
  return kW * t * t * t * t * (1.0 + 2.0 * q);
}

// Exclusive prefix sum over the wavefront's lanes; *total receives the sum.
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t* total) {
  const int lane = threadIdx.x & (WAVE - 1);
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, d, WAVE);
    if (lane >= d) x += y;
  }
  *total = (uint32_t)__builtin_amdgcn_readlane((int)x, WAVE - 1);
  return x - v;
}

// LDS written by some lanes of a wavefront, then read by others
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Candidates of one run's stencil against the run's particles [L, R) of the
// wave.  pre/beg: per stencil cell (27) the prefix of candidate counts and the
// first index; lcl (LOCAL): the row entry of its first particle.  Hits of
// particle p go to its row, counted in lane p's cnt: sorted indices, or (LOCAL)
// entries of staged rows; own: this lane's particle as such an entry.
// candidate slots per lane: four keeps the build at five waves per SIMD (82
// registers with the numbering, 78 and six waves without); eight (four waves) was
// 3 % slower
constexpr int CB = 4;
template <bool LOCAL, class Pos, class Pos4>
__device__ __forceinline__ void run_candidates(const GLB Pos4* x, const uint32_t* pre, const uint32_t* beg,
                                               const uint32_t* lcl, uint32_t M, int L, int R, int wbase, Pos xi,
                                               Pos yi, Pos zi, double cut2, GLB uint32_t* rows, int kr, int off,
                                               int cap, int& cnt, uint32_t own) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & (WAVE - 1);
  for (uint32_t b0 = 0; b0 < M; b0 += (uint32_t)(WAVE * CB)) {
    Pos cx[CB], cy[CB], cz[CB];
    uint32_t cj[CB];
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const uint32_t m = b0 + (uint32_t)(u * WAVE + lane);
      cj[u] = 0xffffffffu;
      cx[u] = cy[u] = cz[u] = (Pos)1e30;   // far: never a hit
      if (m < M) {
        int q = 0;
#pragma unroll
        for (int st = 16; st > 0; st >>= 1)
          if (q + st < 27 && pre[q + st] <= m) q += st;
        const uint32_t j = beg[q] + (m - pre[q]);
        const Pos4 pj = x[j];
        cj[u] = LOCAL ? lcl[q] + 16u * (m - pre[q]) : j;
        cx[u] = pj.x;
        cy[u] = pj.y;
        cz[u] = pj.z;
      }
    }
    const int nu = (int)min((uint32_t)CB, (M - b0 + WAVE - 1) / WAVE);
    for (int p = L; p < R; ++p) {
      const Pos px = rl(xi, p), py = rl(yi, p), pz = rl(zi, p);
      const uint32_t ip = (uint32_t)__builtin_amdgcn_readlane((int)own, p);
      int c = __builtin_amdgcn_readlane(cnt, p);
      GLB uint32_t* row = rows + (int64_t)(wbase + p) * kr + off;
#pragma unroll
      for (int u = 0; u < CB; ++u) {
        if (u >= nu) break;
        const Pos ddx = px - cx[u], ddy = py - cy[u], ddz = pz - cz[u];
        const Pos s2 = ddx * ddx + ddy * ddy;
        const Pos d2 = s2 + ddz * ddz;
        const bool hit = (double)d2 < cut2 && cj[u] != ip;
        const uint64_t mask = __ballot(hit);
        if (hit) {
          const int k = c + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
          if (k < cap) row[k] = cj[u];
        }
        c += __popcll(mask);
      }
      if (lane == p) cnt = c;
    }
  }
}

// The block's candidate cells (BlkHead, BlkItem).  home: the distinct cells of
// the block's particles in order (runs); entry r * 27 + q is cell q of run r's
// stencil.  A cell is numbered where it first appears, so the numbering needs
// no atomics and is the same every time: an entry looks for the first earlier
// run whose stencil holds its cell (a few tens of runs, 16 on the lattice).
constexpr int MAXRUN = 64;
constexpr uint16_t NO_ITEM = 0xffffu, ITEM_REF = 0x8000u;   // no particles; covered by entry (value & 0x7fff)
constexpr int WIDE = 4 * BLOCK;  // threads per block of the widest build
struct RunTab {
  uint32_t runs[BLOCK / WAVE];
};
struct StageTab : RunTab {
  uint32_t home[MAXRUN];
  uint16_t id[2][27 * MAXRUN];       // the entry's item: fluid, solid
  BlkItem item[2][STAGE_ITEMS];
  uint32_t scan[WIDE / WAVE], last[BLOCK / WAVE];
  int cont1;                         // wavefront 1 starts within a run
};

// Fills the table for the runs [r0, r1) and writes the block's head, with the
// given wavefronts staged, and list; returns whether the candidates fit.
template <int NT>
__device__ __forceinline__ bool block_candidates(const SlotDesc& S, StageTab& tb, int lb, int r0, int r1, int waves) {
  const GLB uint32_t* rank = gpc<uint32_t>(S.rank);
  const GLB uint32_t* st[2] = {gpc<uint32_t>(S.start_f), gpc<uint32_t>(S.start_s)};
  const int n = 27 * r1;
  uint32_t done[2] = {0u, 0u};       // (cells << 21) | candidates numbered so far
  bool big = false;
  for (int i0 = 27 * r0; i0 < n; i0 += NT) {
    const int it = i0 + (int)threadIdx.x;
    uint32_t f0[2] = {0u, 0u}, cnt[2] = {0u, 0u};
    int ref = -1;
    if (it < n) {
      const int r = it / 27, q = it - 27 * r;
      const uint32_t hc = tb.home[r];
      const int x = (int)(hc & 1023u) + q % 3 - 1, y = (int)((hc >> 10) & 1023u) + (q / 3) % 3 - 1,
                z = (int)(hc >> 20) + q / 9 - 1;
      if (x >= 0 && y >= 0 && z >= 0 && x < S.dims[0] && y < S.dims[1] && z < S.dims[2]) {
        for (int p = r0; p < r; ++p) {
          const uint32_t h = tb.home[p];
          const uint32_t dx = (uint32_t)(x - (int)(h & 1023u) + 1), dy = (uint32_t)(y - (int)((h >> 10) & 1023u) + 1),
                         dz = (uint32_t)(z - (int)(h >> 20) + 1);
          if (dx <= 2u && dy <= 2u && dz <= 2u) {
            ref = p * 27 + (int)(dz * 9 + dy * 3 + dx);
            break;
          }
        }
        if (ref < 0) {
          const uint32_t rk = rank[cell_linear(S, x, y, z)];
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            f0[a] = st[a][rk];
            cnt[a] = st[a][rk + 1] - f0[a];
            if (cnt[a] > 1023u) {
              cnt[a] = 1023u;
              big = true;
            }
          }
        }
      }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      uint32_t total;
      const uint32_t at = done[a] + block_excl_scan<NT / WAVE>((cnt[a] ? 1u << 21 : 0u) + cnt[a], tb.scan, total);
      done[a] += total;
      const uint32_t e = at >> 21;
      if (it < n) tb.id[a][it] = ref >= 0 ? (uint16_t)(ITEM_REF | ref) : cnt[a] ? (uint16_t)e : NO_ITEM;
      if (cnt[a] && e < (uint32_t)STAGE_ITEMS) tb.item[a][e] = BlkItem{f0[a], (uint16_t)at, (uint16_t)cnt[a]};
    }
  }
  const int nc[2] = {(int)(done[0] & 0x1fffffu), (int)(done[1] & 0x1fffffu)};
  const int ni[2] = {(int)(done[0] >> 21), (int)(done[1] >> 21)};
  const int ns0 = (nc[0] + WAVE - 1) / WAVE * WAVE, nt = ns0 + nc[1];
  const bool ok = !__syncthreads_or(big) && nt <= STAGE_CAP && ni[0] < STAGE_ITEMS && ni[1] < STAGE_ITEMS;
  if (!ok) return false;
  if (threadIdx.x == 0) S.bhead[lb] = BlkHead{nt, ns0, waves, 0};
  uint32_t* list = S.blist + (int64_t)lb * S.list_len;
  if (nc[0] + (int)threadIdx.x < ns0) list[nc[0] + threadIdx.x] = 0u;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    if (a && (int)threadIdx.x < ni[1]) tb.item[1][threadIdx.x].base += (uint16_t)ns0;
    for (int it = 27 * r0 + threadIdx.x; it < n; it += NT) {
      const uint16_t v = tb.id[a][it];
      if (v != NO_ITEM && (v & ITEM_REF)) tb.id[a][it] = tb.id[a][v & 0x7fffu];
    }
  }
  __syncthreads();
  // the list, sixteen lanes per cell
#pragma unroll
  for (int a = 0; a < 2; ++a)
    for (int e = threadIdx.x >> 4; e < ni[a]; e += NT / 16) {
      const BlkItem x = tb.item[a][e];
      for (int k = threadIdx.x & 15; k < x.cnt; k += 16) list[x.base + k] = x.start + (uint32_t)k;
    }
  return true;
}

// NT threads build the rows of BLOCK particles: one thread per particle, each
// wavefront with its own particles' runs, or (WIDE, WIDE / 2) four or two, so
// that as many times the wavefronts share the block's runs.
template <class P, int NT, bool STAGE>
__global__ __launch_bounds__(NT) void k_build(const SlotDesc* table, LaunchTab tab) {
#pragma clang fp contract(off)
  typedef typename P::Pos Pos;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  __shared__ uint32_t lr_all[NT / WAVE][6][32];
  __shared__ typename std::conditional<STAGE, StageTab, RunTab>::type tb;
  // the wavefronts' runs: first particle, cell, run of the block; per particle:
  // row lengths, its own row entry
  __shared__ uint16_t seg_first[BLOCK + 1], seg_run[BLOCK], len[2][BLOCK];
  __shared__ uint32_t seg_cell[BLOCK], own_entry[BLOCK];
  SLOT_FIND(DOM_FLUID);
  if (!live_block(S)) return;
  const int nf = S.nf;
  const int i = lb * BLOCK + threadIdx.x;
  const bool act = threadIdx.x < BLOCK && i < nf;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wv = threadIdx.x / WAVE;
  const GLB Pos4* xa = gpc<Pos4>(S.xa);
  const GLB Pos4* xw = gpc<Pos4>(S.xw);
  uint32_t pc = 0u;
  if (threadIdx.x < BLOCK) {
    const Pos4 x = xa[min(i, nf - 1)];
    int c[3];
    cell_coords<Pos>(S, x.x, x.y, x.z, c);
    if (act) gp<Real4>(S.xo)[i] = cell_offset<P>(S, x.x, x.y, x.z, c);
    pc = pack_cell(c);
  }
  const double cut2 = S.cut2;
  const int kf = S.kf, ks = S.ks;
  // runs of equal cells among each wavefront's particles
  const uint32_t prevc = (uint32_t)__shfl_up((int)pc, 1, WAVE);
  const uint64_t runs = __ballot(act && (lane == 0 || prevc != pc));
  const uint64_t upto = lane == WAVE - 1 ? ~0ull : (2ull << lane) - 1;
  if (wv < BLOCK / WAVE && lane == WAVE - 1) {
    tb.runs[wv] = (uint32_t)__popcll(runs);
    if constexpr (STAGE) tb.last[wv] = pc;
  }
  __syncthreads();
  int nseg = 0, seg = __popcll(runs & upto) - 1, seg0 = 0;   // seg0: the wavefront's own first run
  for (int w = 0; w < BLOCK / WAVE; ++w) {
    if (w < wv) seg0 += (int)tb.runs[w];
    nseg += (int)tb.runs[w];
  }
  seg += seg0;
  const bool head = (runs >> lane) & 1;
  if (head) {
    seg_first[seg] = (uint16_t)threadIdx.x;
    seg_cell[seg] = pc;
  }
  if (threadIdx.x == 0) seg_first[nseg] = (uint16_t)min(BLOCK, nf - lb * BLOCK);
  int waves = 0;   // the particles' wavefronts that are staged
  if constexpr (STAGE) {
    // the block's runs, numbered: a wavefront's first one may continue the last one's
    const bool cont = wv > 0 && wv < BLOCK / WAVE && tb.last[max(wv - 1, 0)] == (uint32_t)__builtin_amdgcn_readlane((int)pc, 0);
    const uint64_t heads = cont ? runs & ~1ull : runs;
    if (wv < BLOCK / WAVE && lane == 0) tb.scan[wv] = (uint32_t)__popcll(heads);
    if (threadIdx.x == WAVE) tb.cont1 = cont;
    __syncthreads();
    int run = __popcll(heads & upto) - 1, nruns = 0, cut1 = 0, cut3 = 0;   // cut1, cut3: runs that start in wavefront 0, in 0 to 2
    for (int w = 0; w < BLOCK / WAVE; ++w) {
      if (w == 1) cut1 = nruns;
      if (w == 3) cut3 = nruns;
      if (w < wv) run += (int)tb.scan[w];
      nruns += (int)tb.scan[w];
    }
    if (head) seg_run[seg] = (uint16_t)run;
    if (nruns <= MAXRUN) {
      if ((heads >> lane) & 1) tb.home[run] = pc;
      __syncthreads();
      // all four wavefronts, or the first or the last three
#pragma unroll 1
      for (int a = 0; a < 3 && !waves; ++a) {
        const int want = a == 0 ? 15 : a == 1 ? 7 : 14;
        if (block_candidates<NT>(S, tb, lb, a == 2 ? cut1 - tb.cont1 : 0, a == 1 ? cut3 : nruns, want)) waves = want;
      }
    }
  }
  if (S.bhead && waves == 0 && threadIdx.x == 0) S.bhead[lb] = BlkHead{0, 0, 0, 0};
  __syncthreads();
  GLB uint32_t* rows = gp<uint32_t>(S.rmaj);
  const GLB uint32_t* rank = gpc<uint32_t>(S.rank);
  const GLB uint32_t* stf = gpc<uint32_t>(S.start_f);
  const GLB uint32_t* sts = gpc<uint32_t>(S.start_s);
  uint32_t (*lr)[32] = lr_all[wv];
  uint32_t *preF = lr[0], *preS = lr[1], *begF = lr[2], *begS = lr[3], *lclF = lr[4], *lclS = lr[5];
  // this lane's offset in a 27-cell stencil
  const int ox = lane % 3 - 1, oy = (lane / 3) % 3 - 1, oz = lane / 9 - 1;
  const int segs = (int)__popcll(runs);
  for (int k = NT > BLOCK ? wv : seg0; k < (NT > BLOCK ? nseg : seg0 + segs); k += NT > BLOCK ? NT / WAVE : 1) {
    const int first = __builtin_amdgcn_readfirstlane((int)seg_first[k]);
    const int R = __builtin_amdgcn_readfirstlane((int)seg_first[k + 1]) - first;
    const uint32_t cell = (uint32_t)__builtin_amdgcn_readfirstlane((int)seg_cell[k]);
    const bool staged = STAGE && ((waves >> (first / WAVE)) & 1);
    const int wbase = lb * BLOCK + first;
    const int q = wbase + min(lane, R - 1);
    const Pos4 xq = xa[q];
    uint32_t own = (uint32_t)q;
    uint32_t f0 = 0, f1 = 0, s0 = 0, s1 = 0, lf = 0, ls = 0;
    if (staged) {
      if constexpr (STAGE) {
        const int e = 27 * __builtin_amdgcn_readfirstlane((int)seg_run[k]);
        const BlkItem h = tb.item[0][tb.id[0][e + 13]];
        own = 16u * (h.base + (uint32_t)q - h.start) | 4u * 13u << 16;
        if (lane < 27) {
          const uint32_t a = tb.id[0][e + lane], b = tb.id[1][e + lane];
          if (a != NO_ITEM) {
            const BlkItem x = tb.item[0][a];
            f0 = x.start;
            f1 = f0 + x.cnt;
            lf = x.base;
          }
          if (b != NO_ITEM) {
            const BlkItem x = tb.item[1][b];
            s0 = x.start;
            s1 = s0 + x.cnt;
            ls = x.base;
          }
        }
      }
    } else {
      const int nx = (int)(cell & 1023u) + ox, ny = (int)((cell >> 10) & 1023u) + oy, nz = (int)(cell >> 20) + oz;
      if (lane < 27 && nx >= 0 && ny >= 0 && nz >= 0 && nx < S.dims[0] && ny < S.dims[1] && nz < S.dims[2]) {
        const uint32_t r = rank[cell_linear(S, nx, ny, nz)];
        f0 = stf[r];
        f1 = stf[r + 1];
        s0 = sts[r];
        s1 = sts[r + 1];
      }
    }
    uint32_t Mf, Ms;
    const uint32_t pf = wave_excl_scan(f1 - f0, &Mf);
    const uint32_t ps = wave_excl_scan(s1 - s0, &Ms);
    if (lane < 27) {
      preF[lane] = pf;
      begF[lane] = f0;
      preS[lane] = ps;
      begS[lane] = s0;
      lclF[lane] = 16u * lf | 4u * (uint32_t)lane << 16;
      lclS[lane] = 16u * ls | 4u * (uint32_t)lane << 16;
    }
    wave_lds_sync();
    const uint32_t none = 0xfffffffeu;   // no solid candidate is the particle itself
    int cf = 0, cs = 0;
    if (staged) {
      run_candidates<true, Pos>(xa, preF, begF, lclF, Mf, 0, R, wbase, xq.x, xq.y, xq.z, cut2, rows, kf + ks, 0, kf, cf, own);
      if (Ms)
        run_candidates<true, Pos>(xw, preS, begS, lclS, Ms, 0, R, wbase, xq.x, xq.y, xq.z, cut2, rows, kf + ks, kf, ks, cs, none);
    } else {
      run_candidates<false, Pos>(xa, preF, begF, nullptr, Mf, 0, R, wbase, xq.x, xq.y, xq.z, cut2, rows, kf + ks, 0, kf, cf, own);
      if (Ms)
        run_candidates<false, Pos>(xw, preS, begS, nullptr, Ms, 0, R, wbase, xq.x, xq.y, xq.z, cut2, rows, kf + ks, kf, ks, cs,
                                   none);
    }
    if (lane < R) {
      own_entry[first + lane] = own;
      len[0][first + lane] = (uint16_t)min(cf, 0xffff);
      len[1][first + lane] = (uint16_t)min(cs, 0xffff);
    }
    wave_lds_sync();
  }
  if (NT > BLOCK) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  // move the rows (written by the block's lanes, still in cache) into the SELL
  // layout: entry k of a wavefront's particles lands contiguous
  const int p = threadIdx.x % BLOCK, part = threadIdx.x / BLOCK;
  const int ip = lb * BLOCK + p;
  if (ip >= nf) return;
  int cf = len[0][p], cs = len[1][p];
  if (part == 0) {
    if (cf > kf || cs > ks) raise_flag(S, F_CAPACITY);
    S.nfc[ip] = (uint32_t)min(cf, kf);
    S.nsc[ip] = (uint32_t)min(cs, ks);
  }
  cf = min(cf, kf);
  cs = min(cs, ks);
  const uint32_t own = own_entry[p];
  const bool staged = STAGE && ((waves >> (p / WAVE)) & 1);
  constexpr int STEP = 4 * (NT / BLOCK);
  const GLB uint32_t* RM = rows + (int64_t)ip * (kf + ks);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int cap = a ? ks : kf, n = a ? cs : cf;
    GLB uint32_t* dst = gp<uint32_t>(a ? S.srec : S.nrec) + (int64_t)(ip >> 6) * cap * WAVE;
    if (a) RM += kf;
    if (staged) {
      // groups of four entries, filled up with the particle itself to a multiple
      // of eight, and to eight at least: the sweeps fetch a row's first eight
      // neighbours before they look at its length
      GLB u4* G = (GLB u4*)dst + lane;
      for (int k = 4 * part; k < max(8, (n + 7) & ~7); k += STEP) {
        u4 e = *(const GLB u4*)(RM + k);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k + u >= n) e[u] = own;
        G[(int64_t)(k >> 2) * WAVE] = e;
      }
    } else {
      GLB uint32_t* RS = dst + lane;
      for (int k = 4 * part; k < n; k += STEP) {
        const u4 e = *(const GLB u4*)(RM + k);
        const uint32_t ev[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k + u < n) RS[(int64_t)(k + u) * WAVE] = ev[u];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// K: kernel sum over the fresh rows, self included (Section 2.4), in FP64
// from the anchors, and the density re-initialisation against the
// perfect-lattice sum S0 (eq. 14 with a free surface, eq. 15 without).  Each
// pair's d^2 is formed exactly as in the cutoff test; the rows are walked in
// order (fluid, then solid) so the sum is reproducible.
// ---------------------------------------------------------------------------
template <class P, bool STAGE>
__global__ __launch_bounds__(BLOCK) void k_sumw(const SlotDesc* table, LaunchTab tab) {
#pragma clang fp contract(off)
  typedef typename P::Pos Pos;
  typedef typename P::Real Real;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  // anchors of the staged candidates (three arrays of coordinates in FP64
  // positions, records in FP32), or the window of the gathering rows
  constexpr int STAGE_BYTES = STAGE ? STAGE_CAP * (sizeof(Pos) == 8 ? 24 : 16) : 0;
  constexpr int SMEM = STAGE_BYTES > WIN * (int)sizeof(Pos4) ? STAGE_BYTES : WIN * (int)sizeof(Pos4);
  __shared__ __attribute__((aligned(32))) char smem[SMEM];
  SLOT_FIND(DOM_FLUID);
  const int i = lb * BLOCK + threadIdx.x;
  const int ii = min(i, S.nf - 1);
  const GLB Pos4* xa = gpc<Pos4>(S.xa);
  const GLB Pos4* xw = gpc<Pos4>(S.xw);
  BlkHead hd;
  StageList sl;
  if constexpr (STAGE) {
    hd = blk_head(S, lb);
    sl = stage_list(S, lb);
  }
  const Pos4 xi4 = xa[ii];
  const int nn = (int)S.nfc[ii], nw = (int)S.nsc[ii];
  if (!live(S)) return;
  const bool staged = STAGE && wave_staged(hd, wave_id());   // this wavefront's rows
  Pos4* wxa = (Pos4*)smem;
  const bool block_gathers = !STAGE || hd.n == 0;
  const Window win = block_gathers ? window_of(lb, S.nf) : Window{0, 0};
  Row8 ef{u4(0), u4(0)}, ew{u4(0), u4(0)};
  if constexpr (STAGE) {
    if (hd.n > 0) {
      if (staged) {
        ef = row_load(row_groups(S, ii), 0);
        ew = row_load(wall_groups(S, ii), 0);
      }
      stage_block(
          hd, sl, [&](bool sol, uint32_t j) { return (sol ? xw : xa)[j]; },
          [&](uint32_t l, const Pos4& x, uint32_t) {
            if constexpr (sizeof(Pos) == 8) {
              Pos* X = (Pos*)smem;
              X[l] = x.x;
              X[STAGE_CAP + l] = x.y;
              X[2 * STAGE_CAP + l] = x.z;
            } else {
              wxa[l] = x;
            }
          });
    }
  }
  if (block_gathers) {
    stage_window(wxa, xa, win);
    __syncthreads();
  }
  if (i >= S.nf) return;
  const Pos xi = xi4.x, yi = xi4.y, zi = xi4.z;
  const double inv_h = 1.0 / S.h, kW = S.kW;
  double sw = kW;   // W(0)
  const int lane = i & (WAVE - 1);
  const int64_t slice = i >> 6;
  auto add = [&](const Pos xj, const Pos yj, const Pos zj, bool real) {
    const Pos ddx = xi - xj, ddy = yi - yj, ddz = zi - zj;
    const Pos s2 = ddx * ddx + ddy * ddy;
    const Pos d2 = s2 + ddz * ddz;
    const double w = kernel_W_d2((double)d2, inv_h, kW);
    if (real) sw += w;
  };
  if (staged) {
    // the fluid row, then the wall row, of the staged candidates
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const GLB u4* G = a ? wall_groups(S, i) : row_groups(S, i);
      Row8 r = a ? ew : ef;
      const int n = a ? nw : nn;
      auto group = [&](int k, auto whole) {
        uint32_t e[8];
        row_entries(r, e);
        if (k + 8 < n) r = row_load(G, k + 8);
        Pos x[8], y[8], z[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if constexpr (sizeof(Pos) == 8) {
            const char* q = smem + ((e[u] & 0xffffu) >> 1);
            x[u] = *(const Pos*)q;
            y[u] = *(const Pos*)(q + 8 * STAGE_CAP);
            z[u] = *(const Pos*)(q + 16 * STAGE_CAP);
          } else {
            const Pos4 o = *(const Pos4*)(smem + (e[u] & 0xffffu));
            x[u] = o.x;
            y[u] = o.y;
            z[u] = o.z;
          }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) add(x[u], y[u], z[u], decltype(whole)::value || k + u < n);
      };
      int k = 0;
      for (; k + 8 <= n; k += 8) group(k, std::true_type{});
      if (k < n) group(k, std::false_type{});
    }
  } else {
    const GLB uint32_t* R = gpc<uint32_t>(S.nrec) + slice * (int64_t)S.kf * WAVE + lane;
    uint32_t jn[ROW_UNROLL];
#pragma unroll
    for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)u * WAVE);
    for (int k = 0; k < nn; k += ROW_UNROLL) {
      Pos4 xj[ROW_UNROLL];
#pragma unroll
      for (int u = 0; u < ROW_UNROLL; ++u) xj[u] = win_get(wxa, xa, k + u < nn ? jn[u] : (uint32_t)i, win);
      if (k + ROW_UNROLL < nn) {
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)(k + ROW_UNROLL + u) * WAVE);
      }
#pragma unroll
      for (int u = 0; u < ROW_UNROLL; ++u) add(xj[u].x, xj[u].y, xj[u].z, k + u < nn);
    }
  }
  GLB Real4* vr = gp<Real4>(S.vr);
  Real4 v = vr[i];
  const double dp3 = S.dp * S.dp * S.dp;
  if (!staged) {
    const int n = nw;
    const GLB uint32_t* R = gpc<uint32_t>(S.srec) + slice * (int64_t)S.ks * WAVE + lane;
    uint32_t wn[SOLID_UNROLL];
#pragma unroll
    for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)u * WAVE);
    for (int k = 0; k < n; k += SOLID_UNROLL) {
      Pos4 xq[SOLID_UNROLL];
#pragma unroll
      for (int u = 0; u < SOLID_UNROLL; ++u) xq[u] = xw[k + u < n ? wn[u] : 0u];
      if (k + SOLID_UNROLL < n) {
#pragma unroll
        for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)(k + SOLID_UNROLL + u) * WAVE);
      }
#pragma unroll
      for (int u = 0; u < SOLID_UNROLL; ++u) add(xq[u].x, xq[u].y, xq[u].z, k + u < n);
    }
  }
  S.sumW[i] = sw;
  const double rre = S.rho0 * (dp3 * sw) / S.S0;
  const double rcur = P::kRel ? S.rho0 + (double)v.w : (double)v.w;
  const double rn = S.free_surface ? fmax(rcur, rre) : rre;
  v.w = P::kRel ? (Real)(rn - S.rho0) : (Real)rn;
  vr[i] = v;
}

// ---------------------------------------------------------------------------
// K: dummy velocity of every solid particle for the wall viscous force
// (eq. 18 with the generalized wall of Section 2.5): v_w = 2 u_w - v~_w, with
// v~_w = (sum_j W_wj v_j) / (sum_j W_wj) the Shepard mean of the step-start
// velocity of the fluid within 2h (the rigid velocity u_w when there is none,
// or with the literal reading of eq. 18).
//
// Solid-centric, with the neighbour build's traversal: a wavefront holds 64
// consecutive solid particles of the Morton order; for each run sharing a
// cell, the fluid candidates of its 27-cell stencil are spread over the lanes
// in chunks of CBW per lane (cell-relative position and velocity loaded
// once); for each chunk the run's particles are taken in turn, every lane
// sums W and W v over its candidates within 2h, and four wave reductions in a
// fixed order add the chunk's share to the particle's sums.  The arithmetic is that of the interaction sweeps (FP32 in
// mixed precision, pair vectors from the frozen cell-relative positions): a
// pair that this test and the FP64 cutoff test of the rows decide differently
// lies within a few ulps of 2h, where W is below 1e-25 W(0).  No atomics: the
// result depends only on the sorted order, so it is the same alone or batched.
// It runs beside the kernel sums, which rewrite only the density component of
// the velocity records read here.
// ---------------------------------------------------------------------------
// candidate slots per lane of the dummy-velocity sweep: four (six waves per
// SIMD) against eight (three waves) took it from 0.29 to 0.20 ms
constexpr int CBW = 4;
template <class P, int NT>
__global__ __launch_bounds__(NT) void k_wallvel(const SlotDesc* table, LaunchTab tab) {
  typedef typename P::Real Real;
  typedef typename P::Real4 Real4;
  __shared__ uint32_t lds_pre[NT / WAVE][32];
  __shared__ uint32_t lds_beg[NT / WAVE][32];
  // WIDE: the block's runs, shared by all wavefronts, and their sums
  __shared__ uint32_t seg_runs[BLOCK / WAVE];
  __shared__ uint16_t seg_first[NT > BLOCK ? BLOCK + 1 : 1];
  __shared__ Real sums[NT > BLOCK ? 4 : 1][NT > BLOCK ? BLOCK : 1];
  SLOT_PROLOGUE(DOM_SOLID);
  const int w = lb * BLOCK + threadIdx.x;
  const int ns = S.ns;
  const bool act = threadIdx.x < BLOCK && w < ns;
  const int ww = act ? w : ns - 1;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wv = threadIdx.x / WAVE;
  const Real4 u = gpc<Real4>(S.vw)[ww];
  // sums of this lane's solid particle: W v (3) and W
  Real acc[4] = {(Real)0, (Real)0, (Real)0, (Real)0};
  if (!S.wall_rigid) {
    const GLB Real4* xo = gpc<Real4>(S.xo);
    const GLB Real4* vr = gpc<Real4>(S.vr);
    const GLB uint32_t* rank = gpc<uint32_t>(S.rank);
    const GLB uint32_t* stf = gpc<uint32_t>(S.start_f);
    const GLB Real4* so = gpc<Real4>(S.so);
    Real4 ow = so[ww];
    const uint32_t cw = unpack_index(ow.w);
    const Real cut2 = (Real)S.cut2, inv_h = (Real)(1.0 / S.h), kW = (Real)S.kW, csr = (Real)S.cs_r;
    uint32_t* pre = lds_pre[wv];
    uint32_t* beg = lds_beg[wv];
    const uint32_t prevc = (uint32_t)__shfl_up((int)cw, 1, WAVE);
    const int nact = __popcll(__ballot(act));
    uint64_t runs = __ballot(act && (lane == 0 || prevc != cw));
    int nseg = 0;
    if (NT > BLOCK) {
      if (wv < BLOCK / WAVE && lane == 0) seg_runs[wv] = (uint32_t)__popcll(runs);
      __syncthreads();
      int seg = __popcll(runs & (lane == WAVE - 1 ? ~0ull : (2ull << lane) - 1)) - 1;
      for (int k = 0; k < BLOCK / WAVE; ++k) {
        if (k < wv) seg += (int)seg_runs[k];
        nseg += (int)seg_runs[k];
      }
      if ((runs >> lane) & 1) seg_first[seg] = (uint16_t)threadIdx.x;
      if (threadIdx.x == 0) seg_first[nseg] = (uint16_t)min(BLOCK, ns - lb * BLOCK);
      __syncthreads();
    }
    const int ox = lane % 3 - 1, oy = (lane / 3) % 3 - 1, oz = lane / 9 - 1;
    for (int k = wv; NT > BLOCK ? k < nseg : runs != 0; k += NT / WAVE) {
      // the run's particles: lanes [L, R)
      int L, R, first = 0;
      if (NT > BLOCK) {
        first = __builtin_amdgcn_readfirstlane((int)seg_first[k]);
        L = 0;
        R = __builtin_amdgcn_readfirstlane((int)seg_first[k + 1]) - first;
        ow = so[lb * BLOCK + first + min(lane, R - 1)];
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] = (Real)0;
      } else {
        L = __builtin_ctzll(runs);
        runs &= runs - 1;
        R = runs ? __builtin_ctzll(runs) : nact;
      }
      const uint32_t cl = (uint32_t)__builtin_amdgcn_readlane((int)unpack_index(ow.w), L);
      const int nx = (int)(cl & 1023u) + ox, ny = (int)((cl >> 10) & 1023u) + oy, nz = (int)(cl >> 20) + oz;
      const bool valid = lane < 27 && nx >= 0 && ny >= 0 && nz >= 0 && nx < S.dims[0] && ny < S.dims[1] &&
                         nz < S.dims[2];
      uint32_t f0 = 0, f1 = 0;
      if (valid) {
        const uint32_t r = rank[cell_linear(S, nx, ny, nz)];
        f0 = stf[r];
        f1 = stf[r + 1];
      }
      uint32_t M;
      const uint32_t pf = wave_excl_scan(f1 - f0, &M);
      if (lane < 27) {
        pre[lane] = pf;
        beg[lane] = f0;
      }
      wave_lds_sync();
      for (uint32_t b0 = 0; b0 < M; b0 += (uint32_t)(WAVE * CBW)) {
        Real4 co[CBW], cv[CBW];
#pragma unroll
        for (int k = 0; k < CBW; ++k) {
          const uint32_t m = b0 + (uint32_t)(k * WAVE + lane);
          co[k] = Real4((Real)1e30);   // far: never within 2h
          co[k].w = pack_index(0u, (Real)0);
          cv[k] = Real4((Real)0);
          if (m < M) {
            int qq = 0;
#pragma unroll
            for (int st = 16; st > 0; st >>= 1)
              if (qq + st < 27 && pre[qq + st] <= m) qq += st;
            const uint32_t j = beg[qq] + (m - pre[qq]);
            co[k] = xo[j];
            cv[k] = vr[j];
          }
        }
        const int nu = (int)min((uint32_t)CBW, (M - b0 + WAVE - 1) / WAVE);
        for (int p = L; p < R; ++p) {
          Real4 op;
          op.x = rl(ow.x, p);
          op.y = rl(ow.y, p);
          op.z = rl(ow.z, p);
          op.w = rl(ow.w, p);
          const uint32_t cp = unpack_index(op.w);
          Real s[4] = {(Real)0, (Real)0, (Real)0, (Real)0};
          bool any = false;
#pragma unroll
          for (int k = 0; k < CBW; ++k) {
            if (k >= nu) break;
            Real rx, ry, rz;
            pair_vec(op, cp, co[k], csr, rx, ry, rz);
            const Real r2 = rx * rx + ry * ry + rz * rz;
            if (r2 < cut2) {
              const Real q = r2 * rsq(r2) * inv_h;
              const Real t = (Real)1 - (Real)0.5 * q;
              const Real wgt = r2 > (Real)0 ? kW * t * t * t * t * ((Real)1 + (Real)2 * q) : kW;
              s[0] += wgt * cv[k].x;
              s[1] += wgt * cv[k].y;
              s[2] += wgt * cv[k].z;
              s[3] += wgt;
              any = true;
            }
          }
          if (!__ballot(any)) continue;
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const Real t = wave_total(s[a]);
            if (lane == p) acc[a] += t;
          }
        }
      }
      wave_lds_sync();
      if (NT > BLOCK && lane < R) {
#pragma unroll
        for (int a = 0; a < 4; ++a) sums[a][first + lane] = acc[a];
      }
    }
    if (NT > BLOCK) {
      __syncthreads();
      if (threadIdx.x < BLOCK) {
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] = sums[a][threadIdx.x];
      }
    }
  }
  if (!act) return;
  Real4 o = u;
  o.w = (Real)0;
  if (!S.wall_rigid && acc[3] > (Real)0) {
    const double inv = 1.0 / (double)acc[3];
    o.x = (Real)(2.0 * (double)u.x - (double)acc[0] * inv);
    o.y = (Real)(2.0 * (double)u.y - (double)acc[1] * inv);
    o.z = (Real)(2.0 * (double)u.z - (double)acc[2] * inv);
    o.w = (Real)((double)acc[3] * (S.dp * S.dp * S.dp));
  }
  gp<Real>(S.vw)[4 * (int64_t)w + 3] = o.w;
  o.w = gpc<Real4>(S.lev)[w].w;   // the body, which the staged record names
  gp<Real4>(S.vd)[w] = o;
}

// ---------------------------------------------------------------------------
// K: contact factor of every solid particle (Section 2.7, eq. 24) after a
// build at the current time, FP64: the sum of V_j W_wj (V_j = m / rho_j) over
// the fluid particles within 2h of the solid particle, over the full-immersion
// reference (the lattice kernel sum over the wall's outer half-space).  The
// solid particle scans its own 27 fluid cells; an observable, not a step
// kernel.
// ---------------------------------------------------------------------------
// zout: the values in the caller's original order (S.zeta when null); part
// (optional, nblk blocks): per-block, per-body sums of the values and of the
// solid-particle counts, quantity-major ([(2 b + k) * nblk + block], k = 0
// sum, 1 count), reduced by k_contact_mean.
template <class P>
__global__ __launch_bounds__(BLOCK) void k_contact(const SlotDesc* table, LaunchTab tab, double* zout,
                                                   double* part) {
#pragma clang fp contract(off)
  typedef typename P::Pos Pos;
  typedef typename P::Pos4 Pos4;
  typedef typename P::Real4 Real4;
  __shared__ double lds[BLOCK / WAVE][NB][2];
  SLOT_PROLOGUE(DOM_SOLID);
  const int w = lb * BLOCK + threadIdx.x;
  double zw = 0.0;
  int bw = -1;
  if (w < S.ns) {
  const GLB Pos4* xa = gpc<Pos4>(S.xa);
  const GLB Real4* vr = gpc<Real4>(S.vr);
  const GLB uint32_t* rank = gpc<uint32_t>(S.rank);
  const GLB uint32_t* stf = gpc<uint32_t>(S.start_f);
  const Pos4 xq = gpc<Pos4>(S.xw)[w];
  int c[3];
  cell_coords<Pos>(S, xq.x, xq.y, xq.z, c);
  const double inv_h = 1.0 / S.h, kW = S.kW, m = S.mass, cut2 = S.cut2;
  double z = 0.0;
  for (int dz = -1; dz <= 1; ++dz)
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        const int nx = c[0] + dx, ny = c[1] + dy, nz = c[2] + dz;
        if (nx < 0 || ny < 0 || nz < 0 || nx >= S.dims[0] || ny >= S.dims[1] || nz >= S.dims[2]) continue;
        const uint32_t r = rank[cell_linear(S, nx, ny, nz)];
        for (uint32_t j = stf[r]; j < stf[r + 1]; ++j) {
          const Pos4 xj = xa[j];
          const Pos ddx = xq.x - xj.x, ddy = xq.y - xj.y, ddz = xq.z - xj.z;
          const Pos s2 = ddx * ddx + ddy * ddy;
          const Pos d2 = s2 + ddz * ddz;
          if ((double)d2 < cut2) {
            const double rw = (double)vr[j].w;
            const double rho = P::kRel ? S.rho0 + rw : rw;
            z += (m / rho) * kernel_W_d2((double)d2, inv_h, kW);
          }
        }
      }
  zw = z / S.zref;
  bw = S.body[w];
  (zout ? zout : S.zeta)[S.sid[w]] = zw;   // in the caller's original order (sid is a permutation)
  }
  if (!part) return;
  // per-body block sums in a fixed order: lanes by shuffle, then the four waves
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
  for (int b = 0; b < S.nbody; ++b) {
    const double sv = wave_sum(bw == b ? zw : 0.0);
    const double cv = (double)__popcll(__ballot(bw == b));
    if (ln == 0) {
      lds[wv][b][0] = sv;
      lds[wv][b][1] = cv;
    }
  }
  __syncthreads();
  const int nblk = S.nblk[DOM_SOLID];
  if (threadIdx.x < 2 * S.nbody) {
    const int b = threadIdx.x / 2, k = threadIdx.x % 2;
    part[(size_t)threadIdx.x * nblk + lb] = ((lds[0][b][k] + lds[1][b][k]) + lds[2][b][k]) + lds[3][b][k];
  }
}

// Mean contact factor of every body from k_contact's block partials: each
// quantity's partials summed over the blocks in a fixed order with Neumaier
// compensation (one wavefront per quantity), then sum / count (0 for a body
// without solid particles).  One block per slot.
__global__ __launch_bounds__(BLOCK) void k_contact_mean(const SlotDesc* table, LaunchTab tab,
                                                        const double* part, double* mean) {
  __shared__ double res[NB][2];
  SLOT_PROLOGUE(DOM_SLOT);
  (void)lb;
  const int nblk = S.nblk[DOM_SOLID];
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
  for (int q = wv; q < 2 * S.nbody; q += BLOCK / WAVE) {
    KS ks{0.0, 0.0};
    for (int k = ln; k < nblk; k += WAVE) ks_add(ks, part[(size_t)q * nblk + k]);
    const KS t = wave_ks(ks);
    if (ln == 0) res[q / 2][q % 2] = t.s + t.c;
  }
  __syncthreads();
  if (threadIdx.x < S.nbody) {
    const int b = threadIdx.x;
    mean[b] = res[b][1] > 0.0 ? res[b][0] / res[b][1] : 0.0;
  }
}

// ---------------------------------------------------------------------------
// K: dual-criteria time step (Section 2.8, eq. 25).  |v|max covers the fluid
// and the bodies' tip speeds; n_ac is capped by shortening dt_ad.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_dt(const SlotDesc* table, LaunchTab tab) {
  __shared__ double red[BLOCK / WAVE];
  SLOT_PROLOGUE(DOM_SLOT);
  (void)lb;
  const int n = S.nblk[DOM_FLUID];
  double m = 0.0;
  for (int k = threadIdx.x; k < n; k += BLOCK) m = fmax(m, S.vmax_part[k]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, WAVE));
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double vm = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  for (int b = 0; b < S.nbody; ++b) vm = fmax(vm, S.btip[b]);
  SlotCtl* C = S.ctl;
  double tad, dt;
  int nac;
  if (S.fixed_dt_ad > 0.0) {
    tad = S.fixed_dt_ad;
    nac = S.fixed_nac > 0 ? S.fixed_nac : 1;
    dt = tad / (double)nac;
  } else {
    const double h = S.h;
    const double visc = h * h / S.nu;
    const double adv = vm > 0.0 ? h / vm : visc;
    tad = S.cfl_ad * (adv < visc ? adv : visc);
    tad = fmin(tad, S.dt_T);   // eq. 26
    const double tac = S.cfl_ac * h / (S.c0 + vm);
    double nn = ceil(tad / tac);
    if (nn < 1.0) nn = 1.0;
    if (nn > (double)S.nac_bound) {
      nn = (double)S.nac_bound;
      tad = nn * tac;
    }
    nac = (int)nn;
    dt = tad / nn;
  }
  C->dt_ad = tad;
  C->dt = dt;
  C->n_ac = nac;
}


// G[a][b] += c dv_a r_b: one pair's term of the SPH velocity gradient
template <class Real>
__device__ __forceinline__ void grad_add(Real* G, Real c, Real dx, Real dy, Real dz, Real rx, Real ry, Real rz) {
  const Real d[3] = {c * dx, c * dy, c * dz};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    G[3 * a] += d[a] * rx;
    G[3 * a + 1] += d[a] * ry;
    G[3 * a + 2] += d[a] * rz;
  }
}

// ---------------------------------------------------------------------------
// K: viscous acceleration (eq. 10 fluid-fluid, eq. 18 fluid-wall) and heat
// conduction rate (eq. 22), both frozen for the advection step.  Per-block
// partials: viscous force and torque on each body and its heat flow into the
// fluid.  Also clears this block's pressure-force accumulators.
// DISS: the launch holds a slot with viscous dissipation heating (eq. 23):
// the velocity gradient G[a][b] = sum V_j (v_j - v_i)_a F_ij r_ij[b] over fluid
// and wall neighbours gives Phi = 2 eta S:S, S = (G + G^T)/2, added to the
// heat rate as Phi/(rho cp); per-block partial of sum V_i Phi_i.
// MAT: the launch holds a slot with several fluid materials: k and cp per
// particle (material index gathered per neighbour), K_ij = 4 k_i k_j /
// (k_i + k_j) from a per-block table.
// MOM0: the same pass also runs the first acoustic sub-step's opening half
// (rho + dt/2 Drho, x + dt/2 v) and its Riemann momentum update, which read
// the same neighbours and frozen pair vectors: each neighbour's half-step
// density is formed from its gathered state and Drho with the arithmetic of
// the separate half update, so the results equal the unfused sequence bit
// for bit.  A fluid pair costs three gathers (cell offset, velocity and
// density, the (T, Drho) record the reorder wrote) instead of the five of
// the separate launches.
// ---------------------------------------------------------------------------
// The staged candidates leave two waves per SIMD, and their 256 registers are
// the budget; with heating, 34 to 36 of them spill in mixed arithmetic (108 to 116
// bytes per lane), 15 to 18 in FP32.  Gathering, the fused sweep without heating
// is held to three waves in FP32 and mixed arithmetic; the rest is the compiler's.
constexpr int visc_min_waves(bool stage, bool mom0, bool diss, bool f64) {
  return stage ? 2 : mom0 && !diss && !f64 ? 3 : 1;
}
template <class P, bool DISS, bool MAT, bool MOM0, bool STAGE>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(
    visc_min_waves(STAGE, MOM0, DISS, std::is_same<typename P::Real, double>::value)))) void
k_visc_heat(const SlotDesc* table, LaunchTab tab) {
  typedef typename P::Real Real;
  typedef typename P::Temp Temp;
  typedef typename P::Real4 Real4;
  // staged candidates, then (after the rows) the block reductions
  constexpr int RED_BYTES = 4 * NB * (7 + (MOM0 ? 6 : 0)) * 8;
  __shared__ __attribute__((aligned(32))) char smem[STAGE ? STAGE_CAP * 32 : RED_BYTES];
  __shared__ float shift[STAGE ? 3 * SHIFT_LD : 1];
  double* lds = (double*)smem;
  double* lds_p = lds + 4 * NB * 7;
  __shared__ double lds_d[BLOCK / WAVE];
  __shared__ Real Ktab[MAT ? NMAT * NMAT : 1];
  __shared__ Real Kwall[(MAT ? NMAT : 1) * NB];   // K_iw of eq. 22 per material and body
  __shared__ Temp Tb[NB];
  SLOT_FIND(DOM_FLUID);
  const int nf = S.nf;
  const int i = lb * BLOCK + threadIdx.x;
  const int ii = min(i, nf - 1);
  const GLB Real4* vr = gpc<Real4>(S.vr);
  const GLB Temp* T = gpc<Temp>(S.T);
  const GLB Real4* xo = gpc<Real4>(S.xo);
  const GLB TempRate<P>* td = gpc<TempRate<P>>(S.td);
  const GLB Real4* vdw = gpc<Real4>(S.vd);   // dummy velocity of eq. 18
  const GLB Real4* vw = gpc<Real4>(S.vw);    // rigid velocity (velocity gradient of eq. 23)
  const GLB Real4* lv = gpc<Real4>(S.lev);
  BlkHead hd;
  StageList sl;
  if constexpr (STAGE) {
    hd = blk_head(S, lb);
    sl = stage_list(S, lb);
  }
  const Real4 vi = vr[ii];
  const Real4 oi = xo[ii];
  const Temp Ti = T[ii];
  const Real drhoi = gpc<Real>(S.drho)[ii];
  const int nn = (int)S.nfc[ii], nw = (int)S.nsc[ii];
  if (!live_block(S)) return;
  const bool staged = STAGE && wave_staged(hd, wave_id());   // this wavefront's rows
  const bool mats = MAT && S.mat != nullptr;
  if (mats) {
    for (int q = threadIdx.x; q < NMAT * NMAT; q += BLOCK) {
      const double ka = S.mk[q / NMAT], kb = S.mk[q % NMAT];
      Ktab[q] = (Real)(4.0 * ka * kb / (ka + kb));
    }
  }
  for (int q = threadIdx.x; q < (mats ? NMAT : 1) * S.nbody; q += BLOCK) {
    const int b = q % S.nbody, mq = q / S.nbody;
    const double k = mats ? S.mk[mq] : S.k_f;
    Kwall[mq * NB + b] = (Real)(4.0 * k * S.bk[b] / (k + S.bk[b]));
    if (mq == 0) Tb[b] = (Temp)S.bT[b];
  }
  Row8 ef{u4(0), u4(0)}, ew{u4(0), u4(0)};
  if constexpr (STAGE) {
    if (hd.n > 0) {
      if (staged) {
        ef = row_load(row_groups(S, ii), 0);
        ew = row_load(wall_groups(S, ii), 0);
      }
      shift_table(shift, (float)S.cs_r);
      const GLB f4* so = gpc<f4>(S.so);
      // the position record's fourth word takes the sorted index, at which the
      // temperature record or the lever arm is gathered
      stage_block(
          hd, sl, [&](bool sol, uint32_t j) { return RecPair{(sol ? so : xo)[j], (sol ? vdw : vr)[j]}; },
          [&](uint32_t l, const RecPair& r, uint32_t j) {
            f4 o = r.a;
            o.w = pack_index(j, 0.0f);
            *(f4*)(smem + 16 * l) = o;
            *(f4*)(smem + 16 * l + 16 * STAGE_CAP) = r.b;
          });
    }
  }
  if (!STAGE || hd.n == 0) __syncthreads();
  const size_t nbf = (size_t)S.nblk[DOM_FLUID];
  if (threadIdx.x < NB * 6) S.press_part[(size_t)threadIdx.x * nbf + lb] = 0.0;
  BodyAcc<7> acc;
  acc.init();
  BodyAcc<6> pacc;   // MOM0: pressure force and torque of the first sub-step
  pacc.init();
  bool wall = false;
  double vphi = 0.0;   // V_i Phi_i
  if (i < nf) {
    const Real m = (Real)S.mass;
    const Real inv_h = (Real)(1.0 / S.h), kF = (Real)S.kF, csr = (Real)S.cs_r;
    const uint32_t ci = unpack_index(oi.w);
    const Real rhoi = rho_abs<P>(S, vi.w);
    const Real c2 = (Real)(2.0 * S.eta) * rcp(rhoi);   // 2 eta V_i / m_i
    const Real Kff = (Real)(4.0 * S.k_f * S.k_f / (S.k_f + S.k_f));
    const uint32_t mi = mats ? S.mat[i] : 0u;
    const double cpI = mats ? S.mcp[mi] : S.cp_f;
    Real ax = 0, ay = 0, az = 0, hs = 0;
    Real G[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) G[q] = 0;
    // MOM0: own half-step state (density opened by dt/2 Drho) and the
    // pressure acceleration of the first sub-step
    Real hdt = 0, wih = 0, rhoih = 0, pih = 0, c2p = 0, c0 = 0;
    Real px = 0, py = 0, pz = 0;
    if constexpr (MOM0) {
      hdt = (Real)(0.5 * S.ctl->dt);
      wih = fma(hdt, drhoi, vi.w);
      rhoih = rho_abs<P>(S, wih);
      pih = press<P>(S, wih);
      c2p = (Real)2 * rcp(rhoih);
      c0 = (Real)S.c0;
    }
    const int lane = i & (WAVE - 1);
    const int64_t slice = i >> 6;
    const Real cc2 = (Real)(S.c0 * S.c0);
    // one fluid pair: its vector, the neighbour's state, temperature, density
    // rate and material
    auto pair = [&](Real rx, Real ry, Real rz, const Real4& vj, Temp Tj, Real dj, uint32_t mj, bool real) {
      const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz), rs = rsq0(r2);
      Real Fk = kernel_F(r2, rs, inv_h, kF);
      Fk = real ? Fk : (Real)0;
      const Real Vj = m * rcp(rho_abs<P>(S, vj.w));
      const Real cv = c2 * Vj * Fk;
      const Real dx = vi.x - vj.x, dy = vi.y - vj.y, dz = vi.z - vj.z;
      ax = fma(cv, dx, ax);
      ay = fma(cv, dy, ay);
      az = fma(cv, dz, az);
      const Real Kij = mats ? Ktab[mi * NMAT + mj] : Kff;
      hs = fma(Vj * Kij * (Real)(Ti - Tj), Fk, hs);
      if (DISS) grad_add(G, Vj * Fk, -dx, -dy, -dz, rx, ry, rz);
      if constexpr (MOM0) {
        // eq. 10-12 at the half-step densities, velocities of the step's start
        const Real wjh = fma(hdt, dj, vj.w);
        const Real sp = mom_factor<P>(S, rhoih, pih, -c2p, c0, cc2, m * rcp(rho_abs<P>(S, wjh)),
                                      dot_fma(dx, dy, dz, rx, ry, rz), rs, wjh, Fk);
        px = fma(sp, rx, px);
        py = fma(sp, ry, py);
        pz = fma(sp, rz, pz);
      }
    };
    // one wall pair: its vector, the dummy velocity, the body, the lever arm
    // and the rigid velocity
    const Real Vw = (Real)S.vol_w;
    const Real rc = rcp(rhoi * (Real)cpI);
    const Real gx0 = (Real)S.g[0], gy0 = (Real)S.g[1], gz0 = (Real)S.g[2];
    const Real rho0 = (Real)S.rho0, ic02 = (Real)(1.0 / (S.c0 * S.c0));
    auto wpair = [&](Real rx, Real ry, Real rz, const Real4& vq, int b, const Real4& lq, const Real4& vg, bool real) {
#pragma clang fp contract(off)
      const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz);
      Real Fk = kernel_F(r2, rsq0(r2), inv_h, kF);
      Fk = real ? Fk : (Real)0;
      const Real cv = c2 * Vw * Fk;
      const Real dx = vi.x - vq.x, dy = vi.y - vq.y, dz = vi.z - vq.z;
      ax = fma(cv, dx, ax);
      ay = fma(cv, dy, ay);
      az = fma(cv, dz, az);
      const Real tk = Vw * Kwall[mi * NB + b] * (Real)(Ti - Tb[b]);
      hs = fma(tk, Fk, hs);
      if (DISS) grad_add(G, Vw * Fk, vg.x - vi.x, vg.y - vi.y, vg.z - vi.z, rx, ry, rz);
      acc.moment(cv * dx, cv * dy, cv * dz, lq);
      acc.v0[6] += (double)(rc * (tk * Fk));
      if constexpr (MOM0) {
        const Real sp = wall_factor(rhoih, pih, c2p, Vw, rho0, ic02, dot_fma(gx0, gy0, gz0, rx, ry, rz), Fk);
        px = fma(sp, rx, px);
        py = fma(sp, ry, py);
        pz = fma(sp, rz, pz);
        pacc.moment(sp * rx, sp * ry, sp * rz, lq);
      }
    };
    wall = nw > 0;
    if (staged) {
      if constexpr (STAGE) {
        // as staged_row, with the temperature records of a set gathered (at the
        // sorted index in its position record) while the set before is used
        const GLB u4* Gr = row_groups(S, i);
        struct Temps {
          Temp T[4];
          Real d[4];
          uint32_t m[4];
        };
        auto gather = [&](Temps& t, const Set4& q) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint32_t j = unpack_index(q.o[u].w);
            if constexpr (MOM0) {
              t.T[u] = td[j].T;
              t.d[u] = td[j].d;
            } else {
              t.T[u] = T[j];
              t.d[u] = 0;
            }
            t.m[u] = mats ? S.mat[j] : 0u;
          }
        };
        auto use = [&](const Set4& q, const Temps& t) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            Real rx, ry, rz;
            set_vec(q, u, oi, rx, ry, rz);
            pair(rx, ry, rz, q.v[u], t.T[u], t.d[u], t.m[u], true);
          }
        };
        Row8 rn = ef;
        if (8 < nn) rn = row_load(Gr, 8);
        Set4 A, B;
        Temps ta, tb;
        set_fetch(A, ef.a, smem, shift);
        set_fetch(B, ef.b, smem, shift);
        gather(ta, A);
        for (int k = 0; k < nn; k += 8) {
          gather(tb, B);
          Row8 rl = rn;
          if (k + 16 < nn) rl = row_load(Gr, k + 16);
          __builtin_amdgcn_sched_barrier(0);
          use(A, ta);
          set_fetch(A, rn.a, smem, shift);
          gather(ta, A);
          __builtin_amdgcn_sched_barrier(0);
          use(B, tb);
          set_fetch(B, rn.b, smem, shift);
          rn = rl;
        }
        staged_wall(wall_groups(S, i), ew, nw, smem, shift, [&](const Set4& W, const bool(&real)[4]) {
          const float w[4] = {W.v[0].w, W.v[1].w, W.v[2].w, W.v[3].w};
          int b[4];
          f4 lq[4], vg[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            lq[u] = vg[u] = f4(0);
            if (real[u]) {
              const uint32_t j = unpack_index(W.o[u].w);
              lq[u] = lv[j];
              if (DISS) vg[u] = vw[j];
            }
          }
          const bool one = acc.current(w, real, b);
          if (MOM0 && pacc.id0 < 0) pacc.id0 = acc.id0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (!one) {
              if (!acc.select(b[u])) raise_flag(S, F_CAPACITY);
              if (MOM0) pacc.select(b[u]);
            }
            Real rx, ry, rz;
            set_vec(W, u, oi, rx, ry, rz);
            wpair(rx, ry, rz, W.v[u], b[u], lq[u], vg[u], real[u]);
          }
        });
      }
    } else {
      const GLB uint32_t* R = gpc<uint32_t>(S.nrec) + slice * (int64_t)S.kf * WAVE + lane;
      uint32_t jn[ROW_UNROLL];
#pragma unroll
      for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)u * WAVE);
      for (int k = 0; k < nn; k += ROW_UNROLL) {
        uint32_t j[ROW_UNROLL];
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) j[u] = k + u < nn ? jn[u] : (uint32_t)i;
        Real4 vj[ROW_UNROLL], oj[ROW_UNROLL];
        Temp Tj[ROW_UNROLL];
        Real dj[ROW_UNROLL];
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) {
          oj[u] = xo[j[u]];
          vj[u] = vr[j[u]];
          if constexpr (MOM0) {
            Tj[u] = td[j[u]].T;
            dj[u] = td[j[u]].d;
          } else {
            Tj[u] = T[j[u]];
            dj[u] = 0;
          }
        }
        if (k + ROW_UNROLL < nn) {
#pragma unroll
          for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)(k + ROW_UNROLL + u) * WAVE);
        }
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) {
          Real rx, ry, rz;
          pair_vec(oi, ci, oj[u], csr, rx, ry, rz);
          pair(rx, ry, rz, vj[u], Tj[u], dj[u], mats ? S.mat[j[u]] : 0u, k + u < nn);
        }
      }
      R = gpc<uint32_t>(S.srec) + slice * (int64_t)S.ks * WAVE + lane;
      const GLB Real4* so = gpc<Real4>(S.so);
      uint32_t wn[VISC_SOLID_UNROLL];
#pragma unroll
      for (int u = 0; u < VISC_SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)u * WAVE);
      for (int k0 = 0; k0 < nw; k0 += VISC_SOLID_UNROLL) {
        Real4 owu[VISC_SOLID_UNROLL], vqu[VISC_SOLID_UNROLL], lqu[VISC_SOLID_UNROLL], vgu[VISC_SOLID_UNROLL];
#pragma unroll
        for (int u = 0; u < VISC_SOLID_UNROLL; ++u) {
          const uint32_t w = k0 + u < nw ? wn[u] : 0u;
          owu[u] = so[w];
          vqu[u] = vdw[w];
          lqu[u] = lv[w];
          if (DISS) vgu[u] = vw[w];
        }
        if (k0 + VISC_SOLID_UNROLL < nw) {
#pragma unroll
          for (int u = 0; u < VISC_SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)(k0 + VISC_SOLID_UNROLL + u) * WAVE);
        }
#pragma unroll
        for (int u = 0; u < VISC_SOLID_UNROLL; ++u) {
          if (k0 + u >= nw) break;
          Real rx, ry, rz;
          pair_vec(oi, ci, owu[u], csr, rx, ry, rz);
          const int b = (int)lqu[u].w;
          if (!acc.select(b)) raise_flag(S, F_CAPACITY);
          if (MOM0) pacc.select(b);
          wpair(rx, ry, rz, vqu[u], b, lqu[u], vgu[u], true);
        }
      }
    }
    {
      if (DISS && S.diss) {
        // Phi = 2 eta S:S with S = (G + G^T)/2
        const Real sxy = (Real)0.5 * (G[1] + G[3]), sxz = (Real)0.5 * (G[2] + G[6]),
                   syz = (Real)0.5 * (G[5] + G[7]);
        const Real ss = (G[0] * G[0] + G[4] * G[4] + G[8] * G[8]) + (Real)2 * ((sxy * sxy + sxz * sxz) + syz * syz);
        const Real phi = (Real)(2.0 * S.eta) * ss;
        hs += phi;
        vphi = (double)(m * rcp(rhoi)) * (double)phi;
      }
      Real4 a;
      a.x = ax;
      a.y = ay;
      a.z = az;
      a.w = rc * hs;
      gp<Real4>(S.ah)[i] = a;
      if constexpr (MOM0) {
        // v_new = v + dt (a_p + a_visc + g); the opening and the closing half
        // drifts x += dt/2 v, x += dt/2 v_new, in that order
        const Real dt = (Real)S.ctl->dt;
        Real4 vn;
        vn.x = vi.x + dt * (px + ax + (Real)S.g[0]);
        vn.y = vi.y + dt * (py + ay + (Real)S.g[1]);
        vn.z = vi.z + dt * (pz + az + (Real)S.g[2]);
        vn.w = wih;
        gp<Real4>(S.vrn)[i] = vn;
        GLB Real4* dr = gp<Real4>(S.drift);
        Real4 d = dr[i];
        d.x += hdt * vi.x;
        d.y += hdt * vi.y;
        d.z += hdt * vi.z;
        d.x += hdt * vn.x;
        d.y += hdt * vn.y;
        d.z += hdt * vn.z;
        dr[i] = d;
      }
    }
  }
  acc.to_force((double)(Real)S.mass);
  pacc.to_force((double)(Real)S.mass);
  {
    // heat flows from the sums of dT/dt
    const uint32_t mi = mats && i < nf ? S.mat[i] : 0u;
    const double mc = (double)(Real)S.mass * (mats ? S.mcp[mi] : S.cp_f);
    acc.v0[6] *= mc;
    acc.v1[6] *= mc;
  }
  if (__syncthreads_or(wall)) {
    block_body_reduce<7>(acc, S.nbody, S.visc_part, nbf, lb, false, lds);
    if constexpr (MOM0) block_body_reduce<6>(pacc, S.nbody, S.press_part, nbf, lb, true, lds_p);
  } else if (threadIdx.x < NB * 7) {
    S.visc_part[(size_t)threadIdx.x * nbf + lb] = 0.0;
  }
  if (DISS && S.diss) {
    const double sw = wave_sum(vphi);
    if ((threadIdx.x & (WAVE - 1)) == 0) lds_d[threadIdx.x / WAVE] = sw;
    __syncthreads();
    if (threadIdx.x == 0)
      S.glob_part[(size_t)NGLOB * nbf + lb] = ((lds_d[0] + lds_d[1]) + lds_d[2]) + lds_d[3];
  }
}

// ---------------------------------------------------------------------------
// K: first half of an acoustic sub-step: rho += dt/2 Drho, x += dt/2 v
// ---------------------------------------------------------------------------
template <class P>
__global__ __launch_bounds__(BLOCK) void k_half_a(const SlotDesc* table, LaunchTab tab, int sub) {
  typedef typename P::Real Real;
  typedef typename P::Real4 Real4;
  SLOT_PROLOGUE(DOM_FLUID);
  if (sub >= S.ctl->n_ac) return;
  const int i = lb * BLOCK + threadIdx.x;
  if (i >= S.nf) return;
  const Real hdt = (Real)(0.5 * S.ctl->dt);
  GLB Real4* vr = gp<Real4>(S.vr);
  Real4 v = vr[i];
  v.w = fma(hdt, gpc<Real>(S.drho)[i], v.w);
  vr[i] = v;
  GLB Real4* dr = gp<Real4>(S.drift);
  Real4 d = dr[i];
  d.x += hdt * v.x;
  d.y += hdt * v.y;
  d.z += hdt * v.z;
  dr[i] = d;
}

// Stages the candidates of a momentum or continuity sweep: cell-relative
// positions with the particle's volume m / rho as the fourth component, then
// the records b (fluid: velocity and density) and ws (solid) at 16 * STAGE_CAP,
// and the shift table.
template <class P>
__device__ __forceinline__ void stage_pairs(const SlotDesc& S, const BlkHead& hd, const StageList& sl,
                                            const GLB f4* b, const GLB f4* ws, char* smem, float* shift) {
  const GLB f4* xo = gpc<f4>(S.xo);
  const GLB f4* so = gpc<f4>(S.so);
  const float m = (float)S.mass;
  shift_table(shift, (float)S.cs_r);
  stage_block(
      hd, sl, [&](bool sol, uint32_t j) { return RecPair{(sol ? so : xo)[j], (sol ? ws : b)[j]}; },
      [&](uint32_t l, const RecPair& r, uint32_t) {
        f4 o = r.a;
        o.w = m * rcp(rho_abs<P>(S, r.b.w));
        *(f4*)(smem + 16 * l) = o;
        *(f4*)(smem + 16 * l + 16 * STAGE_CAP) = r.b;
      });
}

// ---------------------------------------------------------------------------
// K: Riemann momentum (eq. 10-12) with the wall pressure of the one-sided
// problem (eq. 16-19); v_new = v + dt (a_p + a_visc + g), then the second
// half drift x += dt/2 v_new.  Per-block pressure force and torque on each
// body accumulate over the sub-steps.
// ---------------------------------------------------------------------------
template <class P, bool STAGE>
__global__ __launch_bounds__(BLOCK) void k_momentum(const SlotDesc* table, LaunchTab tab, int sub) {
  typedef typename P::Real Real;
  typedef typename P::Real4 Real4;
  // staged candidates, then (after the rows) the block reduction
  __shared__ __attribute__((aligned(32))) char smem[STAGE ? STAGE_CAP * 32 : 4 * NB * 6 * 8];
  __shared__ float shift[STAGE ? 3 * SHIFT_LD : 1];
  double* lds = (double*)smem;
  SLOT_FIND(DOM_FLUID);
  // launches past the step's sub-steps leave before the loads and the barrier (6 us
  // each with them); no launch that reads n_ac writes it
  if (sub >= gpc<SlotCtl>(S.ctl)->n_ac) return;
  const int nf = S.nf;
  const int i = lb * BLOCK + threadIdx.x;
  const int ii = min(i, nf - 1);
  const GLB Real4* vr = gpc<Real4>(S.vr);
  const GLB Real4* xo = gpc<Real4>(S.xo);
  const GLB Real4* lv = gpc<Real4>(S.lev);
  BlkHead hd;
  StageList sl;
  if constexpr (STAGE) {
    hd = blk_head(S, lb);
    sl = stage_list(S, lb);
  }
  const Real4 vi = vr[ii];
  const Real4 oi = xo[ii];
  const int nn = (int)S.nfc[ii], nw = (int)S.nsc[ii];
  if (!live_block(S)) return;
  const bool staged = STAGE && wave_staged(hd, wave_id());   // this wavefront's rows
  Row8 ef{u4(0), u4(0)}, ew{u4(0), u4(0)};
  if constexpr (STAGE) {
    if (hd.n > 0) {
      if (staged) {
        ef = row_load(row_groups(S, ii), 0);
        ew = row_load(wall_groups(S, ii), 0);
      }
      stage_pairs<P>(S, hd, sl, vr, lv, smem, shift);
    }
  }
  BodyAcc<6> acc;
  acc.init();
  bool wall = false;
  if (i < nf) {
    const Real c0 = (Real)S.c0;
    const Real m = (Real)S.mass;
    const uint32_t ci = unpack_index(oi.w);
    const Real rhoi = rho_abs<P>(S, vi.w);
    const Real pi = press<P>(S, vi.w);
    const Real c2 = (Real)2 * rcp(rhoi);   // 2 V_i / m_i
    const Real cc2 = (Real)(S.c0 * S.c0);
    const Real inv_h = (Real)(1.0 / S.h), kF = (Real)S.kF, csr = (Real)S.cs_r;
    Real ax = 0, ay = 0, az = 0;
    const int lane = i & (WAVE - 1);
    const int64_t slice = i >> 6;
    // Vj: the neighbour's volume m / rho_j
    auto pair = [&](Real rx, Real ry, Real rz, const Real4& vj, Real Vj, bool real = true) {
      const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz), rs = rsq0(r2);
      Real Fk = kernel_F(r2, rs, inv_h, kF);
      Fk = real ? Fk : (Real)0;
      const Real sp = mom_factor<P>(S, rhoi, pi, -c2, c0, cc2, Vj,
                                    dot_fma(vi.x - vj.x, vi.y - vj.y, vi.z - vj.z, rx, ry, rz), rs, vj.w, Fk);
      ax = fma(sp, rx, ax);
      ay = fma(sp, ry, ay);
      az = fma(sp, rz, az);
    };
    const Real gx = (Real)S.g[0], gy = (Real)S.g[1], gz = (Real)S.g[2];
    const Real rho0 = (Real)S.rho0, ic02 = (Real)(1.0 / (S.c0 * S.c0)), Vw = (Real)S.vol_w;
    auto wpair = [&](Real rx, Real ry, Real rz, const Real4& lq, bool real) {
#pragma clang fp contract(off)
      const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz);
      Real Fk = kernel_F(r2, rsq0(r2), inv_h, kF);
      Fk = real ? Fk : (Real)0;
      const Real sp = wall_factor(rhoi, pi, c2, Vw, rho0, ic02, dot_fma(gx, gy, gz, rx, ry, rz), Fk);
      ax = fma(sp, rx, ax);
      ay = fma(sp, ry, ay);
      az = fma(sp, rz, az);
      acc.moment(sp * rx, sp * ry, sp * rz, lq);
    };
    wall = nw > 0;
    if (staged) {
      if constexpr (STAGE) {
        staged_row(row_groups(S, i), ef, nn, smem, shift, oi, pair);
        staged_wall(wall_groups(S, i), ew, nw, smem, shift, [&](const Set4& W, const bool(&real)[4]) {
          const float w[4] = {W.v[0].w, W.v[1].w, W.v[2].w, W.v[3].w};
          int b[4];
          const bool one = acc.current(w, real, b);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (!one && !acc.select(b[u])) raise_flag(S, F_CAPACITY);
            Real rx, ry, rz;
            set_vec(W, u, oi, rx, ry, rz);
            wpair(rx, ry, rz, W.v[u], real[u]);
          }
        });
      }
    } else {
      const GLB uint32_t* R = gpc<uint32_t>(S.nrec) + slice * (int64_t)S.kf * WAVE + lane;
      uint32_t jn[ROW_UNROLL];
#pragma unroll
      for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)u * WAVE);
      for (int k = 0; k < nn; k += ROW_UNROLL) {
        uint32_t j[ROW_UNROLL];
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) j[u] = k + u < nn ? jn[u] : (uint32_t)i;
        Real4 vj[ROW_UNROLL], oj[ROW_UNROLL];
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) {
          oj[u] = xo[j[u]];
          vj[u] = vr[j[u]];
        }
        if (k + ROW_UNROLL < nn) {
#pragma unroll
          for (int u = 0; u < ROW_UNROLL; ++u) jn[u] = ldnt(R + (int64_t)(k + ROW_UNROLL + u) * WAVE);
        }
#pragma unroll
        for (int u = 0; u < ROW_UNROLL; ++u) {
          Real rx, ry, rz;
          pair_vec(oi, ci, oj[u], csr, rx, ry, rz);
          pair(rx, ry, rz, vj[u], m * rcp(rho_abs<P>(S, vj[u].w)), k + u < nn);
        }
      }
      R = gpc<uint32_t>(S.srec) + slice * (int64_t)S.ks * WAVE + lane;
      const GLB Real4* so = gpc<Real4>(S.so);
      uint32_t wn[SOLID_UNROLL];
#pragma unroll
      for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)u * WAVE);
      for (int k0 = 0; k0 < nw; k0 += SOLID_UNROLL) {
        Real4 owu[SOLID_UNROLL], lqu[SOLID_UNROLL];
#pragma unroll
        for (int u = 0; u < SOLID_UNROLL; ++u) {
          const uint32_t w = k0 + u < nw ? wn[u] : 0u;
          owu[u] = so[w];
          lqu[u] = lv[w];
        }
        if (k0 + SOLID_UNROLL < nw) {
#pragma unroll
          for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)(k0 + SOLID_UNROLL + u) * WAVE);
        }
#pragma unroll
        for (int u = 0; u < SOLID_UNROLL; ++u) {
          if (k0 + u >= nw) break;
          Real rx, ry, rz;
          pair_vec(oi, ci, owu[u], csr, rx, ry, rz);
          if (!acc.select((int)lqu[u].w)) raise_flag(S, F_CAPACITY);
          wpair(rx, ry, rz, lqu[u], true);
        }
      }
    }
    const Real dt = (Real)S.ctl->dt;
    const Real hdt = (Real)(0.5 * S.ctl->dt);
    const Real4 a = gpc<Real4>(S.ah)[i];
    Real4 vn;
    vn.x = vi.x + dt * (ax + a.x + (Real)S.g[0]);
    vn.y = vi.y + dt * (ay + a.y + (Real)S.g[1]);
    vn.z = vi.z + dt * (az + a.z + (Real)S.g[2]);
    vn.w = vi.w;
    gp<Real4>(S.vrn)[i] = vn;
    GLB Real4* dr = gp<Real4>(S.drift);
    Real4 d = dr[i];
    d.x += hdt * vn.x;
    d.y += hdt * vn.y;
    d.z += hdt * vn.z;
    dr[i] = d;
  }
  acc.to_force((double)(Real)S.mass);
  if (__syncthreads_or(wall))
    block_body_reduce<6>(acc, S.nbody, S.press_part, (size_t)S.nblk[DOM_FLUID], lb, true, lds);
}

// ---------------------------------------------------------------------------
// K: Riemann continuity (eq. 10, 11-13) with (v_i - v*) . e_ij = U* - U_L, and
// the wall's mirror state; writes Drho, commits v <- v_new and applies the
// half updates that close this sub-step and open the next.
// ---------------------------------------------------------------------------
template <class P, bool STAGE>
__global__ __launch_bounds__(BLOCK) void k_continuity(const SlotDesc* table, LaunchTab tab, int sub) {
  typedef typename P::Real Real;
  typedef typename P::Real4 Real4;
  __shared__ __attribute__((aligned(32))) char smem[STAGE ? STAGE_CAP * 32 : 32];
  __shared__ float shift[STAGE ? 3 * SHIFT_LD : 1];
  SLOT_FIND(DOM_FLUID);
  const int i = lb * BLOCK + threadIdx.x;
  const int ii = min(i, S.nf - 1);
  const GLB Real4* vrn = gpc<Real4>(S.vrn);
  const GLB Real4* xo = gpc<Real4>(S.xo);
  const GLB Real4* nuw = gpc<Real4>(S.nuw);
  BlkHead hd;
  StageList sl;
  if constexpr (STAGE) {
    hd = blk_head(S, lb);
    sl = stage_list(S, lb);
  }
  const Real4 vi = vrn[ii];
  const Real4 oi = xo[ii];
  const int nn = (int)S.nfc[ii], nw = (int)S.nsc[ii];
  if (!live_sub(S, sub)) return;
  const bool staged = STAGE && wave_staged(hd, wave_id());   // this wavefront's rows
  Row8 ef{u4(0), u4(0)}, ew{u4(0), u4(0)};
  if constexpr (STAGE) {
    if (hd.n > 0) {
      if (staged) {
        ef = row_load(row_groups(S, ii), 0);
        ew = row_load(wall_groups(S, ii), 0);
      }
      stage_pairs<P>(S, hd, sl, vrn, nuw, smem, shift);
    }
  }
  if (i >= S.nf) return;
  const Real c0 = (Real)S.c0;
  const Real m = (Real)S.mass;
  const uint32_t ci = unpack_index(oi.w);
  const Real rhoi = rho_abs<P>(S, vi.w);
  const Real pi = press<P>(S, vi.w);
  const Real inv_h = (Real)(1.0 / S.h), kF = (Real)S.kF, csr = (Real)S.cs_r;
  const Real cc2 = (Real)(S.c0 * S.c0);
  Real sum = 0;
  const int lane = i & (WAVE - 1);
  const int64_t slice = i >> 6;
  // Vj: the neighbour's volume m / rho_j
  auto pair = [&](Real rx, Real ry, Real rz, const Real4& vj, Real Vj, bool real = true) {
    const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz), rs = rsq0(r2);
    Real Fk = kernel_F(r2, rs, inv_h, kF);
    Fk = real ? Fk : (Real)0;
    sum = fma(cont_factor<P>(S, rhoi, pi, c0, cc2, Vj, dot_fma(vi.x - vj.x, vi.y - vj.y, vi.z - vj.z, rx, ry, rz),
                             r2 * rs, vj.w),
              Fk, sum);
  };
  const Real gx = (Real)S.g[0], gy = (Real)S.g[1], gz = (Real)S.g[2];
  const Real rho0 = (Real)S.rho0, ic02 = (Real)(1.0 / (S.c0 * S.c0)), Vw = (Real)S.vol_w;
  // nq: the wall normal and u_w = -n . v_w
  auto wpair = [&](Real rx, Real ry, Real rz, const Real4& nq, bool real) {
#pragma clang fp contract(off)
    const Real r2 = dot_fma(rx, ry, rz, rx, ry, rz);
    Real Fk = kernel_F(r2, rsq0(r2), inv_h, kF);
    Fk = real ? Fk : (Real)0;
    const Real PR = fma(-rhoi, dot_fma(gx, gy, gz, rx, ry, rz), pi);
    const Real rhoR = fma(PR, ic02, rho0);
    const Real UL = -dot_fma(nq.x, nq.y, nq.z, vi.x, vi.y, vi.z);
    const Real Us = fma(pi - PR, rcp(c0 * (rhoi + rhoR)), nq.w);
    sum = fma(Vw * (Us - UL) * dot_fma(nq.x, nq.y, nq.z, rx, ry, rz), Fk, sum);
  };
  if (staged) {
    if constexpr (STAGE) {
      staged_row(row_groups(S, i), ef, nn, smem, shift, oi, pair);
      staged_wall(wall_groups(S, i), ew, nw, smem, shift, [&](const Set4& W, const bool(&real)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          Real rx, ry, rz;
          set_vec(W, u, oi, rx, ry, rz);
          wpair(rx, ry, rz, W.v[u], real[u]);
        }
      });
      }
  } else {
    constexpr int U = std::is_same<Real, float>::value ? CONT_UNROLL : ROW_UNROLL;
    const GLB uint32_t* R = gpc<uint32_t>(S.nrec) + slice * (int64_t)S.kf * WAVE + lane;
    uint32_t jn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) jn[u] = ldnt(R + (int64_t)u * WAVE);
    for (int k = 0; k < nn; k += U) {
      uint32_t j[U];
#pragma unroll
      for (int u = 0; u < U; ++u) j[u] = k + u < nn ? jn[u] : (uint32_t)i;
      Real4 vj[U], oj[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        oj[u] = xo[j[u]];
        vj[u] = vrn[j[u]];
      }
      if (k + U < nn) {
#pragma unroll
        for (int u = 0; u < U; ++u) jn[u] = ldnt(R + (int64_t)min(k + U + u, S.kf - 1) * WAVE);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        Real rx, ry, rz;
        pair_vec(oi, ci, oj[u], csr, rx, ry, rz);
        pair(rx, ry, rz, vj[u], m * rcp(rho_abs<P>(S, vj[u].w)), k + u < nn);
      }
    }
    R = gpc<uint32_t>(S.srec) + slice * (int64_t)S.ks * WAVE + lane;
    const GLB Real4* so = gpc<Real4>(S.so);
    uint32_t wn[SOLID_UNROLL];
#pragma unroll
    for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)u * WAVE);
    for (int k0 = 0; k0 < nw; k0 += SOLID_UNROLL) {
      Real4 owu[SOLID_UNROLL], nqu[SOLID_UNROLL];
#pragma unroll
      for (int u = 0; u < SOLID_UNROLL; ++u) {
        const uint32_t w = k0 + u < nw ? wn[u] : 0u;
        owu[u] = so[w];
        nqu[u] = nuw[w];
      }
      if (k0 + SOLID_UNROLL < nw) {
#pragma unroll
        for (int u = 0; u < SOLID_UNROLL; ++u) wn[u] = ldnt(R + (int64_t)(k0 + SOLID_UNROLL + u) * WAVE);
      }
#pragma unroll
      for (int u = 0; u < SOLID_UNROLL; ++u) {
        if (k0 + u >= nw) break;
        Real rx, ry, rz;
        pair_vec(oi, ci, owu[u], csr, rx, ry, rz);
        wpair(rx, ry, rz, nqu[u], true);
      }
    }
  }
  // commit v <- v_new and close the sub-step (rho += dt/2 Drho); unless it is
  // the step's last, open the next one (rho += dt/2 Drho, x += dt/2 v).  No
  // thread of this sweep reads vr, so the update is in place.
  const Real dr = (Real)2 * rhoi * sum;
  gp<Real>(S.drho)[i] = dr;
  const Real hdt = (Real)(0.5 * S.ctl->dt);
  Real4 v = vi;
  v.w += hdt * dr;
  if (sub + 1 < S.ctl->n_ac) {
    v.w += hdt * dr;
    GLB Real4* dp = gp<Real4>(S.drift);
    Real4 d = dp[i];
    d.x += hdt * v.x;
    d.y += hdt * v.y;
    d.z += hdt * v.z;
    dp[i] = d;
  }
  gp<Real4>(S.vr)[i] = v;
}

// ---------------------------------------------------------------------------
// K: temperature by explicit Euler over the advection step (eq. 22, 26), and
// per-block totals: mass, kinetic energy, thermal energy, sum rho dp^3, vmax.
// ---------------------------------------------------------------------------
template <class P>
__global__ __launch_bounds__(BLOCK) void k_end(const SlotDesc* table, LaunchTab tab) {
  typedef typename P::Temp Temp;
  typedef typename P::Real4 Real4;
  __shared__ double lds[BLOCK / WAVE][NGLOB];
  SLOT_PROLOGUE(DOM_FLUID);
  const int i = lb * BLOCK + threadIdx.x;
  double q[NGLOB] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (i < S.nf) {
    GLB Temp* T = gp<Temp>(S.T);
    const Temp Tn = T[i] + (Temp)S.ctl->dt_ad * (Temp)gpc<Real4>(S.ah)[i].w;
    T[i] = Tn;
    const Real4 v = gpc<Real4>(S.vr)[i];
    const double vx = v.x, vy = v.y, vz = v.z;
    const double v2 = vx * vx + vy * vy + vz * vz;
    const double r = P::kRel ? S.rho0 + (double)v.w : (double)v.w;
    q[0] = S.mass;
    q[1] = 0.5 * S.mass * v2;
    q[2] = S.mass * (S.mat ? S.mcp[S.mat[i]] : S.cp_f) * (double)Tn;
    q[3] = r * (S.dp * S.dp * S.dp);
    q[4] = sqrt(v2);
    if (!isfinite(v2) || !isfinite(r) || !isfinite((double)Tn)) raise_flag(S, F_NONFINITE);
  }
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
#pragma unroll
  for (int k = 0; k < NGLOB - 1; ++k) {
    const double s = wave_sum(q[k]);
    if (ln == 0) lds[wv][k] = s;
  }
  {
    double md = q[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) md = fmax(md, __shfl_xor(md, o, WAVE));
    if (ln == 0) lds[wv][4] = md;
  }
  __syncthreads();
  if (threadIdx.x < NGLOB) {
    const int k = threadIdx.x;
    double s;
    if (k == 4) s = fmax(fmax(lds[0][4], lds[1][4]), fmax(lds[2][4], lds[3][4]));
    else s = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
    S.glob_part[(size_t)k * S.nblk[DOM_FLUID] + lb] = s;
  }
}

// ---------------------------------------------------------------------------
// K: per-slot reports: compensated sums of the block partials in fixed order,
// per-body force, torque, axial torque, power and heat flow; time integrals;
// advance t and the step counter.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(FINAL_BLOCK) void k_final(const SlotDesc* table, LaunchTab tab) {
  __shared__ double res[NGLOB + NB * 13 + 1];
  __shared__ double bheat[NB];
  __shared__ int bfin[NB];
  SLOT_PROLOGUE(DOM_SLOT);
  (void)lb;
  const int nblk = S.nblk[DOM_FLUID];
  // quantities: the globals, 13 per body, then the dissipated power if on
  const int nq = NGLOB + S.nbody * 13 + (S.diss ? 1 : 0);
  const int q_diss = NGLOB + S.nbody * 13;
  const int wv = threadIdx.x / WAVE, ln = threadIdx.x % WAVE;
  // each wavefront reduces QPW quantities at once (QPW x 8 independent loads
  // in flight per lane), each one's partials added in the same fixed order
  constexpr int QPW = 3;
  for (int q0 = wv * QPW; q0 < nq; q0 += (FINAL_BLOCK / WAVE) * QPW) {
    // quantity qi: global k, or body b component c (7 viscous then 6 pressure)
    // partials are quantity-major: src[q * nblk + block]
    const GLB double* qs[QPW];
    bool use[QPW], mx[QPW];
#pragma unroll
    for (int t = 0; t < QPW; ++t) {
      const int qi = q0 + t;
      use[t] = qi < nq;
      mx[t] = qi == 4;
      const double* src = S.glob_part;
      if (!use[t]) {
      } else if (qi < NGLOB) {
        src = S.glob_part + (size_t)qi * nblk;
      } else if (qi == q_diss) {
        src = S.glob_part + (size_t)NGLOB * nblk;
      } else {
        const int b = (qi - NGLOB) / 13, c = (qi - NGLOB) % 13;
        src = c < 7 ? S.visc_part + (size_t)(b * 7 + c) * nblk : S.press_part + (size_t)(b * 6 + c - 7) * nblk;
      }
      qs[t] = gpc<double>(src);
    }
    KS ks[QPW];
    double m[QPW];
#pragma unroll
    for (int t = 0; t < QPW; ++t) {
      ks[t] = KS{0.0, 0.0};
      m[t] = 0.0;
    }
    for (int k0 = 0; k0 < nblk; k0 += 8 * WAVE) {
      double x[QPW][8];
#pragma unroll
      for (int t = 0; t < QPW; ++t)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int k = k0 + u * WAVE + ln;
          x[t][u] = use[t] && k < nblk ? qs[t][k] : 0.0;
        }
#pragma unroll
      for (int t = 0; t < QPW; ++t) {
        if (mx[t]) {
#pragma unroll
          for (int u = 0; u < 8; ++u) m[t] = fmax(m[t], x[t][u]);
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) ks_add(ks[t], x[t][u]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < QPW; ++t) {
      if (!use[t]) continue;
      if (mx[t]) {
        double v = m[t];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, WAVE));
        if (ln == 0) res[q0 + t] = v;
      } else {
        const KS w = wave_ks(ks[t]);
        if (ln == 0) res[q0 + t] = w.s + w.c;
      }
    }
  }
  __syncthreads();
  // the reports: lane b of the first wavefront finishes body b, lane 0 then
  // the globals; each lane loads the control fields it needs before it
  // stores anything (a store could alias a later load and hold it back)
  if (threadIdx.x >= WAVE) return;
  SlotCtl* C = S.ctl;
  const double tad = C->dt_ad;
  const int32_t nac = C->n_ac;
  const int b = threadIdx.x;
  if (b < S.nbody) {
    double cum[3], cumc[3];
    for (int k = 0; k < 3; ++k) {
      cum[k] = C->cum[b][k];
      cumc[k] = C->cum_c[b][k];
    }
    const double inv_nac = 1.0 / (double)nac;
    const double* r = res + NGLOB + b * 13;
    sph_body_report br;
    for (int k = 0; k < 3; ++k) {
      br.force[k] = r[k] + r[7 + k] * inv_nac;
      br.torque[k] = r[3 + k] + r[10 + k] * inv_nac;
    }
    const double* a = S.ba[b];
    br.torque_axis = a[0] * br.torque[0] + a[1] * br.torque[1] + a[2] * br.torque[2];
    br.power = -S.bom[b] * br.torque_axis;
    br.heat_rate = r[6];
    // running totals over up to 1e5 steps: compensated like the block sums
    const double inc[3] = {tad * br.torque_axis, tad * br.power, tad * br.heat_rate};
    double tot[3];
    for (int k = 0; k < 3; ++k) {
      KS acc{cum[k], cumc[k]};
      ks_add(acc, inc[k]);
      C->cum[b][k] = acc.s;
      C->cum_c[b][k] = acc.c;
      tot[k] = acc.s + acc.c;
    }
    br.torque_axis_int = tot[0];
    br.energy_int = tot[1];
    br.heat_int = tot[2];
    C->brep[b] = br;
    bheat[b] = br.heat_rate;
    bfin[b] = isfinite(br.torque_axis) && isfinite(br.heat_rate) && isfinite(br.force[0]) &&
              isfinite(br.force[1]) && isfinite(br.force[2]);
  }
  wave_lds_sync();
  if (b != 0) return;
  const double dtc = C->dt, t0 = C->t;
  const int64_t step0 = C->step, sub0 = C->substeps;
  const uint32_t flags0 = C->flags;
  KS heat{C->heat_total, C->heat_c}, diss{C->diss_total, C->diss_c};
  double qsum = 0.0;
  bool finite = true;
  for (int q = 0; q < S.nbody; ++q) {
    qsum += bheat[q];
    finite = finite && bfin[q];
  }
  const double t1 = t0 + tad;
  const int64_t step1 = step0 + 1, sub1 = sub0 + nac;
  const double hs = tad * qsum;
  const double ds = S.diss ? tad * res[q_diss] : 0.0;
  ks_add(heat, hs);
  ks_add(diss, ds);
  finite = finite && isfinite(res[1]) && isfinite(res[2]) && isfinite(res[3]) && isfinite(ds);
  const uint32_t flags1 = finite ? flags0 : (flags0 | F_NONFINITE);
  C->t = t1;
  C->step = step1;
  C->substeps = sub1;
  C->heat_total = heat.s;
  C->heat_c = heat.c;
  C->diss_total = diss.s;
  C->diss_c = diss.c;
  if (!finite) C->flags = flags1;
  sph_report R;
  R.t = t1;
  R.step = step1;
  R.n_ac = nac;
  R.dt_ad = tad;
  R.dt = dtc;
  R.mass = res[0];
  R.kinetic = res[1];
  R.thermal = res[2];
  R.mass_proxy = res[3];
  R.vmax = res[4];
  R.heat_step = hs;
  R.heat_total = heat.s + heat.c;
  R.substeps = sub1;
  R.diss_step = ds;
  R.diss_total = diss.s + diss.c;
  R.flags = (int32_t)flags1;
  C->rep = R;
}


// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
int grid_domain(int kid, int which) {
  switch (kid) {
    case SPH_K_CLEAR:
    case SPH_K_SCAN1:
    case SPH_K_SCAN3:
      return DOM_CELL;
    case SPH_K_POSE:
    case SPH_K_CONTACT:
    case SPH_K_WALLVEL:
      return DOM_SOLID;
    case SPH_K_SCAN2:
    case SPH_K_DT:
    case SPH_K_FINAL:
      return DOM_SLOT;
    case SPH_K_SCATTER:
    case SPH_K_CELLSORT:
    case SPH_K_REORDER:
      return which ? DOM_SOLID : DOM_FLUID;
    default:
      return DOM_FLUID;
  }
}

template <class P, bool STAGE>
static hipError_t launch_p(int kid, int which, int sub, const SlotDesc* T, const LaunchTab& L,
                           hipStream_t st) {
  const int dom = grid_domain(kid, which);
  const int nblk = L.blk0[dom][L.n];
  if (nblk <= 0) return hipSuccess;
  const dim3 g(nblk), b(BLOCK);
  switch (kid) {
    case SPH_K_CLEAR: hipLaunchKernelGGL(k_clear, g, b, 0, st, T, L); break;
    case SPH_K_POSE: hipLaunchKernelGGL(k_pose<P>, g, b, 0, st, T, L); break;
    case SPH_K_FOLD: hipLaunchKernelGGL(k_fold<P>, g, b, 0, st, T, L); break;
    case SPH_K_SCAN1: hipLaunchKernelGGL(k_scan1, g, b, 0, st, T, L); break;
    case SPH_K_SCAN2: hipLaunchKernelGGL(k_scan2, g, b, 0, st, T, L); break;
    case SPH_K_SCAN3: hipLaunchKernelGGL(k_scan3, g, b, 0, st, T, L); break;
    case SPH_K_SCATTER: hipLaunchKernelGGL(k_scatter, g, b, 0, st, T, L, which); break;
    case SPH_K_CELLSORT: hipLaunchKernelGGL(k_cellsort, g, b, 0, st, T, L, which); break;
    case SPH_K_REORDER: hipLaunchKernelGGL(k_reorder<P>, g, b, 0, st, T, L, which); break;
    case SPH_K_BUILD:
      // A grid that is resident at once lasts as long as one wavefront's runs, so
      // more wavefronts per block share them: sixteen where every block has a CU
      // of its own (48 blocks: 117 -> 61 us, 196 blocks: 120 -> 69), eight while
      // the blocks of 512 threads still fit together, two per CU in mixed
      // arithmetic, three in FP32 and FP64 (mixed: 313 blocks 133 -> 95 us, 469
      // 147 -> 105, but 664 148 -> 153; FP32, 766 blocks: 152 -> 118, FP64 139 ->
      // 123).  Larger grids fill the CUs by themselves, and there the sharing
      // costs a barrier (7437 blocks: 1047 us against 1014).
      if (g.x <= CUS) hipLaunchKernelGGL((k_build<P, WIDE, STAGE>), g, dim3(WIDE), 0, st, T, L);
      else if (g.x <= (sizeof(typename P::Pos) != sizeof(typename P::Real) ? 2 : 3) * CUS)
        hipLaunchKernelGGL((k_build<P, WIDE / 2, STAGE>), g, dim3(WIDE / 2), 0, st, T, L);
      else hipLaunchKernelGGL((k_build<P, BLOCK, STAGE>), g, b, 0, st, T, L);
      break;
    case SPH_K_SUMW: hipLaunchKernelGGL((k_sumw<P, STAGE>), g, b, 0, st, T, L); break;
    case SPH_K_CONTACT: hipLaunchKernelGGL(k_contact<P>, g, b, 0, st, T, L, nullptr, nullptr); break;
    case SPH_K_WALLVEL:
      // as the build (mixed: 92 blocks 68 -> 28 us, 350 110 -> 76; FP32: 540 89 -> 59;
      // FP64, which spills 20 bytes per lane at 1024 threads: 92 99 -> 49, 214 114 ->
      // 80); three blocks of 512 threads fit a CU in FP32 and mixed arithmetic, one in
      // FP64, which keeps blocks of 256 beyond 256 blocks
      if (g.x <= CUS) {
        hipLaunchKernelGGL((k_wallvel<P, WIDE>), g, dim3(WIDE), 0, st, T, L);
        break;
      }
      if constexpr (sizeof(typename P::Real) == 4) {
        if (g.x <= 3 * CUS) {
          hipLaunchKernelGGL((k_wallvel<P, WIDE / 2>), g, dim3(WIDE / 2), 0, st, T, L);
          break;
        }
      }
      hipLaunchKernelGGL((k_wallvel<P, BLOCK>), g, b, 0, st, T, L);
      break;
    case SPH_K_DT: hipLaunchKernelGGL(k_dt, g, b, 0, st, T, L); break;
    case SPH_K_VISC_HEAT:
      // which = 1: with the first acoustic sub-step's half update and momentum
      if (which == 1) {
        if (L.flags & TAB_MAT) {
          if (L.flags & TAB_DISS) hipLaunchKernelGGL((k_visc_heat<P, true, true, true, STAGE>), g, b, 0, st, T, L);
          else hipLaunchKernelGGL((k_visc_heat<P, false, true, true, STAGE>), g, b, 0, st, T, L);
        } else {
          if (L.flags & TAB_DISS) hipLaunchKernelGGL((k_visc_heat<P, true, false, true, STAGE>), g, b, 0, st, T, L);
          else hipLaunchKernelGGL((k_visc_heat<P, false, false, true, STAGE>), g, b, 0, st, T, L);
        }
      } else if (L.flags & TAB_MAT) {
        if (L.flags & TAB_DISS) hipLaunchKernelGGL((k_visc_heat<P, true, true, false, STAGE>), g, b, 0, st, T, L);
        else hipLaunchKernelGGL((k_visc_heat<P, false, true, false, STAGE>), g, b, 0, st, T, L);
      } else {
        if (L.flags & TAB_DISS) hipLaunchKernelGGL((k_visc_heat<P, true, false, false, STAGE>), g, b, 0, st, T, L);
        else hipLaunchKernelGGL((k_visc_heat<P, false, false, false, STAGE>), g, b, 0, st, T, L);
      }
      break;
    case SPH_K_HALF_A: hipLaunchKernelGGL(k_half_a<P>, g, b, 0, st, T, L, sub); break;
    case SPH_K_MOMENTUM: hipLaunchKernelGGL((k_momentum<P, STAGE>), g, b, 0, st, T, L, sub); break;
    case SPH_K_CONTINUITY: hipLaunchKernelGGL((k_continuity<P, STAGE>), g, b, 0, st, T, L, sub); break;
    case SPH_K_END: hipLaunchKernelGGL(k_end<P>, g, b, 0, st, T, L); break;
    case SPH_K_FINAL: hipLaunchKernelGGL(k_final, g, dim3(FINAL_BLOCK), 0, st, T, L); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// K: the fluid state in the caller's order, FP64.  Bound by the scattered
// stores (64 B per particle); a thread per sorted particle, so that the loads
// are contiguous.  Reading back 0.9 M particles took 26 ms with the reordering
// on the host and takes 6.4, nearly all of it the copy to the host.
template <class P>
__global__ __launch_bounds__(BLOCK) void k_export(const SlotDesc* table, int slot, double* x, double* v, double* rho,
                                                  double* T) {
#pragma clang fp contract(off)
  const SlotDesc& S = table[slot];
  const int k = blockIdx.x * BLOCK + threadIdx.x;
  if (k >= S.nf) return;
  const size_t o = S.fid[k];
  const typename P::Pos4 xk = gpc<typename P::Pos4>(S.xa)[k];
  const typename P::Real4 dk = gpc<typename P::Real4>(S.drift)[k], vk = gpc<typename P::Real4>(S.vr)[k];
  x[3 * o] = (double)xk.x + (double)dk.x;
  x[3 * o + 1] = (double)xk.y + (double)dk.y;
  x[3 * o + 2] = (double)xk.z + (double)dk.z;
  v[3 * o] = (double)vk.x;
  v[3 * o + 1] = (double)vk.y;
  v[3 * o + 2] = (double)vk.z;
  rho[o] = (double)vk.w + (P::kRel ? S.rho0 : 0.0);
  T[o] = (double)gpc<typename P::Temp>(S.T)[k];
}

hipError_t launch_export(int prec, const SlotDesc* table, int slot, int nblk, double* x, double* v, double* rho,
                         double* T, hipStream_t stream) {
  const dim3 g(nblk), b(BLOCK);
  switch (prec) {
    case SPH_PREC_MIXED: hipLaunchKernelGGL(k_export<PMixed>, g, b, 0, stream, table, slot, x, v, rho, T); break;
    case SPH_PREC_FP64: hipLaunchKernelGGL(k_export<PF64>, g, b, 0, stream, table, slot, x, v, rho, T); break;
    case SPH_PREC_FP32: hipLaunchKernelGGL(k_export<PF32>, g, b, 0, stream, table, slot, x, v, rho, T); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class P>
static hipError_t launch_contact_p(const SlotDesc* T, const LaunchTab& L, double* zout, double* part,
                                   double* mean, hipStream_t st) {
  const int nblk = L.blk0[DOM_SOLID][L.n];
  if (nblk > 0) hipLaunchKernelGGL(k_contact<P>, dim3(nblk), dim3(BLOCK), 0, st, T, L, zout, part);
  if (mean && L.blk0[DOM_SLOT][L.n] > 0)
    hipLaunchKernelGGL(k_contact_mean, dim3(L.blk0[DOM_SLOT][L.n]), dim3(BLOCK), 0, st, T, L,
                       (const double*)part, mean);
  return hipGetLastError();
}

hipError_t launch_contact(int prec, const SlotDesc* table, const LaunchTab& tab, double* zout, double* part,
                          double* mean, hipStream_t stream) {
  switch (prec) {
    case SPH_PREC_MIXED: return launch_contact_p<PMixed>(table, tab, zout, part, mean, stream);
    case SPH_PREC_FP64: return launch_contact_p<PF64>(table, tab, zout, part, mean, stream);
    case SPH_PREC_FP32: return launch_contact_p<PF32>(table, tab, zout, part, mean, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_kernel(int prec, int kid, int which, int sub, const SlotDesc* table,
                         const LaunchTab& tab, hipStream_t stream) {
  const bool stage = tab.flags & TAB_STAGE;
  switch (prec) {
    case SPH_PREC_MIXED:
      return stage ? launch_p<PMixed, true>(kid, which, sub, table, tab, stream)
                   : launch_p<PMixed, false>(kid, which, sub, table, tab, stream);
    case SPH_PREC_FP64: return launch_p<PF64, false>(kid, which, sub, table, tab, stream);
    case SPH_PREC_FP32:
      return stage ? launch_p<PF32, true>(kid, which, sub, table, tab, stream)
                   : launch_p<PF32, false>(kid, which, sub, table, tab, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sphk

// sph_device.h -- device-side building blocks shared by the solver kernels
// (sph_kernels.hip) and the particle relaxation (sph_relax.hip): precision
// policies, slot lookup of a batched launch, wave reductions, cell and pair
// geometry of the frozen neighbour rows, and the Wendland C2 kernel factor.
#pragma once
#include <math.h>

#include <type_traits>

#include "sph_internal.h"

namespace sphk {

// ---------------------------------------------------------------------------
// precision policies: position anchors, interaction arithmetic, temperature
// ---------------------------------------------------------------------------
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

struct PMixed {
  typedef double Pos;
  typedef float Real;
  typedef double Temp;
  typedef d4 Pos4;
  typedef f4 Real4;
  static constexpr bool kRel = true;   // density stored as rho - rho0
};
struct PF64 {
  typedef double Pos;
  typedef double Real;
  typedef double Temp;
  typedef d4 Pos4;
  typedef d4 Real4;
  static constexpr bool kRel = true;
};
struct PF32 {
  typedef float Pos;
  typedef float Real;
  typedef float Temp;
  typedef f4 Pos4;
  typedef f4 Real4;
  static constexpr bool kRel = false;  // absolute density in FP32
};

// Arrays live in device global memory; loads through these pointers compile
// to global (not flat) memory instructions.
#define GLB __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ GLB T* gp(void* p) {
  return (GLB T*)p;
}
template <class T>
__device__ __forceinline__ const GLB T* gpc(const void* p) {
  return (const GLB T*)p;
}

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Logical block numbers are laid out so that every XCD runs one
// contiguous range of blocks, i.e. one contiguous range of Morton-sorted
// particles, and the neighbour gathers of adjacent blocks hit the same L2.
constexpr int NXCD = 8;
__device__ __forceinline__ int xcd_block(int b, int g) {
  const int q = g / NXCD, r = g % NXCD;
  const int x = b % NXCD, k = b / NXCD;
  return x * q + min(x, r) + k;
}

__device__ __forceinline__ int find_slot(const LaunchTab& L, int dom, int& lb) {
  const int blk = xcd_block((int)blockIdx.x, (int)gridDim.x);
  int k = 0;
  for (int s = 1; s < L.n; ++s)
    if (blk >= L.blk0[dom][s]) k = s;
  lb = blk - L.blk0[dom][k];
  return L.slot[k];
}

// All words are loaded before any is looked at: a chain of branches would wait
// for memory once per word, at the head of every kernel.
__device__ __forceinline__ bool live(const SlotDesc& S) {
  const GLB SlotCtl* c = gpc<SlotCtl>(S.ctl);
  const uint32_t flags = c->flags;
  const int64_t step = c->step, target = c->target;
  return (flags == 0u) & (step < target);
}
// live, and the acoustic sub-step `sub` is one of this step's
__device__ __forceinline__ bool live_sub(const SlotDesc& S, int sub) {
  const int n_ac = gpc<SlotCtl>(S.ctl)->n_ac;
  return live(S) & (sub < n_ac);
}

// The same, decided once for the whole workgroup (thread 0's reading), with a
// barrier.  For the kernels that raise flags and whose wavefronts take indices
// from each other through LDS: another workgroup may raise a flag between two
// wavefronts' own readings, and the wavefronts that stayed would follow indices
// that the others never wrote.  Elsewhere a launch either raises no flags or
// shares no more than sums, which nobody reads of a faulted solve.
__device__ __forceinline__ bool live_block(const SlotDesc& S) {
  __shared__ int go;
  if (threadIdx.x == 0) go = live(S);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(go) != 0;
}

#define SLOT_FIND(DOM)                              \
  int lb_;                                          \
  const SlotDesc& S = table[find_slot(tab, DOM, lb_)]; \
  const int lb = lb_;
#define SLOT_PROLOGUE(DOM) \
  SLOT_FIND(DOM)           \
  if (!live(S)) return;

__device__ __forceinline__ void raise_flag(const SlotDesc& S, uint32_t f) {
  atomicOr(&S.ctl->flags, f);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
  return v;
}
__device__ __forceinline__ uint32_t wave_sum_u(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// value of lane l (wave-uniform l) as a scalar
__device__ __forceinline__ float rl(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double rl(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the wavefront by DPP lane moves (no LDS traffic), in a fixed
// order: pairs, quads, half-rows and rows of 16 by quad and mirror
// permutations, then row 1 and row 3 take the row before them (row_bcast:15)
// and rows 2 and 3 the first 32 lanes' sum (row_bcast:31).  The total is in
// lane 63; every lane must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_take(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_take(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <class Real>
__device__ __forceinline__ Real wave_total(Real v) {
  v += dpp_take<0xb1, 0xf>(v);    // quad_perm [1,0,3,2]
  v += dpp_take<0x4e, 0xf>(v);    // quad_perm [2,3,0,1]
  v += dpp_take<0x141, 0xf>(v);   // row_half_mirror
  v += dpp_take<0x140, 0xf>(v);   // row_mirror
  v += dpp_take<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_take<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return rl(v, WAVE - 1);
}

// Neumaier-compensated accumulator (additions only, so no contraction applies)
struct KS {
  double s, c;
};
__device__ __forceinline__ void ks_add(KS& k, double x) {
  double t = k.s + x;
  if (fabs(k.s) >= fabs(x)) k.c += (k.s - t) + x;
  else k.c += (x - t) + k.s;
  k.s = t;
}
__device__ __forceinline__ KS wave_ks(KS k) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    double s = __shfl_xor(k.s, o, WAVE);
    double c = __shfl_xor(k.c, o, WAVE);
    ks_add(k, s);
    k.c += c;
  }
  return k;
}

// cell of a point: floor((x - lo)/cs) per axis, FP64, correctly rounded
// division, no contraction.  Out-of-grid points are clamped and reported.
template <class PosT>
__device__ __forceinline__ bool cell_coords(const SlotDesc& S, PosT x, PosT y, PosT z, int c[3]) {
#pragma clang fp contract(off)
  const double p[3] = {(double)x, (double)y, (double)z};
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double f = floor((p[a] - S.lo[a]) / S.cs);
    if (!(f >= 0.0) || f >= (double)S.dims[a]) {
      ok = false;
      f = 0.0;
    }
    c[a] = (int)f;
  }
  return ok;
}

__device__ __forceinline__ int cell_linear(const SlotDesc& S, int cx, int cy, int cz) {
  return (cz * S.dims[1] + cy) * S.dims[0] + cx;
}

template <class P>
__device__ __forceinline__ typename P::Real rho_abs(const SlotDesc& S, typename P::Real s) {
  typedef typename P::Real Real;
  return P::kRel ? (Real)S.rho0 + s : s;
}
template <class P>
__device__ __forceinline__ typename P::Real press(const SlotDesc& S, typename P::Real s) {
  typedef typename P::Real Real;
  const Real c2 = (Real)(S.c0 * S.c0);
  return P::kRel ? c2 * s : c2 * (s - (Real)S.rho0);
}

// Reciprocal and reciprocal square root of the interaction type: the FP32
// hardware instructions (about 1 ulp) in the FP32 sweeps, IEEE operations in
// FP64 mode.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq(double x) { return 1.0 / sqrt(x); }

// A 32-bit integer in the fourth lane of a 4-wide record: its bit pattern in
// FP32 (never a NaN: values stay below 2^30), its exact value in FP64.
__device__ __forceinline__ float pack_index(uint32_t j, float) { return __builtin_bit_cast(float, j); }
__device__ __forceinline__ double pack_index(uint32_t j, double) { return (double)j; }
__device__ __forceinline__ uint32_t unpack_index(float w) { return __builtin_bit_cast(uint32_t, w); }
__device__ __forceinline__ uint32_t unpack_index(double w) { return (uint32_t)w; }

// Cell-relative positions.  At the build every particle stores
// o = x - (lo + c cs_r) rounded to the interaction type, with its cell c
// packed as 10 bits per axis.  A pair's vector is then
//   r_ij = (o_i - o_j) + (c_i - c_j) cs_r,
// where c_i - c_j is -1, 0 or 1 per axis, so the second term is exact and
// r_ij carries only the offsets' roundings (a few ulp of cs_r), however far
// the particles are from the grid origin.
__device__ __forceinline__ uint32_t pack_cell(const int c[3]) {
  return (uint32_t)c[0] | (uint32_t)c[1] << 10 | (uint32_t)c[2] << 20;
}
template <class Real, class Real4>
__device__ __forceinline__ void pair_vec(const Real4 a, uint32_t ca, const Real4 b, Real csr, Real& rx, Real& ry,
                                         Real& rz) {
  const uint32_t cb = unpack_index(b.w);
  const int dx = (int)(ca & 1023u) - (int)(cb & 1023u);
  const int dy = (int)((ca >> 10) & 1023u) - (int)((cb >> 10) & 1023u);
  const int dz = (int)(ca >> 20) - (int)(cb >> 20);
  rx = (a.x - b.x) + (Real)dx * csr;
  ry = (a.y - b.y) + (Real)dy * csr;
  rz = (a.z - b.z) + (Real)dz * csr;
}
template <class P, class Pos>
__device__ __forceinline__ typename P::Real4 cell_offset(const SlotDesc& S, Pos x, Pos y, Pos z, const int c[3]) {
#pragma clang fp contract(off)
  typedef typename P::Real Real;
  typename P::Real4 o;
  o.x = (Real)((double)x - (S.lo[0] + (double)c[0] * S.cs_r));
  o.y = (Real)((double)y - (S.lo[1] + (double)c[1] * S.cs_r));
  o.z = (Real)((double)z - (S.lo[2] + (double)c[2] * S.cs_r));
  o.w = pack_index(pack_cell(c), (Real)0);
  return o;
}

// F = (dW/dr)/r = kF (1 - q/2)^3 of the Wendland C2 kernel from |r|^2 and its
// reciprocal square root
template <class Real>
__device__ __forceinline__ Real kernel_F(Real r2, Real rs, Real inv_h, Real kF) {
  const Real q = r2 * rs * inv_h;
  const Real t = (Real)1 - (Real)0.5 * q;
  return kF * t * t * t;
}
// reciprocal square root kept finite at zero, so that a pair at distance zero
// (a null row entry) has q = 0 and F = kF without a select
__device__ __forceinline__ float rsq0(float r2) { return rsq(fmaxf(r2, 1e-37f)); }
__device__ __forceinline__ double rsq0(double r2) { return rsq(fmax(r2, 1e-300)); }

// One pair's terms of the sweeps.  The fused multiply-adds are written out, so
// a pair gives the same bits in every kernel that forms it (the fused and the
// separate first sub-step, staged and gathered neighbours).
template <class Real>
__device__ __forceinline__ Real dot_fma(Real ax, Real ay, Real az, Real bx, Real by, Real bz) {
  return fma(az, bz, fma(ax, bx, ay * by));
}
// p_i + sign p_j from the neighbour's stored density
template <class P>
__device__ __forceinline__ typename P::Real press_add(typename P::Real pi, typename P::Real sgn_c2, const SlotDesc& S,
                                                      typename P::Real w) {
#pragma clang fp contract(off)
  typedef typename P::Real Real;
  return fma(P::kRel ? w : w - (Real)S.rho0, sgn_c2, pi);
}
// Riemann momentum (eq. 10-12): the factor s with a_i += s r_ij.  dv = v_i - v_j,
// wj and Vj the neighbour's stored density and volume, cm2 = -2 V_i / m_i, c2 the squared sound speed.
template <class P>
__device__ __forceinline__ typename P::Real mom_factor(const SlotDesc& S, typename P::Real rhoi, typename P::Real pi,
                                                       typename P::Real cm2, typename P::Real c0, typename P::Real c2,
                                                       typename P::Real Vj, typename P::Real dot, typename P::Real inv,
                                                       typename P::Real wj, typename P::Real Fk) {
#pragma clang fp contract(off)
  typedef typename P::Real Real;
  const Real rhoj = rho_abs<P>(S, wj);
  const Real dU = -dot * inv;   // U_L - U_R = -(v_i - v_j) . e_ij
  const Real beta = fmin((Real)3 * fmax(dU, (Real)0), c0);
  const Real ps = fma((Real)0.5, press_add<P>(pi, c2, S, wj), rhoi * rhoj * beta * dU * rcp(rhoi + rhoj));
  return cm2 * Vj * ps * Fk;
}
// Riemann continuity (eq. 10, 11-13) per unit F: V_j [ (v_i - v_j) . r / 2 +
// (p_i - p_j) r / (c0 (rho_i + rho_j)) ]
template <class P>
__device__ __forceinline__ typename P::Real cont_factor(const SlotDesc& S, typename P::Real rhoi, typename P::Real pi,
                                                        typename P::Real c0, typename P::Real c2, typename P::Real Vj,
                                                        typename P::Real dot, typename P::Real rr,
                                                        typename P::Real wj) {
#pragma clang fp contract(off)
  typedef typename P::Real Real;
  const Real rhoj = rho_abs<P>(S, wj);
  const Real dv = fma((Real)0.5, dot, press_add<P>(pi, -c2, S, wj) * rr * rcp(c0 * (rhoi + rhoj)));
  return Vj * dv;
}

// Wall pressure of the one-sided Riemann problem (eq. 16-19): the factor s with
// a_i += s r_iw.  The right state of eq. 17: P_R = P_L + rho_f g . (x_w - x_f),
// rho_R from the EoS; then eq. 19.  c2 = 2 V_i / m_i, gr = g . r_iw.
template <class Real>
__device__ __forceinline__ Real wall_factor(Real rhoi, Real pi, Real c2, Real Vw, Real rho0, Real ic02, Real gr,
                                            Real Fk) {
#pragma clang fp contract(off)
  const Real PR = fma(-rhoi, gr, pi);
  const Real rhoR = fma(PR, ic02, rho0);
  const Real ps = fma(rhoi, PR, rhoR * pi) * rcp(rhoi + rhoR);
  return -c2 * Vw * ps * Fk;
}

// rows are streamed once per sweep: non-temporal loads keep them from
// evicting the gathered particle state in L2
template <class T>
__device__ __forceinline__ T ldnt(const GLB T* p) {
  return __builtin_nontemporal_load(p);
}

// ---------------------------------------------------------------------------
// staged candidates of a fluid block (BlkHead): their 16-byte records in LDS
// ---------------------------------------------------------------------------
struct RecPair {
  f4 a, b;
};
__device__ __forceinline__ BlkHead blk_head(const SlotDesc& S, int lb) {
  return __builtin_bit_cast(BlkHead, (u4)gpc<u4>(S.bhead)[lb]);
}

// whether wavefront w's rows hold local indices
__device__ __forceinline__ bool wave_staged(const BlkHead& hd, int w) { return (hd.waves >> w) & 1; }
// this wavefront's index in the block, as a scalar
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x) / WAVE; }

// This thread's candidates t, t + BLOCK, ... of a part's list.  Loaded whole,
// before the block's head is known (entries past the candidates are never
// used): a sweep's first wait covers the head, the list and its own records.
constexpr int STAGE_U = (STAGE_CAP + BLOCK - 1) / BLOCK;
struct StageList {
  uint32_t j[STAGE_U];
};
__device__ __forceinline__ StageList stage_list(const SlotDesc& S, int lb) {
  const int len = S.list_len;
  const GLB uint32_t* list = gpc<uint32_t>(S.blist) + (int64_t)lb * len;
  StageList s;
#pragma unroll
  for (int u = 0; u < STAGE_U; ++u) s.j[u] = list[min(u * BLOCK + (int)threadIdx.x, len - 1)];
  return s;
}

// store(l, load(solid or not, j), j) for every candidate l of the block, j its
// sorted index, and the barrier.  The solids start at a multiple of the
// wavefront, so the source is the same for a wavefront's lanes.  There is no
// branch between the loads (lanes past the candidates take particle 0 and store
// nothing): with one, each load would wait for the one before.  Half of a
// thread's records are in flight together.
template <class Load, class Store>
__device__ __forceinline__ void stage_block(const BlkHead& hd, const StageList& sl, Load&& load, Store&& store) {
  constexpr int U = STAGE_U, H = U / 2;
#pragma unroll
  for (int h = 0; h < U; h += H) {
    decltype(load(false, 0u)) r[H];
    uint32_t j[H];
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const int l = (h + u) * BLOCK + (int)threadIdx.x;
      j[u] = l < hd.n ? sl.j[h + u] : 0u;
      r[u] = load(__builtin_amdgcn_readfirstlane(l) >= hd.ns0 && hd.ns0 < hd.n, j[u]);
    }
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const int l = (h + u) * BLOCK + (int)threadIdx.x;
      if (l < hd.n) store((uint32_t)l, r[u], j[u]);
    }
  }
  __syncthreads();
}

// Shift of a neighbour's cell-relative position into the particle's cell, by
// stencil cell q: minus its offset times the cell edge, components SHIFT_LD
// apart so that a row entry's upper half (4 q) is the byte offset of x.
constexpr int SHIFT_LD = 32;
__device__ __forceinline__ void shift_table(float* shift, float csr) {
  const int q = threadIdx.x;
  if (q < 27) {
    shift[q] = (float)(1 - q % 3) * csr;
    shift[SHIFT_LD + q] = (float)(1 - (q / 3) % 3) * csr;
    shift[2 * SHIFT_LD + q] = (float)(1 - q / 9) * csr;
  }
}

// this lane's groups of four entries of its slice's staged rows (group c at
// [c * WAVE]): fluid, wall
__device__ __forceinline__ const GLB u4* row_groups(const SlotDesc& S, int i) {
  return (const GLB u4*)(gpc<uint32_t>(S.nrec) + (int64_t)(i >> 6) * S.kf * WAVE) + (i & (WAVE - 1));
}
__device__ __forceinline__ const GLB u4* wall_groups(const SlotDesc& S, int i) {
  return (const GLB u4*)(gpc<uint32_t>(S.srec) + (int64_t)(i >> 6) * S.ks * WAVE) + (i & (WAVE - 1));
}
// eight consecutive entries of a staged row
struct Row8 {
  u4 a, b;
};
__device__ __forceinline__ Row8 row_load(const GLB u4* G, int k) {
  const GLB u4* p = G + (int64_t)(k >> 2) * WAVE;
  return Row8{ldnt(p), ldnt(p + WAVE)};
}
__device__ __forceinline__ void row_entries(const Row8& r, uint32_t (&e)[8]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    e[u] = r.a[u];
    e[4 + u] = r.b[u];
  }
}
// four staged neighbours: position records, second records, cell shifts
struct Set4 {
  f4 o[4], v[4];
  float sx[4], sy[4], sz[4];
};
__device__ __forceinline__ void set_fetch(Set4& s, const u4 e, const char* smem, const float* shift) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const char* p = smem + (e[u] & 0xffffu);
    s.o[u] = *(const f4*)p;
    s.v[u] = *(const f4*)(p + 16 * STAGE_CAP);
    const float* q = (const float*)((const char*)shift + (e[u] >> 16));
    s.sx[u] = q[0];
    s.sy[u] = q[SHIFT_LD];
    s.sz[u] = q[2 * SHIFT_LD];
  }
}
// vector from neighbour u to the particle: the cell difference is exact, so
// this is pair_vec's result
__device__ __forceinline__ void set_vec(const Set4& s, int u, const f4 oi, float& rx, float& ry, float& rz) {
  rx = (oi.x - s.o[u].x) + s.sx[u];
  ry = (oi.y - s.o[u].y) + s.sy[u];
  rz = (oi.z - s.o[u].z) + s.sz[u];
}

// Walks a staged row (n entries, groups G, the first eight in r):
// pair(rx, ry, rz, neighbour's second record, its position record's w).  Four
// neighbours' LDS reads are issued before the previous four are used (with two
// waves per SIMD nothing else hides their latency), row groups two ahead.
// Rows are filled up to a multiple of eight with the particle itself, whose
// pair has r = 0 and no velocity, pressure or temperature difference: it adds
// exactly zero to every sum, so there is no mask.
template <class Pair>
__device__ __forceinline__ void staged_row(const GLB u4* G, Row8 r, int n, const char* smem, const float* shift,
                                           const f4 oi, Pair&& pair) {
  auto use = [&](const Set4& s) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float rx, ry, rz;
      set_vec(s, u, oi, rx, ry, rz);
      pair(rx, ry, rz, s.v[u], s.o[u].w);
    }
  };
  Row8 rn = r;
  if (8 < n) rn = row_load(G, 8);
  Set4 A, B;
  set_fetch(A, r.a, smem, shift);
  for (int k = 0; k < n; k += 8) {
    set_fetch(B, r.b, smem, shift);
    Row8 rl = rn;
    if (k + 16 < n) rl = row_load(G, k + 16);
    __builtin_amdgcn_sched_barrier(0);
    use(A);
    set_fetch(A, rn.a, smem, shift);   // past the last group: its entries again
    __builtin_amdgcn_sched_barrier(0);
    use(B);
    r = rn;
    rn = rl;
  }
}
// Walks a staged wall row four entries at a time: four(set, mask of the entries
// below n, as four flags).  Entries past n hold any record; the caller masks
// them, so that the four pairs form one straight run of instructions.
template <class Four>
__device__ __forceinline__ void staged_wall(const GLB u4* G, Row8 r, int n, const char* smem, const float* shift,
                                            Four&& four) {
  for (int k = 0; k < n; k += 8) {
    const Row8 c = r;
    if (k + 8 < n) r = row_load(G, k + 8);
#pragma unroll
    for (int h = 0; h < 8; h += 4) {
      Set4 s;
      set_fetch(s, h ? c.b : c.a, smem, shift);
      bool real[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) real[u] = k + h + u < n;
      four(s, real);
    }
  }
}

// block size of the single-block-per-slot kernels (reports, relaxation step)
constexpr int FINAL_BLOCK = 1024;

}  // namespace sphk

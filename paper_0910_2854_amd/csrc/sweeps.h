// sweeps.h -- HIP kernels of the FISH directional sweeps for gfx950.
//
// Layout: eight SoA arrays (rho, m_x, m_y, m_z, E, b_x, b_y, b_z) of one
// element type, x fastest, all sharing the strides (1, sy, sz).  Along an
// outflow axis every array has one extra layer so that a face array along its
// own normal can hold its last real face n; on a periodic axis face n is face
// 0 and is never stored.  Ghost cells are never stored either: every load
// maps its index (periodic wrap, or clamp for zeroth-order extrapolation).
//
// Both sweeps evaluate the 7-cell stencil of Sect. 3 in one pass, each cell read
// from HBM once but for halos, by one of two policies:
//   Strided (y and z sweeps): a lane owns a pencil segment and walks it as a
//     streaming pipeline: when cell c is loaded, the predictor of cell c-1 and
//     the corrector of cell c-3 are produced, and the value one position back is
//     the lane's own register from the last iteration.  Adjacent lanes are
//     adjacent along x, so every access is coalesced.
//   Lanes (x sweeps, and y and z of small boxes): a lane holds K consecutive cells
//     of a row along the sweep, a wave a window of 64 K of a stream of whole
//     rows, each padded by its ghosts; the scheme runs stage by stage with every
//     value in the lane of its cell, and a neighbour's value is the lane's own or
//     one DPP wave shift away.  The outer lanes of a window are a halo that the
//     neighbouring windows output, so no value crosses windows; the waves of a
//     block that work on one box take the windows of their rows in turn.  Along
//     x every access is coalesced and no row is transposed.
#pragma once

#include "layout.h"
#include "physics.h"

// Multiply-adds are fused only within one source expression (never across
// statements), so the rounding of every value is fixed by the source alone:
// the kernels that run the same arithmetic in different layouts (lanes of one
// cell or two, strided pencils, any work shape) give bitwise the same result.
#pragma clang fp contract(on)

namespace fish {

// The wave's box and its wave index within the box; false past the list
// (the whole wave exits together).
// Blocks are dealt round-robin to the 8 XCDs, each with its own L2.  With
// xcd_remap the list's block order is re-dealt so that the blocks an XCD runs
// are consecutive in the list (neighbouring pencils and rows, whose shared
// halo rows then hit in that XCD's L2); the full rounds of 8 are permuted, a
// ragged tail keeps its order.  With reverse the launch runs from the end of
// the list: every other sweep does, so that it begins with what the sweep
// before it left in the 256 MB cache of the memory (256^3 step, FP32 2.09 ->
// 2.05 ms, FP64 4.00 -> 3.97 ms).
__device__ __forceinline__ int list_block(const WorkList& wl) {
  const int blocks = (wl.nwaves + kBlockWaves - 1) / kBlockWaves;  // the grid of every launch over a list
  int b = (int)blockIdx.x;
  if (wl.reverse) b = blocks - 1 - b;
  if (wl.xcd_remap) {
    const int q = blocks >> 3;
    if (b < (q << 3)) b = (b & 7) * q + (b >> 3);
  }
  return b;
}

// The wave's box.  What a wave loads before its first data are scalar loads that
// miss, each a microsecond or less, and the sweep of a small box lasts five of
// them: so few of them wait for one another.  The launch's arguments (lines of 64
// bytes in host memory) are loaded together by touch(); a table of one box needs
// no look-up of the wave's box before its entry, nor of the entry before its step
// scalars; and the entry's lines and the step scalars are loaded together.  A
// double step before and after: 16^3 FP64 70 -> 60 us (with the launches of the
// start of the step merged), 32^3 FP32 82 -> 77, 64^3 FP32 160 -> 154, 203x77x131
// FP32 326 -> 312.  The entry among the arguments: 65, 80, 159, 318.
__device__ __forceinline__ int scalars_slot(const WorkList& wl, const BoxDesc& d) {
  int slot = wl.slot;
  if (!wl.one) {
    slot = d.slot;
    asm("" : "+s"(slot));
  }
  return slot;
}

template <int KIND, typename L>
__device__ __forceinline__ bool work_item(const L& launch, const BoxDesc*& d, int& lw) {
  const WorkList& wl = launch.wl;
  const int wave =
      __builtin_amdgcn_readfirstlane((int)((list_block(wl) * kBlock + (int)threadIdx.x) >> 6));
  int nwaves = wl.nwaves;
  touch(launch, nwaves);
  if (wave >= nwaves) return false;
  int box = 0;
  if (!wl.one) {
    box = wl.wave_box[wave];
    asm("" : "+s"(box));  // (a branch: as a select it would wait for the load)
  }
  d = wl.boxes + box;
  const Scalars* sc = launch.sc + scalars_slot(wl, *d);
  int first = d->wave0[KIND];
  asm("" : "+s"(first) : "s"(d->g.n[0]), "s"(d->ih[0]), "s"(sc->dt), "s"(sc->kf[0]));
  lw = wave - first;
  return true;
}

// ------------------------------------------------------------ addressing
// A pointer every lane of the wave holds (a stream position of the strided
// sweeps), pinned to scalar registers.  Without the pin the compiler folds the
// per-lane offset into the loop-invariant part of the address and pays a
// 64-bit vector add per load; pinned, the loads take the scalar base + 32-bit
// lane offset form.  The asm is empty: it only names the register class.
template <typename P>
__device__ __forceinline__ P in_sgpr(P p) {
  asm("" : "+s"(p));
  return p;
}

// Load/store at a wave-uniform base pointer plus a 32-bit per-lane byte
// offset (the scalar-base + vector-offset form of the global memory
// instructions: no 64-bit address arithmetic per lane).  The form needs the
// offset's zero extension in the block of the access; the empty asm on the
// offset keeps the compiler from extending a loop-invariant offset once before
// the loop, which would leave a 64-bit vector add per access inside it.  Every
// array the kernels touch is global memory: the address-space cast keeps the
// global form when the compiler cannot see where a pointer came from.
#define FISH_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T ld(const T* p, unsigned off_bytes) {
  asm("" : "+v"(off_bytes));
  return *(const FISH_GLOBAL T*)((const FISH_GLOBAL char*)p + off_bytes);
}
template <typename T>
__device__ __forceinline__ void st(T* p, unsigned off_bytes, T v) {
  asm("" : "+v"(off_bytes));
  *(FISH_GLOBAL T*)((FISH_GLOBAL char*)p + off_bytes) = v;
}
// With ONCE non-temporal, for values that a sweep touches once where
// WorkList::stream is set: the caches are left to the values used again.  A
// kernel of its own: a branch at the access cost 16 bytes of scratch per lane
// in the FP32 y/z fluid sweep.
template <bool ONCE, typename T>
__device__ __forceinline__ T ld_once(const T* p, unsigned off_bytes) {
  if (!ONCE) return ld(p, off_bytes);
  asm("" : "+v"(off_bytes));
  return __builtin_nontemporal_load((const FISH_GLOBAL T*)((const FISH_GLOBAL char*)p + off_bytes));
}
template <bool ONCE, typename T>
__device__ __forceinline__ void st_once(T* p, unsigned off_bytes, T v) {
  if (!ONCE) return st(p, off_bytes, v);
  asm("" : "+v"(off_bytes));
  __builtin_nontemporal_store(v, (FISH_GLOBAL T*)((FISH_GLOBAL char*)p + off_bytes));
}

// ------------------------------------------------------------ position history
// prev(cur, hin, hout): the value this quantity had one stream position
// earlier, read from the history hin; the history for the next position is
// written to hout.  The kernels alternate two history sets (hin/hout swap
// every position), so no register is copied to move the window.
template <typename V>
__device__ __forceinline__ V prev(const V& cur, const V& hin, V& hout) {
  hout = cur;
  return hin;
}

// Lane shifts: lane i takes lane i - 1, lane 0 zero (one DPP move a dword).
__device__ __forceinline__ float lane_shr(float cur) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(cur), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_shr(double cur) {
  const long long cb = __double_as_longlong(cur);
  const int lo = __builtin_amdgcn_mov_dpp((int)(cb & 0xffffffffll), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(cb >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// lane i takes lane i + 1, lane 63 zero
__device__ __forceinline__ float lane_shl(float cur) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(cur), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_shl(double cur) {
  const long long cb = __double_as_longlong(cur);
  const int lo = __builtin_amdgcn_mov_dpp((int)(cb & 0xffffffffll), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(cb >> 32), 0x130, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <typename T, int N>
struct Vec {
  T v[N];
};

// Branch-free maps for indices the stencils reach from a box row, i in
// [-8, n + 8): a clamp on outflow axes, at most one period added or removed
// on periodic ones (boxes thinner than 8 cells take the general wrap).  bc and
// n are uniform across the wave, so the choice of path is a scalar branch.
// The periodic map is the smallest of i, i + n and i - n as unsigned values
// (one of them lies in [0, n), the others are larger or negative), which is
// one three-way minimum.
__device__ __forceinline__ int map_cell_near(int i, int n, int bc) {
  if (bc) return min(max(i, 0), n - 1);
  if (n >= 8) {
    const unsigned a = (unsigned)i, b = (unsigned)(i + n), c = (unsigned)(i - n);
    return (int)min(a, min(b, c));
  }
  return wrap(i, n);
}
__device__ __forceinline__ int map_face_near(int i, int n, int bc) {
  if (bc) return min(max(i, 0), n);
  return map_cell_near(i, n, 0);
}

// ------------------------------------------------------------ L_d pipeline
template <typename T>
struct FluidArgs {
  const T* u[5];
  T* uo[5];
  const T* b[3];
  const T* phi;
  const T* wid[3];  // irregular mesh: cell widths per axis, else null
  Geo g;
  double gamma, alpha;
  int seg, nseg;   // strided: segment length along D and segments per pencil
  int rows_per_wave; // lanes: whole rows per wave
  const Scalars* sc;
  double i2h[3];     // 1 / (2 h_d)
};

// Kernel arguments of a fluid sweep over a batch: the pools and the list.
template <typename T>
struct FluidLaunch {
  const T* u[5];
  T* uo[5];
  const T* b[3];
  const T* phi;
  const T* wid[3];  // irregular meshes: every table box's cell widths per axis (at BoxDesc::woff), else null
  double gamma, alpha;
  WorkList wl;
  Scalars* sc;
};

// The arguments' lines (64 bytes each), loaded together with the first: x is
// what the kernel needs first.
template <typename T>
__device__ __forceinline__ void touch(const FluidLaunch<T>& L, int& x) {
  asm("" : "+s"(x) : "s"(L.u[0]), "s"(L.b[0]), "s"(L.sc));
}

// The per-box view of a launch (pointers at the box, its geometry and step
// scalars).
template <typename T, int KIND>
__device__ __forceinline__ FluidArgs<T> fluid_view(const FluidLaunch<T>& L, const BoxDesc& d) {
  FluidArgs<T> a;
  const long long off = d.off;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    a.u[i] = L.u[i] + off;
    a.uo[i] = L.uo[i] + off;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) a.b[i] = L.b[i] + off;
  a.phi = L.phi ? L.phi + off : nullptr;
#pragma unroll
  for (int i = 0; i < 3; ++i) a.wid[i] = L.wid[i] ? L.wid[i] + d.woff[i] : nullptr;
  a.g = d.g;
  a.gamma = L.gamma;
  a.alpha = L.alpha;
  const int D = KIND - K_FLUID_X;
  a.seg = d.par[KIND];
  a.nseg = d.nseg[KIND];
  a.rows_per_wave = d.par[KIND];
  a.sc = L.sc + scalars_slot(L.wl, d);
#pragma unroll
  for (int i = 0; i < 3; ++i) a.i2h[i] = d.i2h[i];
  (void)D;
  return a;
}

template <typename T>
__device__ __forceinline__ T load_phi(const T* phi, long long base, long long st, int s, int n, int bc) {
  if (s >= 0 && s < n) return phi[base + (long long)s * st];
  if (bc == 0 || n == 1) return phi[base + (long long)wrap(s, n) * st];
  // outflow: linear extrapolation from the two nearest real cells
  if (s < 0) {
    const T p0 = phi[base], p1 = phi[base + st];
    return p0 + (T)s * (p1 - p0);
  }
  const T p0 = phi[base + (long long)(n - 1) * st], p1 = phi[base + (long long)(n - 2) * st];
  return p0 + (T)(s - (n - 1)) * (p0 - p1);
}

// ------------------------------------------------ irregular meshes (Sect. 2.5)
// Width of the cell at stream index i along an axis, mapped as the cell is
// (a ghost takes the width of the cell it copies or wraps to).
template <typename T>
__device__ __forceinline__ T width_at(const T* w, int i, int n, int bc) {
  return w[map_cell(i, n, bc)];
}
// 1/(distance of the centres of the cells either side of a cell)
template <typename T>
__device__ __forceinline__ T inv_span(T wm, T w0, T wp) {
  return rcp(T(0.5) * wm + w0 + T(0.5) * wp);
}
// Per-position factors of the fluid sweep from the widths of cells c-4 .. c
// (w[0..4]): the predictor step of c-1 (dt/(2 dx)), the corrector step of c-3
// (dt/dx), the weights dx_i/(dx_i-1 + dx_i) and dx_i/(dx_i + dx_i+1) that put
// the limited slope of cell c-2 on its interfaces (the 1/2 of Eq. 34 on a
// uniform mesh), and the inverse centre spans of c-1 and c-3 for gravity.
template <typename T>
struct FluidNU {
  T kh1, kf3;
  T wl2, wr2, isp1, isp3;
};
template <typename T>
__device__ __forceinline__ FluidNU<T> fluid_nu(const T* w, T dt) {
  FluidNU<T> n;
  n.kh1 = T(0.5) * dt * rcp(w[3]);
  n.kf3 = dt * rcp(w[1]);
  n.wl2 = w[2] * rcp(w[1] + w[2]);
  n.wr2 = w[2] * rcp(w[2] + w[3]);
  n.isp1 = inv_span(w[2], w[3], w[4]);
  n.isp3 = inv_span(w[0], w[1], w[2]);
  return n;
}

template <typename T>
struct FluidConsts {
  T k_half, k_full;  // dt / (2h) and dt / h
  T half_dt, dt, inv2h, alpha;
  double gamma;
};

template <typename T, bool HSE>
struct FluidHist {
  CellQ<T, HSE> q0, q1;
  FieldQ<T> f;
  Vec<T, 5> F1, ap, am, Lp, bs, F2, ua, ub;
  T ph1, ph2, ph3, ph4, rp1, rp2, mp1, mp2, sp1;
  __device__ void zero() {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      q0.u[k] = q0.F[k] = q1.u[k] = q1.F[k] = T(0);
      F1.v[k] = ap.v[k] = am.v[k] = Lp.v[k] = bs.v[k] = F2.v[k] = ua.v[k] = ub.v[k] = T(0);
    }
    q0.vd = q0.cF = q0.d = q0.cS = q0.xiE = q0.sup = T(0);
    q1.vd = q1.cF = q1.d = q1.cS = q1.xiE = q1.sup = T(0);
    f.b[0] = f.b[1] = f.b[2] = T(0);
    f.b2 = 0.0;
    ph1 = ph2 = ph3 = ph4 = rp1 = rp2 = mp1 = mp2 = sp1 = T(0);
  }
};

// One stream position: loads of cell c in (uc, bc, phc); returns the
// corrected state of cell c-3 in un.
// GRAV: 0 none, 1 unsplit source in the predictor and corrector (Eqs. 41-43),
// 2 split kicks G(dt/2) L G(dt/2) (Eqs. 38-40): the entering cell is kicked
// by gh_c = (dt/2)(phi_c+1 - phi_c-1)/(2h), which the caller computes from
// its own loads for the cell the position maps to (the first positions of a
// stream have no history of phi; a ghost is then the exact copy of its kicked
// cell), before its first use; the output cell c-3 after its corrector, by
// the same factor formed from the history of phi.
// NU: irregular mesh, with the per-position factors in nu (uniform: k).
template <typename T, int D, int GRAV, bool HSE, int LIM, bool NU>
__device__ __forceinline__ void fluid_position(const T* uc_in, const Vec<T, 3>& bcc, T phc, T gh_c, const FluidConsts<T>& k, const FluidNU<T>& nu,
                                               const FluidHist<T, HSE>& hi, FluidHist<T, HSE>& ho, T* un) {
  T phm1 = T(0), phm2 = T(0), phm3 = T(0), phm4 = T(0);
  if (GRAV != 0 || HSE) {
    phm1 = prev(phc, hi.ph1, ho.ph1);
    phm2 = prev(phm1, hi.ph2, ho.ph2);
    phm3 = prev(phm2, hi.ph3, ho.ph3);
    phm4 = prev(phm3, hi.ph4, ho.ph4);
  }
  T uc[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) uc[i] = uc_in[i];
  if (GRAV == 2) gravity_kick<T, D>(uc, gh_c);
  // cell quantities of u at c and c-1
  const FieldQ<T> f0 = field_quantities<T>(bcc.v);
  CellQ<T, HSE> q0;
  cell_quantities<T, D, HSE>(uc, f0, k.gamma, q0);
  const CellQ<T, HSE> q0m = prev(q0, hi.q0, ho.q0);
  const FieldQ<T> f0m = prev(f0, hi.f, ho.f);
  // predictor flux at interface c-1/2 (Eq. 24, dissipation scaled by alpha)
  T Q[5];
  Vec<T, 5> F1;
  dissipation<T, HSE>(q0m, q0, phm1, phc, Q);
#pragma unroll
  for (int i = 0; i < 5; ++i) F1.v[i] = (half_flux<D>(q0m, i) + half_flux<D>(q0, i)) - k.alpha * Q[i];
  const Vec<T, 5> F1m = prev(F1, hi.F1, ho.F1);
  // predictor half step of cell c-1 (Eq. 41; Eq. 69 on an irregular mesh)
  T up[5];
  const T khalf = NU ? nu.kh1 : k.k_half;
  if (GRAV == 1) {
    T S[5];
    gravity_source<T, D>(q0m.u[RHO], q0m.u[MX + D], phc - phm2, NU ? nu.isp1 : k.inv2h, S);
#pragma unroll
    for (int i = 0; i < 5; ++i) up[i] = q0m.u[i] - khalf * (F1.v[i] - F1m.v[i]) + k.half_dt * S[i];
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) up[i] = q0m.u[i] - khalf * (F1.v[i] - F1m.v[i]);
  }
  // cell quantities of the half-step state of c-1 (field unchanged), and of c-2
  CellQ<T, HSE> q1;
  cell_quantities<T, D, HSE>(up, f0m, k.gamma, q1);
  const CellQ<T, HSE> q1m = prev(q1, hi.q1, ho.q1);
  // relaxed flux differences across interface c-3/2 (between c-2 and c-1)
  T Qc[5];
  Vec<T, 5> ap, am, bs;
  dissipation<T, HSE>(q1m, q1, phm2, phm1, Qc);
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const T dF = half_flux<D>(q1, i) - half_flux<D>(q1m, i);
    ap.v[i] = dF + Qc[i];
    am.v[i] = dF - Qc[i];
    bs.v[i] = (half_flux<D>(q1m, i) + half_flux<D>(q1, i)) - Qc[i];
  }
  const Vec<T, 5> apm = prev(ap, hi.ap, ho.ap);
  const Vec<T, 5> amm = prev(am, hi.am, ho.am);
  const Vec<T, 5> bsm = prev(bs, hi.bs, ho.bs);
  // limited second-order flux at interface c-5/2 (Eq. 34); both limiters
  // taken here belong to cell c-2 (its half-step state decides the switch)
  const T sup2 = LIM == 2 ? prev(q1.sup, hi.sp1, ho.sp1) : T(0);
  // (half their limited value; irregular mesh: each difference weighted to put
  // cell c-2's slope on its interfaces, which absorbs that half)
  Vec<T, 5> Lp, F2;
  constexpr T unit = T(NU ? 1.0 : 0.5) * limit_unit<LIM>();
  if (!NU) {
#pragma unroll
    for (int i = 0; i < 5; ++i) Lp.v[i] = limit_scaled<T, LIM>(sup2, apm.v[i], ap.v[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) Lp.v[i] = limit_scaled<T, LIM>(sup2, nu.wl2 * apm.v[i], nu.wr2 * ap.v[i]);
  }
  const Vec<T, 5> Lpm = prev(Lp, hi.Lp, ho.Lp);
  if (!NU) {
#pragma unroll
    for (int i = 0; i < 5; ++i) F2.v[i] = bsm.v[i] + unit * (Lpm.v[i] - limit_scaled<T, LIM>(sup2, amm.v[i], am.v[i]));
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i)
      F2.v[i] = bsm.v[i] + unit * (Lpm.v[i] - limit_scaled<T, LIM>(sup2, nu.wl2 * amm.v[i], nu.wr2 * am.v[i]));
  }
  const Vec<T, 5> F2m = prev(F2, hi.F2, ho.F2);
  // state of cell c-3 before the sweep
  // kick of c-3 (split gravity): phi of c-2 and c-4
  const T gh3 = GRAV == 2 ? k.half_dt * (phm2 - phm4) * (NU ? nu.isp3 : k.inv2h) : T(0);
  Vec<T, 5> um1;
#pragma unroll
  for (int i = 0; i < 5; ++i) um1.v[i] = q0m.u[i];
  const Vec<T, 5> um2 = prev(um1, hi.ua, ho.ua);
  const Vec<T, 5> um3 = prev(um2, hi.ub, ho.ub);
  const T* u3 = um3.v;
  // corrector of cell c-3 (Eq. 43)
  const T kfull = NU ? nu.kf3 : k.k_full;
  if (GRAV == 1) {
    const T rpm2 = prev(up[RHO], hi.rp1, ho.rp1);   // rho' of c-2
    const T rpm3 = prev(rpm2, hi.rp2, ho.rp2);      // rho' of c-3
    const T mpm2 = prev(up[MX + D], hi.mp1, ho.mp1);
    const T mpm3 = prev(mpm2, hi.mp2, ho.mp2);
    T S[5];
    gravity_source<T, D>(rpm3, mpm3, phm2 - phm4, NU ? nu.isp3 : k.inv2h, S);
#pragma unroll
    for (int i = 0; i < 5; ++i) un[i] = u3[i] - kfull * (F2.v[i] - F2m.v[i]) + k.dt * S[i];
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) un[i] = u3[i] - kfull * (F2.v[i] - F2m.v[i]);
    if (GRAV == 2) gravity_kick<T, D>(un, gh3);
  }
  (void)phm3;
}

// The step size of every sub-operator and the factors the sweeps take from
// it, dt / (2 h_d) and dt / h_d per axis (evaluated once per step, not in
// every wave of every sweep).
__device__ __forceinline__ void set_step(Scalars* s, const Geo& g, double dt) {
  s->dt = dt;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    s->kh[d] = dt / (2.0 * g.h[d]);
    s->kf[d] = dt / g.h[d];
  }
}

// The step factors of a sweep along D: dt / (2h) and dt / h from the box's
// step scalars (evaluated once per step with dt), 1 / (2h) from its table entry.
template <typename T>
__device__ __forceinline__ FluidConsts<T> fluid_consts(const FluidArgs<T>& a, int D) {
  const double dt = a.sc->dt;
  FluidConsts<T> k;
  k.k_half = (T)a.sc->kh[D];
  k.k_full = (T)a.sc->kf[D];
  k.half_dt = (T)(0.5 * dt);
  k.dt = (T)dt;
  k.inv2h = (T)a.i2h[D];
  k.alpha = (T)a.alpha;
  k.gamma = a.gamma;
  return k;
}

// Strided policy: wave w walks segment sg of 64 pencils.  The segment (hence
// every position and its boundary mapping along d) is uniform across the wave
// and lives in scalar registers; each lane only adds its pencil offset.
// Returns false for waves beyond the grid (the whole wave exits together).
// Two orders of the pencils (nA along x times nO along the other transverse
// axis, p = o * nA + a): contiguous (64 consecutive pencils per wave), or,
// with row_groups and nA >= 64, the four waves of a block on four
// consecutive rows o over the same 64 values of a, so that the neighbouring
// rows a sweep reads along o are mostly the block's own (L1/L2 hits).
__device__ __forceinline__ bool strided_map(int wave, int nA, int nO, int nseg, int row_groups, int& sg, int& p,
                                            bool& active) {
  const int lane = (int)(threadIdx.x & 63);
  if (row_groups && nA >= 64) {
    const int xc = (nA + 63) >> 6;
    const int per_seg = xc * ((nO + 3) >> 2) * 4;
    sg = wave / per_seg;
    if (sg >= nseg) return false;
    const int w = wave - sg * per_seg;
    const int g = w >> 2;
    const int o = (g / xc) * 4 + (w & 3);
    const int a = (g % xc) * 64 + lane;
    active = a < nA && o < nO;
    p = (o < nO ? o : nO - 1) * nA + (a < nA ? a : nA - 1);
    return true;
  }
  const int P = nA * nO;
  const int wps = (P + 63) >> 6;
  sg = wave / wps;
  if (sg >= nseg) return false;
  const int p0 = (wave - sg * wps) * 64 + lane;
  active = p0 < P;
  p = active ? p0 : P - 1;
  return true;
}

// Strided policy: one lane per pencil segment.  For D = y or z the lanes
// walk along x (each load of a wave is 64 consecutive values); for D = x (an
// alternative to the lanes policy) they walk along y, so that a wave's load
// touches 64 rows, one value of each.
template <typename T, int D, int GRAV, bool HSE, int LIM, bool NU, bool ONCE, bool AHEAD>
__global__ __launch_bounds__(256, sizeof(T) == 4 && GRAV == 0 && LIM != 2 && !NU ? 4 : 1) void fluid_strided_kernel(FluidLaunch<T> L) {
  constexpr int A = D == 0 ? 1 : 0;
  constexpr int O = D == 0 ? 2 : 3 - D;
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const BoxDesc* d;
  int lw;
  if (!work_item<K_FLUID_X + D>(L, d, lw)) return;
  const FluidArgs<T> a = fluid_view<T, K_FLUID_X + D>(L, *d);
  const Geo& g = a.g;
  const int nA = g.n[A], nO = g.n[O], nD = g.n[D];
  int sg, p;
  bool active;
  if (!strided_map(lw, nA, nO, a.nseg, L.wl.row_groups, sg, p, active)) return;
  const int s0 = sg * a.seg;
  const int s1 = min(nD, s0 + a.seg);
  int c[3];
  c[A] = p % nA;
  c[O] = p / nA;
  c[D] = 0;
  const long long stD = g.st[D];
  const int bcD = g.bc[D];
  // lane byte offsets (every array is below 4 GiB)
  const long long lbase = (long long)c[A] * g.st[A] + (long long)c[O] * g.st[O];
  const unsigned base = (unsigned)(lbase * (long long)sizeof(T));
  const unsigned hi1 = (unsigned)((lbase + (long long)(map_face(c[T1] + 1, g.n[T1], g.bc[T1]) - c[T1]) * g.st[T1]) *
                                  (long long)sizeof(T));
  const unsigned hi2 = (unsigned)((lbase + (long long)(map_face(c[T2] + 1, g.n[T2], g.bc[T2]) - c[T2]) * g.st[T2]) *
                                  (long long)sizeof(T));
  const FluidConsts<T> k = fluid_consts(a, D);
  FluidHist<T, HSE> hA, hB;
  hA.zero();
  hB.zero();
  struct In {
    T u[5];
    Vec<T, 3> bc;
    T phi, gh;
    T w[5];  // irregular mesh: widths of cells c-4 .. c
  };
  // inputs of position it (loads only: issued one position ahead of use)
  auto load = [&](int it) {
    In in;
    const int s = s0 - 3 + it;  // uniform
    const long long off = (long long)map_cell(s, nD, bcD) * stD;
#pragma unroll
    for (int i = 0; i < 5; ++i) in.u[i] = ld_once<ONCE>(in_sgpr(a.u[i] + off), base);
    const T* bD0 = in_sgpr(a.b[D] + (long long)map_face(s, nD, bcD) * stD);
    const T* bD1 = in_sgpr(a.b[D] + (long long)map_face(s + 1, nD, bcD) * stD);
    const T* b1 = in_sgpr(a.b[T1] + off);
    const T* b2 = in_sgpr(a.b[T2] + off);
    in.bc.v[D] = T(0.5) * (ld(bD0, base) + ld(bD1, base));
    in.bc.v[T1] = T(0.5) * (ld(b1, base) + ld(b1, hi1));
    in.bc.v[T2] = T(0.5) * (ld(b2, base) + ld(b2, hi2));
    in.phi = GRAV ? load_phi(a.phi, lbase, stD, s, nD, bcD) : T(0);
    if (NU) {
#pragma unroll
      for (int j = 0; j < 5; ++j) in.w[j] = width_at(a.wid[D], s - 4 + j, nD, bcD);
    }
    if (GRAV == 2) {
      // the kick of the cell this position maps to (a ghost is exactly the
      // copy of its kicked cell)
      const int sm = map_cell(s, nD, bcD);
      const T isp0 = NU ? inv_span(width_at(a.wid[D], sm - 1, nD, bcD), width_at(a.wid[D], sm, nD, bcD),
                                   width_at(a.wid[D], sm + 1, nD, bcD))
                        : k.inv2h;
      in.gh = k.half_dt * (load_phi(a.phi, lbase, stD, sm + 1, nD, bcD) -
                           load_phi(a.phi, lbase, stD, sm - 1, nD, bcD)) * isp0;
    } else {
      in.gh = T(0);
    }
    return in;
  };
  auto compute = [&](int it, const In& in, const FluidHist<T, HSE>& hi, FluidHist<T, HSE>& ho) {
    const int s = s0 - 3 + it;
    T un[5];
    const FluidNU<T> nu = NU ? fluid_nu(in.w, k.dt) : FluidNU<T>{};
    fluid_position<T, D, GRAV, HSE, LIM, NU>(in.u, in.bc, in.phi, in.gh, k, nu, hi, ho, un);
    if (it >= 6 && s - 3 < s1 && active) {
      const long long o = (long long)(s - 3) * stD;
#pragma unroll
      for (int i = 0; i < 5; ++i) st_once<ONCE>(in_sgpr(a.uo[i] + o), base, un[i]);
    }
  };
  // positions s0-3 .. s1+2, padded to an even count (the pad writes nothing;
  // the prefetch reads at most two positions past the end, mapped in range)
  const int npos = (s1 - s0) + 6;
  if (!AHEAD) {
    for (int it = 0; it < npos; it += 2) {
      compute(it, load(it), hA, hB);
      compute(it + 1, load(it + 1), hB, hA);
    }
    return;
  }
  In cur = load(0);
  for (int it = 0; it < npos; it += 2) {
    const In nxt = load(it + 1);
    compute(it, cur, hA, hB);
    cur = load(it + 2);
    compute(it + 1, nxt, hB, hA);
  }
}

// Speeds of one cell for Eq. (14)-(15): sp[d] = |v_d| + c_F,d on the active
// axes (0 on an axis with one cell), in the storage precision, with the
// pressure recovered in FP64; also flags a bad state (rho <= 0, p <= 0 or a
// non-finite value).  The pressure takes every conserved value and the cell's
// field, so a non-finite one leaves rho or p non-finite or p <= 0, and a
// speed that is not finite leaves their sum non-finite: four tests instead of
// one per value.  The division by h_d is left to cfl_of: it is monotonic, so
// the maximum of the divided speeds is the divided maximum, bitwise.
template <typename T>
__device__ __forceinline__ void cell_cfl_speeds(const T* u, const T* b, double gamma, const Geo& g, T* sp, int& bad) {
  const double b2 = field_quantities<T>(b).b2;
  const T p = pressure<T>(u, b2, gamma - 1.0);
  const T ri = rcp(u[RHO]);
  const T a2 = (T)gamma * p * ri;
  const T q = a2 + (T)b2 * ri;
  T sum = T(0);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    sp[d] = T(0);
    if (g.n[d] > 1) {
      sp[d] = fabs(u[MX + d] * ri) + fast_speed(q, a2, b[d], ri);
      sum += sp[d];
    }
  }
  const bool ok = u[RHO] > T(0) && p > T(0) && isfinite(u[RHO]) && isfinite(p) && isfinite(sum);
  if (!ok) bad = 1;
}

// max over the active axes of smax[d] / h_d (Eq. 15).
template <typename T>
__device__ __forceinline__ double cfl_of(const T* smax, const Geo& g) {
  double c = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.n[d] > 1) c = fmax(c, (double)smax[d] / g.h[d]);
  return c;
}

// Eq. (70), the CFL condition on an irregular mesh: max over the active axes
// of one cell's speed over its own width along that axis.
template <typename T>
__device__ __forceinline__ double cfl_of_cell(const T* sp, double wx, double wy, double wz, const Geo& g) {
  const double w[3] = {wx, wy, wz};
  double c = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.n[d] > 1) c = fmax(c, (double)sp[d] / w[d]);
  return c;
}

// The CFL reduction of a launch ends in one address per box, where atomics of
// all waves serialise (5.5 ns each: 181 us of a 256^3 FP32 sweep of 32768
// waves).  So the waves of a block that work on one box combine in LDS, the
// last of them publishes, and only where it exceeds what the box has already.
struct CflShared {
  unsigned long long bits;
  int bad, done;
};
// Every thread of the block calls this before any wave leaves the kernel.
__device__ __forceinline__ void cfl_shared_init(CflShared* sh) {
  if (threadIdx.x == 0) {
    sh->bits = 0ull;
    sh->bad = sh->done = 0;
  }
  __syncthreads();
}

// Reduce (cmax, bad) over the wave and publish it.  Every lane of the wave
// must reach this call.
__device__ __forceinline__ void publish_cfl(double cmax, int bad, Scalars* sc, const WorkList& wl, CflShared* sh) {
  unsigned long long bits = __double_as_longlong(cmax);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(bits, off, 64);
    bits = o > bits ? o : bits;
    bad |= __shfl_xor(bad, off, 64);
  }
  if ((threadIdx.x & 63) != 0) return;
  const int w0 = list_block(wl) * kBlockWaves;  // the block's waves w0 .. w1
  const int w1 = min(w0 + kBlockWaves, wl.nwaves) - 1;
  if (wl.one || wl.wave_box[w0] == wl.wave_box[w1]) {  // boxes are consecutive in the list
    __hip_atomic_fetch_max(&sh->bits, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(&sh->bad, bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__hip_atomic_fetch_add(&sh->done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) != w1 - w0) return;
    bits = __hip_atomic_load(&sh->bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    bad = __hip_atomic_load(&sh->bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // the published maximum only grows during a launch: an older value is safe
  if (bits > __hip_atomic_load(&sc->cmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&sc->cmax_bits, bits);
  if (bad) atomicOr(&sc->status, 1);
}

// ------------------------------------------------------------ L_x
// Lanes policy (D = x).  A lane holds K consecutive cells of an x row, a wave
// 64 K of a stream of whole rows, each padded by its ghosts.  A value of the
// neighbouring cell is the lane's own register or, at the lane's edge, the
// neighbour lane's by one DPP shift (folded into the instruction that uses it
// where that is possible).  The outer lanes of a window are a halo that the
// neighbouring windows output.
//   K = 2: both cells of a lane in one 8-byte (FP64: 16-byte) load and store,
//   and half the shifts, index arithmetic and halo of K = 1.  256^3: 200 us
//   (FP64 356), K = 1 233 (384) and K = 2 with single-cell loads 234 (393); with
//   the next window's loads ahead 261 (409), at 5 waves per SIMD instead of 6.
//   The waves of a block that work on one box take the windows of their rows in
//   turn: windows end inside the 128-byte lines of ten arrays, and the wave
//   that reads the rest of a line should do so while it is still in the L1 or
//   L2.  With a stretch of rows per wave the lines had left both (24 waves per
//   CU): the 256^3 FP32 sweep fetched 937 MB of its 537, now 714.
template <typename T, int K>
__device__ __forceinline__ void from_left(const T (&x)[K], T (&o)[K]) {
  o[0] = lane_shr(x[K - 1]);
#pragma unroll
  for (int j = 1; j < K; ++j) o[j] = x[j - 1];
}
template <typename T, int K>
__device__ __forceinline__ void from_right(const T (&x)[K], T (&o)[K]) {
#pragma unroll
  for (int j = 0; j + 1 < K; ++j) o[j] = x[j + 1];
  o[K - 1] = lane_shl(x[0]);
}
template <typename T, int K>
__device__ __forceinline__ void from_left(const Vec<T, 5> (&x)[K], Vec<T, 5> (&o)[K]) {
#pragma unroll
  for (int i = 0; i < 5; ++i) o[0].v[i] = lane_shr(x[K - 1].v[i]);
#pragma unroll
  for (int j = 1; j < K; ++j) o[j] = x[j - 1];
}
template <typename T, int K>
__device__ __forceinline__ void from_right(const Vec<T, 5> (&x)[K], Vec<T, 5> (&o)[K]) {
#pragma unroll
  for (int j = 0; j + 1 < K; ++j) o[j] = x[j + 1];
#pragma unroll
  for (int i = 0; i < 5; ++i) o[K - 1].v[i] = lane_shl(x[0].v[i]);
}
template <int D, typename T, bool HSE, int K>
__device__ __forceinline__ void cells_from_right(const CellQ<T, HSE> (&x)[K], CellQ<T, HSE> (&o)[K]) {
#pragma unroll
  for (int j = 0; j + 1 < K; ++j) o[j] = x[j + 1];
  const CellQ<T, HSE>& c = x[0];
  CellQ<T, HSE>& r = o[K - 1];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    r.u[i] = lane_shl(c.u[i]);
    r.F[i] = i == RHO ? r.F[i] : lane_shl(c.F[i]);
  }
  r.F[RHO] = T(0);
  r.d = lane_shl(c.d);
  r.sup = T(0);
  if (HSE) {
    r.vd = lane_shl(c.vd);
    r.cF = lane_shl(c.cF);
    r.cS = lane_shl(c.cS);
    r.xiE = lane_shl(c.xiE);
  } else {
    r.vd = r.cF = r.cS = r.xiE = T(0);
  }
}

// Per-cell factors of an irregular mesh from the widths of the cell and its
// neighbours (as FluidNU, which serves cells of several positions).
template <typename T>
struct CellNU {
  T kh, kf, wl, wr, isp;
};
template <typename T>
__device__ __forceinline__ CellNU<T> cell_nu(T wm, T w0, T wp, T dt) {
  CellNU<T> n;
  n.kh = T(0.5) * dt * rcp(w0);
  n.kf = dt * rcp(w0);
  n.wl = w0 * rcp(wm + w0);
  n.wr = w0 * rcp(w0 + wp);
  n.isp = inv_span(wm, w0, wp);
  return n;
}

// The sweep of a window: un of the lane's cells from their states u, field
// products f, potential phi and (split gravity) kicks gh; the arithmetic of
// fluid_position, with every value kept in the lane of its cell.  Interface j
// is the one right of cell j.
template <typename T, int D, int GRAV, bool HSE, int LIM, bool NU, int K>
__device__ __forceinline__ void fluid_window(const T (&u_in)[K][5], const FieldQ<T> (&f)[K], const T (&phi)[K],
                                             const T (&gh)[K], const CellNU<T> (&nu)[K], const FluidConsts<T>& k,
                                             T (&un)[K][5]) {
  T phl[K], phr[K];
  from_left(phi, phl);
  from_right(phi, phr);
  T u[K][5];
  CellQ<T, HSE> q[K], qr[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
#pragma unroll
    for (int i = 0; i < 5; ++i) u[j][i] = u_in[j][i];
    if (GRAV == 2) gravity_kick<T, D>(u[j], gh[j]);
    cell_quantities<T, D, HSE>(u[j], f[j], k.gamma, q[j]);
  }
  cells_from_right<D>(q, qr);
  // predictor
  Vec<T, 5> F[K], Fl[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    T Q[5];
    dissipation<T, HSE>(q[j], qr[j], phi[j], phr[j], Q);
#pragma unroll
    for (int i = 0; i < 5; ++i) F[j].v[i] = (half_flux<D>(q[j], i) + half_flux<D>(qr[j], i)) - k.alpha * Q[i];
  }
  from_left(F, Fl);
  T up[K][5];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const T khalf = NU ? nu[j].kh : k.k_half;
    if (GRAV == 1) {
      T S[5];
      gravity_source<T, D>(u[j][RHO], u[j][MX + D], phr[j] - phl[j], NU ? nu[j].isp : k.inv2h, S);
#pragma unroll
      for (int i = 0; i < 5; ++i) up[j][i] = u[j][i] - khalf * (F[j].v[i] - Fl[j].v[i]) + k.half_dt * S[i];
    } else {
#pragma unroll
      for (int i = 0; i < 5; ++i) up[j][i] = u[j][i] - khalf * (F[j].v[i] - Fl[j].v[i]);
    }
    cell_quantities<T, D, HSE>(up[j], f[j], k.gamma, q[j]);
  }
  cells_from_right<D>(q, qr);
  // corrector
  Vec<T, 5> ap[K], am[K], bs[K], al[K], Lp[K], Lm[K], Lmr[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    T Q[5];
    dissipation<T, HSE>(q[j], qr[j], phi[j], phr[j], Q);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const T dF = half_flux<D>(qr[j], i) - half_flux<D>(q[j], i);
      ap[j].v[i] = dF + Q[i];
      am[j].v[i] = dF - Q[i];
      bs[j].v[i] = (half_flux<D>(q[j], i) + half_flux<D>(qr[j], i)) - Q[i];
    }
  }
  from_left(ap, al);
#pragma unroll
  for (int j = 0; j < K; ++j) {
#pragma unroll
    for (int i = 0; i < 5; ++i)
      Lp[j].v[i] = NU ? limit_scaled<T, LIM>(q[j].sup, nu[j].wl * al[j].v[i], nu[j].wr * ap[j].v[i])
                      : limit_scaled<T, LIM>(q[j].sup, al[j].v[i], ap[j].v[i]);
  }
  from_left(am, al);
#pragma unroll
  for (int j = 0; j < K; ++j) {
#pragma unroll
    for (int i = 0; i < 5; ++i)
      Lm[j].v[i] = NU ? limit_scaled<T, LIM>(q[j].sup, nu[j].wl * al[j].v[i], nu[j].wr * am[j].v[i])
                      : limit_scaled<T, LIM>(q[j].sup, al[j].v[i], am[j].v[i]);
  }
  from_right(Lm, Lmr);
  constexpr T unit = T(NU ? 1.0 : 0.5) * limit_unit<LIM>();
#pragma unroll
  for (int j = 0; j < K; ++j) {
#pragma unroll
    for (int i = 0; i < 5; ++i) F[j].v[i] = bs[j].v[i] + unit * (Lp[j].v[i] - Lmr[j].v[i]);
  }
  from_left(F, Fl);
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const T kfull = NU ? nu[j].kf : k.k_full;
    if (GRAV == 1) {
      T S[5];
      gravity_source<T, D>(up[j][RHO], up[j][MX + D], phr[j] - phl[j], NU ? nu[j].isp : k.inv2h, S);
#pragma unroll
      for (int i = 0; i < 5; ++i) un[j][i] = u[j][i] - kfull * (F[j].v[i] - Fl[j].v[i]) + k.dt * S[i];
    } else {
#pragma unroll
      for (int i = 0; i < 5; ++i) un[j][i] = u[j][i] - kfull * (F[j].v[i] - Fl[j].v[i]);
      if (GRAV == 2) gravity_kick<T, D>(un[j], gh[j]);
    }
  }
}

// The rows of a block's waves that work on one box, as one stream of rows
// padded to L positions, dealt to those waves in turn by windows.
struct RowStream {
  int L, first, rows;  // positions per row; first row (y + z ny) and number of rows
  int turn, waves;     // this wave's turn among the group's waves
  float invL, inv_n;
  int n;               // rows per plane (n_y, or the face rows)
  __device__ void init(int lw, int box_waves, int rows_per_wave, int L_, int n_, int nrows) {
    const int in_block = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g0 = max(lw - in_block, 0);
    const int g1 = min(lw - in_block + kBlockWaves, box_waves);
    turn = lw - g0;
    waves = g1 - g0;
    first = g0 * rows_per_wave;
    rows = min(waves * rows_per_wave, nrows - first);
    L = L_;
    n = n_;
    invL = 1.0f / (float)L;
    inv_n = 1.0f / (float)n;
  }
  // a / b for 0 <= a < 2^24 and its remainder, from the rounded reciprocal
  __device__ static int divide(int a, int b, float inv, int& rem) {
    int q = (int)((float)a * inv);
    rem = a - q * b;
    if (rem < 0) {
      --q;
      rem += b;
    }
    if (rem >= b) {
      ++q;
      rem -= b;
    }
    return q;
  }
  // position in its row, y and z of stream position pos (0 <= pos < rows L)
  __device__ void locate(int pos, int& cp, int& y, int& z) const {
    const int rr = divide(pos, L, invL, cp);
    const int z0 = first / n;  // uniform
    z = z0 + divide(first - z0 * n + rr, n, inv_n, y);
  }
};

// Load/store of two consecutive elements (ld, st), aligned as one.
template <typename T>
struct PairOf {
  typedef T type __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};
template <typename T>
__device__ __forceinline__ void ld2(const T* p, unsigned off_bytes, T& v0, T& v1) {
  asm("" : "+v"(off_bytes));
  const typename PairOf<T>::type v =
      *(const FISH_GLOBAL typename PairOf<T>::type*)((const FISH_GLOBAL char*)p + off_bytes);
  v0 = v.x;
  v1 = v.y;
}
template <typename T>
__device__ __forceinline__ void st2(T* p, unsigned off_bytes, T v0, T v1) {
  asm("" : "+v"(off_bytes));
  typename PairOf<T>::type v;
  v.x = v0;
  v.y = v1;
  *(FISH_GLOBAL typename PairOf<T>::type*)((FISH_GLOBAL char*)p + off_bytes) = v;
}
template <typename T>
__device__ __forceinline__ void st2_once(T* p, unsigned off_bytes, T v0, T v1) {
  asm("" : "+v"(off_bytes));
  typename PairOf<T>::type v;
  v.x = v0;
  v.y = v1;
  __builtin_nontemporal_store(v, (FISH_GLOBAL typename PairOf<T>::type*)((FISH_GLOBAL char*)p + off_bytes));
}

// With CFL the sweep also reduces the CFL speed of the state it writes (the
// last sub-operator of a double step leaves the next step's time step ready).
template <typename T, int D, int GRAV, bool HSE, int LIM, bool CFL, bool NU, int K>
__global__ __launch_bounds__(256) void fluid_lanes_kernel(FluidLaunch<T> FL) {
  static_assert(D == 0 || !CFL, "the last sweep of a step is along x");
  constexpr int A = D == 0 ? 1 : 0, O = D == 0 ? 2 : 3 - D;  // rows: A fast
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  // an output depends on 3 cells to its left and 3 to its right, the last of
  // which takes its right face from a fourth
  constexpr int HL = (3 + K - 1) / K, HR = (4 + K - 1) / K;
  constexpr int OFF = HL * K;               // position of a row's cell 0
  constexpr int STEP = (64 - HL - HR) * K;  // cells a window outputs
  constexpr unsigned z4 = sizeof(T);
  __shared__ CflShared sh;
  if (CFL) cfl_shared_init(&sh);
  const BoxDesc* d;
  int lw;
  if (!work_item<K_FLUID_X + D>(FL, d, lw)) return;
  const FluidArgs<T> a = fluid_view<T, K_FLUID_X + D>(FL, *d);
  const Geo& g = a.g;
  const int n = g.n[D], bcD = g.bc[D];
  const int nrows = g.n[A] * g.n[O];  // < 2^32 bytes of cells
  const int rpw = a.rows_per_wave;
  RowStream rs;
  rs.init(lw, (nrows + rpw - 1) / rpw, rpw, (OFF + n + 4 + K - 1) / K * K, g.n[A], nrows);
  const int npos = rs.rows * rs.L;
  const int lane = threadIdx.x & 63;
  const FluidConsts<T> k = fluid_consts(a, D);
  T smax[3] = {T(0), T(0), T(0)};  // per axis, the largest |v_d| + c_F,d of the lane's cells
  double cnu = 0.0;  // irregular mesh: the CFL speed over widths, per cell
  int bad = 0;
  // byte offsets (arrays < 2^32 bytes): along the row, between rows, and to the
  // face above the row's cells along T1 and T2 (the next row, or on a periodic
  // axis from the last one back to the first)
  const unsigned sD = (unsigned)g.st[D] * z4, sA = (unsigned)g.st[A] * z4, sO = (unsigned)g.st[O] * z4;
  const unsigned up1 = (unsigned)g.st[T1] * z4, last1 = g.bc[T1] ? up1 : (unsigned)(1 - g.n[T1]) * up1;
  const unsigned up2 = (unsigned)g.st[T2] * z4, last2 = g.bc[T2] ? up2 : (unsigned)(1 - g.n[T2]) * up2;
  struct In {
    T u[K][5], bD[K], b1[K][2], b2[K][2];
    T phi[K], gh[K];
    T w[K], wt[2];   // irregular mesh: the cells' widths along D; the row's along T1 and T2
    unsigned o[K];   // byte offsets of the cells (mapped into the box)
    int c0;          // index of the first along D; out of the row: no output
  };
  auto load = [&](int win) {
    In in;
    const int pos = win * STEP + (lane - HL) * K;
    int cp, ra, ro;
    // positions before the stream or past it are moved onto it; they output nothing
    rs.locate(min(max(pos, 0), npos - K), cp, ra, ro);
    in.c0 = lane >= HL && lane < 64 - HR && pos < npos ? cp - OFF : -K;
    const unsigned base = (unsigned)ra * sA + (unsigned)ro * sO;
    const int c1 = T1 == A ? ra : ro, c2 = T2 == A ? ra : ro;
    const unsigned d1 = c1 + 1 < g.n[T1] ? up1 : last1, d2 = c2 + 1 < g.n[T2] ? up2 : last2;
    unsigned f[K];  // the cells' low faces along D
#pragma unroll
    for (int j = 0; j < K; ++j) {
      in.o[j] = base + (unsigned)map_cell_near(cp - OFF + j, n, bcD) * sD;
      f[j] = base + (unsigned)map_face_near(cp - OFF + j, n, bcD) * sD;
    }
    const unsigned* o = in.o;
    // along x a pair is split only where the row's ghosts wrap or are copies
    bool pairs = false;
    if constexpr (D == 0 && K == 2) pairs = __all(o[1] == o[0] + z4 && f[1] == f[0] + z4);
    if (D == 0 && K == 2 && pairs) {
      constexpr int J = K - 1;
#pragma unroll
      for (int i = 0; i < 5; ++i) ld2(a.u[i], o[0], in.u[0][i], in.u[J][i]);
      ld2(a.b[D], f[0], in.bD[0], in.bD[J]);
      ld2(a.b[T1], o[0], in.b1[0][0], in.b1[J][0]);
      ld2(a.b[T1], o[0] + d1, in.b1[0][1], in.b1[J][1]);
      ld2(a.b[T2], o[0], in.b2[0][0], in.b2[J][0]);
      ld2(a.b[T2], o[0] + d2, in.b2[0][1], in.b2[J][1]);
    } else {
#pragma unroll
      for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int i = 0; i < 5; ++i) in.u[j][i] = ld(a.u[i], o[j]);
        in.bD[j] = ld(a.b[D], f[j]);
        in.b1[j][0] = ld(a.b[T1], o[j]);
        in.b1[j][1] = ld(a.b[T1], o[j] + d1);
        in.b2[j][0] = ld(a.b[T2], o[j]);
        in.b2[j][1] = ld(a.b[T2], o[j] + d2);
      }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const int c = cp - OFF + j;
      const long long row = base / z4, st = g.st[D];
      in.phi[j] = GRAV ? load_phi(a.phi, row, st, c, n, bcD) : T(0);
      if (NU) in.w[j] = width_at(a.wid[D], c, n, bcD);
      if (GRAV == 2) {
        // the kick of the cell this position maps to (a ghost is exactly the
        // copy of its kicked cell)
        const int cm = map_cell(c, n, bcD);
        const T isp0 = NU ? inv_span(width_at(a.wid[D], cm - 1, n, bcD), width_at(a.wid[D], cm, n, bcD),
                                     width_at(a.wid[D], cm + 1, n, bcD))
                          : k.inv2h;
        in.gh[j] = k.half_dt * (load_phi(a.phi, row, st, cm + 1, n, bcD) - load_phi(a.phi, row, st, cm - 1, n, bcD)) *
                   isp0;
      } else {
        in.gh[j] = T(0);
      }
    }
    if (NU && CFL) {
      in.wt[0] = width_at(a.wid[T1], c1, g.n[T1], g.bc[T1]);
      in.wt[1] = width_at(a.wid[T2], c2, g.n[T2], g.bc[T2]);
    }
    return in;
  };
  auto compute = [&](const In& in) {
    T bDr[K], un[K][5], bc[K][3];
    from_right(in.bD, bDr);
    FieldQ<T> f[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      bc[j][D] = T(0.5) * (in.bD[j] + bDr[j]);
      bc[j][T1] = T(0.5) * (in.b1[j][0] + in.b1[j][1]);
      bc[j][T2] = T(0.5) * (in.b2[j][0] + in.b2[j][1]);
      f[j] = field_quantities<T>(bc[j]);
    }
    CellNU<T> nu[K]{};
    if (NU) {
      T wl[K], wr[K];
      from_left(in.w, wl);
      from_right(in.w, wr);
#pragma unroll
      for (int j = 0; j < K; ++j) nu[j] = cell_nu(wl[j], in.w[j], wr[j], k.dt);
    }
    fluid_window<T, D, GRAV, HSE, LIM, NU, K>(in.u, f, in.phi, in.gh, nu, k, un);
    // OFF is a multiple of K, so a row's cell 0 is the first of its lane, and
    // only the last lane of a row can hold a single cell of it
    bool out[K];
#pragma unroll
    for (int j = 0; j < K; ++j) out[j] = in.c0 >= 0 && in.c0 + j < n;
    if (K == 2 && out[K - 1]) {
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        if (D != 0) {
          st(a.uo[i], in.o[0], un[0][i]);
          st(a.uo[i], in.o[K - 1], un[K - 1][i]);
        } else if (FL.wl.stream) {
          st2_once(a.uo[i], in.o[0], un[0][i], un[K - 1][i]);
        } else {
          st2(a.uo[i], in.o[0], un[0][i], un[K - 1][i]);
        }
      }
    } else if (out[0]) {
#pragma unroll
      for (int i = 0; i < 5; ++i) st(a.uo[i], in.o[0], un[0][i]);
    }
    if (CFL) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        int cell_bad = 0;
        T sp[3];
        cell_cfl_speeds<T>(un[j], bc[j], a.gamma, g, sp, cell_bad);
        if (out[j]) {
          if (NU) {
            cnu = fmax(cnu, cfl_of_cell(sp, (double)in.w[j], (double)in.wt[0], (double)in.wt[1], g));
          } else {
#pragma unroll
            for (int dd = 0; dd < 3; ++dd) smax[dd] = fmax(smax[dd], sp[dd]);
          }
          bad |= cell_bad;
        }
      }
    }
  };
  const int nwin = (npos + STEP - 1) / STEP;
  for (int win = rs.turn; win < nwin; win += rs.waves) compute(load(win));
  if (CFL) publish_cfl(NU ? cnu : cfl_of(smax, g), bad, const_cast<Scalars*>(a.sc), FL.wl, &sh);
}

// ------------------------------------------------------------ B_d (fused)
// One kernel per field sweep: the transverse advection of b_t1 and b_t2 and
// the constraint update of b_d from the same edge fluxes (Eq. 64), without
// an edge-flux array in HBM.  A thread owns the face rows (t1-face c1, t2-cell
// c2) of b_t1, (t1-cell c1, t2-face c2) of b_t2 and (c1, c2) of b_d; the edge
// fluxes of the neighbouring rows c1+1 and c2+1 that the constraint needs are
// recomputed from the same inputs (bitwise the values their owners compute).
template <typename T>
struct FieldArgs {
  const T* rho;
  const T* md;             // momentum along d (the fluid state is held fixed)
  const T* bt[2];          // b_t1, b_t2 (input)
  const T* bd;             // b_d (input)
  T* bto[2];               // outputs
  T* bdo;
  const T* wid[3];         // irregular mesh: cell widths per axis, else null
  Geo g;
  int seg, nseg;           // strided policy
  int rows_per_wave;       // lanes policy
  const Scalars* sc;
  double ih[3];            // 1 / h_d
};

template <typename T>
struct FieldLaunch {
  const T* rho;
  const T* md;
  const T* bt[2];
  const T* bd;
  T* bto[2];
  T* bdo;
  const T* wid[3];  // irregular meshes: every table box's cell widths per axis (at BoxDesc::woff), else null
  WorkList wl;
  Scalars* sc;
};
template <typename T>
__device__ __forceinline__ void touch(const FieldLaunch<T>& L, int& x) {
  asm("" : "+s"(x) : "s"(L.rho), "s"(L.sc));
}

template <typename T, int KIND>
__device__ __forceinline__ FieldArgs<T> field_view(const FieldLaunch<T>& L, const BoxDesc& d) {
  FieldArgs<T> a;
  const long long off = d.off;
  a.rho = L.rho + off;
  a.md = L.md + off;
  a.bt[0] = L.bt[0] + off;
  a.bt[1] = L.bt[1] + off;
  a.bd = L.bd + off;
  a.bto[0] = L.bto[0] + off;
  a.bto[1] = L.bto[1] + off;
  a.bdo = L.bdo + off;
#pragma unroll
  for (int i = 0; i < 3; ++i) a.wid[i] = L.wid[i] ? L.wid[i] + d.woff[i] : nullptr;
  a.g = d.g;
  const int D = KIND - K_FIELD_X;
  a.seg = d.par[KIND];
  a.nseg = d.nseg[KIND];
  a.rows_per_wave = d.par[KIND];
  a.sc = L.sc + scalars_slot(L.wl, d);
#pragma unroll
  for (int i = 0; i < 3; ++i) a.ih[i] = d.ih[i];
  (void)D;
  return a;
}

template <typename T>
struct RowHist {
  T w1, w2, b1, b2, b3, b4, f2, p1, vb1, vb2, vb3, fp3, fp4, d34, lim4, P2;
  __device__ void zero() { w1 = w2 = b1 = b2 = b3 = b4 = f2 = p1 = vb1 = vb2 = vb3 = fp3 = fp4 = d34 = lim4 = P2 = T(0); }
};

// One position of one face row of b_t along d: Eq. (65) face velocity w0 at
// cell c, Eq. (66) smoothing, Eq. (68) interface velocity, Eq. (67)
// first-order upwind predictor flux, second-order limited upwind corrector
// flux (end of Sect. 2.4), Eq. (63).  Gives the edge flux at d-face c-3 (the
// interface between c-4 and c-3) and, for NEED_BN, the new b_t of cell c-4.
// Irregular mesh (Sect. 2.5): the weights that put the limited slope of cell
// c-3 on its interfaces, as in the fluid corrector; k_half and k_full are then those of cells c-2 and c-4.
template <typename T>
struct FieldW {
  T wl3, wr3;
};

template <typename T, int LIM, bool NEED_BN, bool NU>
__device__ __forceinline__ T row_position(T w0, T bb, T k_half, T k_full, const FieldW<T>& fw,
                                          const RowHist<T>& hi, RowHist<T>& ho, T& bn) {
  const T w1 = prev(w0, hi.w1, ho.w1);
  const T w2 = prev(w1, hi.w2, ho.w2);
  // outer neighbours first: an odd face velocity gives exact negatives here
  // and V = 0 exactly, which the <= 0 branch of Eq. (67) decides
  const T vbc = T(0.25) * ((w2 + w0) + T(2) * w1);   // v-bar of c-1
  const T b1 = prev(bb, hi.b1, ho.b1);                   // b of c-1
  const T fc = vbc * b1;                            // f of c-1
  const T vb1 = prev(vbc, hi.vb1, ho.vb1);                // v-bar of c-2
  const T V = vb1 + vbc;                            // twice that of interface c-3/2
  const T f2 = prev(fc, hi.f2, ho.f2);              // f of c-2
  const T P1 = V > T(0) ? f2 : fc;                  // Phi1 at c-3/2
  const T p1 = prev(P1, hi.p1, ho.p1);              // Phi1 at c-5/2
  const T b2 = prev(b1, hi.b2, ho.b2);              // b of c-2
  const T bp = b2 - k_half * (P1 - p1);             // b' of c-2
  const T fp2 = vb1 * bp;                           // f' of c-2
  const T vb2 = prev(vb1, hi.vb2, ho.vb2);          // v-bar of c-3
  const T vb3 = prev(vb2, hi.vb3, ho.vb3);          // v-bar of c-4
  const T V7 = vb3 + vb2;                           // twice that of interface c-7/2
  const T fp3 = prev(fp2, hi.fp3, ho.fp3);
  const T fp4 = prev(fp3, hi.fp4, ho.fp4);
  // the limited slope of cell c-3; that of c-4 is the one the last position took
  const T d23 = fp2 - fp3;
  const T d34 = prev(d23, hi.d34, ho.d34);
  const T lim3 = NU ? limit_scaled<T, LIM>(T(0), fw.wl3 * d34, fw.wr3 * d23) : limit_scaled<T, LIM>(T(0), d34, d23);
  const T lim4 = prev(lim3, hi.lim4, ho.lim4);
  constexpr T unit = T(NU ? 1.0 : 0.5) * limit_unit<LIM>();
  const T up = fp4 + unit * lim4;
  const T dn = fp3 - unit * lim3;
  const T P2c = V7 > T(0) ? up : dn;                // Phi2 at c-7/2
  if (NEED_BN) {
    const T P2 = prev(P2c, hi.P2, ho.P2);                // Phi2 at c-9/2
    const T b3 = prev(b2, hi.b3, ho.b3);
    const T b4 = prev(b3, hi.b4, ho.b4);
    bn = b4 - k_full * (P2c - P2);
  }
  return P2c;
}

template <typename T>
struct FieldConsts {
  T k_half, k_full, dt, ih1, ih2;
};

// The step factors of a field sweep along D (see fluid_consts).
template <typename T, int D>
__device__ __forceinline__ FieldConsts<T> field_consts(const FieldArgs<T>& a) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  FieldConsts<T> k;
  k.k_half = (T)a.sc->kh[D];
  k.k_full = (T)a.sc->kf[D];
  k.dt = (T)a.sc->dt;
  k.ih1 = (T)a.ih[T1];
  k.ih2 = (T)a.ih[T2];
  return k;
}

// Offsets a position needs besides the d offset.  Cells are relative to the
// thread's own cell (c1, c2) mapped into the box (on the outflow face rows
// c = n_t the mapped cell is n_t - 1, exactly the ghost the boundary copies);
// faces are relative to the face-row base (c1, c2).
struct FieldOffsets {
  long long c1m, c1p, c2m, c2p;   // cells (c1-1, c2), (c1+1, c2), (c1, c2-1), (c1, c2+1)
  long long f1p, f2p;             // t1-face c1+1, t2-face c2+1
};

template <int D>
__device__ __forceinline__ FieldOffsets field_offsets(const Geo& g, int c1, int c2) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  FieldOffsets o;
  const int m1 = map_cell(c1, g.n[T1], g.bc[T1]);
  const int m2 = map_cell(c2, g.n[T2], g.bc[T2]);
  o.c1m = (long long)(map_cell(c1 - 1, g.n[T1], g.bc[T1]) - m1) * g.st[T1];
  o.c1p = (long long)(map_cell(c1 + 1, g.n[T1], g.bc[T1]) - m1) * g.st[T1];
  o.c2m = (long long)(map_cell(c2 - 1, g.n[T2], g.bc[T2]) - m2) * g.st[T2];
  o.c2p = (long long)(map_cell(c2 + 1, g.n[T2], g.bc[T2]) - m2) * g.st[T2];
  o.f1p = (long long)(map_face(c1 + 1, g.n[T1], g.bc[T1]) - c1) * g.st[T1];
  o.f2p = (long long)(map_face(c2 + 1, g.n[T2], g.bc[T2]) - c2) * g.st[T2];
  return o;
}

// Byte offsets of everything one position reads, relative to the arrays'
// base pointers (which carry the d offset when it is wave-uniform).
struct FieldLane {
  unsigned cc, c1m, c1p, c2m, c2p;  // cells (c1, c2) and its four transverse neighbours
  unsigned fA, fB, fC, fD;          // b_t1 at t1-faces c1, c1+1; b_t2 at t2-faces c2, c2+1
};

template <typename T>
__device__ __forceinline__ FieldLane field_lane(long long base, long long ownc, const FieldOffsets& o, long long off) {
  constexpr long long z = sizeof(T);
  FieldLane l;
  l.cc = (unsigned)((ownc + off) * z);
  l.c1m = (unsigned)((ownc + off + o.c1m) * z);
  l.c1p = (unsigned)((ownc + off + o.c1p) * z);
  l.c2m = (unsigned)((ownc + off + o.c2m) * z);
  l.c2p = (unsigned)((ownc + off + o.c2p) * z);
  l.fA = (unsigned)((base + off) * z);
  l.fB = (unsigned)((base + off + o.f1p) * z);
  l.fC = l.fA;
  l.fD = (unsigned)((base + off + o.f2p) * z);
  return l;
}

// Inputs of one position of the four face rows (loads only, so that they can
// be issued a position ahead of their use).
template <typename T>
struct FieldIn {
  T md[5], rho[5];  // cells (c1, c2), (c1-1, c2), (c1+1, c2), (c1, c2-1), (c1, c2+1)
  T b[4];           // b_t1 at t1-faces c1, c1+1; b_t2 at t2-faces c2, c2+1
  T bd3;            // b_d at d-face c-3, which the constraint update of this position rewrites
};

template <typename T>
__device__ __forceinline__ FieldIn<T> field_load(const T* md, const T* rho, const T* bt0, const T* bt1,
                                                  const FieldLane& l) {
  FieldIn<T> in;
  const unsigned c[5] = {l.cc, l.c1m, l.c1p, l.c2m, l.c2p};
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    in.md[i] = ld(md, c[i]);
    in.rho[i] = ld(rho, c[i]);
  }
  in.b[0] = ld(bt0, l.fA);
  in.b[1] = ld(bt0, l.fB);
  in.b[2] = ld(bt1, l.fC);
  in.b[3] = ld(bt1, l.fD);
  in.bd3 = T(0);
  return in;
}

// Irregular mesh: the factors of one face row set (fixed along the pencil):
// per t-face the weights of its low and high cell in the interpolation of
// Eq. (65) (each the other cell's width over their sum), and 1/width of the
// thread's cell across t1 and t2 for Eq. (64).
template <typename T>
struct FieldRowNU {
  T a[4][2];  // faces A (t1-face c1), B (c1+1), C (t2-face c2), D (c2+1): low, high
  T ih1, ih2;
};
template <typename T>
__device__ __forceinline__ FieldRowNU<T> field_row_nu(T w1m, T w10, T w1p, T w2m, T w20, T w2p) {
  FieldRowNU<T> r;
  const T sA = rcp(w1m + w10), sB = rcp(w10 + w1p), sC = rcp(w2m + w20), sD = rcp(w20 + w2p);
  r.a[0][0] = w10 * sA;
  r.a[0][1] = w1m * sA;
  r.a[1][0] = w1p * sB;
  r.a[1][1] = w10 * sB;
  r.a[2][0] = w20 * sC;
  r.a[2][1] = w2m * sC;
  r.a[3][0] = w2p * sD;
  r.a[3][1] = w20 * sD;
  r.ih1 = rcp(w10);
  r.ih2 = rcp(w20);
  return r;
}
// Irregular mesh: the per-position factors from the widths of cells c-5 .. c-2.
template <typename T>
struct FieldPosNU {
  T kh, kf;
  FieldW<T> w;
};
template <typename T>
__device__ __forceinline__ FieldPosNU<T> field_pos_nu(const T* w, T dt) {
  FieldPosNU<T> f;
  f.kh = T(0.5) * dt * rcp(w[3]);
  f.kf = dt * rcp(w[1]);
  f.w.wl3 = w[2] * rcp(w[1] + w[2]);
  f.w.wr3 = w[2] * rcp(w[2] + w[3]);
  return f;
}
// Eq. (65) on an irregular mesh: linear interpolation between the two cell
// centres, two separate products (never fused, so the value is exactly odd
// when the velocities and widths are mirrored).
template <typename T>
__device__ __forceinline__ T face_interp(T alo, T vlo, T ahi, T vhi) {
  const T p = alo * vlo;
  const T q = ahi * vhi;
  return p + q;
}

// v_d of the five cells around the thread's pencil (Sect. 2.4: the fluid state
// current at B_d) and Eq. (65) on its four t-faces.
template <typename T, bool NU>
__device__ __forceinline__ void field_velocities(const FieldIn<T>& in, const FieldRowNU<T>& rn, T* w) {
  T v[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) v[i] = in.md[i] * rcp(in.rho[i]);
  if (!NU) {
    w[0] = T(0.5) * (v[1] + v[0]);
    w[1] = T(0.5) * (v[0] + v[2]);
    w[2] = T(0.5) * (v[3] + v[0]);
    w[3] = T(0.5) * (v[0] + v[4]);
  } else {
    w[0] = face_interp(rn.a[0][0], v[1], rn.a[0][1], v[0]);
    w[1] = face_interp(rn.a[1][0], v[0], rn.a[1][1], v[2]);
    w[2] = face_interp(rn.a[2][0], v[3], rn.a[2][1], v[0]);
    w[3] = face_interp(rn.a[3][0], v[0], rn.a[3][1], v[4]);
  }
}
// Eq. (64), physical signs: d/dt b_d = d_t1 Phi^t1 + d_t2 Phi^t2, from the edge
// fluxes of the four faces
template <typename T, bool NU>
__device__ __forceinline__ T field_change(T eA, T eB, T eC, T eD, const FieldConsts<T>& k, const FieldRowNU<T>& rn) {
  return k.dt * ((eB - eA) * (NU ? rn.ih1 : k.ih1) + (eD - eC) * (NU ? rn.ih2 : k.ih2));
}

// All four face rows at one position.
template <typename T, int LIM, bool NU>
__device__ __forceinline__ void field_compute(const FieldIn<T>& in, const FieldConsts<T>& k, const FieldRowNU<T>& rn,
                                              const FieldPosNU<T>& pn, const RowHist<T>* hi, RowHist<T>* ho, T& bn1,
                                              T& bn2, T& dbd) {
  T w[4];
  field_velocities<T, NU>(in, rn, w);
  const T kh = NU ? pn.kh : k.k_half, kf = NU ? pn.kf : k.k_full;
  T dummy;
  const T eA = row_position<T, LIM, true, NU>(w[0], in.b[0], kh, kf, pn.w, hi[0], ho[0], bn1);
  const T eB = row_position<T, LIM, false, NU>(w[1], in.b[1], kh, kf, pn.w, hi[1], ho[1], dummy);
  const T eC = row_position<T, LIM, true, NU>(w[2], in.b[2], kh, kf, pn.w, hi[2], ho[2], bn2);
  const T eD = row_position<T, LIM, false, NU>(w[3], in.b[3], kh, kf, pn.w, hi[3], ho[3], dummy);
  dbd = field_change<T, NU>(eA, eB, eC, eD, k, rn);
}

// Strided policy (d = y or z).
template <typename T, int D, int LIM, bool NU, bool ONCE>
__global__ __launch_bounds__(256) void field_strided_kernel(FieldLaunch<T> FL) {
  static_assert(D != 0, "x sweeps use the lanes policy");
  constexpr int A = 0;
  constexpr int O = 3 - D;
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const BoxDesc* d;
  int lw;
  if (!work_item<K_FIELD_X + D>(FL, d, lw)) return;
  const FieldArgs<T> a = field_view<T, K_FIELD_X + D>(FL, *d);
  const Geo& g = a.g;
  const int nD = g.n[D];
  const int rA = g.n[A] + g.bc[A];  // outflow adds the face row n
  const int rO = g.n[O] + g.bc[O];
  int sg, p;
  bool active;
  if (!strided_map(lw, rA, rO, a.nseg, FL.wl.row_groups, sg, p, active)) return;
  const int s0 = sg * a.seg;
  const int s1 = min(nD, s0 + a.seg);
  const bool last = (s1 == nD);
  const bool outD = g.bc[D] == 1;
  int c[3];
  c[A] = p % rA;
  c[O] = p / rA;
  c[D] = 0;
  const int c1 = c[T1], c2 = c[T2];
  const bool own1 = active && c2 < g.n[T2];   // b_t1 row is real
  const bool own2 = active && c1 < g.n[T1];   // b_t2 row is real
  const bool ownd = own1 && own2;             // b_d row is real
  const long long stD = g.st[D];
  const long long base = (long long)c1 * g.st[T1] + (long long)c2 * g.st[T2];
  const long long ownc = (long long)map_cell(c1, g.n[T1], g.bc[T1]) * g.st[T1] +
                         (long long)map_cell(c2, g.n[T2], g.bc[T2]) * g.st[T2];
  const FieldOffsets oc = field_offsets<D>(g, c1, c2);
  const FieldConsts<T> k = field_consts<T, D>(a);
  RowHist<T> hA[4], hB[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    hA[q].zero();
    hB[q].zero();
  }
  const FieldLane l = field_lane<T>(base, ownc, oc, 0);  // lane byte offsets, fixed along the pencil
  FieldRowNU<T> rn{};
  if (NU) {
    const T* w1 = a.wid[T1];
    const T* w2 = a.wid[T2];
    const int n1 = g.n[T1], n2 = g.n[T2], b1 = g.bc[T1], b2 = g.bc[T2];
    rn = field_row_nu(width_at(w1, c1 - 1, n1, b1), width_at(w1, c1, n1, b1), width_at(w1, c1 + 1, n1, b1),
                      width_at(w2, c2 - 1, n2, b2), width_at(w2, c2, n2, b2), width_at(w2, c2 + 1, n2, b2));
  }
  if (nD == 1) {
    // every ghost along d is the cell itself: the smoothing, the predictor and
    // the limited slopes leave v b of the cell as the edge flux, exactly, and
    // b_t as it was; a walk of nine positions otherwise (512^2 FP32: 21 us)
    const FieldIn<T> in = field_load<T>(a.md, a.rho, a.bt[0], a.bt[1], l);
    T w[4];
    field_velocities<T, NU>(in, rn, w);
    const T dbd = field_change<T, NU>(w[0] * in.b[0], w[1] * in.b[1], w[2] * in.b[2], w[3] * in.b[3], k, rn);
    if (own1) st(a.bto[0], l.fA, in.b[0]);
    if (own2) st(a.bto[1], l.fA, in.b[2]);
    if (ownd) {
      st(a.bdo, l.fA, ld(a.bd, l.fA) + dbd);
      if (outD) st(a.bdo + stD, l.fA, ld(a.bd + stD, l.fA) + dbd);
    }
    return;
  }
  auto load = [&](int it) {
    const int s = s0 - 4 + it;  // uniform
    const long long off = (long long)map_cell(s, nD, g.bc[D]) * stD;
    FieldIn<T> in = field_load<T>(in_sgpr(a.md + off), in_sgpr(a.rho + off), in_sgpr(a.bt[0] + off),
                                  in_sgpr(a.bt[1] + off), l);
    // b_d at d-face s-3, issued with the other loads (the constraint update
    // of this position rewrites it); the mapped face is in range everywhere
    const T* bd3 = in_sgpr(a.bd + (long long)map_face(s - 3, nD, g.bc[D]) * stD);
    in.bd3 = ld_once<ONCE>(bd3, l.fA);
    return in;
  };
  auto compute = [&](int it, const FieldIn<T>& in, const RowHist<T>* hi, RowHist<T>* ho) {
    const int s = s0 - 4 + it;
    T bn1, bn2, dbd;
    FieldPosNU<T> pn{};
    if (NU) {
      T w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = width_at(a.wid[D], s - 5 + j, nD, g.bc[D]);
      pn = field_pos_nu(w, k.dt);
    }
    field_compute<T, LIM, NU>(in, k, rn, pn, hi, ho, bn1, bn2, dbd);
    if (it >= 8 && s - 4 < s1) {
      const long long ob = (long long)(s - 4) * stD;
      if (own1) st_once<ONCE>(in_sgpr(a.bto[0] + ob), l.fA, bn1);
      if (own2) st_once<ONCE>(in_sgpr(a.bto[1] + ob), l.fA, bn2);
    }
    const int fd = s - 3;
    if (ownd && it >= 7 && (fd < s1 || (last && outD && fd == nD))) {
      const long long of = (long long)fd * stD;
      st_once<ONCE>(in_sgpr(a.bdo + of), l.fA, in.bd3 + dbd);
    }
  };
  // positions s0-4 .. s1+3, padded to an even count (the pad writes nothing;
  // the lookahead reads at most two positions past the end, mapped in range).
  // The lookahead costs one wave per SIMD in FP32 (5 -> 4) and hides more
  // than that (measured).
  const int npos = (s1 - s0) + 8;
  FieldIn<T> cur = load(0);
  for (int it = 0; it < npos; it += 2) {
    const FieldIn<T> nxt = load(it + 1);
    compute(it, cur, hA, hB);
    cur = load(it + 2);
    compute(it + 1, nxt, hB, hA);
  }
}

// ------------------------------------------------------------ B_x
// Lanes policy (D = x), as L_x: two cells of a face row per lane, windows dealt
// to the waves of a block, every value in the lane of its cell.  256^3: 160 us
// FP32, 277 us FP64 at one row per wave (one position per lane, streamed a row
// per wave: 220 and 385 us).  Bound by its loads, ten of fifteen of which are
// of the neighbouring rows: with sums in place of the scheme it takes 157 us,
// with the row's own values in place of the neighbours' 109.
//
// One face row of b_t: Eq. (65) face velocity w, Eq. (66) smoothing, Eq. (68)
// interface velocity, Eq. (67) first-order upwind predictor flux, second-order
// limited upwind corrector flux (end of Sect. 2.4), Eq. (63); the arithmetic of
// row_position.  e is the edge flux right of each cell; el and bn (the edge
// flux left of it, the new b_t) only with NEED_BN.
template <typename T, int LIM, bool NEED_BN, bool NU, int K>
__device__ __forceinline__ void face_row(const T (&w)[K], const T (&b)[K], const FieldConsts<T>& k,
                                         const CellNU<T> (&nu)[K], T (&e)[K], T (&bn)[K]) {
  T l[K], r[K], vb[K], vbr[K], f[K], fr[K], P[K], fp[K], fpr[K], d[K], lim[K];
  bool right[K];  // the interface velocity is positive: the left cell is upwind
  from_left(w, l);
  from_right(w, r);
#pragma unroll
  for (int j = 0; j < K; ++j) {
    // outer neighbours first: an odd face velocity gives exact negatives here
    // and an interface velocity of exactly 0, which the <= 0 branch decides
    vb[j] = T(0.25) * ((l[j] + r[j]) + T(2) * w[j]);
    f[j] = vb[j] * b[j];
  }
  from_right(vb, vbr);
  from_right(f, fr);
#pragma unroll
  for (int j = 0; j < K; ++j) {
    right[j] = vb[j] + vbr[j] > T(0);
    P[j] = right[j] ? f[j] : fr[j];
  }
  from_left(P, l);
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const T bp = b[j] - (NU ? nu[j].kh : k.k_half) * (P[j] - l[j]);
    fp[j] = vb[j] * bp;
  }
  from_right(fp, fpr);
#pragma unroll
  for (int j = 0; j < K; ++j) d[j] = fpr[j] - fp[j];
  from_left(d, l);
#pragma unroll
  for (int j = 0; j < K; ++j)
    lim[j] = NU ? limit_scaled<T, LIM>(T(0), nu[j].wl * l[j], nu[j].wr * d[j])
                : limit_scaled<T, LIM>(T(0), l[j], d[j]);
  from_right(lim, r);
  constexpr T unit = T(NU ? 1.0 : 0.5) * limit_unit<LIM>();
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const T up = fp[j] + unit * lim[j];
    const T dn = fpr[j] - unit * r[j];
    e[j] = right[j] ? up : dn;
  }
  if (NEED_BN) {
    from_left(e, l);
#pragma unroll
    for (int j = 0; j < K; ++j) bn[j] = b[j] - (NU ? nu[j].kf : k.k_full) * (e[j] - l[j]);
  }
}

template <typename T, int D, int LIM, bool NU, int K>
__global__ __launch_bounds__(256) void field_lanes_kernel(FieldLaunch<T> FL) {
  constexpr int A = D == 0 ? 1 : 0;  // rows: A fast
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  // an output depends on 4 cells either side
  constexpr int H = (4 + K - 1) / K;
  constexpr int OFF = H * K;               // position of a row's cell 0
  constexpr int STEP = (64 - 2 * H) * K;   // cells a window outputs
  constexpr unsigned z4 = sizeof(T);
  const BoxDesc* d;
  int lw;
  if (!work_item<K_FIELD_X + D>(FL, d, lw)) return;
  const FieldArgs<T> a = field_view<T, K_FIELD_X + D>(FL, *d);
  const Geo& g = a.g;
  const int n = g.n[D], bcD = g.bc[D], n1 = g.n[T1], n2 = g.n[T2];
  const int r1 = n1 + g.bc[T1], r2 = n2 + g.bc[T2];  // face rows
  const int nrows = r1 * r2;
  const int rpw = a.rows_per_wave;
  RowStream rs;
  rs.init(lw, (nrows + rpw - 1) / rpw, rpw, (n + 2 * OFF + K - 1) / K * K, T1 == A ? r1 : r2, nrows);
  const int npos = rs.rows * rs.L;
  const int lane = threadIdx.x & 63;
  const FieldConsts<T> k = field_consts<T, D>(a);
  // byte offsets to the cells and faces beside a row along T1 and T2: inside
  // the box one row, at its ends the wrap (periodic) or the copy (outflow); all
  // in unsigned arithmetic, where a negative offset wraps and wraps back
  const unsigned sD = (unsigned)g.st[D] * z4, s1 = (unsigned)g.st[T1] * z4, s2 = (unsigned)g.st[T2] * z4;
  const unsigned lo1 = g.bc[T1] ? 0u : (unsigned)(n1 - 1) * s1, hi1 = 0u - lo1;
  const unsigned lo2 = g.bc[T2] ? 0u : (unsigned)(n2 - 1) * s2, hi2 = 0u - lo2;
  for (int win = rs.turn; win * STEP < npos; win += rs.waves) {
    const int pos = win * STEP + (lane - H) * K;
    int cp, ra, ro;
    // positions before the stream or past it are moved onto it; they output nothing
    rs.locate(min(max(pos, 0), npos - K), cp, ra, ro);
    const int y = T1 == A ? ra : ro, z = T1 == A ? ro : ra;  // the row's indices along T1 and T2
    const int c0 = lane >= H && lane < 64 - H && pos < npos ? cp - OFF : -K;
    const unsigned row = (unsigned)z * s2 + (unsigned)y * s1;
    // the row past an outflow axis's last cell has faces only: its cell is the last one
    const bool end1 = y == n1, end2 = z == n2;
    const unsigned own = row - (end1 ? s1 : 0u) - (end2 ? s2 : 0u);
    const unsigned c1m = end1 ? 0u : (y == 0 ? lo1 : 0u - s1);
    const unsigned c1p = end1 ? 0u : (y == n1 - 1 ? hi1 : s1);
    const unsigned c2m = end2 ? 0u : (z == 0 ? lo2 : 0u - s2);
    const unsigned c2p = end2 ? 0u : (z == n2 - 1 ? hi2 : s2);
    const unsigned f1p = end1 ? 0u : (y == n1 - 1 && !g.bc[T1] ? hi1 : s1);
    const unsigned f2p = end2 ? 0u : (z == n2 - 1 && !g.bc[T2] ? hi2 : s2);
    unsigned x[K], xf[K];  // byte offsets in the row of the cells and of their low faces along D
#pragma unroll
    for (int j = 0; j < K; ++j) {
      x[j] = (unsigned)map_cell_near(cp - OFF + j, n, bcD) * sD;
      xf[j] = (unsigned)map_face_near(cp - OFF + j, n, bcD) * sD;
    }
    const unsigned c[5] = {own, own + c1m, own + c1p, own + c2m, own + c2p};
    T md[5][K], rho[5][K], b[4][K], bd[K];
    // along x a pair is split only where the row's ghosts wrap or are copies
    constexpr int J = K - 1;
    bool pairs = false;
    if constexpr (D == 0 && K == 2) pairs = __all(x[J] == x[0] + z4 && xf[J] == xf[0] + z4);
    if (D == 0 && K == 2 && pairs) {
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        ld2(a.md, c[i] + x[0], md[i][0], md[i][J]);
        ld2(a.rho, c[i] + x[0], rho[i][0], rho[i][J]);
      }
      ld2(a.bt[0], row + x[0], b[0][0], b[0][J]);
      ld2(a.bt[0], row + f1p + x[0], b[1][0], b[1][J]);
      ld2(a.bt[1], row + x[0], b[2][0], b[2][J]);
      ld2(a.bt[1], row + f2p + x[0], b[3][0], b[3][J]);
      ld2(a.bd, row + xf[0], bd[0], bd[J]);
    } else {
#pragma unroll
      for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          md[i][j] = ld(a.md, c[i] + x[j]);
          rho[i][j] = ld(a.rho, c[i] + x[j]);
        }
        b[0][j] = ld(a.bt[0], row + x[j]);
        b[1][j] = ld(a.bt[0], row + f1p + x[j]);
        b[2][j] = ld(a.bt[1], row + x[j]);
        b[3][j] = ld(a.bt[1], row + f2p + x[j]);
        bd[j] = ld(a.bd, row + xf[j]);
      }
    }
    FieldRowNU<T> rn{};
    CellNU<T> nu[K]{};
    if (NU) {
      rn = field_row_nu(width_at(a.wid[T1], y - 1, n1, g.bc[T1]), width_at(a.wid[T1], y, n1, g.bc[T1]),
                        width_at(a.wid[T1], y + 1, n1, g.bc[T1]), width_at(a.wid[T2], z - 1, n2, g.bc[T2]),
                        width_at(a.wid[T2], z, n2, g.bc[T2]), width_at(a.wid[T2], z + 1, n2, g.bc[T2]));
      T w[K], wl[K], wr[K];
#pragma unroll
      for (int j = 0; j < K; ++j) w[j] = width_at(a.wid[D], cp - OFF + j, n, bcD);
      from_left(w, wl);
      from_right(w, wr);
#pragma unroll
      for (int j = 0; j < K; ++j) nu[j] = cell_nu(wl[j], w[j], wr[j], k.dt);
    }
    T w[4][K];  // v_D on the t1-faces c1 and c1+1 and the t2-faces c2 and c2+1
#pragma unroll
    for (int j = 0; j < K; ++j) {
      FieldIn<T> in;
      T wj[4];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        in.md[i] = md[i][j];
        in.rho[i] = rho[i][j];
      }
      field_velocities<T, NU>(in, rn, wj);
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q][j] = wj[q];
    }
    T e[4][K], bn1[K], bn2[K], none[K];
    face_row<T, LIM, true, NU>(w[0], b[0], k, nu, e[0], bn1);
    face_row<T, LIM, false, NU>(w[1], b[1], k, nu, e[1], none);
    face_row<T, LIM, true, NU>(w[2], b[2], k, nu, e[2], bn2);
    face_row<T, LIM, false, NU>(w[3], b[3], k, nu, e[3], none);
    // the change of b_D at the face right of the cell; a cell's own face is the
    // one left of it
    T dr[K], dbd[K];
#pragma unroll
    for (int j = 0; j < K; ++j) dr[j] = field_change<T, NU>(e[0][j], e[1][j], e[2][j], e[3][j], k, rn);
    from_left(dr, dbd);
    // cells [0, n) of b_t, faces [0, n) of b_D and on an outflow axis face n
    const bool own1 = !end2, own2 = !end1;
    auto put = [&](T* p, unsigned o0, unsigned o1, T v0, T v1) {
      if (D != 0) {
        st(p, o0, v0);
        st(p, o1, v1);
      } else if (FL.wl.stream) {
        st2_once(p, o0, v0, v1);
      } else {
        st2(p, o0, v0, v1);
      }
    };
    if (K == 2 && c0 >= 0 && c0 + 1 < n) {
      if (own1) put(a.bto[0], row + x[0], row + x[J], bn1[0], bn1[J]);
      if (own2) put(a.bto[1], row + x[0], row + x[J], bn2[0], bn2[J]);
    } else if ((unsigned)c0 < (unsigned)n) {
      if (own1) st(a.bto[0], row + x[0], bn1[0]);
      if (own2) st(a.bto[1], row + x[0], bn2[0]);
    }
    if (own1 && own2) {
      const int nf = n + (bcD ? 1 : 0);
      if (K == 2 && c0 >= 0 && c0 + 1 < nf)
        put(a.bdo, row + xf[0], row + xf[J], bd[0] + dbd[0], bd[J] + dbd[J]);
      else if ((unsigned)c0 < (unsigned)nf)
        st(a.bdo, row + xf[0], bd[0] + dbd[0]);
    }
  }
}

// ------------------------------------------------------------ CFL + state check
template <typename T>
struct CheckLaunch {
  const T* u[5];
  const T* b[3];
  const T* wid[3];  // irregular meshes: every table box's cell widths per axis (at BoxDesc::woff), else null
  double gamma;
  WorkList wl;
  Scalars* sc;
};
template <typename T>
__device__ __forceinline__ void touch(const CheckLaunch<T>& L, int& x) {
  asm("" : "+s"(x) : "s"(L.u[0]), "s"(L.sc));
}

// Eq. (14)-(15) on the stored state: the CFL speed of every cell (the same
// function, hence bitwise the same value, as the reduction fused into the
// last sweep of a step) and the state check (rho > 0, p > 0, every value
// finite).  A wave covers 64 * par consecutive cells of its box (x fastest);
// each lane steps its cell index by 64, never dividing inside the loop.
template <typename T>
__global__ __launch_bounds__(256) void check_cfl_kernel(CheckLaunch<T> L) {
  __shared__ CflShared sh;
  cfl_shared_init(&sh);
  const BoxDesc* d;
  int lw;
  if (!work_item<K_CHECK>(L, d, lw)) return;
  const Geo g = d->g;
  const long long off = d->off;
  const int n0 = g.n[0], n1 = g.n[1], n2 = g.n[2];
  const long long ncell = (long long)n0 * n1 * n2;
  const long long c0 = (long long)lw * 64 * d->par[K_CHECK];
  const long long c1 = min(ncell, c0 + 64ll * d->par[K_CHECK]);
  const T* u[5];
  const T* b[3];
#pragma unroll
  for (int f = 0; f < 5; ++f) u[f] = L.u[f] + off;
#pragma unroll
  for (int f = 0; f < 3; ++f) b[f] = L.b[f] + off;
  const unsigned st1 = (unsigned)g.st[1], st2 = (unsigned)g.st[2];
  constexpr unsigned z4 = sizeof(T);
  long long c = c0 + (threadIdx.x & 63);
  int x = (int)(c % n0);
  const long long r = c / n0;
  int y = (int)(r % n1);
  int zz = (int)(r / n1);
  T smax[3] = {T(0), T(0), T(0)};
  double cnu = 0.0;                      // irregular mesh: per-cell speeds over widths
  const bool nu = L.wid[0] != nullptr;   // uniform across the launch
  const T* wx = nu ? L.wid[0] + d->woff[0] : nullptr;
  const T* wy = nu ? L.wid[1] + d->woff[1] : nullptr;
  const T* wz = nu ? L.wid[2] + d->woff[2] : nullptr;
  int bad = 0;
  for (; c < c1; c += 64) {
    const unsigned s = (unsigned)x + (unsigned)y * st1 + (unsigned)zz * st2;
    const unsigned o = s * z4;
    T uc[5], bc[3];
#pragma unroll
    for (int f = 0; f < 5; ++f) uc[f] = ld(u[f], o);
    const unsigned sx = (unsigned)(map_face_near(x + 1, n0, g.bc[0]) - x);
    const unsigned sy = (unsigned)(map_face_near(y + 1, n1, g.bc[1]) - y) * st1;
    const unsigned sz = (unsigned)(map_face_near(zz + 1, n2, g.bc[2]) - zz) * st2;
    bc[0] = T(0.5) * (ld(b[0], o) + ld(b[0], (s + sx) * z4));
    bc[1] = T(0.5) * (ld(b[1], o) + ld(b[1], (s + sy) * z4));
    bc[2] = T(0.5) * (ld(b[2], o) + ld(b[2], (s + sz) * z4));
    T sp[3];
    cell_cfl_speeds<T>(uc, bc, L.gamma, g, sp, bad);
    if (nu) {
      cnu = fmax(cnu, cfl_of_cell(sp, (double)wx[x], (double)wy[y], (double)wz[zz], g));
    } else {
#pragma unroll
      for (int dd = 0; dd < 3; ++dd) smax[dd] = fmax(smax[dd], sp[dd]);
    }
    x += 64;
    while (x >= n0) {
      x -= n0;
      if (++y == n1) {
        y = 0;
        ++zz;
      }
    }
  }
  publish_cfl(nu ? cnu : cfl_of(smax, g), bad, L.sc + scalars_slot(L.wl, *d), L.wl, &sh);
}

}  // namespace fish

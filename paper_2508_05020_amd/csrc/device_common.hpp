// Device helpers shared by the HIP kernels of libamr: patch-pool
// addressing, physical-boundary mapping, same-level cell lookup through the
// level maps, MC-limited prolongation, the CFL rate of a cell, a block-wide
// maximum, and the XCD-contiguous block-to-work-item mapping.
//
// Included by the .hip sources only, after their fp-contract pragma.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "amr_internal.hpp"

namespace amr {
namespace {


constexpr int NG = kNG;

__device__ __forceinline__ int bc_map(int g, int N, int periodic) {
  if (periodic) {
    g %= N;
    return g < 0 ? g + N : g;
  }
  return g < 0 ? 0 : (g >= N ? N - 1 : g);
}

// bc_map for an index at most one period outside the domain
__device__ __forceinline__ int bc_near(int g, int N, int periodic) {
  if (periodic) return g < 0 ? g + N : (g >= N ? g - N : g);
  return g < 0 ? 0 : (g >= N ? N - 1 : g);
}

template <int D>
__device__ __forceinline__ int box_off(int full, int x, int y, int z) {
  // offsets inside one patch fit 32 bits, and the factors 24 (one full-rate
  // 24-bit multiply-add each instead of 64-bit products)
  if constexpr (D == 1) return x;
  if constexpr (D == 2) return __mul24(y, full) + x;
  return __mul24(__mul24(z, full) + y, full) + x;
}

template <int D>
__device__ __forceinline__ int var_stride(int full) {
  if constexpr (D == 1) return full;
  if constexpr (D == 2) return __mul24(full, full);
  return __mul24(__mul24(full, full), full);
}

__device__ __forceinline__ long long patch_base(const DevMesh& m, int pid, int l) {
  return m.lv[l].pool_off + (long long)(pid - m.lv[l].pid_base) * m.lv[l].stride;
}

template <int D>
__device__ __forceinline__ int map_at(const DevMesh& m, int l, const int q[3]) {
  const LevelC& L = m.lv[l];
  int idx = q[0];
  if constexpr (D >= 2) idx += L.np * q[1];
  if constexpr (D >= 3) idx += L.np * L.np * q[2];
  return m.map[L.map_off + idx];
}

// v / d for 0 <= v where mul = ceil(2^32 / d) gives the exact quotient (one
// product instead of an integer division of about 25 instructions), or by
// division where mul is 0
__device__ __forceinline__ int div_by(int v, int d, unsigned mul) {
  return mul ? (int)__umulhi((unsigned)v, mul) : v / d;
}

// Same-level patches around the patch at pc, by offset code (o0+1) + 3 (o1+1)
// + 9 (o2+1), o in {-1,0,1}^D (periodic wrap), as the offsets of their data in
// the state buffer (-1 where no patch or outside a non-periodic domain); one
// per thread of the first 3^D.
template <int D>
__device__ __forceinline__ void load_neighbours(const DevMesh& m, int l, const int pc[3],
                                                long long* sNB) {
  constexpr int NO = D == 1 ? 3 : (D == 2 ? 9 : 27);
  const int t = threadIdx.x;
  if (t < NO) {
    const int np = m.lv[l].np;
    int q[3] = {0, 0, 0};
    bool in = true;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int o = (j == 0 ? t : (j == 1 ? t / 3 : t / 9)) % 3 - 1;
      int v = pc[j] + o;
      if (v < 0 || v >= np) {
        if (m.periodic[j]) v = (v + np) % np;
        else in = false;
      }
      q[j] = v;
    }
    const int pid = in ? map_at<D>(m, l, q) : -1;
    sNB[t] = pid >= 0 ? patch_base(m, pid, l) : -1;
  }
}

// Pressure from conserved values in the reference operation order:
// u_j = m_j / rho, ke = 0.5 * (m_x u_x + m_y u_y + m_z u_z), p = (gamma-1)(E - ke).
template <int D>
__device__ __forceinline__ double pressure_exact(const double* u, double gm1) {
  const double rho = u[0];
  double ke = u[1] * (u[1] / rho);
#pragma unroll
  for (int j = 1; j < D; ++j) ke = ke + u[1 + j] * (u[1 + j] / rho);
  ke = 0.5 * ke;
  return gm1 * (u[D + 1] - ke);
}

// Quotients by one divisor d from its reciprocal: r refined by two Newton
// steps, q = a r and one correction by the residual, fma(fma(-d, q, a), r, q)
// (Markstein 1990), which is the correctly rounded quotient, as the division is, while no scaling is needed
// (d, and a unless it is zero, in [2^-300, 2^300]: takes(a)).
struct Divisor {
  double d, r;
  bool ok;
  __device__ __forceinline__ explicit Divisor(double v) : d(v) {
    ok = in_range(v);
    r = __builtin_amdgcn_rcp(v);
    r = fma(fma(-v, r, 1.0), r, r);
    r = fma(fma(-v, r, 1.0), r, r);
  }
  static __device__ __forceinline__ bool in_range(double a) {
    return fabs(a) > 0x1p-300 && fabs(a) < 0x1p300;
  }
  __device__ __forceinline__ bool takes(double a) const { return ok && (in_range(a) || a == 0.0); }
  __device__ __forceinline__ double operator()(double a) const {  // takes(a)
    const double q = a * r;
    return fma(fma(-d, q, a), r, q);
  }
};

// sqrt(x), correctly rounded, for x where no scaling is needed (2^-700 .. 2^700):
// one Goldschmidt step on the hardware estimate of 1/sqrt(x), then two residual
// corrections.
__device__ __forceinline__ double sqrt_in_range(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, x), h, g);
  return fma(fma(-g, g, x), h, g);
}

// Centre value phi and MC-limited slopes sl of the level-lc cell at in-domain
// index gc, for its conservative linear prolongation: a child on the sides
// sig_j = +-1 is phi + sum_j (sig_j / 4) sl_j, terms added in the order x, y,
// z.  All slopes are zero when any of the 2^D children would have rho <= 0 or
// p <= 0.  False when a cell of the stencil has no patch.
template <int D>
__device__ __forceinline__ bool prolong_coarse(const DevMesh& m, const double* __restrict__ U,
                                               int lc, const int gc[3], double phi[D + 2],
                                               double sl[D][D + 2]) {
  constexpr int NV = D + 2;
  constexpr int NS = 2 * D + 1;  // coarse stencil: centre, then (+1, -1) per direction
  const LevelC& C = m.lv[lc];
  // the centre's patch and cell; a stencil cell leaves the patch by one cell
  // at most (periodic wrap of the patch position; at a transmissive boundary
  // the clamped position is the centre itself)
  int q[3] = {0, 0, 0}, c[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < D; ++j) {
    q[j] = div_by(gc[j], C.n, C.n_mul);
    c[j] = gc[j] - q[j] * C.n;
  }
  const int vs = var_stride<D>(C.full);
  const int step[3] = {1, C.full, __mul24(C.full, C.full)};
  const int mstep[3] = {1, C.np, C.np * C.np};
  int at = q[0], off0 = box_off<D>(C.full, c[0] + NG, c[1] + NG, c[2] + NG);
  if constexpr (D >= 2) at += C.np * q[1];
  if constexpr (D >= 3) at += C.np * C.np * q[2];
  // all map lookups first, then all loads, so the latencies overlap
  int pids[NS], offs[NS];
  const int* map = m.map + C.map_off;
  pids[0] = map[at];
  offs[0] = off0;
#pragma unroll
  for (int j = 0; j < D; ++j) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int o = k == 0 ? 1 : -1, cj = c[j] + o;
      int am = at, of = off0 + o * step[j];
      if ((unsigned)cj >= (unsigned)C.n) {
        int qj = q[j] + o;
        if ((unsigned)qj >= (unsigned)C.np) {
          if (m.periodic[j]) qj -= o * C.np;
        }
        if ((unsigned)qj >= (unsigned)C.np) {
          of = off0;
        } else {
          am = at + (qj - q[j]) * mstep[j];
          of = off0 - o * (C.n - 1) * step[j];
        }
      }
      pids[1 + 2 * j + k] = map[am];
      offs[1 + 2 * j + k] = of;
    }
  }
  bool found = true;
#pragma unroll
  for (int s = 0; s < NS; ++s) found &= pids[s] >= 0;
  if (!found) return false;
  double val[NS][NV];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const double* P = U + patch_base(m, pids[s], lc) + offs[s];
#pragma unroll
    for (int v = 0; v < NV; ++v) val[s][v] = P[v * vs];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) phi[v] = val[0][v];
#pragma unroll
  for (int j = 0; j < D; ++j) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double a = val[1 + 2 * j][v] - phi[v];
      const double b = phi[v] - val[2 + 2 * j][v];
      const bool same = (a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0);
      const double mag = fmin(fmin(2.0 * fabs(a), 2.0 * fabs(b)), 0.5 * fabs(a + b));
      sl[j][v] = same ? copysign(mag, a) : 0.0;
    }
  }
  // Every child lies within dev = sum_j |sl_j| / 4 of phi in every variable.
  // Where the smallest density and energy within that are at least 1e-3 of the
  // cell's own (so that their rounding stays below 1e-12 of them) and give
  // 2 rho E > |m|^2 with the largest momenta by a margin far above it, every
  // child passes the exact test; only the other cells (and NaN) go through the
  // children one by one.
  double lo[2], mm = 0.0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double dev = fabs(sl[0][v]);
#pragma unroll
    for (int j = 1; j < D; ++j) dev = dev + fabs(sl[j][v]);
    if (v == 0 || v == NV - 1) {
      lo[v == 0 ? 0 : 1] = phi[v] - 0.25 * dev;
    } else {
      const double hi = fabs(phi[v]) + 0.25 * dev;
      mm = mm + hi * hi;
    }
  }
  if (!(lo[0] > 1e-3 * phi[0] && lo[1] > 1e-3 * phi[NV - 1] &&
        2.0 * lo[0] * lo[1] > mm * (1.0 + 1e-10))) {
    bool bad = false;
    for (int k = 0; k < (1 << D); ++k) {
      double ch[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        double x = phi[v];
#pragma unroll
        for (int j = 0; j < D; ++j) x = x + (((k >> j) & 1) ? 0.25 : -0.25) * sl[j][v];
        ch[v] = x;
      }
      const double p = pressure_exact<D>(ch, m.gm1);
      if (!(ch[0] > 0.0 && p > 0.0)) bad = true;
    }
    if (bad) {
#pragma unroll
      for (int j = 0; j < D; ++j)
#pragma unroll
        for (int v = 0; v < NV; ++v) sl[j][v] = 0.0;
    }
  }
  return true;
}

// The level-lf cell at mapped global index g prolonged from level lf-1.
template <int D>
__device__ __forceinline__ bool prolong_cell(const DevMesh& m, const double* __restrict__ U, int lf,
                                             const int g[3], double out[D + 2]) {
  int gc[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < D; ++j) gc[j] = g[j] >> 1;
  double phi[D + 2], sl[D][D + 2];
  if (!prolong_coarse<D>(m, U, lf - 1, gc, phi, sl)) return false;
#pragma unroll
  for (int v = 0; v < D + 2; ++v) {
    double x = phi[v];
#pragma unroll
    for (int j = 0; j < D; ++j) x = x + ((g[j] & 1) ? 0.25 : -0.25) * sl[j][v];
    out[v] = x;
  }
  return true;
}

// The 2^D children of a coarse cell into a patch at box offset off (of the
// lowest child): side sg[j][f] = +-1 of child f (0 low, 1 high) along j; NaN
// when `ok` is false.  x pairs go out as one 16-byte store: every offset here
// is even (even patch edges and box rows, ghost width 4, pools of whole
// patches behind an even head pad) and the state buffers are 256-byte aligned.
template <int D>
__device__ __forceinline__ void store_children(double* P, int vs, int full, int off, bool ok,
                                               const double phi[D + 2], const double sl[D][D + 2],
                                               const double sg[3][2]) {
#pragma unroll
  for (int f = 0; f < (1 << (D - 1)); ++f) {
    const int o = off + (f & 1 ? full : 0) + (f & 2 ? __mul24(full, full) : 0);
#pragma unroll
    for (int v = 0; v < D + 2; ++v) {
      double2 x;
      x.x = phi[v] + (sg[0][0] * 0.25) * sl[0][v];
      x.y = phi[v] + (sg[0][1] * 0.25) * sl[0][v];
#pragma unroll
      for (int j = 1; j < D; ++j) {
        const double t = (sg[j][(f >> (j - 1)) & 1] * 0.25) * sl[j][v];
        x.x = x.x + t;
        x.y = x.y + t;
      }
      if (!ok) x.x = x.y = __builtin_nan("");
      *reinterpret_cast<double2*>(P + v * vs + o) = x;
    }
  }
}

// Signal speed sum_j (|u_j| + c) of a cell as bits in ascending order (IEEE bits
// of a non-negative double as an unsigned integer); NaN maps to the largest
// value so that it propagates.  The quotients and the root are those of the
// divisions and of sqrt, from one reciprocal of rho.
constexpr unsigned long long kNanBits = 0x7ff8000000000000ull;

template <int D>
__device__ __forceinline__ unsigned long long cell_speed_bits(const double* u, const DevMesh& m) {
  const Divisor rho(u[0]);
  bool ok = true;
#pragma unroll
  for (int j = 0; j < D; ++j) ok = ok && rho.takes(u[1 + j]);
  double uj[D];
#pragma unroll
  for (int j = 0; j < D; ++j) uj[j] = ok ? rho(u[1 + j]) : u[1 + j] / u[0];
  double ke = u[1] * uj[0];
#pragma unroll
  for (int j = 1; j < D; ++j) ke = ke + u[1 + j] * uj[j];
  ke = 0.5 * ke;
  const double gp = m.gamma * (m.gm1 * (u[D + 1] - ke));
  // in range: gp is positive, and gp / rho between 2^-600 and 2^600
  const double c = ok && gp > 0x1p-300 && gp < 0x1p300 && u[0] > 0.0 ? sqrt_in_range(rho(gp))
                                                                      : sqrt(gp / u[0]);
  double s = fabs(uj[0]) + c;
#pragma unroll
  for (int j = 1; j < D; ++j) s = s + (fabs(uj[j]) + c);
  return s >= 0.0 ? (unsigned long long)__double_as_longlong(s) : kNanBits;
}

// Maximum over a wave by lane shifts (row_shr 1, 2, 4, 8, then row_bcast 15 and
// 31): the high words first, then the low words of the lanes that hold the
// largest high word.
__device__ __forceinline__ unsigned wave_max(unsigned v) {
#define AMR_DPP_MAX(ctrl) \
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false))
  AMR_DPP_MAX(0x111);
  AMR_DPP_MAX(0x112);
  AMR_DPP_MAX(0x114);
  AMR_DPP_MAX(0x118);
  AMR_DPP_MAX(0x142);
  AMR_DPP_MAX(0x143);
#undef AMR_DPP_MAX
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
  const unsigned hi = (unsigned)(v >> 32);
  const unsigned top = wave_max(hi);
  const unsigned low = wave_max(hi == top ? (unsigned)v : 0u);
  return ((unsigned long long)top << 32) | low;
}

// The block's largest cell speed over the cell size h (the rate; division by h
// keeps the order, so one division per block serves all its cells), into this
// XCD's part of the rate slot `lam`.  What a block waits for at its end keeps
// the next one off its CU: with five divisions per cell, LDS shuffles and one
// address for all atomics the stage kernel's third stage took 26.1 us (2D, 0.28 M
// cells), 170 (2.75 M) and 2112 (3D, 20.4 M), and k_max_rate 17, 48 and 463;
// 21.8, 162 and 2045, and 7.4, 30 and 338 so.
__device__ __forceinline__ void block_max_rate(unsigned long long best, double h,
                                               unsigned long long* __restrict__ lam) {
  __shared__ unsigned long long red[16];
  const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  best = wave_max(best);
  if (waves > 1) {
    if (lane == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    best = wave_max(lane < waves ? red[lane] : 0ull);
  }
  const double r = __longlong_as_double((long long)best) / h;
  best = r >= 0.0 ? (unsigned long long)__double_as_longlong(r) : kNanBits;
  if (lane == 0 && best) atomicMax(lam + blockIdx.x % kXcds * kRateStride, best);
}

// The rate in a slot.
__device__ __forceinline__ double slot_rate(const unsigned long long* __restrict__ lam) {
  unsigned long long best = lam[0];
#pragma unroll
  for (int x = 1; x < kXcds; ++x) {
    const unsigned long long b = lam[x * kRateStride];
    best = b > best ? b : best;
  }
  return __longlong_as_double((long long)best);
}

__device__ __forceinline__ void clear_rate(unsigned long long* __restrict__ lam) {
#pragma unroll
  for (int x = 0; x < kXcds; ++x) lam[x * kRateStride] = 0ull;
}

// The entries and live count of a list (see ListArg).  The count is loaded with
// `dir`, not behind the branch, and the recorded form stands outside the eager
// launches' path.
__device__ __forceinline__ void live_list(ListArg& a) {
  asm("" : "+s"(a.count));
  if (__builtin_expect(a.dir == nullptr, 1)) return;
  a.ptr += a.dir[0];
  a.count = a.dir[1];
}

// Work item of this block.  Workgroups are dealt to the chip's XCDs in
// turn (block b runs on XCD b mod kXcds) and each XCD has its own L2: XCD x
// takes the contiguous items [x per, (x + 1) per), per = ceil(count /
// kXcds), in dispatch order, so tiles of one patch and of neighbouring
// patches (the list is in brick order), which read each other's cells as
// halos, share an L2.  The grid holds at least kXcds per blocks; it may hold
// more (a launch recorded for a longer list), and a block without an item
// gets -1.
__device__ __forceinline__ int xcd_item(int count) {
  const int per = (count + kXcds - 1) / kXcds;
  const int k = (int)blockIdx.x / kXcds;
  const int item = ((int)blockIdx.x % kXcds) * per + k;
  return (k < per && item < count) ? item : -1;
}

// Work item of this block where items differ in size: chunks of C consecutive
// items go to the XCDs in turn (block b runs on XCD b mod kXcds), so that an
// XCD's items at any time are neighbours in the list and every XCD gets a
// share of each part of it.  The grid is whole groups of kXcds C blocks.
template <int C>
__device__ __forceinline__ int xcd_chunk(int count, int b = (int)blockIdx.x) {
  const int g = b / (kXcds * C) * (kXcds * C);
  const int item = g + (b % kXcds) * C + (b / kXcds) % C;
  return item < count ? item : -1;
}

}  // namespace
}  // namespace amr

// HIP kernels of libamr for gfx950 (CDNA4, wave64), except the fused stage
// kernel (stage.hip): ghost fill, refluxing, restriction, CFL rate, tagging,
// prolongation of new patches, checks.
//
// Every kernel works on the patch pools described in amr_internal.hpp: a
// patch of level l stores nvar * (n_l + 8)^dim doubles, var-major, x fastest,
// with 4 ghost layers.  Work lists (pids or (pid, tile) pairs) are device
// arrays built by the host after each regrid, so one launch covers the
// patches of every level.
//
// Floating-point contract: implicit contraction is disabled; the refluxing
// correction writes its fused multiply-add out with fma().  The
// prolongation, restriction, tag and time-step paths use the operation order
// of the definitions they implement (no fma), so that integer decisions (tags,
// positivity switches) are taken on the same values as the FP64 reference.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <stdexcept>

#include "amr_internal.hpp"

// no implicit contraction anywhere in this file (see the header comment)
#pragma clang fp contract(off)

#include "device_common.hpp"

namespace amr {
namespace {

// Consecutive patches whose ghosts an XCD copies at a time (xcd_chunk): they
// read each other's cells.  3D, 4288 patches of 8^3 and 448 of 16^3: 336 us
// with patch b on XCD b mod 8, 478 us with a contiguous eighth of the list per
// XCD (the first holds all the large patches), 306 us with chunks of 32.
constexpr int kCopyChunk = 32;

// ---------------------------------------------------------------------------
// ghost fill
// ---------------------------------------------------------------------------
// Ghost cells of one patch that lie in a same-level patch, by the whole block:
// copied from that patch (neighbour table sNB by offset code), x pairs as
// 16-byte accesses (a pair lies on one side of every region boundary and, but
// for the clamp at a transmissive wall, in one source row).  Regions without a
// same-level patch are prolonged elsewhere.  The cells read are interior
// cells, the cells written ghosts.  Bound by memory: 40 B written per 3D cell.
template <int D, int NT>
__device__ __forceinline__ void copy_ghosts(const DevMesh& m, const double* __restrict__ Uin,
                                            double* __restrict__ U, int pid, long long* sNB) {
  constexpr int NV = D + 2;
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n, full = L.full, vs = var_stride<D>(full);
  const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
  load_neighbours<D>(m, l, pc, sNB);
  __syncthreads();
  double* P = U + patch_base(m, pid, l);
#pragma unroll 2
  for (int pair = threadIdx.x; pair < vs / 2; pair += NT) {
    const int idx = 2 * pair;
    const int r = D >= 2 ? div_by(idx, full, L.full_mul) : 0;
    const int rz = D >= 3 ? div_by(r, full, L.full_mul) : 0;
    const int c[3] = {idx - r * full - NG, D >= 2 ? r - rz * full - NG : 0, rz - NG};
    int code = 0, mul = 1, loc[3] = {0, 0, 0};
    bool ghost = false, dup = false;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      int o = c[j] < 0 ? -1 : (c[j] >= n ? 1 : 0);
      ghost |= o != 0;
      loc[j] = c[j] - o * n;
      if (o != 0 && !m.periodic[j] && (unsigned)(pc[j] + o) >= (unsigned)L.np) {
        loc[j] = o < 0 ? 0 : n - 1;
        if (j == 0) dup = true;
        o = 0;
      }
      code += (o + 1) * mul;
      mul *= 3;
    }
    if (!ghost) continue;
    const long long sb = sNB[code];
    if (sb < 0) continue;
    const double* S = Uin + sb;
    const int src = box_off<D>(full, loc[0] + NG, loc[1] + NG, loc[2] + NG);
    double2 x[NV];
    if (dup) {
#pragma unroll
      for (int v = 0; v < NV; ++v) x[v].x = x[v].y = S[v * vs + src];
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) x[v] = *reinterpret_cast<const double2*>(S + v * vs + src);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double* to = P + v * vs + idx;
      if constexpr (D == 3) {
        // ghosts are the larger part of a 3D box: stored past the L2, which
        // keeps the interiors for the neighbours (312 to 291 us, and the
        // prolongation after it 72 to 54 us)
        typedef double d2 __attribute__((ext_vector_type(2)));
        const d2 y = {x[v].x, x[v].y};
        __builtin_nontemporal_store(y, reinterpret_cast<d2*>(to));
      } else {
        *reinterpret_cast<double2*>(to) = x[v];
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_copy3(DevMesh m, const double* __restrict__ Uin,
                                                    double* __restrict__ U, ListArg list) {
  __shared__ long long sNB[27];
  live_list(list);
  const int item = xcd_chunk<kCopyChunk>(list.count);
  if (item >= 0) copy_ghosts<3, 256>(m, Uin, U, list.ptr[item], sNB);
}

// Ghost cells without a same-level source: one work item per (leaf, ghost
// region), region = neighbour offset r in {-1,0,1}^D coded as
// (r0+1) + 3 (r1+1) + 9 (r2+1); the host lists only regions whose source
// position (after the physical-boundary clamp) holds no same-level patch, so
// every cell of the region is prolonged from level l-1.
template <int D, int NT>
__device__ __forceinline__ void fill_cf_region(const DevMesh& m, double* __restrict__ U,
                                               const int* __restrict__ list, int item,
                                               int* __restrict__ err) {
  constexpr int NV = D + 2;
  const int pid = list[2 * item];
  const int code = list[2 * item + 1];
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n, full = L.full;
  const int vs = var_stride<D>(full);
  double* P = U + patch_base(m, pid, l);
  const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
  int start[3] = {0, 0, 0}, ext[3] = {1, 1, 1};
  int total = 1;
  for (int j = 0; j < D; ++j) {
    const int r = (j == 0 ? code : (j == 1 ? code / 3 : code / 9)) % 3 - 1;
    start[j] = r < 0 ? -NG : (r == 0 ? 0 : n);
    ext[j] = r == 0 ? n : NG;
    total *= ext[j];
  }
  for (int idx = threadIdx.x; idx < total; idx += NT) {
    int c[3] = {start[0] + idx % ext[0], 0, 0};
    if constexpr (D >= 2) c[1] = start[1] + (idx / ext[0]) % ext[1];
    if constexpr (D >= 3) c[2] = start[2] + idx / (ext[0] * ext[1]);
    int g[3] = {0, 0, 0};
    for (int j = 0; j < D; ++j) g[j] = bc_near(pc[j] * n + c[j], L.cells, m.periodic[j]);
    double val[NV];
    const bool ok = (l > 0) && prolong_cell<D>(m, U, l, g, val);
    if (!ok) {
      err[0] = 1;
      for (int v = 0; v < NV; ++v) val[v] = __builtin_nan("");
    }
    const int off = box_off<D>(full, c[0] + NG, c[1] + NG, c[2] + NG);
#pragma unroll
    for (int v = 0; v < NV; ++v) P[v * vs + off] = val[v];
  }
}

// One block per region.
template <int D, int NT>
__global__ __launch_bounds__(NT) void k_fill_cf(DevMesh m,
                                                double* __restrict__ U, ListArg regions,
                                                int* __restrict__ err) {
  live_list(regions);
  if ((int)blockIdx.x < regions.count) fill_cf_region<D, NT>(m, U, regions.ptr, blockIdx.x, err);
}

// The same regions by coarse cell (2D and 3D).  A region's start and extent
// are even in every dimension, so its fine cells come in aligned blocks of
// 2^D, and both cells of an aligned pair have the same coarse cell also
// after the boundary mapping (a periodic wrap of an even cell count keeps
// pairs together; the clamp sends a whole out-of-domain pair to one edge
// cell).  One thread computes the coarse stencil, the MC slopes and the
// positivity test once and forms each of the 2^D fine values as
// prolong_cell does, in the same operation order, so the values are bitwise
// those of the per-fine-cell fill.  A block takes G consecutive regions and
// spreads all their coarse cells over its lanes: a 3D region covers as few
// as 8 coarse cells (a corner).
template <int G>
struct RegionGroup {
  int pid[G], code[G], lev[G], pc[G][3], pre[G + 1];
};

template <int D, int NT, int G>
__device__ __forceinline__ void fill_cf_coarse_group(const DevMesh& m, double* __restrict__ U,
                                                     const int* __restrict__ list, int count,
                                                     int first, int* __restrict__ err,
                                                     RegionGroup<G>& s) {
  constexpr int NV = D + 2;
  static_assert(G <= 64 && (G & (G - 1)) == 0, "one wave scans the group's counts");
  if (threadIdx.x < 64) {
    const int t = threadIdx.x, i = first + t;
    int cnt = 0;
    if (t < G && i < count) {
      const int pid = list[2 * i], code = list[2 * i + 1];
      const int l = m.level[pid];
      const int n = m.lv[l].n;
      cnt = 1;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int r = (j == 0 ? code : (j == 1 ? code / 3 : code / 9)) % 3 - 1;
        cnt *= (r == 0 ? n : NG) / 2;
        s.pc[t][j] = m.coord[3 * pid + j];
      }
      s.pid[t] = pid;
      s.code[t] = code;
      s.lev[t] = l;
    }
    int sum = cnt;
#pragma unroll
    for (int d = 1; d < G; d *= 2) {
      const int o = __shfl_up(sum, d);
      if (t >= d) sum += o;
    }
    if (t < G) s.pre[t + 1] = sum;
    if (t == 0) s.pre[0] = 0;
  }
  __syncthreads();
  const int total = s.pre[G];
  for (int idx = threadIdx.x; idx < total; idx += NT) {
    int it = 0;  // the region with pre[it] <= idx < pre[it + 1]
#pragma unroll
    for (int d = G / 2; d > 0; d /= 2)
      if (idx >= s.pre[it + d]) it += d;
    const int pid = s.pid[it], code = s.code[it], lev = s.lev[it];
    const int local = idx - s.pre[it];
    // one pass per level among the wave's lanes (nearly always one: the list
    // is in level order), so that the level's constants are scalar
    for (bool done = false; !done;) {
      const int l = __builtin_amdgcn_readfirstlane(lev);
      if (lev != l) continue;
      done = true;
      const LevelC& L = m.lv[l];
      const int n = L.n, full = L.full;
      double* P = U + patch_base(m, pid, l);
      int start[3] = {0, 0, 0}, half[3] = {1, 1, 1};
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int r = (j == 0 ? code : (j == 1 ? code / 3 : code / 9)) % 3 - 1;
        start[j] = r < 0 ? -NG : (r == 0 ? 0 : n);
        half[j] = (r == 0 ? n : NG) / 2;
      }
      // half is n / 2 or 2 in every direction
      auto by_half = [&](int v, int h) { return h == NG / 2 ? v / (NG / 2) : div_by(2 * v, n, L.n_mul); };
      const int r0 = D >= 2 ? by_half(local, half[0]) : 0;
      const int r1 = D >= 3 ? by_half(r0, half[1]) : 0;
      const int k[3] = {local - r0 * half[0], D >= 2 ? r0 - r1 * half[1] : 0, r1};
      int c0[3] = {0, 0, 0}, gc[3] = {0, 0, 0};
      double sg[3][2] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
      for (int j = 0; j < D; ++j) {
        c0[j] = start[j] + 2 * k[j];
        const int g = s.pc[it][j] * n + c0[j];
        const int g0 = bc_near(g, L.cells, m.periodic[j]);
        const int g1 = bc_near(g + 1, L.cells, m.periodic[j]);
        gc[j] = g0 >> 1;
        sg[j][0] = (g0 & 1) ? 1.0 : -1.0;
        sg[j][1] = (g1 & 1) ? 1.0 : -1.0;
      }
      double phi[NV] = {}, sl[D][NV] = {};
      const bool ok = l > 0 && prolong_coarse<D>(m, U, l - 1, gc, phi, sl);
      if (!ok) err[0] = 1;
      store_children<D>(P, var_stride<D>(full), full,
                        box_off<D>(full, c0[0] + NG, c0[1] + NG, c0[2] + NG), ok, phi, sl, sg);
    }
  }
}

// A block takes a group of G consecutive regions.
template <int D, int NT, int G>
__global__ __launch_bounds__(NT) void k_fill_cf_coarse(DevMesh m,
                                                       double* __restrict__ U, ListArg regions,
                                                       int* __restrict__ err) {
  __shared__ RegionGroup<G> s;
  live_list(regions);
  const int first = (int)blockIdx.x * G;
  if (first < regions.count)
    fill_cf_coarse_group<D, NT, G>(m, U, regions.ptr, regions.count, first, err, s);
}

// The whole fill in one launch (1D, 2D): prolonged regions (groups of G, by
// coarse cell; in 1D a region per block) in the first blocks, whose chains of
// dependent loads the copies of the others cover.  They write different ghosts
// and both read interior cells only.  2D, 240^2 base with three levels of 24^2
// patches: 5.6 + 5.7 us in two launches (copies with 256 threads), 7.2 in one.  In 3D the prolongation's 126
// VGPRs would halve the waves of the copies, which are bound by memory: 384 us
// against 290 + 57 (64^3 base, 16^3/16^3/8^3 patches), so two launches there.
constexpr int fill_threads(int dim) { return dim == 1 ? 64 : 128; }
constexpr int kFillGroup = 4;

template <int D>
__global__ __launch_bounds__(fill_threads(D)) void k_fill(DevMesh m, const double* __restrict__ Uin,
                                                          double* __restrict__ U, ListArg list,
                                                          ListArg regions, int rblocks,
                                                          int* __restrict__ err) {
  constexpr int NT = fill_threads(D);
  __shared__ RegionGroup<kFillGroup> s;
  __shared__ long long sNB[27];
  const int b = (int)blockIdx.x;
  if (b < rblocks) {
    live_list(regions);
    if constexpr (D == 1) {
      if (b < regions.count) fill_cf_region<D, NT>(m, U, regions.ptr, b, err);
    } else {
      if (b * kFillGroup < regions.count)
        fill_cf_coarse_group<D, NT, kFillGroup>(m, U, regions.ptr, regions.count, b * kFillGroup,
                                                err, s);
    }
  } else {
    live_list(list);
    const int item = xcd_chunk<kCopyChunk>(list.count, b - rblocks);
    if (item >= 0) copy_ghosts<D, NT>(m, Uin, U, list.ptr[item], sNB);
  }
}

// ---------------------------------------------------------------------------
// coarse/fine flux correction: list of RefluxItem; a cell's faces are corrected
// in the order x-, x+, y-, y+, z-, z+ so that corner cells see a fixed order
// ---------------------------------------------------------------------------
// The fine side of a coarse cell's c/f face: the same-level position of the
// fine patch that holds the face's 2^(D-1) sub-faces in its patch map, and the
// offsets of the face in the two patches' flux registers (variable 0).
struct FinePart {
  int map, coarse, fine;
};

template <int D>
__device__ __forceinline__ FinePart fine_part(const DevMesh& m, int l, const int pc[3],
                                              const int c[3], int j, int side) {
  constexpr int NV = D + 2;
  const LevelC& Fv = m.lv[l + 1];
  const int n = m.lv[l].n, nf = Fv.n, Nf = Fv.cells;
  const int nface = (D == 1) ? 1 : (D == 2 ? n : n * n);
  const int nfface = (D == 1) ? 1 : (D == 2 ? nf : nf * nf);
  // fine cell column adjacent to the face (periodic wrap on the high side,
  // and on the low side of the domain)
  const int F = 2 * (pc[j] * n + (side ? n : 0));
  const int cj = side ? (F == Nf ? 0 : F) : (F == 0 ? Nf : F) - 1;
  // tangential coordinates in ascending dimension order: of the cell, and of
  // its fine sub-faces 2 g and 2 g + 1, which one fine patch holds (even edges)
  int t = 0, ft = 0, at = div_by(cj, nf, Fv.n_mul) * (j == 0 ? 1 : (j == 1 ? Fv.np : Fv.np * Fv.np));
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (d == j) continue;
    const bool second = d - (d > j ? 1 : 0) == 1;
    const int g = 2 * (pc[d] * n + c[d]);
    const int q = div_by(g, nf, Fv.n_mul);
    t += c[d] * (second ? n : 1);
    ft += (g - q * nf) * (second ? nf : 1);
    at += q * (d == 0 ? 1 : (d == 1 ? Fv.np : Fv.np * Fv.np));
  }
  return {Fv.map_off + at, (j * 2 + side) * NV * nface + t,
          (j * 2 + (side ? 0 : 1)) * NV * nfface + ft};
}

// Correction of the coarse cell values u by one c/f face (fine patch fpid):
// coef (G_c - mean of the 2^(D-1) fine sub-face fluxes), signed +1 on the high
// face and -1 on the low face.
template <int D>
__device__ __forceinline__ void face_correct(const DevMesh& m, const double* __restrict__ fr,
                                             const double* __restrict__ frc, int l,
                                             const FinePart& fp, int fpid, int side, double coef,
                                             double u[D + 2]) {
  constexpr int NV = D + 2;
  const LevelC& Fv = m.lv[l + 1];
  const int n = m.lv[l].n, nf = Fv.n;
  const int nface = (D == 1) ? 1 : (D == 2 ? n : n * n);
  const int nfface = (D == 1) ? 1 : (D == 2 ? nf : nf * nf);
  const double* gcp = frc + fp.coarse;
  const double* frf = fr + Fv.fr_off +
                      (long long)((fpid < 0 ? Fv.pid_base : fpid) - Fv.pid_base) * Fv.fr_stride +
                      fp.fine;
  const double sgn = side ? 1.0 : -1.0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    // sub-face pairs as 16-byte loads (every offset is even, as nf is)
    const double* sub = frf + v * nfface;
    double avg;
    if constexpr (D == 1) {
      avg = sub[0];
    } else {
      const double2 a = *reinterpret_cast<const double2*>(sub);
      if constexpr (D == 2) {
        avg = (a.x + a.y) * 0.5;
      } else {
        const double2 b = *reinterpret_cast<const double2*>(sub + nf);
        avg = ((a.x + a.y) + (b.x + b.y)) * 0.25;
      }
    }
    if (fpid < 0) avg = __builtin_nan("");
    u[v] = fma(coef, sgn * (gcp[v * nface] - avg), u[v]);
  }
}

// Refluxing on the items of leaves with c/f faces.  Every cell on a masked face is
// owned by one thread (the first masked face containing it in the order
// x-, x+, y-, y+, z-, z+), which applies the corrections of all masked faces
// containing the cell in that order; at stage 3 it also feeds the corrected
// cell's CFL rate to the next step's maximum.  Bound by its chain of dependent
// loads: a cell is on at most one face per direction, and the fine patches of
// all of them are looked up before any register is read (a cell on the edge of
// two masked faces took one such chain after the other, and its wave with it);
// the level and position come with the item.  k_post with both, and with the
// restriction of the corrected faces alone (see there): 1D 3.6 to 2.9 us (20
// tiles), 2D 7.2 to 6.1 (0.28 M cells) and 14.8 to 12.0 (2.75 M), 3D 18.0 to
// 15.3 (0.7 M) and 76 to 67 (20.4 M).
template <int D, int NT>
__device__ __forceinline__ void reflux_item(const DevMesh& m, int mode, double* __restrict__ out,
                                            const double* __restrict__ fr, const RefluxItem& ri,
                                            const double* __restrict__ dtp, double w,
                                            unsigned long long* __restrict__ lam_next) {
  constexpr int NV = D + 2;
  const int pid = ri.pid, mask = ri.mask, l = ri.level;
  const LevelC& L = m.lv[l];
  const int n = L.n;
  const int nface = (D == 1) ? 1 : (D == 2 ? n : n * n);
  const int* pc = ri.pc;
  const double* frc = fr + L.fr_off + (long long)(pid - L.pid_base) * L.fr_stride;
  double* P = out + patch_base(m, pid, l);
  const int vs = var_stride<D>(L.full);
  const double coef = (mode == kModeRHS) ? L.inv_h : (w * dtp[0]) * L.inv_h;
  const bool want_rate = lam_next != nullptr && mode == kModeStage3;
  unsigned long long best = 0ull;
  // one item per cell of a masked face (a front crosses one to three of them)
  const int items = __popc(mask) * nface;
  for (int it = threadIdx.x; it < items; it += NT) {
    const int row = D >= 2 ? div_by(it, n, L.n_mul) : it;
    const int nth = D >= 3 ? div_by(row, n, L.n_mul) : row;
    int left = mask;
    for (int k = 0; k < nth; ++k) left &= left - 1;
    const int f = __ffs(left) - 1;
    // cell on face f: normal coordinate 0 or n-1, tangential ones in ascending
    // dimension order
    const int t0 = D >= 2 ? it - row * n : 0, t1 = D >= 3 ? row - nth * n : 0;
    int c[3] = {0, 0, 0};
    // per direction, whether the cell is on a masked face and on which side
    bool on[3] = {false, false, false};
    int side[3];
    bool owned = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int j = f >> 1, k = d - (d > j ? 1 : 0);
      c[d] = (d == j) ? ((f & 1) ? n - 1 : 0) : (k == 0 ? t0 : t1);
      side[d] = c[d] == 0 ? 0 : 1;
      on[d] = (c[d] == 0 || c[d] == n - 1) && (mask >> (2 * d + side[d]) & 1);
      if (d < j) owned &= !on[d];
    }
    if (!owned) continue;
    // the cell's values stay in registers through all of its corrections
    const int off = box_off<D>(L.full, c[0] + NG, c[1] + NG, c[2] + NG);
    FinePart fp[D];
    int fpid[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      fp[d] = fine_part<D>(m, l, pc, c, d, side[d]);
      fpid[d] = -1;
      if (on[d]) fpid[d] = m.map[fp[d].map];
    }
    double u[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = P[v * vs + off];
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (on[d]) face_correct<D>(m, fr, frc, l, fp[d], fpid[d], side[d], coef, u);
#pragma unroll
    for (int v = 0; v < NV; ++v) P[v * vs + off] = u[v];
    if (want_rate) {
      const unsigned long long bits = cell_speed_bits<D>(u, m);
      best = bits > best ? bits : best;
    }
  }
  if (want_rate) block_max_rate(best, L.h, lam_next);
}

template <int D, int NT>
__global__ __launch_bounds__(NT) void k_reflux(DevMesh m, int mode, double* __restrict__ out,
                                               const double* __restrict__ fr,
                                               const RefluxItem* __restrict__ list, int count,
                                               const int* __restrict__ dir,
                                               const double* __restrict__ dtp, double w,
                                               unsigned long long* __restrict__ lam_next) {
  if (dir) {
    list = reinterpret_cast<const RefluxItem*>(reinterpret_cast<const int*>(list) + dir[0]);
    count = dir[1];
  }
  if ((int)blockIdx.x >= count) return;
  reflux_item<D, NT>(m, mode, out, fr, list[blockIdx.x], dtp, w, lam_next);
}

// Where a child patch (level lf >= 1) is restricted to: the offset in a state
// buffer of the first parent cell it covers.
template <int D>
__device__ __forceinline__ long long restrict_target(const DevMesh& m, int cpid, int lf) {
  const LevelC& C = m.lv[lf - 1];
  const int ppid = m.parent[cpid];
  int q[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < D; ++j)
    q[j] = m.coord[3 * cpid + j] * (m.lv[lf].n / 2) - m.coord[3 * ppid + j] * C.n + NG;
  return patch_base(m, ppid, lf - 1) + box_off<D>(C.full, q[0], q[1], q[2]);
}

// Restriction into one covered parent cell ((a, b, c) among those the child
// covers): the sum of its 2^D child cells in pairs, x, then y, then z, times
// 2^-D.
template <int D>
__device__ __forceinline__ void restrict_cell(const DevMesh& m, double* __restrict__ U, int cpid,
                                              long long target, int lf, int a, int b, int c) {
  constexpr int NV = D + 2;
  const LevelC& F = m.lv[lf];
  const LevelC& C = m.lv[lf - 1];
  const double* Pc = U + patch_base(m, cpid, lf);
  double* Pp = U + target;
  const long long vsf = var_stride<D>(F.full), vsc = var_stride<D>(C.full);
  const long long dst = box_off<D>(C.full, a, b, c);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double* S = Pc + v * vsf;
    // sum of the x-pair (2a, 2a + 1) of fine row (y, z), read as one 16-byte
    // load: every offset here is even (even patch edges, ghost width 4, pools
    // of whole patches) and the state buffer is 256-byte aligned
    auto xsum = [&](int y, int z) {
      const double2 t = *reinterpret_cast<const double2*>(
          S + box_off<D>(F.full, 2 * a + NG, 2 * b + y + NG, 2 * c + z + NG));
      return t.x + t.y;
    };
    double r;
    if constexpr (D == 1) r = xsum(0, 0) * 0.5;
    else if constexpr (D == 2)
      r = (xsum(0, 0) + xsum(1, 0)) * 0.25;
    else
      r = ((xsum(0, 0) + xsum(1, 0)) + (xsum(0, 1) + xsum(1, 1))) * 0.125;
    Pp[v * vsc + dst] = r;
  }
}

// idx / (n / 2) of a level
__device__ __forceinline__ int div_half(int idx, const LevelC& L) {
  return div_by(2 * idx, L.n, L.n_mul);
}

// restriction of patch cpid (level lf) into its parent, by the whole block
template <int D>
__device__ __forceinline__ void restrict_patch(const DevMesh& m, double* __restrict__ U,
                                               int cpid, int lf, long long target) {
  const LevelC& F = m.lv[lf];
  const int h = F.n / 2;
  int total = h;
  if constexpr (D >= 2) total *= h;
  if constexpr (D >= 3) total *= h;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int row = D >= 2 ? div_half(idx, F) : 0;
    const int c = D >= 3 ? div_half(row, F) : 0;
    restrict_cell<D>(m, U, cpid, target, lf, idx - row * h, D >= 2 ? row - c * h : 0, c);
  }
}

// the covered parent cells along the masked faces of a leaf, by the whole block
// (cells on an edge of two faces are written from both, with the same value)
template <int D>
__device__ __forceinline__ void restrict_faces(const DevMesh& m, double* __restrict__ U, int cpid,
                                               int lf, long long target, int mask) {
  const LevelC& F = m.lv[lf];
  const int h = F.n / 2;
  const int face = (D == 1) ? 1 : (D == 2 ? h : h * h);
  const int total = __popc(mask) * face;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int row = D >= 2 ? div_half(idx, F) : idx;
    const int nth = D >= 3 ? div_half(row, F) : row;
    int left = mask;
    for (int k = 0; k < nth; ++k) left &= left - 1;
    const int f = __ffs(left) - 1, j = f >> 1;
    const int t0 = D >= 2 ? idx - row * h : 0, t1 = D >= 3 ? row - nth * h : 0;
    int q[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k = d - (d > j ? 1 : 0);
      q[d] = (d == j) ? ((f & 1) ? h - 1 : 0) : (k == 0 ? t0 : t1);
    }
    restrict_cell<D>(m, U, cpid, target, lf, q[0], q[1], q[2]);
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_restrict(DevMesh m, double* __restrict__ U,
                                                  ListArg list) {
  live_list(list);
  if ((int)blockIdx.x >= list.count) return;
  const int pid = list.ptr[blockIdx.x], l = m.level[pid];
  restrict_patch<D>(m, U, pid, l, restrict_target<D>(m, pid, l));
}

// After a stage, in one launch: refluxing, and what it changes of the
// restriction of the leaves (the stage kernel restricts every leaf as it writes
// it), and the restriction of level L-2 into L-3.  Blocks:
//  [0, nref)       reflux items; the parent cells along the
//                  corrected faces are then formed again;
//  [nref, +npair)  level-(L-2) patches with children: restrict into the parent
//                  (their children, on the finest level, are never refluxed:
//                  the stage kernel has restricted their final values).
// A block's restriction after refluxing reads only what the same block wrote
// (block barrier between); the blocks touch disjoint cells otherwise:
// refluxing changes leaf cells, restriction writes non-leaf cells.  Recorded,
// `dir` has the entries of both lists, in order (one load), and rlist is the
// list buffer.
// Restricting the corrected leaves whole, here and in the coarser levels'
// launches: 76 and 26 us (3D, 20.4 M cells), 67 and 16 so.
template <int D, int NT>
__global__ __launch_bounds__(NT) void k_post(DevMesh m, int mode,
                                             double* __restrict__ out,
                                             const double* __restrict__ fr,
                                             const RefluxItem* __restrict__ rlist, int nref,
                                             const int* __restrict__ plist, int npair,
                                             const int* __restrict__ dir,
                                             const double* __restrict__ dtp, double w,
                                             unsigned long long* __restrict__ lam_next) {
  if (dir) {
    const int* buf = reinterpret_cast<const int*>(rlist);
    rlist = reinterpret_cast<const RefluxItem*>(buf + dir[0]);
    nref = dir[1];
    plist = buf + dir[2];
    npair = dir[3];
  }
  const int b = blockIdx.x;
  if (b < nref) {
    const RefluxItem& ri = rlist[b];
    reflux_item<D, NT>(m, mode, out, fr, ri, dtp, w, lam_next);
    if (ri.level >= 1) {
      __syncthreads();
      restrict_faces<D>(m, out, ri.pid, ri.level, ri.target, ri.mask);
    }
  } else if (b - nref < npair) {
    const int pid = plist[b - nref], l = m.level[pid];
    restrict_patch<D>(m, out, pid, l, restrict_target<D>(m, pid, l));
  }
}

// ---------------------------------------------------------------------------
// CFL rate: max over leaf cells of sum_j (|u_j| + c) / h, as IEEE bits of a
// non-negative double (order-preserving): the cells' speeds reduced by lane
// shifts and LDS, one division by h and one 64-bit atomic max per block, into
// the part of the rate slot that its XCD owns (block_max_rate)
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_max_rate(DevMesh m, const double* __restrict__ U,
                                                  ListArg list,
                                                  unsigned long long* __restrict__ lam) {
  constexpr int NV = D + 2;
  live_list(list);
  if ((int)blockIdx.x >= list.count) return;
  unsigned long long best = 0ull;
  const int pid = list.ptr[blockIdx.x], l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n;
  const double* P = U + patch_base(m, pid, l);
  const int vs = var_stride<D>(L.full);
  // pairs along x (even patch edges), one 16-byte load per variable
  int total = n / 2;
  if constexpr (D >= 2) total *= n;
  if constexpr (D >= 3) total *= n;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int row = D >= 2 ? div_half(idx, L) : 0;
    const int z = D >= 3 ? div_by(row, n, L.n_mul) : 0;
    const int x = 2 * (idx - row * (n / 2)), y = row - z * n;
    const int off = box_off<D>(L.full, x + NG, y + NG, z + NG);
    double2 u[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = *reinterpret_cast<const double2*>(P + v * vs + off);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double c[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) c[v] = h == 0 ? u[v].x : u[v].y;
      const unsigned long long bits = cell_speed_bits<D>(c, m);
      best = bits > best ? bits : best;
    }
  }
  block_max_rate(best, L.h, lam);
}

__global__ void k_zero_rate(unsigned long long* slot) { clear_rate(slot); }

__global__ void k_dt_from_rate(const unsigned long long* __restrict__ lam, double cfl,
                               double* __restrict__ dt, unsigned long long* __restrict__ clear) {
  dt[0] = cfl / slot_rate(lam);
  if (clear) clear_rate(clear);
}

// ---------------------------------------------------------------------------
// tagging: per leaf, any cell within tag_buffer of the interior with
// |phi+ - phi-| > theta (|phi+| + |phi-|) for phi in {rho, p}, any direction
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void rho_p_at(const DevMesh& m, const double* P, long long vs,
                                         long long off, double& rho, double& p) {
  double u[D + 2];
#pragma unroll
  for (int v = 0; v < D + 2; ++v) u[v] = P[v * vs + off];
  rho = u[0];
  p = pressure_exact<D>(u, m.gm1);
}

// rho and p at patch-local cell c of patch P (level l, patch position pc);
// with FUSE a cell outside the patch is read from the same-level patch that
// holds it (neighbour table sN by offset code, periodic wrap and transmissive
// clamp applied), else from P's own ghost layer (prolonged values).
template <int D, bool FUSE>
__device__ __forceinline__ void rho_p_node(const DevMesh& m, const double* __restrict__ U,
                                           const double* __restrict__ P, long long vs, int full,
                                           int n, int l, const int pc[3], const int* sN,
                                           const int c[3], double& rho, double& p) {
  if constexpr (FUSE) {
    bool inside = true;
    for (int j = 0; j < D; ++j) inside &= (c[j] >= 0 && c[j] < n);
    if (!inside) {
      const LevelC& L = m.lv[l];
      int code = 0, loc[3] = {0, 0, 0}, mul = 1;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int g = bc_map(pc[j] * n + c[j], L.cells, m.periodic[j]);
        const int q = g / n;
        int o = q - pc[j];
        if (o > 1) o -= L.np;
        if (o < -1) o += L.np;
        loc[j] = g - q * n;
        code += (o + 1) * mul;
        mul *= 3;
      }
      const int src = sN[code];
      if (src >= 0) {
        rho_p_at<D>(m, U + patch_base(m, src, l), vs,
                    box_off<D>(full, loc[0] + NG, loc[1] + NG, loc[2] + NG), rho, p);
        return;
      }
    }
  }
  rho_p_at<D>(m, P, vs, box_off<D>(full, c[0] + NG, c[1] + NG, c[2] + NG), rho, p);
}

template <int D, bool FUSE>
__global__ __launch_bounds__(256) void k_tag(DevMesh m, const double* __restrict__ U,
                                             ListArg list, uint8_t* __restrict__ has_tag,
                                             uint8_t* __restrict__ raw, int lds_nodes) {
  live_list(list);
  if ((int)blockIdx.x >= list.count) return;
  const int pid = list.ptr[blockIdx.x];
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n, b = m.tag_buffer, w = n + 2 * b;
  const double* P = U + patch_base(m, pid, l);
  const int vs = var_stride<D>(L.full);
  const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
  // same-level neighbours by offset code (o0+1) + 3 (o1+1) + 9 (o2+1)
  __shared__ int sN[27];
  if constexpr (FUSE) {
    constexpr int NO = D == 1 ? 3 : (D == 2 ? 9 : 27);
    const int t = threadIdx.x;
    if (t < NO) {
      int q[3] = {0, 0, 0};
      bool in = true;
      for (int j = 0; j < D; ++j) {
        const int o = (j == 0 ? t : (j == 1 ? t / 3 : t / 9)) % 3 - 1;
        int v = pc[j] + o;
        if (v < 0 || v >= L.np) {
          if (m.periodic[j]) v = (v + L.np) % L.np;
          else in = false;
        }
        q[j] = v;
      }
      sN[t] = in ? map_at<D>(m, l, q) : -1;
    }
    __syncthreads();
  }
  int total = w;
  if constexpr (D >= 2) total *= w;
  if constexpr (D >= 3) total *= w;
  int any = 0;
  uint8_t* rp = raw ? raw + L.tag_off + (long long)(pid - L.pid_base) * vs : nullptr;
  // rho and p of every node of the box [-b-1, n+b]^D once, in LDS (dynamic,
  // sized on the host for the largest patch edge whose box fits; always in
  // 1D/2D), then the tests read LDS; larger 3D patches compute each cell's
  // neighbours directly below
  const int wn = w + 2;
  int nodes = wn;
  if constexpr (D >= 2) nodes *= wn;
  if constexpr (D >= 3) nodes *= wn;
  if (nodes <= lds_nodes) {
    extern __shared__ double stag[];
    double* sr = stag;
    double* sp = stag + nodes;
    for (int idx = threadIdx.x; idx < nodes; idx += blockDim.x) {
      const int c[3] = {idx % wn - b - 1, D >= 2 ? (idx / wn) % wn - b - 1 : 0,
                        D >= 3 ? idx / (wn * wn) - b - 1 : 0};
      rho_p_node<D, FUSE>(m, U, P, vs, L.full, n, l, pc, sN, c, sr[idx], sp[idx]);
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
      const int c0 = idx % w - b;
      const int c1 = D >= 2 ? (idx / w) % w - b : 0;
      const int c2 = D >= 3 ? idx / (w * w) - b : 0;
      const int node = (c0 + b + 1) + (D >= 2 ? (c1 + b + 1) * wn : 0) +
                       (D >= 3 ? (c2 + b + 1) * wn * wn : 0);
      bool t = false;
      for (int j = 0; j < D; ++j) {
        const int st = j == 0 ? 1 : (j == 1 ? wn : wn * wn);
        const double rp_ = sr[node + st], rm_ = sr[node - st];
        const double pp_ = sp[node + st], pm_ = sp[node - st];
        t |= fabs(rp_ - rm_) > m.theta * (fabs(rp_) + fabs(rm_));
        t |= fabs(pp_ - pm_) > m.theta * (fabs(pp_) + fabs(pm_));
      }
      any |= t;
      if (rp) rp[box_off<D>(L.full, c0 + NG, c1 + NG, c2 + NG)] = t ? 1 : 0;
    }
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) has_tag[pid] = any ? 1 : 0;
    return;
  }
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    int c[3] = {idx % w - b, 0, 0};
    if constexpr (D >= 2) c[1] = (idx / w) % w - b;
    if constexpr (D >= 3) c[2] = idx / (w * w) - b;
    bool t = false;
    for (int j = 0; j < D; ++j) {
      int cp[3] = {c[0], c[1], c[2]}, cm[3] = {c[0], c[1], c[2]};
      cp[j] += 1;
      cm[j] -= 1;
      double rp_, pp_, rm_, pm_;
      rho_p_node<D, FUSE>(m, U, P, vs, L.full, n, l, pc, sN, cp, rp_, pp_);
      rho_p_node<D, FUSE>(m, U, P, vs, L.full, n, l, pc, sN, cm, rm_, pm_);
      t |= fabs(rp_ - rm_) > m.theta * (fabs(rp_) + fabs(rm_));
      t |= fabs(pp_ - pm_) > m.theta * (fabs(pp_) + fabs(pm_));
    }
    any |= t;
    if (rp) rp[box_off<D>(L.full, c[0] + NG, c[1] + NG, c[2] + NG)] = t ? 1 : 0;
  }
  any = __syncthreads_or(any);
  if (threadIdx.x == 0) has_tag[pid] = any ? 1 : 0;
}

// Dilation of the cell tags, one block per tile of a leaf (blocks of the levels
// as in k_tag_cells; a block past its leaf's tiles ends): the tags of the tile
// and tag_buffer cells around it in LDS, then the maximum along x, y and z in
// turn.  SHARED: raw holds each cell's tag once, in its own patch, so that cells
// outside the patch are read from the same-level patch that holds them; a cell
// beyond a transmissive wall has no tag that the boundary cell lacks; where no
// patch is, and for SHARED false everywhere, the leaf's own ghost places hold
// the tags.  With (2 b + 1)^D reads of memory per cell 201 us (3D, 64^3 base and
// three levels of 16^3 and 8^3 patches, b = 2; the tags before it 473 us of each
// leaf's own dilated box, 211 shared) and 12.8 us (2D, 384^2 base), 91 and 8.8 so.
constexpr int cell_tile(int dim) { return dim == 1 ? 256 : (dim == 2 ? 32 : 8); }

// Entry of a list in level order whose tile is block b's, -1 past the last one;
// b becomes the tile, l the entry's level in `tl`.  (Branches marked as rare keep
// the recorded form out of the eager launches' instruction lines.)
__device__ __forceinline__ int level_item(const DevMesh& m, const TagLevels& tl, ListArg& list,
                                          int& b, int& l) {
  int first = 0;
  l = 0;
  if (__builtin_expect(tl.dir != nullptr, 0)) {
    for (; l < m.nlev - 1; ++l) {
      const int here = __builtin_amdgcn_readfirstlane(tl.dir[2 * l]);
      if (b < here * tl.tiles[l]) break;
      b -= here * tl.tiles[l];
      first += here;
    }
    live_list(list);
    if (first + b / tl.tiles[l] >= list.count) return -1;
  } else {
    for (; l < m.nlev - 1 && b >= tl.count[l] * tl.tiles[l]; ++l) {
      b -= tl.count[l] * tl.tiles[l];
      first += tl.count[l];
    }
  }
  const int item = first + b / tl.tiles[l];
  b %= tl.tiles[l];
  return item;
}

template <int D, bool SHARED>
__global__ __launch_bounds__(256) void k_cell_tags(DevMesh m, const uint8_t* __restrict__ raw,
                                                   ListArg leaves, TagLevels tl,
                                                   uint8_t* __restrict__ out) {
  constexpr int T = cell_tile(D), MAXB = 3, B = T + 2 * MAXB;
  constexpr int NODES = D == 1 ? B : (D == 2 ? B * B : B * B * B);
  constexpr int CENTRE = D == 1 ? 1 : (D == 2 ? 4 : 13);
  __shared__ uint8_t sa[NODES], sb[NODES];
  __shared__ int sN[27];
  int bl = blockIdx.x, k;
  const int item = level_item(m, tl, leaves, bl, k);
  if (item < 0) return;
  const int tile = bl, pid = leaves.ptr[item];
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n, b = m.tag_buffer, vs = var_stride<D>(L.full), nt = (n + T - 1) / T;
  if (tile >= (D == 1 ? nt : (D == 2 ? nt * nt : nt * nt * nt))) return;
  const int o[3] = {tile % nt * T, D >= 2 ? tile / nt % nt * T : 0, D >= 3 ? tile / (nt * nt) * T : 0};
  int e[3] = {1, 1, 1};  // cells of the tile (the last tile of an edge may be partial)
#pragma unroll
  for (int j = 0; j < D; ++j) e[j] = min(T, n - o[j]);
  const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
  if constexpr (SHARED) {
    constexpr int NO = D == 1 ? 3 : (D == 2 ? 9 : 27);
    const int t = threadIdx.x;
    if (t < NO) {
      int q[3] = {0, 0, 0};
      bool in = true;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int d = (j == 0 ? t : (j == 1 ? t / 3 : t / 9)) % 3 - 1;
        q[j] = pc[j] + d;
        if ((unsigned)q[j] >= (unsigned)L.np) {
          if (m.periodic[j]) q[j] -= d * L.np;
          else in = false;
        }
      }
      sN[t] = in ? map_at<D>(m, l, q) : -1;
    }
    __syncthreads();
  }
  // places up to the tile's last row or plane (small patches and the last tiles
  // fill a part of the LDS box)
  const int live = D == 1 ? e[0] + 2 * b : (D == 2 ? B * (e[1] + 2 * b) : B * B * (e[2] + 2 * b));
  const uint8_t* level = raw + L.tag_off;
  const uint8_t* own = level + (long long)(pid - L.pid_base) * vs;
  for (int idx = threadIdx.x; idx < live; idx += 256) {
    const int t[3] = {idx % B, D >= 2 ? idx / B % B : 0, D >= 3 ? idx / (B * B) : 0};
    int c[3] = {0, 0, 0};
    bool in = true;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      in = in && t[j] < e[j] + 2 * b;
      c[j] = o[j] + t[j] - b;
    }
    if (!in) continue;
    const uint8_t* src = own;
    bool wall = false;
    if constexpr (SHARED) {
      int code = 0, mul = 1, loc[3] = {0, 0, 0};
#pragma unroll
      for (int j = 0; j < D; ++j) {
        int d = c[j] < 0 ? -1 : (c[j] >= n ? 1 : 0);
        loc[j] = c[j] - d * n;
        if (d != 0 && !m.periodic[j] && (unsigned)(pc[j] + d) >= (unsigned)L.np) {
          wall = true;
          d = 0;
        }
        code += (d + 1) * mul;
        mul *= 3;
      }
      const int nb = code == CENTRE ? pid : sN[code];
      wall = wall && nb >= 0;
      if (!wall && nb >= 0) {
        src = level + (long long)(nb - L.pid_base) * vs;
#pragma unroll
        for (int j = 0; j < D; ++j) c[j] = loc[j];
      }
    }
    sa[idx] = wall ? (uint8_t)0 : src[box_off<D>(L.full, c[0] + NG, c[1] + NG, c[2] + NG)];
  }
  __syncthreads();
  // along direction j (T_j cells from T_j + 2 b places; the others keep theirs)
  auto dilate = [&](int j, const uint8_t* from, auto put) {
    const int st = j == 0 ? 1 : (j == 1 ? B : B * B);
    for (int idx = threadIdx.x; idx < live; idx += 256) {
      const int t[3] = {idx % B, D >= 2 ? idx / B % B : 0, D >= 3 ? idx / (B * B) : 0};
      bool in = true;
#pragma unroll
      for (int d = 0; d < D; ++d) in = in && t[d] < e[d] + (d > j ? 2 * b : 0);
      if (!in) continue;
      int v = 0;
      for (int q = 0; q <= 2 * b; ++q) v |= from[idx + q * st];
      put(idx, t, (uint8_t)(v ? 1 : 0));
    }
  };
  uint8_t* op = out + L.tag_off + (long long)(pid - L.pid_base) * vs;
  auto result = [&](int, const int t[3], uint8_t v) {
    op[box_off<D>(L.full, o[0] + t[0] + NG, o[1] + t[1] + NG, o[2] + t[2] + NG)] = v;
  };
  if constexpr (D == 1) {
    dilate(0, sa, result);
  } else {
    dilate(0, sa, [&](int idx, const int*, uint8_t v) { sb[idx] = v; });
    __syncthreads();
    if constexpr (D == 2) {
      dilate(1, sb, result);
    } else {
      dilate(1, sb, [&](int idx, const int*, uint8_t v) { sa[idx] = v; });
      __syncthreads();
      dilate(2, sa, result);
    }
  }
}

// ---------------------------------------------------------------------------
// 3D tag flags in three passes (fused halo; with `raw` also each cell's own tag).  A patch has a
// tag when a cell within tag_buffer = b cells of its interior is tagged; a cell
// of the dilated box that lies in a same-level patch has there the tag it has
// here (the same cell values around it), so every cell is tested once, by its
// own patch, and the patches share the outcome:
//  k_tag_cells    each patch's cells, as a 27-bit mask: bit (r0+1) + 3 (r1+1) +
//                 9 (r2+1) is set when a tagged cell lies within b cells of
//                 the low (r = -1) or high (r = 1) side in each direction
//                 with r != 0;
//  k_tag_regions  the cells of ghost regions without a same-level patch
//                 (prolonged values), b deep, of leaves without a tag of their
//                 own;
//  k_tag_flags    a patch's flag from its own mask, its regions' flag and the
//                 facing bits of its neighbours' masks.
// A position beyond a transmissive wall repeats the boundary cell along the
// wall and adds no difference across it: its tag implies the boundary cell's.
// One block per patch over the dilated box evaluated 5 nodes per 8^3 patch cell
// (2744 for 512) with three divisions each, and 6 per cell without LDS for
// larger patches: 908 us for 13.8 k leaves (11.8 M cells) and 218 us for 195
// coarsening candidates, against 542 us for the three passes (309, 214 and 7)
// with the clear and the requests.
// ---------------------------------------------------------------------------
constexpr int kTagTile = 8;   // cells per tile edge of k_tag_cells

// pressure_exact with one reciprocal for the D quotients (see Divisor).
template <int D>
__device__ __forceinline__ double pressure_fast(const double* u, double gm1) {
  const Divisor rho(u[0]);
  bool ok = true;
#pragma unroll
  for (int j = 0; j < D; ++j) ok = ok && rho.takes(u[1 + j]);
  if (!ok) return pressure_exact<D>(u, gm1);
  double ke = u[1] * rho(u[1]);
#pragma unroll
  for (int j = 1; j < D; ++j) ke = ke + u[1 + j] * rho(u[1 + j]);
  ke = 0.5 * ke;
  return gm1 * (u[D + 1] - ke);
}

__device__ __forceinline__ bool differs(double a, double b, double theta) {
  return fabs(a - b) > theta * (fabs(a) + fabs(b));
}

// rho and p at patch-local cell c (at most 4 cells outside patch P of the
// neighbour table sNB): in the same-level patch that holds it, else in P's own
// ghost layer.
__device__ __forceinline__ void tag_node(const DevMesh& m, const double* __restrict__ U,
                                         const double* __restrict__ P, int n, int full, int vs,
                                         int np, const int pc[3], const long long* sNB,
                                         const int c[3], double& rho, double& p) {
  int code = 0, mul = 1, loc[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    int o = c[j] < 0 ? -1 : (c[j] >= n ? 1 : 0);
    loc[j] = c[j] - o * n;
    if (o != 0 && !m.periodic[j] && (unsigned)(pc[j] + o) >= (unsigned)np) {
      loc[j] = o < 0 ? 0 : n - 1;
      o = 0;
    }
    code += (o + 1) * mul;
    mul *= 3;
  }
  const long long sb = sNB[code];
  const double* src = U + sb;
  int off = box_off<3>(full, loc[0] + NG, loc[1] + NG, loc[2] + NG);
  if (sb < 0) {
    src = P;
    off = box_off<3>(full, c[0] + NG, c[1] + NG, c[2] + NG);
  }
  double u[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) u[v] = src[v * vs + off];
  rho = u[0];
  p = pressure_fast<3>(u, m.gm1);
}

// One block per 8^3 tile of every active patch (`list` in level order; the
// level of a block and its patch and tile follow from the blocks per level):
// rho and p of the tile and one layer around it in LDS, then the tile's cells.
// Bound by memory: the 64-byte rows of an 8^3 patch are fetched as 128-byte
// lines, 9.2 of the 13.8 KB of a variable for 4 KB of cells.  Chunks of 16
// consecutive tiles per XCD, so that x neighbours share their cells in one L2:
// 14.6 M cells 425 us in launch order, 309 so (64 and 128 the same).
constexpr int kTagChunk = 16;

__global__ __launch_bounds__(256) void k_tag_cells(DevMesh m, const double* __restrict__ U,
                                                   ListArg list, TagLevels tl, int blocks,
                                                   int* __restrict__ mask,
                                                   uint8_t* __restrict__ raw) {
  constexpr int B = kTagTile + 2;
  __shared__ long long sNB[27];
  __shared__ double sr[B * B * B], sp[B * B * B];
  __shared__ int sm;
  int b = xcd_chunk<kTagChunk>(blocks), l;
  if (b < 0) return;
  const int item = level_item(m, tl, list, b, l);
  if (item < 0) return;
  const int tile = b, pid = list.ptr[item];
  const LevelC& L = m.lv[l];
  const int n = L.n, full = L.full, vs = var_stride<3>(full);
  const int nt = (n + kTagTile - 1) / kTagTile;
  const int o[3] = {tile % nt * kTagTile, tile / nt % nt * kTagTile, tile / (nt * nt) * kTagTile};
  const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
  load_neighbours<3>(m, l, pc, sNB);
  if (threadIdx.x == 0) sm = 0;
  __syncthreads();
  const double* P = U + patch_base(m, pid, l);
  int e[3];  // cells of the tile (the last tile of an edge may be partial)
#pragma unroll
  for (int j = 0; j < 3; ++j) e[j] = min(kTagTile, n - o[j]);
#pragma unroll 2
  for (int idx = threadIdx.x; idx < B * B * B; idx += 256) {
    const int t[3] = {idx % B - 1, idx / B % B - 1, idx / (B * B) - 1};
    int outside = 0;
    bool in = true;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      outside += t[j] < 0 || t[j] >= e[j];
      in = in && t[j] <= e[j];
    }
    if (outside > 1 || !in) continue;  // edges and corners are not tested
    const int c[3] = {o[0] + t[0], o[1] + t[1], o[2] + t[2]};
    tag_node(m, U, P, n, full, vs, L.np, pc, sNB, c, sr[idx], sp[idx]);
  }
  __syncthreads();
  int bits = 0;
  const int tb = m.tag_buffer;
  for (int idx = threadIdx.x; idx < kTagTile * kTagTile * kTagTile; idx += 256) {
    const int t[3] = {idx % kTagTile, idx / kTagTile % kTagTile, idx / (kTagTile * kTagTile)};
    if (t[0] >= e[0] || t[1] >= e[1] || t[2] >= e[2]) continue;
    const int node = t[0] + 1 + B * (t[1] + 1 + B * (t[2] + 1));
    bool tag = false;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int st = j == 0 ? 1 : (j == 1 ? B : B * B);
      tag |= differs(sr[node + st], sr[node - st], m.theta);
      tag |= differs(sp[node + st], sp[node - st], m.theta);
    }
    if (raw)
      raw[L.tag_off + (long long)(pid - L.pid_base) * vs +
          box_off<3>(full, o[0] + t[0] + NG, o[1] + t[1] + NG, o[2] + t[2] + NG)] = tag ? 1 : 0;
    if (!tag) continue;
    // sides the cell is near, per direction: bit 0 low, 1 always, 2 high
    int side[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int c = o[j] + t[j];
      side[j] = 2 | (c < tb ? 1 : 0) | (c >= n - tb ? 4 : 0);
    }
    int m9 = 0, m27 = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) m9 |= (side[1] >> k & 1) ? side[0] << (3 * k) : 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) m27 |= (side[2] >> k & 1) ? m9 << (9 * k) : 0;
    bits |= m27;
  }
  if (bits) atomicOr(&sm, bits);
  __syncthreads();
  if (threadIdx.x == 0 && sm) atomicOr(mask + pid, sm);
}

// Ghost regions without a same-level patch, 4 per block: bit 27 of the leaf's
// mask is set when a cell of the region within tag_buffer of the leaf is
// tagged (values prolonged into the leaf's ghost layer by the fill).  Bound by
// the lines it fetches (1.4 GB for 205 us, mostly ghost rows of 32 bytes);
// consecutive groups share an XCD as in k_tag_cells (214 us in launch order).
__global__ __launch_bounds__(128) void k_tag_regions(DevMesh m, const double* __restrict__ U,
                                                     ListArg regions, int* __restrict__ mask,
                                                     uint8_t* __restrict__ raw) {
  constexpr int G = 4, CENTRE = 1 << 13;
  __shared__ long long sNB[G][27];
  __shared__ int s_pid[G], s_code[G], s_lev[G], s_pc[G][3], s_pre[G + 1];
  live_list(regions);
  const int* list = regions.ptr;
  const int b = m.tag_buffer, count = regions.count;
  const int bb = xcd_chunk<kTagChunk>((count + G - 1) / G);
  if (bb < 0) return;
  {
    // one neighbour table per region, by the threads [27 g, 27 g + 27)
    const int g = (int)threadIdx.x / 27, t = (int)threadIdx.x - 27 * g;
    const int i = bb * G + g;
    if (g < G && i < count) {
      const int pid = list[2 * i], l = m.level[pid], np = m.lv[l].np;
      int q[3];
      bool in = true;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int o = (j == 0 ? t : (j == 1 ? t / 3 : t / 9)) % 3 - 1;
        q[j] = m.coord[3 * pid + j] + o;
        if (t == 13) s_pc[g][j] = q[j];
        if ((unsigned)q[j] >= (unsigned)np) {
          if (m.periodic[j]) q[j] -= o * np;
          else in = false;
        }
      }
      const int nb = in ? map_at<3>(m, l, q) : -1;
      sNB[g][t] = nb >= 0 ? patch_base(m, nb, l) : -1;
    }
  }
  if (threadIdx.x == 0) {
    s_pre[0] = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int i = bb * G + g;
      int cells = 0;
      if (i < count) {
        const int pid = list[2 * i], code = list[2 * i + 1], l = m.level[pid];
        s_pid[g] = pid;
        s_code[g] = code;
        s_lev[g] = l;
        // a leaf with a tag of its own needs no more (but its cells' tags)
        if (raw || !(mask[pid] & CENTRE)) {
          cells = 1;
#pragma unroll
          for (int j = 0; j < 3; ++j)
            cells *= (j == 0 ? code : (j == 1 ? code / 3 : code / 9)) % 3 == 1 ? m.lv[l].n : b;
        }
      }
      s_pre[g + 1] = s_pre[g] + cells;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < s_pre[G]; idx += 128) {
    int it = idx >= s_pre[2] ? 2 : 0;
    if (idx >= s_pre[it + 1]) ++it;
    const int local = idx - s_pre[it], code = s_code[it];
    const LevelC& L = m.lv[s_lev[it]];
    const int n = L.n, full = L.full, vs = var_stride<3>(full);
    const double* P = U + sNB[it][13];
    const int pc[3] = {s_pc[it][0], s_pc[it][1], s_pc[it][2]};
    int c[3], left = local;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int r = (j == 0 ? code : (j == 1 ? code / 3 : code / 9)) % 3 - 1;
      const int ext = r == 0 ? n : b;
      const int k = left % ext;
      left /= ext;
      c[j] = r < 0 ? k - b : (r == 0 ? k : n + k);
    }
    bool tag = false;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      int cp[3] = {c[0], c[1], c[2]}, cm[3] = {c[0], c[1], c[2]};
      cp[j] += 1;
      cm[j] -= 1;
      double rp, pp, rm, pm;
      tag_node(m, U, P, n, full, vs, L.np, pc, sNB[it], cp, rp, pp);
      tag_node(m, U, P, n, full, vs, L.np, pc, sNB[it], cm, rm, pm);
      tag |= differs(rp, rm, m.theta);
      tag |= differs(pp, pm, m.theta);
    }
    if (tag) atomicOr(mask + s_pid[it], 1 << 27);
    if (raw)
      raw[L.tag_off + (long long)(s_pid[it] - L.pid_base) * vs +
          box_off<3>(full, c[0] + NG, c[1] + NG, c[2] + NG)] = tag ? 1 : 0;
  }
}

// Tag flag of every patch of `list`: a tagged cell of its own, one of its
// prolonged regions, or one of a neighbour within tag_buffer of it (the
// neighbour at offset code k faces it with its side 26 - k).  8 lanes a patch.
__global__ __launch_bounds__(256) void k_tag_flags(DevMesh m, ListArg list,
                                                   const int* __restrict__ mask,
                                                   uint8_t* __restrict__ has_tag) {
  live_list(list);
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x) >> 3, lane = threadIdx.x & 7;
  int any = 0, pid = -1;
  if (i < list.count) {
    pid = list.ptr[i];
    const int l = m.level[pid], np = m.lv[l].np;
    const int pc[3] = {m.coord[3 * pid], m.coord[3 * pid + 1], m.coord[3 * pid + 2]};
    if (lane == 0) any = mask[pid] & (1 << 13 | 1 << 27);
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 8) {
      const int k = k0 + lane;
      int q[3];
      bool in = k < 27 && k != 13;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int o = (j == 0 ? k : (j == 1 ? k / 3 : k / 9)) % 3 - 1;
        q[j] = pc[j] + o;
        if ((unsigned)q[j] >= (unsigned)np) {
          if (m.periodic[j]) q[j] -= o * np;
          else in = false;
        }
      }
      const int nb = in ? map_at<3>(m, l, q) : -1;
      if (nb >= 0) any |= mask[nb] >> (26 - k) & 1;
    }
  }
  for (int d = 4; d > 0; d >>= 1) any |= __shfl_xor(any, d);
  if (lane == 0 && pid >= 0) has_tag[pid] = any ? 1 : 0;
}

// One wave, a sum of terms after the other: recorded at the end of a caller's
// recording of a call.  In the kernels themselves (the check at their end, the
// flag in DevMesh) it cost every 2D step 0.6 %, recorded by the caller or not.
__global__ void k_check_covers(const int* __restrict__ dir, CoverTerms c, int* __restrict__ err) {
  int sum = 0;
  for (int i = 0; i < c.n; ++i) {
    sum += dir[c.t[i].at] * c.t[i].weight;
    if (c.t[i].cover < 0) continue;
    if (sum > c.t[i].cover) err[0] = 1;
    sum = 0;
  }
}

__global__ void k_zero_int(int* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// refine request: active leaf below the finest level with a tag;
// coarsen request: patch whose children are all leaves without tags.  8 lanes a
// patch: a 3D patch has up to 64 children, whose flags one lane would read in
// a chain of 64 (20 us for 16 k slots, 6.8 us now).
__global__ __launch_bounds__(256) void k_requests(DevMesh m, const uint8_t* __restrict__ has_tag,
                                                  const uint8_t* __restrict__ active_leaf,
                                                  int nslots, uint8_t* __restrict__ refine,
                                                  uint8_t* __restrict__ coarsen) {
  const int pid = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 3), lane = threadIdx.x & 7;
  if (pid >= nslots) return;  // whole groups of 8 lanes
  const uint8_t al = active_leaf[pid];  // 0 inactive, 1 leaf, 2 non-leaf
  int rq = 0, cq = 0;
  if (al == 1) {
    rq = (has_tag[pid] && m.level[pid] < m.nlev - 1) ? 1 : 0;
  } else if (al == 2) {
    // a coarsening candidate (all children leaves) was tagged on its own
    // restricted data as well; it is coarsened only if that is untagged too
    cq = has_tag[pid] ? 0 : 1;
    const int nc = m.nchild[pid];
#pragma unroll 4
    for (int k = lane; k < nc; k += 8) {
      const int c = m.child[(long long)pid * m.maxc + k];
      cq &= (active_leaf[c] == 1 && !has_tag[c]) ? 1 : 0;
    }
  }
  for (int d = 4; d > 0; d >>= 1) cq &= __shfl_xor(cq, d);
  if (lane == 0) {
    if (refine) refine[pid] = (uint8_t)rq;
    if (coarsen) coarsen[pid] = (uint8_t)cq;
  }
}

// prolongation of the interiors of newly created patches of one level, by
// coarse cell: one thread forms the limited slopes of a coarse cell and its
// 2^D children (84.7 us for 3456 patches of 8^3 with a thread per fine cell,
// 30.3 us now)
template <int D, int NT>
__global__ __launch_bounds__(NT) void k_prolong_new(DevMesh m, const double* __restrict__ Uin,
                                                    double* __restrict__ U, ListArg list,
                                                    int* __restrict__ err) {
  constexpr int NV = D + 2;
  if ((int)blockIdx.x >= list.count) return;
  const int pid = list.ptr[blockIdx.x];
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n, h = n / 2;
  double* P = U + patch_base(m, pid, l);
  const int vs = var_stride<D>(L.full);
  const double sg[3][2] = {{-1.0, 1.0}, {-1.0, 1.0}, {-1.0, 1.0}};
  int total = h;
  if constexpr (D >= 2) total *= h;
  if constexpr (D >= 3) total *= h;
  for (int idx = threadIdx.x; idx < total; idx += NT) {
    // 2 idx / n = idx / h
    const int r = D >= 2 ? div_by(2 * idx, n, L.n_mul) : 0;
    const int z = D >= 3 ? div_by(2 * r, n, L.n_mul) : 0;
    const int k[3] = {idx - r * h, D >= 2 ? r - z * h : 0, z};
    int gc[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < D; ++j) gc[j] = m.coord[3 * pid + j] * h + k[j];
    double phi[NV] = {}, sl[D][NV] = {};
    const bool ok = prolong_coarse<D>(m, Uin, l - 1, gc, phi, sl);
    if (!ok) err[0] = 1;
    store_children<D>(P, vs, L.full,
                      box_off<D>(L.full, 2 * k[0] + NG, 2 * k[1] + NG, 2 * k[2] + NG), ok, phi, sl,
                      sg);
  }
}

__global__ void k_count_nonzero(const uint8_t* __restrict__ a, int n, int* __restrict__ out) {
  int c = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    c += a[i] ? 1 : 0;
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(out, c);
}

__global__ void k_scatter_int(int* __restrict__ dst, const int* __restrict__ pairs, int npairs) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < npairs) dst[pairs[2 * i]] = pairs[2 * i + 1];
}

template <int D>
__global__ __launch_bounds__(256) void k_check(DevMesh m, const double* __restrict__ U,
                                               ListArg list, int* __restrict__ bad) {
  constexpr int NV = D + 2;
  live_list(list);
  if ((int)blockIdx.x >= list.count) return;
  const int pid = list.ptr[blockIdx.x];
  const int l = m.level[pid];
  const LevelC& L = m.lv[l];
  const int n = L.n;
  const double* P = U + patch_base(m, pid, l);
  const int vs = var_stride<D>(L.full);
  int total = n;
  if constexpr (D >= 2) total *= n;
  if constexpr (D >= 3) total *= n;
  int cnt = 0;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int x = idx % n;
    const int y = D >= 2 ? (idx / n) % n : 0;
    const int z = D >= 3 ? idx / (n * n) : 0;
    double u[NV];
    const int off = box_off<D>(L.full, x + NG, y + NG, z + NG);
    for (int v = 0; v < NV; ++v) u[v] = P[v * vs + off];
    const double p = pressure_exact<D>(u, m.gm1);
    if (!(u[0] > 0.0 && p > 0.0)) ++cnt;
  }
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
  if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(bad, cnt);
}

}  // namespace

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
#define AMR_DISPATCH_DIM(dim, KERNEL, GRID, BLOCK, STREAM, ...)                         \
  do {                                                                                  \
    if ((dim) == 1) hipLaunchKernelGGL(KERNEL<1>, GRID, BLOCK, 0, STREAM, __VA_ARGS__); \
    else if ((dim) == 2) hipLaunchKernelGGL(KERNEL<2>, GRID, BLOCK, 0, STREAM, __VA_ARGS__); \
    else hipLaunchKernelGGL(KERNEL<3>, GRID, BLOCK, 0, STREAM, __VA_ARGS__);             \
  } while (0)

// Whether the coarse/fine fill launch of this mesh works by coarse cell, and
// its regions per block (the kernel choice of fill_cf below).
static bool fill_cf_by_coarse(const DevMesh& m) {
  int nmax = 0;
  for (int l = 1; l < m.nlev; ++l) nmax = std::max(nmax, m.lv[l].n);
  return m.dim == 3 || (m.dim == 2 && nmax > 16);
}

static int fill_cf_per_block(const DevMesh& m) {
  if (!fill_cf_by_coarse(m)) return 1;
  return m.dim == 2 ? 2 : 4;
}

int Kernels::fill_cf_grid(const DevMesh& m, int count) {
  const int g = fill_cf_per_block(m);
  return (count + g - 1) / g;
}

void Kernels::fill_cf(const DevMesh& m, double* U, const ListArg& regions, int* err,
                      hipStream_t s) {
  if (regions.count <= 0) return;
  // one block per region (group of regions)
  auto launch = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3(fill_cf_grid(m, regions.count)), dim3(threads), 0, s, m, U, regions,
                       err);
  };
  switch (m.dim) {
    case 1: launch(k_fill_cf<1, 64>, 64); break;
    case 2: {
      // refined patches of edge 16 or less: one fine cell per thread (a side
      // region is 4 n = 64 cells); wider ones: by coarse cell, two regions
      // per wave (a side region of a 32^2 patch is 64 coarse cells).  Level 0
      // has no prolonged ghosts.  Per launch on a 3-level 2D hierarchy of
      // base 256^2 with 32/16/16 patches (484 side regions): 5.2 us per fine
      // cell, 5.6 us by coarse cell; on a 5-level one of base 512^2 with 32^2
      // patches (1808): 11.0 us by coarse cell with 2 regions per wave, 10.9
      // with 4 per two waves, 12.9 with 4 per wave.
      if (fill_cf_by_coarse(m))
        launch(k_fill_cf_coarse<2, 64, 2>, 64);
      else
        launch(k_fill_cf<2, 64>, 64);
      break;
    }
    default:
      // one thread per coarse cell, 4 regions per two waves: a side region of
      // an 8^3 patch covers 32 coarse cells and one of a 16^3 patch 128 (side
      // regions of four-level hierarchies of base 64^3 with 32/16/16/8 patches:
      // 114 us with 4 regions per 128 threads, 135 with 4 per 64, 118 with 8
      // per 256, 145 with 8 per 128; 16.3 / 23.3 / 20.9 / 24.9 us on a two-level
      // one of 12^3 patches)
      launch(k_fill_cf_coarse<3, 128, 4>, 128);
      break;
  }
}

void Kernels::fill(const DevMesh& m, double* U, const ListArg& list, const ListArg& regions,
                   int* err, hipStream_t s) {
  const int group = kXcds * kCopyChunk;  // blocks per group of chunks (xcd_chunk)
  const int copies = (list.count + group - 1) / group * group;
  if (m.dim == 3) {
    if (copies > 0)
      hipLaunchKernelGGL(k_fill_copy3, dim3(copies), dim3(256), 0, s, m, U, U, list);
    fill_cf(m, U, regions, err, s);
    return;
  }
  const int per = m.dim == 1 ? 1 : kFillGroup;
  // whole groups of kXcds blocks, so that a copy block's XCD follows its index
  const int rblocks = ((regions.count + per - 1) / per + kXcds - 1) / kXcds * kXcds;
  if (rblocks + copies <= 0) return;
  if (m.dim == 1)
    hipLaunchKernelGGL(k_fill<1>, dim3(rblocks + copies), dim3(fill_threads(1)), 0, s, m, U, U, list,
                       regions, rblocks, err);
  else
    hipLaunchKernelGGL(k_fill<2>, dim3(rblocks + copies), dim3(fill_threads(2)), 0, s, m, U, U, list,
                       regions, rblocks, err);
}

void Kernels::reflux(const DevMesh& m, int mode, double* out, const double* fr,
                     const ListArg& list, const double* dt, double w,
                     unsigned long long* lam_next, hipStream_t s) {
  if (list.count <= 0) return;
  auto launch = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3(list.count), dim3(threads), 0, s, m, mode, out, fr,
                       reinterpret_cast<const RefluxItem*>(list.ptr), list.count, list.dir, dt, w,
                       lam_next);
  };
  switch (m.dim) {
    case 1: launch(k_reflux<1, 64>, 64); break;
    case 2: launch(k_reflux<2, 64>, 64); break;
    default: launch(k_reflux<3, 512>, 512); break;
  }
}

void Kernels::post(const DevMesh& m, int mode, double* out, const double* fr,
                   const ListArg& rlist, const ListArg& plist, const double* dt, double w,
                   unsigned long long* lam_next, hipStream_t s) {
  const int nb = rlist.count + plist.count;
  if (nb <= 0) return;
  auto launch = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3(nb), dim3(threads), 0, s, m, mode, out, fr,
                       reinterpret_cast<const RefluxItem*>(rlist.ptr), rlist.count, plist.ptr,
                       plist.count, rlist.dir, dt, w, lam_next);
  };
  switch (m.dim) {
    case 1: launch(k_post<1, 64>, 64); break;
    case 2: launch(k_post<2, 256>, 256); break;
    // 3D: the cells of two 16^3 faces (256 threads took 22 % longer, 1024 the
    // same within 5 %)
    default: launch(k_post<3, 512>, 512); break;
  }
}

void Kernels::restrict_level(const DevMesh& m, double* U, const ListArg& list, hipStream_t s) {
  if (list.count <= 0) return;
  // one block per child patch, one thread per covered parent cell
  auto launch = [&](auto kern, int threads) {
    hipLaunchKernelGGL(kern, dim3(list.count), dim3(threads), 0, s, m, U, list);
  };
  switch (m.dim) {
    case 1: launch(k_restrict<1>, 64); break;
    // 2D: a 32^2 patch covers 256 parent cells
    case 2: launch(k_restrict<2>, 256); break;
    default: launch(k_restrict<3>, 256); break;
  }
}

void Kernels::max_rate(const DevMesh& m, const double* U, const ListArg& list,
                       unsigned long long* lam, hipStream_t s) {
  if (list.count <= 0) return;
  AMR_DISPATCH_DIM(m.dim, k_max_rate, dim3(list.count), dim3(256), s, m, U, list, lam);
}

void Kernels::zero_rate(unsigned long long* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_rate, dim3(1), dim3(1), 0, s, slot);
}

void Kernels::dt_from_rate(const DevMesh& m, const unsigned long long* lam, double* dt,
                           unsigned long long* clear, hipStream_t s) {
  hipLaunchKernelGGL(k_dt_from_rate, dim3(1), dim3(1), 0, s, lam, m.cfl, dt, clear);
}

void Kernels::tag(const DevMesh& m, const double* U, const ListArg& list, uint8_t* has_tag,
                  uint8_t* raw, bool fuse, hipStream_t s) {
  const int nb = list.count;
  if (nb <= 0) return;
  // LDS for rho and p on the box [-b-1, n+b]^D of the largest patch edge
  // (1D/2D), or of the largest edge whose box fits 64 KB (3D)
  int lds_nodes = 0;
  for (int l = 0; l < m.nlev; ++l) {
    const long long wn = (long long)m.lv[l].n + 2 * m.tag_buffer + 2;
    const long long nodes = m.dim == 1 ? wn : (m.dim == 2 ? wn * wn : wn * wn * wn);
    if (m.dim <= 2 || nodes * 2 * (long long)sizeof(double) <= 64 * 1024)
      lds_nodes = std::max<long long>(lds_nodes, nodes);
  }
  const size_t lds = 2 * (size_t)lds_nodes * sizeof(double);
  if (lds > 160 * 1024) throw std::runtime_error("tagging box exceeds LDS");
  if (lds > 64 * 1024) {
    static bool big = false;
    if (!big) {
      big = true;
      (void)hipFuncSetAttribute((const void*)k_tag<1, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      (void)hipFuncSetAttribute((const void*)k_tag<1, false>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      (void)hipFuncSetAttribute((const void*)k_tag<2, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      (void)hipFuncSetAttribute((const void*)k_tag<2, false>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    }
  }
#define AMR_TAG(D)                                                                           \
  do {                                                                                       \
    if (fuse) k_tag<D, true><<<nb, 256, lds, s>>>(m, U, list, has_tag, raw, lds_nodes);      \
    else k_tag<D, false><<<nb, 256, lds, s>>>(m, U, list, has_tag, raw, lds_nodes);          \
  } while (0)
  if (m.dim == 1) AMR_TAG(1);
  else if (m.dim == 2) AMR_TAG(2);
  else AMR_TAG(3);
#undef AMR_TAG
}

int Kernels::tag_tiles(int n) {
  const int nt = (n + kTagTile - 1) / kTagTile;
  return nt * nt * nt;
}

int Kernels::cell_tiles(int dim, int n) {
  const int nt = (n + cell_tile(dim) - 1) / cell_tile(dim);
  return dim == 1 ? nt : (dim == 2 ? nt * nt : nt * nt * nt);
}

void Kernels::check_covers(const int* dir, const CoverTerms& c, int* err, hipStream_t s) {
  hipLaunchKernelGGL(k_check_covers, dim3(1), dim3(1), 0, s, dir, c, err);
}

void Kernels::tag_flags3(const DevMesh& m, const double* U, const ListArg& list,
                         const int* level_count, const int* level_dir, const ListArg& regions,
                         int* mask, uint8_t* has_tag, uint8_t* raw, hipStream_t s) {
  const int count = list.count;
  if (count <= 0) return;
  TagLevels tl{};
  if (list.dir) tl.dir = level_dir;
  int blocks = 0;
  for (int l = 0; l < m.nlev; ++l) {
    tl.count[l] = level_count[l];
    tl.tiles[l] = tag_tiles(m.lv[l].n);
    blocks += tl.count[l] * tl.tiles[l];
  }
  hipLaunchKernelGGL(k_zero_int, dim3((m.max_patches + 255) / 256), dim3(256), 0, s, mask,
                     m.max_patches);
  const int group = kXcds * kTagChunk;  // blocks per group of chunks (xcd_chunk)
  hipLaunchKernelGGL(k_tag_cells, dim3((blocks + group - 1) / group * group), dim3(256), 0, s, m, U,
                     list, tl, blocks, mask, raw);
  // without dilation no ghost cell counts
  if (regions.count > 0 && m.tag_buffer > 0)
    hipLaunchKernelGGL(k_tag_regions, dim3(((regions.count + 3) / 4 + group - 1) / group * group),
                       dim3(128), 0, s, m, U, regions, mask, raw);
  hipLaunchKernelGGL(k_tag_flags, dim3((count + 31) / 32), dim3(256), 0, s, m, list, mask, has_tag);
}

void Kernels::cell_tags(const DevMesh& m, const uint8_t* raw, const ListArg& leaves,
                        const int* level_leaves, const int* level_dir, bool shared, uint8_t* out,
                        hipStream_t s) {
  const int count = leaves.count;
  if (count <= 0) return;
  TagLevels tl{};
  if (leaves.dir) tl.dir = level_dir;
  int most = 0, blocks = 0;
  for (int l = 0; l < m.nlev; ++l) {
    tl.tiles[l] = cell_tiles(m.dim, m.lv[l].n);
    most = std::max(most, tl.tiles[l]);
    tl.count[l] = level_leaves ? level_leaves[l] : 0;
    blocks += tl.count[l] * tl.tiles[l];
  }
  if (!level_leaves) {
    // leaves of any level: blocks for the most tiles
    tl.count[0] = count;
    tl.tiles[0] = most;
    blocks = count * most;
  }
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, m, raw, leaves, tl, out);
  };
  switch (m.dim) {
    case 1: launch(k_cell_tags<1, false>); break;
    case 2: launch(k_cell_tags<2, false>); break;
    default:
      if (shared) launch(k_cell_tags<3, true>);
      else launch(k_cell_tags<3, false>);
  }
}

void Kernels::requests(const DevMesh& m, const uint8_t* has_tag, const uint8_t* active_leaf,
                       int nslots, uint8_t* refine, uint8_t* coarsen, hipStream_t s) {
  if (nslots <= 0) return;
  hipLaunchKernelGGL(k_requests, dim3((nslots + 31) / 32), dim3(256), 0, s, m, has_tag,
                     active_leaf, nslots, refine, coarsen);
}

void Kernels::prolong_new(const DevMesh& m, double* U, const ListArg& list, int* err,
                          hipStream_t s) {
  const int nb = list.count;
  if (nb <= 0) return;
  // a new patch of 8^3 has 64 coarse cells, one wave's worth
  switch (m.dim) {
    case 1: k_prolong_new<1, 64><<<nb, 64, 0, s>>>(m, U, U, list, err); break;
    case 2: k_prolong_new<2, 64><<<nb, 64, 0, s>>>(m, U, U, list, err); break;
    default: k_prolong_new<3, 64><<<nb, 64, 0, s>>>(m, U, U, list, err); break;
  }
}

void Kernels::count_nonzero(const uint8_t* a, int n, int* out, hipStream_t s) {
  if (n <= 0) return;
  const int blocks = std::min(1024, (n + 255) / 256);
  hipLaunchKernelGGL(k_count_nonzero, dim3(blocks), dim3(256), 0, s, a, n, out);
}

void Kernels::scatter_int(int* dst, const int* pairs, int npairs, hipStream_t s) {
  if (npairs <= 0) return;
  hipLaunchKernelGGL(k_scatter_int, dim3((npairs + 255) / 256), dim3(256), 0, s, dst, pairs,
                     npairs);
}

void Kernels::check(const DevMesh& m, const double* U, const ListArg& list, int* bad,
                    hipStream_t s) {
  if (list.count <= 0) return;
  AMR_DISPATCH_DIM(m.dim, k_check, dim3(list.count), dim3(256), s, m, U, list, bad);
}

}  // namespace amr

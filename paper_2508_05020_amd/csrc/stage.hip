// The fused stage kernel of libamr for gfx950 (CDNA4, wave64): per (patch,
// tile) work item, primitives of the tile and its halos in LDS, WENO5-JS
// interpolation and the Rusanov flux at every edge (Eq. (10)-(12)), the
// face fluxes and divergence of Eq. (9) in flux form, and the SSP-RK3 stage
// combination; also the tile variants the autotuner chooses from.
//
// Floating-point contract: implicit contraction is off and every fused
// multiply-add is written with fma(), so a cell's operation sequence is fixed
// by this source and identical for every tile variant, fused or explicit
// halo, per-patch or batched launch.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "amr_internal.hpp"

// no implicit contraction anywhere in this file
#pragma clang fp contract(off)

#include "device_common.hpp"

namespace amr {
namespace {

// ---------------------------------------------------------------------------
// fused right-hand side + SSP-RK3 stage on (pid, tile) work items
// ---------------------------------------------------------------------------

// threadIdx.x hidden from the optimiser: the index arithmetic of a phase is
// then formed in that phase instead of being shared with another direction's
// phase and held in registers across the edge phases, where they run out
__device__ __forceinline__ int phase_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// 1/x from the hardware reciprocal estimate r (relative error e near 2^-24)
// and one third-order step, r (1 + e + e^2): the remaining error e^3 is below
// the rounding (relative error near one ulp).  One operation less than two
// Newton steps.  Used where correct rounding is not required.
__device__ __forceinline__ double rcp_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// sqrt(x) for x > 0 from the hardware reciprocal square-root estimate
// (relative error near 2^-24): one coupled Goldschmidt step for sqrt(x) and
// 1/(2 sqrt(x)), then one Newton correction of the root (a few ulp).  Used
// for the sound speed in the Rusanov dissipation only.
__device__ __forceinline__ double sqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y;
  double h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  const double d = fma(-g, g, x);
  return fma(d, h, g);
}

// sqrt(x) and 1/sqrt(x) for x > 0 from the hardware reciprocal square-root
// estimate: two coupled Goldschmidt steps for sqrt(x) and 1/(2 sqrt(x)),
// then one Newton correction of the root (both within a few ulp).
__device__ __forceinline__ void sqrt_rsqrt_nr(double x, double& s, double& is) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y;
  double h = 0.5 * y;
  double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  s = fma(fma(-g, g, x), h, g);
  is = 2.0 * h;
}

// Numerator and denominator of the nonlinear WENO5-JS combination of three
// candidates q_k from e_k = eps + b_k (b_k the smoothness indicators): the
// value is sum(alpha_k q_k) / sum(alpha_k) with alpha_k = d_k / t_k, t_k =
// e_k^2 and d = (1, 10, 5)/16, evaluated as cross products (alpha_k times
// t0 t1 t2 / 16): num = t2 (t1 q0 + 10 t0 q1) + 5 t0 t1 q2, den = t2 (t1 +
// 10 t0) + 5 t0 t1.
__device__ __forceinline__ void weno_num_den(double e0, double e1, double e2, double q0, double q1,
                                             double q2, double& num, double& den) {
  const double t0 = e0 * e0, t1 = e1 * e1, t2 = e2 * e2;
  const double c0 = 10.0 * t0;
  const double p5 = 5.0 * (t0 * t1);
  den = fma(t2, c0 + t1, p5);
  num = fma(t2, fma(c0, q1, t1 * q0), p5 * q2);
}

// WENO5-JS point values on both sides of the edge between v2 and v3 from the
// six nodes v0..v5: the left-biased value from v0..v4 and the right-biased
// value from the mirrored stencil v5..v1.  Candidates: the quadratic through
// three consecutive nodes evaluated at the edge (x8), two of which the sides
// share.  Indicators (x4): 13/12 k^2 + 1/4 s^2 of the Jiang-Shu definition
// for the window (a, b, c), with k = a - 2b + c and s the first-derivative
// form at the node the edge adjoins: a - 4b + 3c (window left of the edge),
// a - c (centred), 3a - 4b + c (window right of it).  With the first
// differences d_i = v_(i+1) - v_i, k_w = d_(w+1) - d_w and the three forms
// are k + 2 d_(w+1), -(d_w + d_(w+1)) and k - 2 d_w, so the four windows
// share their differences.  The curvature term of a window (with eps) is
// shared by the two sides where both use the window.  One reciprocal serves
// both sides: 1/(den_L den_R) (the indicators are bounded below by eps, and
// eps is at least 1e-20, so the product stays a normal number) times the
// other side's denominator, and with it the final 1/8.  The scalings are
// powers of two.
__device__ __forceinline__ void weno5_pair(double v0, double v1, double v2, double v3, double v4,
                                           double v5, double eps4, double& L, double& R) {
  const double qa = fma(15.0, v2, fma(-10.0, v1, 3.0 * v0));  // left, nodes v0..v2
  const double qb = fma(3.0, v3, fma(6.0, v2, -v1));          // nodes v1..v3 (both sides)
  const double qc = fma(6.0, v3, fma(3.0, v2, -v4));          // nodes v2..v4 (both sides)
  const double qd = fma(15.0, v3, fma(-10.0, v4, 3.0 * v5));  // right, nodes v3..v5
  const double d0 = v1 - v0, d1 = v2 - v1, d2 = v3 - v2, d3 = v4 - v3, d4 = v5 - v4;
  const double k0 = d1 - d0, k1 = d2 - d1, k2 = d3 - d2, k3 = d4 - d3;
  constexpr double c4 = 4.0 * (13.0 / 12.0);
  // eps + curvature term of windows v0..v2, v1..v3, v2..v4, v3..v5
  const double h0 = fma(c4 * k0, k0, eps4);
  const double h1 = fma(c4 * k1, k1, eps4);
  const double h2 = fma(c4 * k2, k2, eps4);
  const double h3 = fma(c4 * k3, k3, eps4);
  const double sl0 = fma(2.0, d1, k0);   // window v0..v2, node v2
  const double sl1 = d1 + d2;            // window v1..v3, centred
  const double sl2 = fma(-2.0, d2, k2);  // window v2..v4, node v2
  const double sr0 = fma(-2.0, d3, k3);  // window v3..v5, node v3
  const double sr1 = d2 + d3;            // window v2..v4, centred
  const double sr2 = fma(2.0, d2, k1);   // window v1..v3, node v3
  double nl, dl, nr, dr;
  weno_num_den(fma(sl0, sl0, h0), fma(sl1, sl1, h1), fma(sl2, sl2, h2), qa, qb, qc, nl, dl);
  weno_num_den(fma(sr0, sr0, h3), fma(sr1, sr1, h2), fma(sr2, sr2, h1), qd, qc, qb, nr, dr);
  const double inv = rcp_nr(dl * dr) * 0.125;
  L = nl * (dr * inv);
  R = nr * (dl * inv);
}

// WENO5-JS point values of a node's two edges from the five nodes a..e around
// it (c the node): L, the left-biased value at the edge towards d, and R, the
// right-biased value at the edge towards b.  Both use the same three windows
// (a,b,c), (b,c,d), (c,d,e) with the same smoothness indicators; only the
// linear weights are mirrored.  A window's parabola about the node is c +
// (s/2) x + (k/2) x^2 with k its second difference and s its slope form at the
// node (a - 4b + 3c, d - b, -3c + 4d - e), so its candidates times 8 are 8 c
// + k + 2 s (at x = 1/2) and 8 c + k - 2 s (at x = -1/2), and the indicators
// times 4 are (13/3) k^2 + s^2.  The weights are cross products (1/t_w times
// t0 t1 t2, t = (eps + indicator)^2), shared by the two values; one reciprocal
// of den_L den_R serves both (eps is at least 1e-20, so the product stays a
// normal number).  The values are formed as c plus a weighted correction: a
// constant stencil gives c exactly.  58 operations and the estimate per node,
// against 76 per edge for weno5_pair, which forms every indicator twice (once
// per edge of its node).
__device__ __forceinline__ void weno5_node(double a, double b, double c, double d, double e,
                                           double eps4, double& L, double& R) {
  const double d0 = b - a, d1 = c - b, d2 = d - c, d3 = e - d;
  const double k0 = d1 - d0, k1 = d2 - d1, k2 = d3 - d2;
  const double s0 = fma(2.0, d1, k0), s1 = d1 + d2, s2 = fma(2.0, d2, -k2);
  constexpr double c4 = 4.0 * (13.0 / 12.0);
  const double e0 = fma(s0, s0, fma(c4 * k0, k0, eps4));
  const double e1 = fma(s1, s1, fma(c4 * k1, k1, eps4));
  const double e2 = fma(s2, s2, fma(c4 * k2, k2, eps4));
  const double t0 = e0 * e0, t1 = e1 * e1, t2 = e2 * e2;
  // weights times 16 t0 t1 t2: (t1 t2, 10 t0 t2, 5 t0 t1) for L and the
  // mirrored (5 t1 t2, 10 t0 t2, t0 t1) for R
  const double w12 = t1 * t2, w02 = 10.0 * (t0 * t2), w01 = t0 * t1;
  const double v01 = 5.0 * w01, v12 = 5.0 * w12;
  const double dl = (w12 + w02) + v01;
  const double dr = (w01 + w02) + v12;
  const double nl = fma(w12, fma(2.0, s0, k0), fma(w02, fma(2.0, s1, k1), v01 * fma(2.0, s2, k2)));
  const double nr =
      fma(w01, fma(-2.0, s2, k2), fma(w02, fma(-2.0, s1, k1), v12 * fma(-2.0, s0, k0)));
  const double inv = rcp_nr(dl * dr) * 0.125;
  L = fma(nl, dr * inv, c);
  R = fma(nr, dl * inv, c);
}

__device__ __forceinline__ double central4(double b, double c, double d, double e) {
  return fma(9.0, c + d, -(b + e)) * 0.0625;
}

template <int D>
struct EdgeState {
  double p, T, u[D];
};

// Density, total energy and direction-J signal speed |u_J| + c of an edge
// state (Eq. (5)-(7), T = p / rho).
template <int D, int J>
__device__ __forceinline__ void edge_thermo(const DevMesh& m, const EdgeState<D>& w, double& rho,
                                            double& E, double& speed) {
  rho = w.p * rcp_nr(w.T);
  double uu = w.u[0] * w.u[0];
#pragma unroll
  for (int i = 1; i < D; ++i) uu = fma(w.u[i], w.u[i], uu);
  E = fma(0.5 * rho, uu, w.p * m.igm1);
  speed = sqrt_nr(m.gamma * w.T) + fabs(w.u[J]);
}

// Variable v of the conserved state and of the direction-J flux of an edge
// state (Eq. (1)-(3)).
template <int D, int J>
__device__ __forceinline__ void edge_uf(const EdgeState<D>& w, double rho, double E, int v,
                                        double& U, double& F) {
  if (v == 0) {
    U = rho;
    F = rho * w.u[J];
  } else if (v == D + 1) {
    U = E;
    F = (E + w.p) * w.u[J];
  } else {
    const int i = v - 1;
    double ui = w.u[0];
#pragma unroll
    for (int k = 1; k < D; ++k)
      if (k == i) ui = w.u[k];
    const double mi = rho * ui;
    U = mi;
    F = (i == J) ? fma(mi, w.u[J], w.p) : mi * w.u[J];
  }
}

template <int D, int TX, int TY, int TZ>
struct TileShape {
  static constexpr int T0 = TX;
  static constexpr int T1 = D >= 2 ? TY : 1;
  static constexpr int T2 = D >= 3 ? TZ : 1;
  static constexpr int NCELL = T0 * T1 * T2;
  // Row pitch (doubles) of the node arrays in LDS: the union box of 1D/2D
  // tiles and the x-extended box of 3D tiles have rows of T0 + 8 nodes, a
  // multiple of 8 for the tile widths used; an odd pitch starts successive
  // rows in different banks, so the lanes of a wave that read or write
  // neighbouring rows do not collide.  The y- and z-extended 3D boxes are
  // read in runs of whole rows and keep their width.
  static constexpr int UPITCH = D == 1 ? T0 + 8 : ((T0 + 8) | 1);
  static constexpr int NUNION = UPITCH * (D >= 2 ? T1 + 8 : 1);
  // smallest pitch >= p with the residue r modulo 16 (the doubles of one LDS
  // pass): planes of r-wide rows then start in successive banks
  static constexpr int pad16(int p, int r) { return p % 16 == r % 16 ? p : pad16(p + 1, r); }
  // 3D tile extended by 4 nodes on both sides along j: row and plane pitch.
  // The lanes of a wave take the cross-section of j (see edges_dir): across x
  // they read one node of successive rows, across y one row of successive
  // planes, so those pitches are odd and padded; across z they read whole
  // planes.
  static constexpr int xpitch(int j) { return j == 0 ? ((T0 + 8) | 1) : T0; }
  static constexpr int xplane(int j) {
    return j == 1 ? pad16(T0 * (T1 + 8), T0) : xpitch(j) * T1;
  }
  static constexpr int ext(int j) { return xplane(j) * (T2 + (j == 2 ? 8 : 0)); }
  // layout index of tile node (t0, t1, t2) in the box extended along j
  template <int J>
  static __device__ __forceinline__ int node(int t0, int t1, int t2) {
    return (t0 + (J == 0 ? 4 : 0)) + xpitch(J) * (t1 + (J == 1 ? 4 : 0)) +
           xplane(J) * (t2 + (J == 2 ? 4 : 0));
  }
  // Flux array of direction j: slot a (0 .. T_j + 3) of a line belongs to node
  // a - 2 and holds its right-biased values, then the flux of the edge on its
  // low side (a >= 1); pitches as for the nodes.
  static constexpr int fpitch(int j) { return j == 0 ? ((T0 + 4) | 1) : T0; }
  static constexpr int fplane(int j) {
    return j == 1 ? pad16(T0 * (T1 + 4), T0) : fpitch(j) * T1;
  }
  static constexpr int slots(int j) {
    return D < 3 ? fpitch(j) * (T1 + (j == 1 ? 4 : 0)) : fplane(j) * (T2 + (j == 2 ? 4 : 0));
  }
  static constexpr int fstep(int j) { return j == 0 ? 1 : (j == 1 ? fpitch(1) : fplane(2)); }
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int EXTMAX = cmax(ext(0), cmax(D >= 2 ? ext(1) : 0, D >= 3 ? ext(2) : 0));
  static constexpr int FXMAX =
      cmax(slots(0), cmax(D >= 2 ? slots(1) : 0, D >= 3 ? slots(2) : 0));
};

// Primitives (p, T, u_j) of one node from its conserved values.
template <int D>
__device__ __forceinline__ void node_primitives(const DevMesh& m, const double* u, double* q) {
  const double r = rcp_nr(u[0]);
  double ke = 0.0;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const double ui = u[1 + i] * r;
    ke = (i == 0) ? u[1] * ui : fma(u[1 + i], ui, ke);
    q[2 + i] = ui;
  }
  const double p = m.gm1 * fma(-0.5, ke, u[D + 1]);
  q[0] = p;
  q[1] = p * r;
}

// What the edge phase reads of a node: its primitives (p, T, u_j), or for
// the characteristic scheme its conserved values, at sP[k NEXT + idx].
template <int D, bool CHAR>
__device__ __forceinline__ void node_store(const DevMesh& m, const double* u, double* sP, int next,
                                           int idx) {
  if constexpr (CHAR) {
#pragma unroll
    for (int v = 0; v < D + 2; ++v) sP[v * next + idx] = u[v];
  } else {
    double q[D + 2];
    node_primitives<D>(m, u, q);
#pragma unroll
    for (int k = 0; k < D + 2; ++k) sP[k * next + idx] = q[k];
  }
}


// Where the values of a node outside the patch along one direction are read by
// the ghost-fill rule, from the patch nb across that face (a pid or kNbNone,
// kNbWall) and the node's coordinate c along the direction: in nb, at the
// nearest cell of this patch beyond a transmissive boundary, or (no patch there:
// prolonged) at the node's own place in this patch's ghost layer.  Returns the
// patch's data and the coordinate in it.
__device__ __forceinline__ const double* across(const DevMesh& m, const double* Uin,
                                                const double* Pin, int l, int n, int nb, int& c) {
  const int cw = c < 0 ? 0 : n - 1;      // nearest cell
  const int cn = c < 0 ? c + n : c - n;  // the same position seen from nb
  c = nb >= 0 ? cn : (nb == kNbWall ? cw : c);
  return nb >= 0 ? Uin + patch_base(m, nb, l) : Pin;
}

// 1D/2D: where the values of the node at patch-local cell c are read (it may lie
// in the halo, at most 4 cells outside the patch along one direction);
// `prolonged`: the value comes from the level below.
template <int D, bool FUSE>
__device__ __forceinline__ void node_source(const DevMesh& m, const double* Uin, const double* Pin,
                                            int n, int full, const int cell[3],
                                            const StageItem& it, const double*& src, int& off,
                                            bool& prolonged) {
  int c[3] = {cell[0], cell[1], cell[2]};
  src = Pin;
  prolonged = false;
  if constexpr (FUSE) {
    const bool x = (unsigned)c[0] >= (unsigned)n, y = D >= 2 && (unsigned)c[1] >= (unsigned)n;
    if (x || y) {
      int cj = x ? c[0] : c[1];
      const int nb = cj < 0 ? (x ? it.nb[0] : it.nb[2]) : (x ? it.nb[1] : it.nb[3]);
      src = across(m, Uin, Pin, it.level, n, nb, cj);
      prolonged = nb == kNbNone;
      if (x) c[0] = cj;
      else c[1] = cj;
    }
  }
  off = box_off<D>(full, c[0] + NG, c[1] + NG, c[2] + NG);
}

// Conserved values of a node of a 3D tile's halo along J (or of the tile
// itself), by the ghost-fill rule: only its J component can lie outside the
// patch.
template <int D, int J, bool FUSE>
__device__ __forceinline__ void node_conserved_dir(const DevMesh& m,
                                                   const double* __restrict__ Uin,
                                                   const double* __restrict__ Pin, int n,
                                                   int full, const int c[3], const StageItem& it,
                                                   double* u) {
  constexpr int NV = D + 2;
  const int vs = var_stride<D>(full);
  const double* src = Pin;
  int cj = c[J];
  if (FUSE && (unsigned)cj >= (unsigned)n)
    src = across(m, Uin, Pin, it.level, n, cj < 0 ? it.nb[2 * J] : it.nb[2 * J + 1], cj);
  const int off = box_off<D>(full, (J == 0 ? cj : c[0]) + NG, (J == 1 ? cj : c[1]) + NG,
                             (J == 2 ? cj : c[2]) + NG);
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = src[v * vs + off];
}

// 1D/2D: primitives of the tile plus 4-node halos in every direction (corner
// nodes are used by no stencil), loaded once per launch.  The nodes are the
// tile's rows with their x halos, then the y halo rows; a thread issues the
// loads of all its nodes before it converts any.  Nodes without a same-level
// source (fused halo): in 1D they are prolonged here, each by the one thread
// that loads it, and also written to the patch's ghost layer (Pg in the source
// buffer; no kernel reads that layer in this mode), which saves the fill
// launch before the stage: 20 tiles, 3.6 + 6.3 us per stage in two launches,
// 7.4 in one.  In 2D they come from the ghost layer that the fill launch has
// written: prolonged here they cost the kernel 80 VGPRs and a spill, 27.8 us
// against 5.1 + 21.6 (0.28 M cells) and 204 against 11 + 164 (2.75 M).
template <int D, int TX, int TY, int NT, bool FUSE, bool CHAR>
__device__ __forceinline__ void load_union(const DevMesh& m, const double* __restrict__ Uin,
                                           const double* __restrict__ Pin, double* Pg, int* err,
                                           int n, int full, const StageItem& it, double* sP) {
  using S = TileShape<D, TX, TY, 1>;
  constexpr int NV = D + 2;
  constexpr int T0 = TX, T1 = D >= 2 ? TY : 1;
  constexpr int U0 = T0 + 8;
  constexpr int NROWS = U0 * T1;                        // nodes of the tile's rows
  constexpr int NU = NROWS + (D >= 2 ? 8 * T0 : 0);
  constexpr int ITER = (NU + NT - 1) / NT;
  constexpr bool PROLONG = FUSE && D == 1;
  const int* o = it.o;
  const int vs = var_stride<D>(full);
  double u[ITER][NV];
  int e0[ITER], e1[ITER];
  bool pro[ITER];
#pragma unroll
  for (int k = 0; k < ITER; ++k) {
    const int idx = threadIdx.x + k * NT;
    pro[k] = false;
    e0[k] = -1;
    if (idx >= NU) continue;
    if (D == 1 || idx < NROWS) {
      e0[k] = idx % U0;
      e1[k] = D >= 2 ? 4 + idx / U0 : 0;
    } else {
      const int r = (idx - NROWS) / T0;
      e0[k] = 4 + (idx - NROWS) % T0;
      e1[k] = r < 4 ? r : T1 + r;
    }
    const int c[3] = {o[0] + e0[k] - 4, D >= 2 ? o[1] + e1[k] - 4 : 0, 0};
    const double* src;
    int off;
    node_source<D, FUSE>(m, Uin, Pin, n, full, c, it, src, off, pro[k]);
#pragma unroll
    for (int v = 0; v < NV; ++v) u[k][v] = src[v * vs + off];
  }
#pragma unroll
  for (int k = 0; k < ITER; ++k) {
    if (e0[k] < 0) continue;
    if (PROLONG && pro[k]) {
      const int l = it.level, x = o[0] + e0[k] - 4;
      const int g[3] = {bc_near(it.px * n + x, m.lv[l].cells, m.periodic[0]), 0, 0};
      if (!(l > 0 && prolong_cell<D>(m, Uin, l, g, u[k]))) {
        err[0] = 1;
#pragma unroll
        for (int v = 0; v < NV; ++v) u[k][v] = __builtin_nan("");
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Pg[v * vs + x + NG] = u[k][v];
    }
    node_store<D, CHAR>(m, u[k], sP, S::NUNION, e0[k] + S::UPITCH * e1[k]);
  }
}

// Rusanov flux (Eq. (11)-(12)) of direction J from the two edge states,
// stored doubled at sF[v NED + e], one variable at a time.
template <int D, int J, int NED>
__device__ __forceinline__ void edge_rusanov(const DevMesh& m, const EdgeState<D>& wl,
                                             const EdgeState<D>& wr, double* sF, int e) {
  constexpr int NV = D + 2;
  double rl, El, sl, rr, Er, sr;
  edge_thermo<D, J>(m, wl, rl, El, sl);
  edge_thermo<D, J>(m, wr, rr, Er, sr);
  const double S = fmax(sr, sl);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double UL, FL, UR, FR;
    edge_uf<D, J>(wl, rl, El, v, UL, FL);
    edge_uf<D, J>(wr, rr, Er, v, UR, FR);
    sF[v * NED + e] = fma(-S, UR - UL, FR + FL);
  }
}

// Primitives of one node in LDS (NEXT nodes per primitive).
template <int D, int NEXT>
__device__ __forceinline__ void node_state(const double* sP, int idx, EdgeState<D>& w) {
  w.p = sP[idx];
  w.T = sP[NEXT + idx];
#pragma unroll
  for (int i = 0; i < D; ++i) w.u[i] = sP[(2 + i) * NEXT + idx];
}

// Both WENO5-JS values of every primitive at one node (layout index idx, STEP
// between neighbours along the direction): the left-biased ones stay in
// registers for the edge above the node, the right-biased ones go to the
// node's slot e of sF for the thread of the node below.
template <int D, int NEXT, int STEP, int NED>
__device__ __forceinline__ void node_values(const DevMesh& m, const double* sP, int idx,
                                            double* left, double* sF, int e) {
  const double eps4 = 4.0 * m.eps;
#pragma unroll
  for (int q = 0; q < D + 2; ++q) {
    const double* col = sP + q * NEXT + idx;
    double r;
    weno5_node(col[-2 * STEP], col[-STEP], col[0], col[STEP], col[2 * STEP], eps4, left[q], r);
    sF[q * NED + e] = r;
  }
}

// Flux of the edge between the node idx (whose left-biased values are `left`)
// and the next one, from the next node's right-biased values in its slot e of
// sF, which the flux then replaces (no other thread reads the slot).  Where p
// or T is not positive on a side the edge takes the states of its two nodes.
template <int D, int J, int NEXT, int STEP, int NED>
__device__ __forceinline__ void node_edge(const DevMesh& m, const double* sP, int idx,
                                          const double* left, double* sF, int e) {
  EdgeState<D> wl, wr;
  wl.p = left[0];
  wl.T = left[1];
#pragma unroll
  for (int i = 0; i < D; ++i) wl.u[i] = left[2 + i];
  node_state<D, NED>(sF, e, wr);
  if (!((wl.p > 0.0) && (wl.T > 0.0) && (wr.p > 0.0) && (wr.T > 0.0))) {
    node_state<D, NEXT>(sP, idx, wl);
    node_state<D, NEXT>(sP, idx + STEP, wr);
  }
  edge_rusanov<D, J, NED>(m, wl, wr, sF, e);
}

// Riemann flux of direction J at one edge with the central interpolation of
// Eq. (8); the edge's nodes are idx and idx + STEP.
template <int D, int J, int NEXT, int STEP, int NED>
__device__ __forceinline__ void edge_central(const DevMesh& m, const double* sP, int idx,
                                             double* sF, int e) {
  double w[D + 2];
#pragma unroll
  for (int q = 0; q < D + 2; ++q) {
    const double* col = sP + q * NEXT + idx;
    w[q] = central4(col[-STEP], col[0], col[STEP], col[2 * STEP]);
  }
  EdgeState<D> wl, wr;
  if ((w[0] > 0.0) && (w[1] > 0.0)) {
    wl.p = w[0];
    wl.T = w[1];
#pragma unroll
    for (int i = 0; i < D; ++i) wl.u[i] = w[2 + i];
    wr = wl;
  } else {
    node_state<D, NEXT>(sP, idx, wl);
    node_state<D, NEXT>(sP, idx + STEP, wr);
  }
  edge_rusanov<D, J, NED>(m, wl, wr, sF, e);
}

// Physical flux of direction J (Eq. (1)-(3)) of one conserved edge state
// and its signal speed |u_J| + c (Eq. (7)), variable v of the flux in F[v].
template <int D, int J>
__device__ __forceinline__ void conserved_flux(const DevMesh& m, const double* U, double* F,
                                               double& speed) {
  const double ir = rcp_nr(U[0]);
  double u[D];
  double q2 = 0.0;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    u[i] = U[1 + i] * ir;
    q2 = (i == 0) ? u[0] * u[0] : fma(u[i], u[i], q2);
  }
  const double p = m.gm1 * fma(-0.5 * U[0], q2, U[D + 1]);
  F[0] = U[1 + J];
#pragma unroll
  for (int i = 0; i < D; ++i) F[1 + i] = (i == J) ? fma(U[1 + i], u[J], p) : U[1 + i] * u[J];
  F[D + 1] = (U[D + 1] + p) * u[J];
  speed = sqrt_nr(m.gamma * p * ir) + fabs(u[J]);
}

// Riemann flux of direction J at one edge from characteristic variables (the
// shock-capturing variant of Section 2.2): the conserved states of the
// window nodes i-2 .. i+3 (in LDS, NEXT nodes per variable, STEP between
// neighbours along J) are projected on the left eigenvectors of the flux
// Jacobian A_J at the mean of nodes i and i+1, each characteristic field is
// interpolated by WENO5-JS (left value from i-2..i+2, right value from the
// mirrored stencil), and the edge states are projected back with the right
// eigenvectors.  Fields in the order u_J - c, entropy, shear (tangential
// directions ascending), u_J + c.  An edge where an interpolated rho or p is
// not positive on either side takes the states of nodes i and i+1.  The
// Rusanov flux (Eq. (11)-(12)) is stored doubled at sF[v NED + e].
template <int D, int J, int NEXT, int STEP, int NED>
__device__ __forceinline__ void edge_char(const DevMesh& m, const double* sP, int base, double* sF,
                                          int e) {
  constexpr int NV = D + 2;
  const double eps4 = 4.0 * m.eps;
  const double* col = sP + base;  // variable v of window node k at col[v NEXT + k STEP]
  // eigensystem at the mean state: u, c, 1/c, H = (E + p) / rho,
  // b1 = (gamma - 1) / c^2, b2 = b1 u.u / 2
  double ub[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v)
    ub[v] = 0.5 * (col[v * NEXT + 2 * STEP] + col[v * NEXT + 3 * STEP]);
  const double ir = rcp_nr(ub[0]);
  double u[D];
  double q2 = 0.0;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    u[i] = ub[1 + i] * ir;
    q2 = (i == 0) ? u[0] * u[0] : fma(u[i], u[i], q2);
  }
  const double pb = m.gm1 * fma(-0.5 * ub[0], q2, ub[D + 1]);
  double c, ic;
  sqrt_rsqrt_nr(m.gamma * pb * ir, c, ic);
  const double H = (ub[D + 1] + pb) * ir;
  const double b1 = m.gm1 * (ic * ic);
  const double b2 = 0.5 * b1 * q2;
  // per node, s = b1 (E - u.m) + b2 rho and a = (u_J rho - m_J) / c: the
  // acoustic fields are (s + a) / 2 (u_J - c) and (s - a) / 2 (u_J + c), the
  // entropy field rho - s; the shear field of a tangential t is m_t - u_t rho
  double sv[6], av[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double* nk = col + k * STEP;
    double um = u[0] * nk[NEXT];
#pragma unroll
    for (int i = 1; i < D; ++i) um = fma(u[i], nk[(1 + i) * NEXT], um);
    sv[k] = fma(b1, nk[(D + 1) * NEXT] - um, b2 * nk[0]);
    av[k] = fma(u[J], nk[0], -nk[(1 + J) * NEXT]) * ic;
  }
  double wl[NV], wr[NV];
  weno5_pair(0.5 * (sv[0] + av[0]), 0.5 * (sv[1] + av[1]), 0.5 * (sv[2] + av[2]),
             0.5 * (sv[3] + av[3]), 0.5 * (sv[4] + av[4]), 0.5 * (sv[5] + av[5]), eps4, wl[0],
             wr[0]);
  weno5_pair(0.5 * (sv[0] - av[0]), 0.5 * (sv[1] - av[1]), 0.5 * (sv[2] - av[2]),
             0.5 * (sv[3] - av[3]), 0.5 * (sv[4] - av[4]), 0.5 * (sv[5] - av[5]), eps4,
             wl[NV - 1], wr[NV - 1]);
  weno5_pair(col[0] - sv[0], col[STEP] - sv[1], col[2 * STEP] - sv[2], col[3 * STEP] - sv[3],
             col[4 * STEP] - sv[4], col[5 * STEP] - sv[5], eps4, wl[1], wr[1]);
  int f = 2;
#pragma unroll
  for (int t = 0; t < D; ++t) {
    if (t == J) continue;
    const double* mt = col + (1 + t) * NEXT;
    weno5_pair(fma(-u[t], col[0], mt[0]), fma(-u[t], col[STEP], mt[STEP]),
               fma(-u[t], col[2 * STEP], mt[2 * STEP]), fma(-u[t], col[3 * STEP], mt[3 * STEP]),
               fma(-u[t], col[4 * STEP], mt[4 * STEP]), fma(-u[t], col[5 * STEP], mt[5 * STEP]),
               eps4, wl[f], wr[f]);
    ++f;
  }
  // back to conserved states: rho = W- + We + W+, m_J = u_J rho + c (W+ - W-),
  // m_t = u_t rho + W_t, E = H (W- + W+) + u_J c (W+ - W-) + q2/2 We + sum_t u_t W_t
  double UX[2][NV];
  bool ok = true;
#pragma unroll
  for (int X = 0; X < 2; ++X) {
    const double* w = X == 0 ? wl : wr;
    double* U = UX[X];
    const double A = w[0] + w[NV - 1];
    const double B = w[NV - 1] - w[0];
    const double rho = A + w[1];
    double Et = 0.5 * q2 * w[1];
    int g = 2;
#pragma unroll
    for (int t = 0; t < D; ++t) {
      if (t == J) {
        U[1 + t] = fma(u[J], rho, c * B);
      } else {
        U[1 + t] = fma(u[t], rho, w[g]);
        Et = fma(u[t], w[g], Et);
        ++g;
      }
    }
    U[0] = rho;
    U[D + 1] = fma(H, A, fma(u[J] * c, B, Et));
    const double irx = rcp_nr(rho);
    double ke = U[1] * (U[1] * irx);
#pragma unroll
    for (int i = 1; i < D; ++i) ke = fma(U[1 + i], U[1 + i] * irx, ke);
    const double px = m.gm1 * fma(-0.5, ke, U[D + 1]);
    ok = ok && (rho > 0.0) && (px > 0.0);
  }
  if (!ok) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      UX[0][v] = col[v * NEXT + 2 * STEP];
      UX[1][v] = col[v * NEXT + 3 * STEP];
    }
  }
  double FL[NV], FR[NV], sl, sr;
  conserved_flux<D, J>(m, UX[0], FL, sl);
  conserved_flux<D, J>(m, UX[1], FR, sr);
  const double S = fmax(sr, sl);
#pragma unroll
  for (int v = 0; v < NV; ++v) sF[v * NED + e] = fma(-S, UX[1][v] - UX[0][v], FR[v] + FL[v]);
}

// Divergence of the face fluxes G = F - (F_- - 2 F + F_+) / 24 of direction J
// (flux form of Eq. (9)) from the edge fluxes in sF into acc, as the difference
// F_0 - F_-1 and the correction of it (five operations per variable; the two
// face fluxes first took eight: 2D, 2.75 M cells 160.4 against 158.3 us, 0.28 M
// 22.2 against 21.2 us; 3D the same within 0.5 %), and the face fluxes
// themselves on patch boundaries with flux registers, by their few threads.
template <int D, int TX, int TY, int TZ, int NT, int J>
__device__ __forceinline__ void cells_at(const double* sF, double* __restrict__ frp, int n,
                                         const int o[3], double acc[][D + 2], double inv_h,
                                         int wmask) {
  using S = TileShape<D, TX, TY, TZ>;
  constexpr int NV = D + 2;
  constexpr int NED = S::slots(J);
  constexpr int CPT = (S::NCELL + NT - 1) / NT;
  const int tid = threadIdx.x;
  const int nface = (D == 1) ? 1 : (D == 2 ? n : n * n);
  constexpr double c24 = 1.0 / 24.0;
  const double half_inv_h = 0.5 * inv_h;
  // patch-boundary faces whose flux registers refluxing reads
  const bool lo_reg = (wmask >> (2 * J)) & 1, hi_reg = (wmask >> (2 * J + 1)) & 1;
#pragma unroll
  for (int cc = 0; cc < CPT; ++cc) {
    const int cell = tid + cc * NT;
    if (cell >= S::NCELL) break;
    const int t0 = cell % S::T0;
    const int t1 = (cell / S::T0) % S::T1;
    const int t2 = cell / (S::T0 * S::T1);
    const int tj = J == 0 ? t0 : (J == 1 ? t1 : t2);
    // slot of edge (t_J - 2) + 1/2, the first of the cell's four
    constexpr int ESTEP = S::fstep(J);
    const int eb = t0 + S::fpitch(J) * t1 + S::fplane(J) * t2 + ESTEP;
    const int i = o[J] + tj;
    int tang = 0;
    if constexpr (D == 2) tang = (J == 0) ? (o[1] + t1) : (o[0] + t0);
    if constexpr (D == 3) {
      if constexpr (J == 0) tang = (o[1] + t1) + __mul24(n, o[2] + t2);
      else if constexpr (J == 1) tang = (o[0] + t0) + __mul24(n, o[2] + t2);
      else tang = (o[0] + t0) + __mul24(n, o[1] + t1);
    }
    // the flux registers of this face (variable v at v nface + tang of the
    // face's block; 32-bit offsets, 24-bit products), written per variable
    const bool lo = i == 0 && lo_reg, hi = i == n - 1 && hi_reg;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      // edge fluxes are stored doubled (the Rusanov 1/2 is applied here, as
      // 1/2 inv_h, and to the boundary faces; power-of-two scaling is exact)
      const double* F = sF + v * NED + eb;
      const double Fm2 = F[0], Fm1 = F[ESTEP], F0 = F[2 * ESTEP], Fp1 = F[3 * ESTEP];
      const double d = F0 - Fm1;
      const double dG = fma(c24, fma(3.0, d, Fm2 - Fp1), d);
      acc[cc][v] = fma(-dG, half_inv_h, acc[cc][v]);
    }
    if (lo || hi) {
      double* fb = frp + __mul24((J * 2 + (hi ? 1 : 0)) * NV, nface) + tang;
#pragma unroll 1
      for (int v = 0; v < NV; ++v) {
        const double* F = sF + v * NED + eb + (hi ? ESTEP : 0);
        fb[__mul24(v, nface)] = 0.5 * fma(-c24, fma(-2.0, F[ESTEP], F[0]) + F[2 * ESTEP], F[ESTEP]);
      }
    }
  }
}

// Where thread item t of a direction-J phase works: node a - 2 along J
// (a = 0 .. T_J + 3) of line c of the tile's cross-section.  The cross-section
// varies fastest, so that in 3D a wave holds one node position of 64 lines:
// its LDS accesses meet the padded pitches without bank conflicts, and the
// edge phase, which has one item less per line, leaves whole waves idle.
template <int D, int TX, int TY, int TZ, int J, bool UNION>
struct Line {
  using S = TileShape<D, TX, TY, TZ>;
  static constexpr int TJ = J == 0 ? S::T0 : (J == 1 ? S::T1 : S::T2);
  static constexpr int NCROSS = S::NCELL / TJ;
  static constexpr int NNODE = NCROSS * (TJ + 4);     // items of the node phase
  static constexpr int NEXT = UNION ? S::NUNION : S::ext(J);
  static constexpr int STEP =
      J == 0 ? 1 : (UNION ? S::UPITCH : (J == 1 ? S::xpitch(1) : S::xplane(2)));
  static constexpr int NED = S::slots(J);
  int idx, slot;  // layout index of the node and of its slot
  __device__ __forceinline__ explicit Line(int t) {
    const int a = t / NCROSS, c = t % NCROSS;
    if constexpr (J == 0) {
      const int c1 = c % S::T1, c2 = c / S::T1;
      idx = UNION ? (D >= 2 ? (c1 + 4) * S::UPITCH : 0) + a + 2
                  : a + 2 + S::xpitch(0) * c1 + S::xplane(0) * c2;
      slot = a + S::fpitch(0) * c1 + S::fplane(0) * c2;
    } else if constexpr (J == 1) {
      const int c0 = c % S::T0, c2 = c / S::T0;
      idx = UNION ? (a + 2) * S::UPITCH + c0 + 4
                  : c0 + S::xpitch(1) * (a + 2) + S::xplane(1) * c2;
      slot = c0 + S::fpitch(1) * a + S::fplane(1) * c2;
    } else {
      const int c0 = c % S::T0, c1 = c / S::T0;
      idx = c0 + S::xpitch(2) * c1 + S::xplane(2) * (a + 2);
      slot = c0 + S::fpitch(2) * c1 + S::fplane(2) * a;
    }
  }
};

// Riemann flux at every edge i+1/2, i = o_J-2 .. o_J+T_J, of direction J
// from the node values in sP (the union layout in 1D/2D, the tile extended
// along J in 3D), into sF.  WENO5 of the primitives: a node phase (one thread
// per node forms both of its edge values) and, after a block barrier, an edge
// phase (one thread per edge).  The 8x8x8 tile has 768 nodes per direction, a
// thread each, and 704 edges.  With one phase of 704 edges, each forming the
// indicators of both its nodes, a stage launch took 2225 us against 1959 us
// (3D, 20.4 M leaf cells, mostly 8^3 patches; 44.2 against 37.6 wave
// instructions per cell, 37.0 with the later steps), 180 against
// 163 us (2D, 2.75 M cells in 32^2 patches) and 24.2 against 21.4 us (2D, 0.28 M
// cells).
template <int D, int TX, int TY, int TZ, int NT, int J, bool UNION, bool CHAR>
__device__ __forceinline__ void edges_dir(const DevMesh& m, const double* sP, double* sF) {
  using G = Line<D, TX, TY, TZ, J, UNION>;
  constexpr int NEDGE = G::NNODE - G::NCROSS;
  if constexpr (CHAR) {
    for (int t = threadIdx.x; t < NEDGE; t += NT) {
      const G g(t);
      edge_char<D, J, G::NEXT, G::STEP, G::NED>(m, sP, g.idx - 2 * G::STEP, sF,
                                                g.slot + TileShape<D, TX, TY, TZ>::fstep(J));
    }
  } else if (m.scheme == AMR_SCHEME_CENTRAL) {
    for (int t = threadIdx.x; t < NEDGE; t += NT) {
      const G g(t);
      edge_central<D, J, G::NEXT, G::STEP, G::NED>(m, sP, g.idx, sF,
                                                   g.slot + TileShape<D, TX, TY, TZ>::fstep(J));
    }
  } else {
    constexpr int ITER = (G::NNODE + NT - 1) / NT;
    double left[ITER][D + 2];
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
      const int t = threadIdx.x + k * NT;
      if (t < G::NNODE) {
        const G g(t);
        node_values<D, G::NEXT, G::STEP, G::NED>(m, sP, g.idx, left[k], sF, g.slot);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
      const int t = threadIdx.x + k * NT;
      if (t < NEDGE) {
        const G g(t);
        node_edge<D, J, G::NEXT, G::STEP, G::NED>(m, sP, g.idx, left[k], sF,
                                                  g.slot + TileShape<D, TX, TY, TZ>::fstep(J));
      }
    }
  }
}

// 3D, characteristic scheme: the conserved values of the tile extended by 4
// nodes on both sides along J, into sP in the extended-box layout.  The
// tile's own nodes come first in the thread order and the 8 halo layers
// after them, so that a wave holds nodes of one kind (the tile's own nodes
// are read straight from the patch); every thread issues the loads of all
// its nodes before storing any.
template <int D, int TX, int TY, int TZ, int NT, int J, bool FUSE>
__device__ __forceinline__ void load_dir(const DevMesh& m, const double* __restrict__ Uin,
                                         const double* __restrict__ Pin, int n, int full,
                                         const StageItem& it, double* sP) {
  using S = TileShape<D, TX, TY, TZ>;
  constexpr int NV = D + 2;
  constexpr int NEXT = S::ext(J);
  constexpr int NC = S::NCELL;
  constexpr int TJ = J == 0 ? S::T0 : (J == 1 ? S::T1 : S::T2);
  constexpr int HL = NC / TJ;                  // nodes of one layer across J
  constexpr int CA = J == 0 ? S::T1 : S::T0;   // extent of the lower cross direction
  constexpr int NNODE = NC + 8 * HL;           // nodes of the extended box
  constexpr int ITER = (NNODE + NT - 1) / NT;
  double u[ITER][NV];
  int lidx[ITER];
#pragma unroll
  for (int k = 0; k < ITER; ++k) {
    const int idx = threadIdx.x + k * NT;
    lidx[k] = -1;
    if (idx >= NNODE) continue;
    int t[3];
    if (idx < NC) {
      t[0] = idx % S::T0;
      t[1] = (idx / S::T0) % S::T1;
      t[2] = idx / (S::T0 * S::T1);
    } else {
      const int hh = idx - NC;
      const int layer = hh / HL;                // -4..-1, then T_J..T_J+3
      const int r = hh - layer * HL;
      const int a = r % CA, b = r / CA;         // the two other directions, lower first
      t[J] = layer < 4 ? layer - 4 : TJ + layer - 4;
      t[J == 0 ? 1 : 0] = a;
      t[J == 2 ? 1 : 2] = b;
    }
    const int c[3] = {it.o[0] + t[0], it.o[1] + t[1], it.o[2] + t[2]};
    lidx[k] = S::template node<J>(t[0], t[1], t[2]);
    node_conserved_dir<D, J, FUSE>(m, Uin, Pin, n, full, c, it, u[k]);
  }
#pragma unroll
  for (int k = 0; k < ITER; ++k)
    if (lidx[k] >= 0) node_store<D, true>(m, u[k], sP, NEXT, lidx[k]);
}

// 3D primitive schemes: thread t < NCELL loads the conserved values of tile
// node t once, first in the item (they need no neighbour table), and keeps
// them in `keep` for the three directions and as the stage input of cell t
// in the epilogue.
template <int D, int TX, int TY, int TZ>
__device__ __forceinline__ void own_load(const double* __restrict__ Pin, int full, const int o[3],
                                         double* keep) {
  using S = TileShape<D, TX, TY, TZ>;
  const int tid = threadIdx.x;
  if (tid < S::NCELL) {
    const int t0 = tid % S::T0, t1 = (tid / S::T0) % S::T1, t2 = tid / (S::T0 * S::T1);
    const int off = box_off<D>(full, o[0] + t0 + NG, o[1] + t1 + NG, o[2] + t2 + NG);
    const int vs = var_stride<D>(full);
#pragma unroll
    for (int v = 0; v < D + 2; ++v) keep[v] = Pin[v * vs + off];
  }
}

// 3D primitive schemes: the 8 halo layers of the tile extended along J (its
// own nodes are kept in registers).  For y and z their loads are issued
// (halo_issue) before the previous direction's divergence is formed and
// converted and stored (halo_store) after it, so that they are in flight
// meanwhile.  Halo node h (layers -4..-1, then T_J..T_J+3, the two other
// directions lower first) is item h / NT of thread h mod NT.
template <int D, int TX, int TY, int TZ, int NT, int J>
struct DirHalo {
  using S = TileShape<D, TX, TY, TZ>;
  static constexpr int NV = D + 2;
  static constexpr int TJ = J == 0 ? S::T0 : (J == 1 ? S::T1 : S::T2);
  static constexpr int HL = S::NCELL / TJ;                  // nodes of one layer
  static constexpr int NH = 8 * HL;
  static constexpr int ITER = (NH + NT - 1) / NT;
  double u[ITER][NV];
  int lidx[ITER];
};

template <int D, int TX, int TY, int TZ, int NT, int J, bool FUSE>
__device__ __forceinline__ void halo_issue(const DevMesh& m, const double* __restrict__ Uin,
                                           const double* __restrict__ Pin, int n, int full,
                                           const StageItem& it, DirHalo<D, TX, TY, TZ, NT, J>& h) {
  using S = TileShape<D, TX, TY, TZ>;
  using H = DirHalo<D, TX, TY, TZ, NT, J>;
  constexpr int CA = J == 0 ? S::T1 : S::T0;   // extent of the lower cross direction
  const int tid = phase_tid();
#pragma unroll
  for (int k = 0; k < H::ITER; ++k) {
    // threads past the last halo node load node NH - 1 again (no branch
    // around the loads) and store nothing
    const int h0 = tid + k * NT;
    const int hh = h0 < H::NH ? h0 : H::NH - 1;
    const int layer = hh / H::HL;
    const int r = hh - layer * H::HL;
    int t[3];
    t[J] = layer < 4 ? layer - 4 : H::TJ + layer - 4;
    t[J == 0 ? 1 : 0] = r % CA;
    t[J == 2 ? 1 : 2] = r / CA;
    const int c[3] = {it.o[0] + t[0], it.o[1] + t[1], it.o[2] + t[2]};
    h.lidx[k] = h0 < H::NH ? S::template node<J>(t[0], t[1], t[2]) : -1;
    node_conserved_dir<D, J, FUSE>(m, Uin, Pin, n, full, c, it, h.u[k]);
  }
}

template <int D, int TX, int TY, int TZ, int NT, int J>
__device__ __forceinline__ void halo_store(const DevMesh& m, const DirHalo<D, TX, TY, TZ, NT, J>& h,
                                           const double* keep, double* sP) {
  using S = TileShape<D, TX, TY, TZ>;
  using H = DirHalo<D, TX, TY, TZ, NT, J>;
  constexpr int NEXT = S::ext(J);
  const int tid = phase_tid();
  if (tid < S::NCELL) {
    const int t0 = tid % S::T0, t1 = (tid / S::T0) % S::T1, t2 = tid / (S::T0 * S::T1);
    node_store<D, false>(m, keep, sP, NEXT, S::template node<J>(t0, t1, t2));
  }
#pragma unroll
  for (int k = 0; k < H::ITER; ++k)
    if (h.lidx[k] >= 0) node_store<D, false>(m, h.u[k], sP, NEXT, h.lidx[k]);
}

// 1D/2D: edge fluxes and their divergence for direction J from the union
// layout loaded once for all directions.
template <int D, int TX, int TY, int TZ, int NT, int J, bool CHAR>
__device__ __forceinline__ void stage_direction(const DevMesh& m, double* __restrict__ frp, int n,
                                                const int o[3], double* sP, double* sF,
                                                double acc[][D + 2], double inv_h, int wmask) {
  edges_dir<D, TX, TY, TZ, NT, J, true, CHAR>(m, sP, sF);
  __syncthreads();
  cells_at<D, TX, TY, TZ, NT, J>(sF, frp, n, o, acc, inv_h, wmask);
  __syncthreads();
}

// 2D union layout, both directions at once: the x and y nodes (and then
// edges) form one work range, x first, then every cell takes its x and then
// its y divergence, the order of the direction-by-direction path.
template <int D, int TX, int TY, int NT, bool CHAR>
__device__ __forceinline__ void stage_both(const DevMesh& m, double* __restrict__ frp, int n,
                                           const int o[3], const double* sP, double* sFx,
                                           double* sFy, double acc[][D + 2], double inv_h,
                                           int wmask) {
  static_assert(D == 2, "combined sweep is 2D");
  using S = TileShape<D, TX, TY, 1>;
  using GX = Line<D, TX, TY, 1, 0, true>;
  using GY = Line<D, TX, TY, 1, 1, true>;
  constexpr int NX = GX::NNODE, EX = NX - GX::NCROSS, EY = GY::NNODE - GY::NCROSS;
  auto both = [&](int t, int nx, auto fx, auto fy) {
    if (t < nx) fx(GX(t));
    else fy(GY(t - nx));
  };
  if constexpr (CHAR) {
    for (int t = threadIdx.x; t < EX + EY; t += NT)
      both(t, EX,
           [&](const GX& g) {
             edge_char<D, 0, GX::NEXT, GX::STEP, GX::NED>(m, sP, g.idx - 2 * GX::STEP, sFx,
                                                          g.slot + S::fstep(0));
           },
           [&](const GY& g) {
             edge_char<D, 1, GY::NEXT, GY::STEP, GY::NED>(m, sP, g.idx - 2 * GY::STEP, sFy,
                                                          g.slot + S::fstep(1));
           });
  } else if (m.scheme == AMR_SCHEME_CENTRAL) {
    for (int t = threadIdx.x; t < EX + EY; t += NT)
      both(t, EX,
           [&](const GX& g) {
             edge_central<D, 0, GX::NEXT, GX::STEP, GX::NED>(m, sP, g.idx, sFx,
                                                             g.slot + S::fstep(0));
           },
           [&](const GY& g) {
             edge_central<D, 1, GY::NEXT, GY::STEP, GY::NED>(m, sP, g.idx, sFy,
                                                             g.slot + S::fstep(1));
           });
  } else {
    // the nodes of both phases keep their items: node item t has edge item t
    // wherever its line has an edge above it
    constexpr int ITER = (NX + GY::NNODE + NT - 1) / NT;
    double left[ITER][D + 2];
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
      const int t = threadIdx.x + k * NT;
      if (t < NX + GY::NNODE)
        both(t, NX,
             [&](const GX& g) {
               node_values<D, GX::NEXT, GX::STEP, GX::NED>(m, sP, g.idx, left[k], sFx, g.slot);
             },
             [&](const GY& g) {
               node_values<D, GY::NEXT, GY::STEP, GY::NED>(m, sP, g.idx, left[k], sFy, g.slot);
             });
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITER; ++k) {
      const int t = threadIdx.x + k * NT;
      if (t < EX || (t >= NX && t < NX + EY))
        both(t, NX,
             [&](const GX& g) {
               node_edge<D, 0, GX::NEXT, GX::STEP, GX::NED>(m, sP, g.idx, left[k], sFx,
                                                            g.slot + S::fstep(0));
             },
             [&](const GY& g) {
               node_edge<D, 1, GY::NEXT, GY::STEP, GY::NED>(m, sP, g.idx, left[k], sFy,
                                                            g.slot + S::fstep(1));
             });
    }
  }
  __syncthreads();
  cells_at<D, TX, TY, 1, NT, 0>(sFx, frp, n, o, acc, inv_h, wmask);
  cells_at<D, TX, TY, 1, NT, 1>(sFy, frp, n, o, acc, inv_h, wmask);
}

// Restriction of a tile into its parent patch, from the new values of its
// cells (sR: variable v of tile cell i at sR[v NCELL + i]): each parent cell
// is the mean of its 2^D children, summed as the post-stage restriction sums
// them (x pairs first, then y, then z).  SERIAL: one variable at a time
// (unrolled, the reads of all variables are issued at once and can take more
// registers than the primitive schemes' kernels have).
template <int D, int TX, int TY, int TZ, int NT, bool SERIAL>
__device__ __forceinline__ void restrict_tile(const DevMesh& m, double* __restrict__ out,
                                              const StageItem& it, const double* sR) {
  using S = TileShape<D, TX, TY, TZ>;
  constexpr int NV = D + 2;
  constexpr int NC = S::NCELL;
  constexpr int H0 = S::T0 / 2, H1 = D >= 2 ? S::T1 / 2 : 1, H2 = D >= 3 ? S::T2 / 2 : 1;
  constexpr int NP = H0 * H1 * H2;
  static_assert(S::T0 % 2 == 0 && (D < 2 || S::T1 % 2 == 0) && (D < 3 || S::T2 % 2 == 0),
                "tiles cover whole 2^D groups of children");
  const LevelC& C = m.lv[it.level - 1];
  double* Pp = out + it.parent;
  const int vsc = var_stride<D>(C.full);
  for (int k = threadIdx.x; k < NP; k += NT) {
    const int a = k % H0, b = (k / H0) % H1, c = k / (H0 * H1);
    const int dst = box_off<D>(C.full, a, b, c);
    auto at = [&](int v, int x, int y, int z) {
      return sR[v * NC + (2 * a + x) + S::T0 * ((2 * b + y) + S::T1 * (2 * c + z))];
    };
    auto one = [&](int v) {
      auto xsum = [&](int y, int z) { return at(v, 0, y, z) + at(v, 1, y, z); };
      double r;
      if constexpr (D == 1) r = xsum(0, 0) * 0.5;
      else if constexpr (D == 2) r = (xsum(0, 0) + xsum(1, 0)) * 0.25;
      else r = ((xsum(0, 0) + xsum(1, 0)) + (xsum(0, 1) + xsum(1, 1))) * 0.125;
      Pp[v * vsc + dst] = r;
    };
    if constexpr (SERIAL) {
#pragma unroll 1
      for (int v = 0; v < NV; ++v) one(v);
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) one(v);
    }
  }
}

// One (pid, tile) work item: the whole RHS of the tile and its stage
// combination; `best` collects the signal speed bits of the item's cells.
template <int D, int TX, int TY, int TZ, int NT, bool FUSE, bool BOTH, bool CHAR>
__device__ __forceinline__ void stage_item(const DevMesh& m, int mode,
                                           const double* __restrict__ Uin, double* Ug, int* err,
                                           const double* Un, double* out, double* __restrict__ fr,
                                           const StageItem& it, bool first,
                                           const double* __restrict__ dtp,
                                           unsigned long long* __restrict__ lam_next,
                                           const unsigned long long* __restrict__ lam_in,
                                           double* __restrict__ dt_out, double* sP, double* sF,
                                           unsigned long long& best) {
  using S = TileShape<D, TX, TY, TZ>;
  constexpr int NV = D + 2;
  constexpr int CPT = (S::NCELL + NT - 1) / NT;
  constexpr bool UNION = D <= 2;
  const int pid = it.pid, l = it.level;
  const int* o = it.o;
  const LevelC& L = m.lv[l];
  const int n = L.n, full = L.full;
  const long long base = patch_base(m, pid, l);
  const double* Pin = Uin + base;
  double* frp = fr + L.fr_off + (long long)(pid - L.pid_base) * L.fr_stride;
  const int wmask = it.regs;
  double acc[CPT][NV];
#pragma unroll
  for (int cc = 0; cc < CPT; ++cc)
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[cc][v] = 0.0;

  // 3D primitive schemes: the conserved values of this thread's tile node,
  // loaded first and kept for the three directions and the epilogue
  // (own_load), and U^n of its cell
  constexpr bool KEPT = !UNION && !CHAR;
  double keep[NV], un0[NV];
  static_assert(!KEPT || NT >= S::NCELL, "a thread per tile node holds its values");
  if constexpr (KEPT) own_load<D, TX, TY, TZ>(Pin, full, o, keep);
  if constexpr (UNION) {
    load_union<D, TX, TY, NT, FUSE, CHAR>(m, Uin, Pin, Ug + base, err, n, full, it, sP);
    __syncthreads();
    if constexpr (BOTH && D == 2) {
      stage_both<D, TX, TY, NT, CHAR>(m, frp, n, o, sP, sF,
                                      sF + (D + 2) * S::slots(0), acc, L.inv_h, wmask);
    } else {
      stage_direction<D, TX, TY, TZ, NT, 0, CHAR>(m, frp, n, o, sP, sF, acc, L.inv_h, wmask);
      if constexpr (D >= 2)
        stage_direction<D, TX, TY, TZ, NT, 1, CHAR>(m, frp, n, o, sP, sF, acc, L.inv_h, wmask);
    }
  } else {
    // 3D, direction by direction: the next direction's nodes are loaded in
    // the phase that forms the previous direction's divergence (sP is free
    // once the edges are done, sF is read), two block barriers per direction
    if constexpr (KEPT) {
      DirHalo<D, TX, TY, TZ, NT, 0> h;
      halo_issue<D, TX, TY, TZ, NT, 0, FUSE>(m, Uin, Pin, n, full, it, h);
      halo_store<D, TX, TY, TZ, NT, 0>(m, h, keep, sP);
    } else {
      load_dir<D, TX, TY, TZ, NT, 0, FUSE>(m, Uin, Pin, n, full, it, sP);
    }
    __syncthreads();
    edges_dir<D, TX, TY, TZ, NT, 0, false, CHAR>(m, sP, sF);
    __syncthreads();
    if constexpr (KEPT) {
      DirHalo<D, TX, TY, TZ, NT, 1> h;
      halo_issue<D, TX, TY, TZ, NT, 1, FUSE>(m, Uin, Pin, n, full, it, h);
      cells_at<D, TX, TY, TZ, NT, 0>(sF, frp, n, o, acc, L.inv_h, wmask);
      halo_store<D, TX, TY, TZ, NT, 1>(m, h, keep, sP);
    } else {
      load_dir<D, TX, TY, TZ, NT, 1, FUSE>(m, Uin, Pin, n, full, it, sP);
      cells_at<D, TX, TY, TZ, NT, 0>(sF, frp, n, o, acc, L.inv_h, wmask);
    }
    __syncthreads();
    edges_dir<D, TX, TY, TZ, NT, 1, false, CHAR>(m, sP, sF);
    __syncthreads();
    if constexpr (KEPT) {
      DirHalo<D, TX, TY, TZ, NT, 2> h;
      halo_issue<D, TX, TY, TZ, NT, 2, FUSE>(m, Uin, Pin, n, full, it, h);
      cells_at<D, TX, TY, TZ, NT, 1>(sF, frp, n, o, acc, L.inv_h, wmask);
      halo_store<D, TX, TY, TZ, NT, 2>(m, h, keep, sP);
    } else {
      load_dir<D, TX, TY, TZ, NT, 2, FUSE>(m, Uin, Pin, n, full, it, sP);
      cells_at<D, TX, TY, TZ, NT, 1>(sF, frp, n, o, acc, L.inv_h, wmask);
    }
    __syncthreads();
    edges_dir<D, TX, TY, TZ, NT, 2, false, CHAR>(m, sP, sF);
    __syncthreads();
    if constexpr (KEPT) {
      // U^n of the thread's own cell for the combination, loaded while the
      // last divergence is formed (the kept stage input when U^n is it)
      const int tid = threadIdx.x;
      if (mode != kModeRHS && tid < S::NCELL) {
        if (Un == Uin) {
#pragma unroll
          for (int v = 0; v < NV; ++v) un0[v] = keep[v];
        } else {
          const int t0 = tid % S::T0, t1 = (tid / S::T0) % S::T1, t2 = tid / (S::T0 * S::T1);
          const double* p = Un + base + box_off<D>(full, o[0] + t0 + NG, o[1] + t1 + NG,
                                                   o[2] + t2 + NG);
          const int vs = var_stride<D>(full);
#pragma unroll
          for (int v = 0; v < NV; ++v) un0[v] = __builtin_nontemporal_load(p + v * vs);
        }
      }
    }
    cells_at<D, TX, TY, TZ, NT, 2>(sF, frp, n, o, acc, L.inv_h, wmask);
  }

  const int vs = var_stride<D>(full);
  // stage 1 of a step may take dt = CFL / rate from the rate slot itself
  // (every block computes it; the first work item publishes it for the rest
  // of the step and clears the slot stage 3 accumulates into)
  double dt;
  if (mode == kModeRHS) {
    dt = 0.0;
  } else if (lam_in) {
    dt = m.cfl / slot_rate(lam_in);
    if (first && threadIdx.x == 0) {
      dt_out[0] = dt;
      clear_rate(lam_next);
    }
  } else {
    dt = dtp[0];
  }
  constexpr double c23 = 2.0 / 3.0;
  // next step's CFL rate from the final leaf values; cells on coarse/fine
  // faces are left to the flux-correction kernel, which changes them
  const bool want_rate = lam_next != nullptr && mode == kModeStage3;
  const int fmask = it.cf;
  // the tile of a leaf is restricted into its parent here, from the values it
  // writes (staged in sF, free once every thread has read its edge fluxes),
  // instead of being read back by the post-stage launches; refluxing forms the
  // parent cells along the faces it corrects again
  const bool restrict_here = mode != kModeRHS && l >= 1;
  static_assert(S::NCELL <= S::FXMAX, "the staged cell values fit sF");
  double* sR = sF;
  if (restrict_here) __syncthreads();
#pragma unroll
  for (int cc = 0; cc < CPT; ++cc) {
    const int cell = threadIdx.x + cc * NT;
    if (cell >= S::NCELL) break;
    const int t0 = cell % S::T0;
    const int t1 = (cell / S::T0) % S::T1;
    const int t2 = cell / (S::T0 * S::T1);
    const long long off = base + box_off<D>(full, o[0] + t0 + NG, o[1] + t1 + NG, o[2] + t2 + NG);
    double r[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const long long a = off + v * vs;
      const double Lv = acc[cc][v];
      if (mode == kModeRHS) {
        r[v] = Lv;
      } else if (mode == kModeStage1) {
        // U^n and the stage input of the cell: held for the thread's own
        // cell (cc = 0) in 3D, else loaded
        const double un = (KEPT && cc == 0) ? un0[v] : Un[a];
        r[v] = fma(dt, Lv, un);
      } else {
        const double un = (KEPT && cc == 0) ? un0[v] : Un[a];
        const double ui = (KEPT && cc == 0) ? keep[v] : Uin[a];
        r[v] = fma(mode == kModeStage2 ? 0.25 : c23, fma(dt, Lv, ui) - un, un);
      }
      // 3D: a non-temporal store, which keeps the stage input's halo rows
      // in L2 for the neighbouring tiles
      if constexpr (UNION)
        out[a] = r[v];
      else
        __builtin_nontemporal_store(r[v], out + a);
      if (restrict_here) sR[v * S::NCELL + cell] = r[v];
    }
    if (want_rate) {
      const int c3[3] = {o[0] + t0, o[1] + t1, o[2] + t2};
      bool on_cf = false;
      for (int j = 0; j < D; ++j)
        on_cf |= ((fmask >> (2 * j)) & 1) && c3[j] == 0 || ((fmask >> (2 * j + 1)) & 1) && c3[j] == n - 1;
      if (!on_cf) {
        const unsigned long long bits = cell_speed_bits<D>(r, m);
        best = bits > best ? bits : best;
      }
    }
  }
  if (restrict_here) {
    __syncthreads();
    restrict_tile<D, TX, TY, TZ, NT, KEPT>(m, out, it, sR);
  }
}

// The fused stage kernel over (pid, tile) work items, one item per block.
// With `dir` (recorded launches) the live count is read from the device list
// directory {offset, count}, so that a launch recorded once stays valid when a
// regrid rewrites the items (its grid may then hold more blocks than items).
// A block's first loads of cells depend on its item alone (StageItem): two
// dependent loads instead of four, and no block barrier before them.  2D 21.2
// to 20.0 us (0.28 M cells) and 158.3 to 153.1 (2.75 M), 1D 7.6 to 6.8 (20
// items), characteristic 3D 101 to 98; 3D with 12-wave blocks the same: it
// issues FP64 at nine tenths of the rate that a loop of independent FMAs reaches
// on the card (2.27 ns per wave operation and SIMD).  XCD x (block b runs on XCD b mod 8)
// takes one contiguous eighth of the list, which is in brick order, so the
// items in flight on an XCD are neighbours that read each other's cells as
// halos from that XCD's L2.
template <int D, int TX, int TY, int TZ, int NT, bool FUSE, bool BOTH, bool CHAR>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(CHAR ? 4 : 6))) void k_stage(DevMesh m, int mode, const double* __restrict__ Uin,
                                              double* Ug, int* err, const double* Un, double* out,
                                              double* __restrict__ fr,
                                              const StageItem* __restrict__ items, int count,
                                              const int* __restrict__ dir,
                                              const double* __restrict__ dtp,
                                              unsigned long long* __restrict__ lam_next,
                                              const unsigned long long* __restrict__ lam_in,
                                              double* __restrict__ dt_out) {
  using S = TileShape<D, TX, TY, TZ>;
  constexpr bool UNION = D <= 2;
  constexpr int NU = S::NUNION;
  // edge fluxes: one direction at a time, or x and y together (BOTH)
  constexpr int NEDXY = S::slots(0) + S::slots(1);
  __shared__ double sP[(D + 2) * (UNION ? NU : S::EXTMAX)];
  __shared__ double sF[(D + 2) * (BOTH ? NEDXY : S::FXMAX)];
  const int item = xcd_item(dir ? dir[1] : count);
  if (item < 0) return;
  unsigned long long best = 0ull;
  stage_item<D, TX, TY, TZ, NT, FUSE, BOTH, CHAR>(m, mode, Uin, Ug, err, Un, out, fr, items[item],
                                                  item == 0, dtp, lam_next, lam_in, dt_out, sP, sF,
                                                  best);
  if (lam_next != nullptr && mode == kModeStage3)
    block_max_rate(best, m.lv[items[item].level].h, lam_next);
}

// Items of a (pid, tile) list, a thread each (see StageItem).
template <int D>
__global__ __launch_bounds__(64) void k_item_tables(DevMesh m, const int* __restrict__ tiles,
                                                    int count, int tx, int ty, int tz,
                                                    const uint8_t* __restrict__ cfmask,
                                                    StageItem* __restrict__ items) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= count) return;
  StageItem it;
  it.pid = tiles[2 * i];
  const int tile = tiles[2 * i + 1];
  it.level = m.level[it.pid];
  const LevelC& L = m.lv[it.level];
  it.cf = cfmask[it.pid];
  it.regs = cfmask[m.max_patches + it.pid];
  const int nt0 = L.n / tx, nt1 = D >= 2 ? L.n / ty : 1;
  it.o[0] = tile % nt0 * tx;
  it.o[1] = D >= 2 ? tile / nt0 % nt1 * ty : 0;
  it.o[2] = D >= 3 ? tile / (nt0 * nt1) * tz : 0;
  int pc[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < D; ++j) pc[j] = m.coord[3 * it.pid + j];
  it.px = pc[0];
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    const int j = f >> 1;
    it.nb[f] = kNbNone;
    if (j >= D) continue;
    int q[3] = {pc[0], pc[1], pc[2]};
    q[j] += f & 1 ? 1 : -1;
    const bool out = (unsigned)q[j] >= (unsigned)L.np;
    if (out && !m.periodic[j]) {
      it.nb[f] = kNbWall;
    } else {
      if (out) q[j] = f & 1 ? 0 : L.np - 1;
      it.nb[f] = map_at<D>(m, it.level, q);
    }
  }
  it.parent = 0;
  if (it.level > 0) {
    const int ppid = m.parent[it.pid];
    const LevelC& C = m.lv[it.level - 1];
    int q[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < D; ++j)
      q[j] = pc[j] * (L.n / 2) - m.coord[3 * ppid + j] * C.n + it.o[j] / 2 + NG;
    it.parent = patch_base(m, ppid, it.level - 1) + box_off<D>(C.full, q[0], q[1], q[2]);
  }
  items[i] = it;
}

}  // namespace

void Kernels::stage_items(const DevMesh& m, const int* tiles, int count, const uint8_t* cfmask,
                          StageItem* items, hipStream_t s) {
  if (count <= 0) return;
  const TileVariant& t = variant(m.tile);
  const dim3 grid((count + 63) / 64), block(64);
  switch (t.dim) {
    case 1: hipLaunchKernelGGL(k_item_tables<1>, grid, block, 0, s, m, tiles, count, t.tx, t.ty, t.tz, cfmask, items); break;
    case 2: hipLaunchKernelGGL(k_item_tables<2>, grid, block, 0, s, m, tiles, count, t.tx, t.ty, t.tz, cfmask, items); break;
    default: hipLaunchKernelGGL(k_item_tables<3>, grid, block, 0, s, m, tiles, count, t.tx, t.ty, t.tz, cfmask, items); break;
  }
}

// Tile variants: thread counts cover the nodes (T_J + 4 per line) of one
// direction of the tile in one pass, in whole waves (the 8x8x4 tile's z
// direction takes two); the 8x8x8 tile's 768 nodes are 12 waves, which also
// spread evenly over a CU's 4 SIMDs.
static const Kernels::TileVariant kVariants[] = {
    {1, 16, 1, 1, 64}, {1, 8, 1, 1, 64},                                   // 1D
    {2, 16, 16, 1, 320}, {2, 16, 8, 1, 192}, {2, 8, 8, 1, 128},           // 2D
    {3, 8, 8, 8, 768}, {3, 8, 8, 4, 448}, {3, 4, 4, 4, 128},              // 3D
    // 2D, x and y edges in one sweep (stage_both)
    {2, 16, 16, 1, 320, 1}, {2, 16, 8, 1, 192, 1}, {2, 8, 8, 1, 128, 1},
};

int Kernels::num_variants() { return (int)(sizeof(kVariants) / sizeof(kVariants[0])); }

Kernels::TileVariant Kernels::variant(int v) { return kVariants[v]; }

bool Kernels::variant_fits(int v, int dim, const int* n, int nlev) {
  if (v < 0 || v >= num_variants() || kVariants[v].dim != dim) return false;
  const TileVariant& t = kVariants[v];
  for (int l = 0; l < nlev; ++l) {
    if (n[l] % t.tx) return false;
    if (dim >= 2 && n[l] % t.ty) return false;
    if (dim >= 3 && n[l] % t.tz) return false;
  }
  return true;
}

int Kernels::default_variant(int dim, const int* n, int nlev) {
  for (int v = 0; v < num_variants(); ++v)
    if (variant_fits(v, dim, n, nlev)) return v;
  return -1;
}

int Kernels::tiles_per_patch(int v, int n) {
  const TileVariant& t = kVariants[v];
  int r = n / t.tx;
  if (t.dim >= 2) r *= n / t.ty;
  if (t.dim >= 3) r *= n / t.tz;
  return r;
}

void Kernels::stage(const DevMesh& m, int mode, double* Uin, int* err, const double* Un,
                    double* out, double* fr, const StageItem* items, int count, const int* dir,
                    const double* dt, bool fuse, unsigned long long* lam_next, hipStream_t s,
                    hipEvent_t ev0, hipEvent_t ev1,
                    const unsigned long long* lam_in, double* dt_out) {
  if (count <= 0) return;
  // one block per work item (`count` may exceed the live count read from the
  // directory), in whole groups of kXcds blocks (see xcd_item)
  const int nb = stage_grid(count);
  const bool chr = m.scheme == AMR_SCHEME_CHAR;
#define AMR_STAGE_K(D, TX, TY, TZ, NT, F, B, C)                                                \
  do {                                                                                          \
    auto kern = k_stage<D, TX, TY, TZ, NT, F, B, C>;                                            \
    if (ev0)                                                                                    \
      hipExtLaunchKernelGGL(kern, dim3(nb), dim3(NT), 0, s, ev0, ev1, 0, m, mode, Uin, Uin, err, Un, \
                            out, fr, items, count, dir, dt, lam_next, lam_in, dt_out);          \
    else                                                                                        \
      hipLaunchKernelGGL(kern, dim3(nb), dim3(NT), 0, s, m, mode, Uin, Uin, err, Un, out, fr, items, \
                         count, dir, dt, lam_next, lam_in, dt_out);                             \
  } while (0)
#define AMR_STAGE_F(D, TX, TY, TZ, NT, F, B)          \
  do {                                                \
    if (chr)                                          \
      AMR_STAGE_K(D, TX, TY, TZ, NT, F, B, true);     \
    else                                              \
      AMR_STAGE_K(D, TX, TY, TZ, NT, F, B, false);    \
  } while (0)
#define AMR_STAGE(D, TX, TY, TZ, NT, B)        \
  do {                                         \
    if (fuse)                                  \
      AMR_STAGE_F(D, TX, TY, TZ, NT, true, B); \
    else                                       \
      AMR_STAGE_F(D, TX, TY, TZ, NT, false, B);\
  } while (0)
  switch (m.tile) {
    case 0: AMR_STAGE(1, 16, 1, 1, 64, false); break;
    case 1: AMR_STAGE(1, 8, 1, 1, 64, false); break;
    case 2: AMR_STAGE(2, 16, 16, 1, 320, false); break;
    case 3: AMR_STAGE(2, 16, 8, 1, 192, false); break;
    case 4: AMR_STAGE(2, 8, 8, 1, 128, false); break;
    case 5: AMR_STAGE(3, 8, 8, 8, 768, false); break;
    case 6: AMR_STAGE(3, 8, 8, 4, 448, false); break;
    case 7: AMR_STAGE(3, 4, 4, 4, 128, false); break;
    case 8: AMR_STAGE(2, 16, 16, 1, 320, true); break;
    case 9: AMR_STAGE(2, 16, 8, 1, 192, true); break;
    default: AMR_STAGE(2, 8, 8, 1, 128, true); break;
  }
#undef AMR_STAGE
#undef AMR_STAGE_F
#undef AMR_STAGE_K
}

}  // namespace amr

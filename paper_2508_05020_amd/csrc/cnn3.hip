// Learned refinement predictor (3D): BF16 inputs/weights/activations, FP32
// accumulation on the MFMA units of gfx950.
//
// The network works on tiles of 8^3 output cells, so that one patch of edge
// 8, 16 or 32 is 1, 8 or 64 tiles and every tile's activations fit in LDS.
// Input per tile: normalised (rho, u, v, w, p) on the tile plus a halo of 3
// cells, [14]^3 voxels stored with 8 channels (the last 3 zero) so that the
// 4 consecutive channels an MFMA lane needs are one 8-byte load.  Three valid
// 3x3x3 convolutions 5 -> 8 -> 8 -> 1 with bias, ReLU after the first two,
// give one logit per tile cell.
//
// Convolutions as implicit GEMM on the 16x16x32 MFMA: rows = 16 output
// voxels, columns = output channels (8 of 16 used), K = (tap, input channel)
// with 4 taps x 8 channels per chunk, a lane's 8 values being one voxel's
// channels (one 16-byte read), 7 chunks for 27 taps.  Weight gradients swap the
// roles: rows = output channel, columns = (tap of a pair, input channel), K =
// voxels.  Operand layout: see cnn_device.hpp.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "amr_internal.hpp"
#include "cnn_device.hpp"
#include "cnn_internal.hpp"

namespace amr {
namespace {

using namespace cnnd;

constexpr int NG = kNG;
constexpr int T = CNN3_TILE;
constexpr int CH = CNN3_CH;
constexpr int W0 = T + 6, W1 = T + 4, W2 = T + 2;
constexpr int P0 = CNN3_P0, P1 = CNN3_P1, P2 = CNN3_P2, P3 = CNN3_P3;
constexpr int KCH = 7;     // K chunks of a convolution: taps 4 kc .. 4 kc + 3
constexpr int WPAIRS = 14;  // tap pairs of a weight gradient
// weights of one convolution in LDS as B operands: [28 taps][8 columns][8 K
// channels], tap 27 zero
constexpr int OPS = 4 * KCH * 8 * 8;
// threads per block: the loops stride over the block's waves, so more waves
// shorten a tile's latency (a training batch is only tens of tiles)
constexpr int FWD_THREADS = 1024;
constexpr int TRAIN_THREADS = 1024;
constexpr int TRAIN_WAVES = TRAIN_THREADS / 64;

static_assert(CH == 8, "a lane's 8 K values are one voxel's channels");
static_assert(P1 % 16 == 0, "layer-1 voxels in whole MFMA row blocks");

// ---------------------------------------------------------------------------
// gather: normalised BF16 input tiles from the FP64 state (ghosts filled)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_cnn3_gather(DevMesh m, const double* __restrict__ U,
                                                     const int* __restrict__ items, int count,
                                                     CnnNorm norm,
                                                     unsigned short* __restrict__ X) {
#pragma clang fp contract(off)
  const long long total = (long long)count * P0;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(t / P0);
    const int v = (int)(t - (long long)b * P0);
    const int item = items[b];
    const int pid = item / CNN3_MAX_TILES, tile = item - pid * CNN3_MAX_TILES;
    const LevelC& L = m.lv[m.level[pid]];
    const int nt = L.n / T;
    const int tz = tile / (nt * nt), ty = (tile / nt) % nt, tx = tile % nt;
    const int z = v / (W0 * W0), y = (v / W0) % W0, x = v % W0;
    // interior cell coordinates -3 .. n + 2: inside the 4 ghost layers
    const int cz = T * tz + z - 3, cy = T * ty + y - 3, cx = T * tx + x - 3;
    const double* P = U + L.pool_off + (long long)(pid - L.pid_base) * L.stride;
    const long long vs = (long long)L.full * L.full * L.full;
    const long long off = ((long long)(cz + NG) * L.full + (cy + NG)) * L.full + (cx + NG);
    const double rho = P[off], mx = P[vs + off], my = P[2 * vs + off], mz = P[3 * vs + off];
    const double E = P[4 * vs + off];
    const double ux = mx / rho, uy = my / rho, uz = mz / rho;
    double ke = mx * ux;
    ke = ke + my * uy;
    ke = ke + mz * uz;
    ke = 0.5 * ke;
    const double pr = m.gm1 * (E - ke);
    const double f[5] = {rho, ux, uy, uz, pr};
    unsigned short h[8];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      const double zc = (f[c] - (double)norm.mean[c]) * (double)norm.istd[c];
      h[c] = f2bf((float)zc);
    }
    h[5] = h[6] = h[7] = 0;
    uint4 o;
    o.x = h[0] | ((unsigned)h[1] << 16);
    o.y = h[2] | ((unsigned)h[3] << 16);
    o.z = h[4] | ((unsigned)h[5] << 16);
    o.w = h[6] | ((unsigned)h[7] << 16);
    reinterpret_cast<uint4*>(X)[(long long)b * P0 + v] = o;
  }
}

// ---------------------------------------------------------------------------
// forward of one tile per block (16 waves); activations in LDS
// ---------------------------------------------------------------------------

// A operands of a 3x3x3 convolution over a box of edge WI with 8 channels per
// voxel: chunk kc holds the taps 4 kc + kq of the lane groups kq, FLIP reading
// tap t at the mirrored place.  Tap 27 does not exist: zero.
template <int WI, bool FLIP>
struct TapReads {
  int off[KCH];  // voxels from the voxel at tap 0 (2 2 2 of a mirrored one)
  bool last;     // the lane has a tap in the last chunk
  __device__ __forceinline__ explicit TapReads(int kq) : last(kq < 3) {
#pragma unroll
    for (int kc = 0; kc < KCH; ++kc) {
      const int t = min(4 * kc + kq, 26), tap = FLIP ? 26 - t : t;
      off[kc] = ((tap / 9) * WI + (tap / 3) % 3) * WI + tap % 3;
    }
  }
  __device__ __forceinline__ u4 operator()(const unsigned short* voxel, int kc) const {
    u4 a = *reinterpret_cast<const u4*>(voxel + off[kc] * CH);
    if (kc == KCH - 1 && !last) a = u4{0u, 0u, 0u, 0u};
    return a;
  }
};

// The B operands of a convolution into LDS, by the whole block: column j, K
// channel k and tap t from w[(j SJ + k SK) 27 + t], k < NK.
template <int SJ, int SK, int NK>
__device__ __forceinline__ void stage_operands(unsigned short* ops, const unsigned short* w) {
  for (int t = threadIdx.x; t < OPS; t += blockDim.x) {
    const int k = t & 7, j = (t >> 3) & 7, tap = t >> 6;
    ops[t] = tap < 27 && k < NK ? w[(j * SJ + k * SK) * 27 + tap] : (unsigned short)0;
  }
}

struct Operands {
  u4 b[KCH];
  __device__ __forceinline__ Operands(const unsigned short* ops, int i, int kq) {
#pragma unroll
    for (int kc = 0; kc < KCH; ++kc)
      b[kc] = reinterpret_cast<const u4*>(ops)[(4 * kc + kq) * 8 + (i & 7)];
  }
};

// valid 3x3x3 convolution, 8 output channels, from a voxel-major LDS input of
// edge WI with 8 stored channels to edge WI - 2 (bias, ReLU, BF16).
template <int WI>
__device__ __forceinline__ void conv3(const unsigned short* __restrict__ in,
                                      unsigned short* __restrict__ out,
                                      const unsigned short* __restrict__ ops,
                                      const float* __restrict__ bias) {
  constexpr int WO = WI - 2;
  constexpr int P = WO * WO * WO;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int i = lane & 15, kq = lane >> 4;
  const Operands w(ops, i, kq);
  const TapReads<WI, false> a(kq);
  const float bcol = bias[i & 7];
  constexpr int nblk = (P + 15) / 16;
  for (int blk = wave; blk < nblk; blk += nw) {
    const int p = 16 * blk + i;
    const int pc = p < P ? p : P - 1;
    const int pz = pc / (WO * WO), r = pc - pz * WO * WO;
    const int py = r / WO, px = r - py * WO;
    const unsigned short* voxel = in + ((pz * WI + py) * WI + px) * CH;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KCH; ++kc) acc = mfma32(a(voxel, kc), w.b[kc], acc);
    if (i < 8) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = 16 * blk + 4 * kq + e;
        const float v = acc[e] + bcol;
        if (q < P) out[q * CH + i] = f2bf_hw(v > 0.f ? v : 0.f);
      }
    }
  }
}

// A tile's latency is the sum of its phases: with 8 waves, weights packed by
// every wave from global memory, 16-wide K chunks and layer-3 weights read per
// tap, 256 tiles took 30.4 us; 14.8 now.
// LDS (bytes)
constexpr int FL_X = 0;
constexpr int FL_A1 = FL_X + P0 * CH * 2;
constexpr int FL_W1 = FL_A1 + P1 * CH * 2;
constexpr int FL_W2 = FL_W1 + OPS * 2;
constexpr int FL_W3 = FL_W2 + OPS * 2;
constexpr int FL_TOTAL = FL_W3 + 27 * 8 * 4;
static_assert(2 * FL_TOTAL <= 160 * 1024, "two blocks per CU");

__global__ __launch_bounds__(FWD_THREADS) void k_cnn3_fwd(int count, const unsigned short* __restrict__ X,
                                                      const unsigned short* __restrict__ Wb,
                                                      const float* __restrict__ params,
                                                      float* __restrict__ Z) {
  extern __shared__ __align__(16) unsigned char fwd_smem[];
  const int b = blockIdx.x;
  if (b >= count) return;
  unsigned short* sx = (unsigned short*)(fwd_smem + FL_X);   // P0 x 8
  unsigned short* s1 = (unsigned short*)(fwd_smem + FL_A1);  // P1 x 8
  unsigned short* s2 = sx;                                   // P2 x 8, over sx once layer 1 is done
  unsigned short* w1 = (unsigned short*)(fwd_smem + FL_W1);
  unsigned short* w2 = (unsigned short*)(fwd_smem + FL_W2);
  float* w3 = (float*)(fwd_smem + FL_W3);                    // [27][8]
  const uint4* xg = reinterpret_cast<const uint4*>(X) + (long long)b * P0;
  for (int t = threadIdx.x; t < P0; t += FWD_THREADS) reinterpret_cast<uint4*>(sx)[t] = xg[t];
  stage_operands<5, 1, 5>(w1, Wb + CNN3_W1);
  stage_operands<8, 1, 8>(w2, Wb + CNN3_W2);
  if (threadIdx.x < 27 * 8) w3[(threadIdx.x % 27) * 8 + threadIdx.x / 27] = bf2f(Wb[CNN3_W3 + threadIdx.x]);
  __syncthreads();
  conv3<W0>(sx, s1, w1, params + CNN3_B1);
  __syncthreads();
  conv3<W1>(s1, s2, w2, params + CNN3_B2);
  __syncthreads();
  // layer 3 (8 -> 1) on the VALU
  const float b3 = params[CNN3_B3];
  for (int p = threadIdx.x; p < P3; p += FWD_THREADS) {
    const int pz = p / (T * T), py = (p / T) % T, px = p % T;
    const unsigned short* base = s2 + ((pz * W2 + py) * W2 + px) * CH;
    float acc = 0.f;
#pragma unroll
    for (int tap = 0; tap < 27; ++tap) {
      const u4 a = *reinterpret_cast<const u4*>(base + (((tap / 9) * W2 + (tap / 3) % 3) * W2 + tap % 3) * CH);
      const float4 wa = *reinterpret_cast<const float4*>(w3 + tap * 8);
      const float4 wb = *reinterpret_cast<const float4*>(w3 + tap * 8 + 4);
      const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
      for (int c = 0; c < 8; ++c)
        acc += bf2f((unsigned short)(a[c >> 1] >> (16 * (c & 1)))) * w[c];
    }
    Z[(long long)b * P3 + p] = acc + b3;
  }
}

// ---------------------------------------------------------------------------
// training: forward, loss and backward of one tile per block, the per-tile
// parameter gradients and loss to global memory (the 3D form of k_cnn_train)
// ---------------------------------------------------------------------------
// One tile's latency per launch: the forward (29 us for 64 tiles), the loss
// (4.6 us) and the backward (124 us) were launches of their own, with
// activations through memory, bounds checks per tap and serial sums per
// parameter; one launch now, 45.6 us with 16-wide K chunks and weights packed by
// every wave, 39.4 with 32-wide chunks and operands staged once, 37.9 with the
// blocks of dz1 taken as the waves come, 37.4 with weights of dz2 read for two
// voxels; clearing the activations past the grid in dW2 takes 0.2 us of that.
//
// LDS (bytes): dz1 takes the place of the second activation,
// the logit gradients and the FP32 copy of W3; dz2 has a border of two zero
// voxels.
constexpr int TL_X = 0;
constexpr int TL_A1 = TL_X + P0 * CH * 2;
constexpr int TL_A2 = TL_A1 + (P1 + 2) * CH * 2;  // two zero voxels behind a1 (see dW2)
constexpr int TL_G = TL_A2 + P2 * CH * 2;
constexpr int TL_W3 = TL_G + P3 * 4;
constexpr int TL_DZ1 = TL_A2;
constexpr int TL_DZ2 = TL_DZ1 + P1 * CH * 2;
constexpr int TL_RED = TL_DZ2 + P0 * CH * 2;      // dz2 with its border is as large as the input
constexpr int RED_N = 8 * 27 + 1;                 // dW3 and db3 of one wave
constexpr int TL_W2F = TL_RED + ((TRAIN_WAVES * RED_N * 4 + 15) / 16) * 16;  // W2, mirrored
constexpr int TL_NEXT = TL_W2F + OPS * 2;  // block counter of dz1
constexpr int TL_TOTAL = TL_NEXT + 16;
constexpr int TL_W1 = TL_DZ2, TL_W2 = TL_W1 + OPS * 2;  // until the forward convolutions are done
static_assert(TL_W3 + 27 * 8 * 4 <= TL_DZ2, "a2, g and W3 fit under dz1");
static_assert(TL_TOTAL <= 160 * 1024, "one block per CU");
static_assert(W2 + 4 == W0, "dz2 with its border has the input's shape");

__global__ __launch_bounds__(TRAIN_THREADS) void k_cnn3_train(
    int count, const unsigned short* __restrict__ X, const uint8_t* __restrict__ Y,
    const unsigned short* __restrict__ Wg, const float* __restrict__ params, float pos_weight,
    float inv_total, float* __restrict__ partials, float* __restrict__ loss_part) {
  extern __shared__ __align__(16) unsigned char train_smem[];
  const int b = blockIdx.x;
  if (b >= count) return;
  unsigned short* x = (unsigned short*)(train_smem + TL_X);
  unsigned short* a1 = (unsigned short*)(train_smem + TL_A1);
  unsigned short* a2 = (unsigned short*)(train_smem + TL_A2);
  float* g = (float*)(train_smem + TL_G);
  float* w3 = (float*)(train_smem + TL_W3);                       // [27][8]
  unsigned short* dz1 = (unsigned short*)(train_smem + TL_DZ1);   // [P1][8]
  unsigned short* dz2 = (unsigned short*)(train_smem + TL_DZ2);   // [W0^3][8]
  float* red = (float*)(train_smem + TL_RED);
  unsigned short* w1 = (unsigned short*)(train_smem + TL_W1);
  unsigned short* w2 = (unsigned short*)(train_smem + TL_W2);
  unsigned short* w2f = (unsigned short*)(train_smem + TL_W2F);
  int* next = (int*)(train_smem + TL_NEXT);
  float* part = partials + (long long)b * CNN3_NPARAM;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, kq = lane >> 4;

  {
    const uint4* gx = reinterpret_cast<const uint4*>(X) + (long long)b * P0;
    const uint4 z = {0u, 0u, 0u, 0u};
    for (int t = tid; t < P0; t += TRAIN_THREADS) {
      reinterpret_cast<uint4*>(x)[t] = gx[t];
    }
    stage_operands<5, 1, 5>(w1, Wg + CNN3_W1);
    stage_operands<8, 1, 8>(w2, Wg + CNN3_W2);
    stage_operands<1, 8, 8>(w2f, Wg + CNN3_W2);
    if (tid == 0) next[0] = 0;
    if (tid < 2) reinterpret_cast<uint4*>(a1 + P1 * CH)[tid] = z;
    if (tid < 27 * 8) w3[(tid % 27) * 8 + tid / 27] = bf2f(Wg[CNN3_W3 + tid]);
  }
  __syncthreads();
  conv3<W0>(x, a1, w1, params + CNN3_B1);
  __syncthreads();
  conv3<W1>(a1, a2, w2, params + CNN3_B2);
  __syncthreads();
  for (int t = tid; t < P0; t += TRAIN_THREADS) reinterpret_cast<uint4*>(dz2)[t] = uint4{0u, 0u, 0u, 0u};

  // --- layer 3 and the loss: 2 lanes per voxel, 4 channels each
  {
    static_assert(2 * P3 == TRAIN_THREADS, "one layer-3 item per thread");
    const int p = tid >> 1, c4 = 4 * (tid & 1);
    const int pz = p / (T * T), py = (p / T) % T, px = p % T;
    const unsigned short* base = a2 + ((pz * W2 + py) * W2 + px) * CH + c4;
    float acc = 0.f;
#pragma unroll
    for (int tap = 0; tap < 27; ++tap) {
      const s4 a = load4(base + (((tap / 9) * W2 + (tap / 3) % 3) * W2 + tap % 3) * CH);
      const float4 w = *reinterpret_cast<const float4*>(w3 + tap * 8 + c4);
      acc += bf2f((unsigned short)a.x) * w.x;
      acc += bf2f((unsigned short)a.y) * w.y;
      acc += bf2f((unsigned short)a.z) * w.z;
      acc += bf2f((unsigned short)a.w) * w.w;
    }
    acc += __shfl_xor(acc, 1);
    float loss = 0.f;
    if ((tid & 1) == 0) {
      const float z = acc + params[CNN3_B3];
      const float yv = Y[(long long)b * P3 + p] ? 1.f : 0.f;
      const float tail = log1pf(expf(-fabsf(z)));
      loss = pos_weight * yv * (fmaxf(-z, 0.f) + tail) + (1.f - yv) * (fmaxf(z, 0.f) + tail);
      const float s = 1.f / (1.f + expf(-z));
      g[p] = (pos_weight * yv * (s - 1.f) + (1.f - yv) * s) * inv_total;
    }
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
    if (lane == 0) red[wave] = loss;
  }
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
    for (int k = 0; k < TRAIN_WAVES; ++k) s += red[k];
    loss_part[b] = s * inv_total;
  }
  __syncthreads();

  // --- dW3[c][tap] = sum_p a2[p + tap][c] g[p], db3 = sum_p g[p]: a wave takes
  // x rows, a lane one tap and 4 channels (54 lanes; lane 54 sums g); partial
  // sums per wave into red
  if (lane <= 54) {
    const int tap = lane < 54 ? lane >> 1 : 0, c4 = 4 * (lane & 1);
    const unsigned short* at = a2 + (((tap / 9) * W2 + (tap / 3) % 3) * W2 + tap % 3) * CH + c4;
    float acc[4] = {0.f, 0.f, 0.f, 0.f}, gs = 0.f;
    for (int r = wave; r < T * T; r += TRAIN_WAVES) {
      const unsigned short* ar = at + ((r / T) * W2 + r % T) * W2 * CH;
#pragma unroll
      for (int px = 0; px < T; ++px) {
        const float gv = g[r * T + px];
        const s4 a = load4(ar + px * CH);
        gs += gv;
        acc[0] += bf2f((unsigned short)a.x) * gv;
        acc[1] += bf2f((unsigned short)a.y) * gv;
        acc[2] += bf2f((unsigned short)a.z) * gv;
        acc[3] += bf2f((unsigned short)a.w) * gv;
      }
    }
    if (lane < 54) {
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave * RED_N + (c4 + e) * 27 + tap] = acc[e];
    } else {
      red[wave * RED_N + 8 * 27] = gs;
    }
  }
  // --- dz2 = relu'(z2) * (W3 (x) g) on the layer-2 grid, 4 channels per item, two
  // items per thread (t and t + TRAIN_THREADS), which share each weight read
  {
    static_assert(2 * P2 <= 2 * TRAIN_THREADS, "two items per thread cover the grid");
    const int c4 = 4 * (tid & 1);
    int q[2], qz[2], qy[2], qx[2];
    float acc[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      q[k] = (tid + k * TRAIN_THREADS) >> 1;
      qz[k] = q[k] / (W2 * W2);
      qy[k] = (q[k] / W2) % W2;
      qx[k] = q[k] % W2;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[k][e] = 0.f;
    }
#pragma unroll 1  // the weights of 9 taps at a time in registers
    for (int tz = 0; tz < 3; ++tz) {
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        const float4 w = *reinterpret_cast<const float4*>(w3 + (9 * tz + t9) * 8 + c4);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int pz = qz[k] - tz, py = qy[k] - t9 / 3, px = qx[k] - t9 % 3;
          // read in any case (no branch around the loads), zero outside
          const bool in = (unsigned)pz < (unsigned)T && (unsigned)py < (unsigned)T && (unsigned)px < (unsigned)T;
          const float gr = g[in ? (pz * T + py) * T + px : 0];
          const float gv = in ? gr : 0.f;
          acc[k][0] += w.x * gv;
          acc[k][1] += w.y * gv;
          acc[k][2] += w.z * gv;
          acc[k][3] += w.w * gv;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (q[k] >= P2) continue;
      const s4 on = load4(a2 + q[k] * CH + c4);  // a2 = relu(z2) in BF16: nonzero iff z2 > 0
      uint2 o;
      o.x = f2bf_hw(on.x ? acc[k][0] : 0.f) | ((unsigned)f2bf_hw(on.y ? acc[k][1] : 0.f) << 16);
      o.y = f2bf_hw(on.z ? acc[k][2] : 0.f) | ((unsigned)f2bf_hw(on.w ? acc[k][3] : 0.f) << 16);
      *reinterpret_cast<uint2*>(dz2 + (((qz[k] + 2) * W0 + qy[k] + 2) * W0 + qx[k] + 2) * CH + c4) = o;
    }
  }
  __syncthreads();

  if (tid < RED_N) {
    float s = 0.f;
    for (int k = 0; k < TRAIN_WAVES; ++k) s += red[k * RED_N + tid];
    part[CNN3_W3 + tid] = s;  // db3 follows W3
  }
  static_assert(CNN3_B3 == CNN3_W3 + 8 * 27 && WPAIRS < TRAIN_WAVES,
                "a wave per tap pair and one for the bias sums");
  // column j of a weight-gradient product: (tap of the pair, input channel);
  // in transposed reads this lane points at voxel i / 4 of its K group of 4 x
  // neighbours and at 4 columns of it: channels c4 of tap `ltap` (the second
  // tap of the last pair does not exist: its columns are not used)
  const int wtap = 2 * wave + (i >> 3), wc = i & 7;
  const int gx = i >> 2, c4 = 4 * (i & 1);
  const int ltap = min(2 * wave + ((i >> 1) & 1), 26);

  // --- dW2[o][c][tap] = sum_p dz2[p][o] a1[p + tap][c]: D[i = o][j = (tap, c)],
  // K = layer-2 voxels, a tap pair per wave; db2 by the wave after them.  A
  // step's 4 K groups are 4 rows y of one plane (the last two rows of two
  // planes together), the same x in each, so that a step's reads differ from
  // the lane's first by a wave-uniform offset; x runs to 12: dz2's border is
  // zero there, a1 reads at most two voxels past its end, and what it reads for
  // those x is cleared (zero times an infinite activation would be NaN).
  if (wave < WPAIRS) {
    const int tz = ltap / 9, ty = (ltap / 3) % 3, tx = ltap % 3;
    const unsigned short* za = dz2 + ((2 * W0 + 2 + kq) * W0 + 2 + gx) * CH + c4;
    const unsigned short* aa = a1 + ((tz * W1 + ty + kq) * W1 + tx + gx) * CH + c4;
    // the same for rows 8 and 9 of planes z and z + 1
    const int ky = 8 + (kq & 1), kz = kq >> 1;
    const unsigned short* zb = dz2 + (((2 + kz) * W0 + 2 + ky) * W0 + 2 + gx) * CH + c4;
    const unsigned short* ab = a1 + (((tz + kz) * W1 + ty + ky) * W1 + tx + gx) * CH + c4;
    f4 acc[3] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    static_assert(W2 == 10, "rows 0 .. 7 in blocks of four, 8 and 9 in pairs of planes");
    auto act = [](const unsigned short* p, int xg) {
      s4 v = load4_tr(p);
      if (xg == 2) v.z = v.w = 0;  // x = 10 and 11
      return v;
    };
    for (int z = 0; z < W2; ++z) {
#pragma unroll
      for (int xg = 0; xg < 3; ++xg)
        acc[xg] = mfma32(join(load4_tr(za + (z * W0 * W0 + 4 * xg) * CH),
                              load4_tr(za + ((z * W0 + 4) * W0 + 4 * xg) * CH)),
                         join(act(aa + (z * W1 * W1 + 4 * xg) * CH, xg),
                              act(aa + ((z * W1 + 4) * W1 + 4 * xg) * CH, xg)), acc[xg]);
      if (z & 1) continue;
#pragma unroll
      for (int xg = 0; xg < 3; ++xg)
        acc[xg] = mfma(load4_tr(zb + (z * W0 * W0 + 4 * xg) * CH),
                       act(ab + (z * W1 * W1 + 4 * xg) * CH, xg), acc[xg]);
    }
    if (wtap < 27) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = 4 * kq + e;
        if (o < 8) part[CNN3_W2 + (o * 8 + wc) * 27 + wtap] = (acc[0][e] + acc[1][e]) + acc[2][e];
      }
    }
  } else if (wave == WPAIRS) {
    const int o = lane & 7;
    float s = 0.f;
#pragma unroll 4
    for (int p = lane >> 3; p < P2; p += 8) {
      const int pz = p / (W2 * W2), py = (p / W2) % W2, px = p % W2;
      s += bf2f(dz2[(((pz + 2) * W0 + py + 2) * W0 + px + 2) * CH + o]);
    }
    s += __shfl_xor(s, 8);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lane < 8) part[CNN3_B2 + o] = s;
  }

  // --- dz1[q][c] = relu'(z1) sum_tap sum_o W2[o][c][tap] dz2[q - tap][o]:
  // D[i = voxel][j = c], K = (tap, o), 4 taps x 8 channels per chunk
  {
    const Operands w(w2f, i, kq);
    const TapReads<W0, true> a(kq);
    constexpr int nblk = P1 / 16;
    // blocks as the waves come: those with a tap pair above arrive last
    for (int blk = take(next); blk < nblk; blk = take(next)) {
      const int q = 16 * blk + i;
      const int qz = q / (W1 * W1), qy = (q / W1) % W1, qx = q % W1;
      const unsigned short* voxel = dz2 + ((qz * W0 + qy) * W0 + qx) * CH;
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < KCH; ++kc) acc = mfma32(a(voxel, kc), w.b[kc], acc);
      if (i < 8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int q = 16 * blk + 4 * kq + e;
          dz1[q * CH + i] = f2bf_hw(a1[q * CH + i] != 0 ? acc[e] : 0.f);
        }
      }
    }
  }
  __syncthreads();

  // --- dW1[o][c][tap] = sum_p dz1[p][o] x[p + tap][c], db1 by the wave after
  if (wave < WPAIRS) {
    const unsigned short* da = dz1 + (kq * W1 + gx) * CH + c4;
    const unsigned short* xa = x + (((ltap / 9) * W0 + (ltap / 3) % 3 + kq) * W0 + ltap % 3 + gx) * CH + c4;
    f4 acc[3] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    static_assert(W1 == 12, "three blocks of four rows and of four voxels in x");
    for (int z = 0; z < W1; z += 2)
#pragma unroll
      for (int yb = 0; yb < 3; ++yb)
#pragma unroll
        for (int xg = 0; xg < 3; ++xg) {
          const unsigned short* d = da + ((z * W1 + 4 * yb) * W1 + 4 * xg) * CH;
          const unsigned short* v = xa + ((z * W0 + 4 * yb) * W0 + 4 * xg) * CH;
          acc[xg] = mfma32(join(load4_tr(d), load4_tr(d + W1 * W1 * CH)),
                           join(load4_tr(v), load4_tr(v + W0 * W0 * CH)), acc[xg]);
        }
    if (wtap < 27 && wc < 5) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = 4 * kq + e;
        if (o < 8) part[CNN3_W1 + (o * 5 + wc) * 27 + wtap] = (acc[0][e] + acc[1][e]) + acc[2][e];
      }
    }
  } else if (wave == WPAIRS) {
    const int o = lane & 7;
    float s = 0.f;
#pragma unroll 4
    for (int q = lane >> 3; q < P1; q += 8) s += bf2f(dz1[q * CH + o]);
    s += __shfl_xor(s, 8);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lane < 8) part[CNN3_B1 + o] = s;
  }
}

// per-tile refine request: any logit above the threshold flags the tile's patch
__global__ __launch_bounds__(256) void k_cnn3_requests(int count, const float* __restrict__ Z,
                                                       const int* __restrict__ items, float zt,
                                                       uint8_t* __restrict__ flag) {
  const int b = blockIdx.x;
  if (b >= count) return;
  int any = 0;
  for (int p = threadIdx.x; p < P3; p += blockDim.x) any |= Z[(long long)b * P3 + p] > zt;
  any = __syncthreads_or(any);
  // several tiles of one patch may store the same value
  if (threadIdx.x == 0 && any) flag[items[b] / CNN3_MAX_TILES] = 1;
}

}  // namespace

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
size_t Cnn3::fwd_lds() { return FL_TOTAL; }

static void allow_large_lds3() {
  static bool done = false;
  if (done) return;
  done = true;
  (void)hipFuncSetAttribute((const void*)k_cnn3_fwd, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
  (void)hipFuncSetAttribute((const void*)k_cnn3_train, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
}

void Cnn3::gather(const DevMesh& m, const double* U, const int* items, int count,
                  const CnnNorm& norm, unsigned short* X, hipStream_t s) {
  if (count <= 0) return;
  const long long total = (long long)count * P0;
  const int blocks = (int)std::min<long long>((total + 255) / 256, 65535);
  hipLaunchKernelGGL(k_cnn3_gather, dim3(blocks), dim3(256), 0, s, m, U, items, count, norm, X);
}

void Cnn3::forward(int count, const unsigned short* X, const unsigned short* Wb, const float* params,
                   float* Z, hipStream_t s) {
  if (count <= 0) return;
  allow_large_lds3();
  hipLaunchKernelGGL(k_cnn3_fwd, dim3(count), dim3(FWD_THREADS), fwd_lds(), s, count, X, Wb, params,
                     Z);
}

void Cnn3::train(int count, const unsigned short* X, const uint8_t* Y, const unsigned short* Wb,
                 const float* params, float pos_weight, float* partials, float* loss_part,
                 hipStream_t s) {
  if (count <= 0) return;
  allow_large_lds3();
  const float inv_total = 1.0f / (float)((long long)count * P3);
  hipLaunchKernelGGL(k_cnn3_train, dim3(count), dim3(TRAIN_THREADS), TL_TOTAL, s, count, X, Y, Wb,
                     params, pos_weight, inv_total, partials, loss_part);
}

void Cnn3::requests(int count, const float* Z, const int* items, float zt, uint8_t* flag,
                    hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_cnn3_requests, dim3(count), dim3(256), 0, s, count, Z, items, zt, flag);
}

}  // namespace amr

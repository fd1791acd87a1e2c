// Learned refinement predictor (2D): BF16 inputs/weights/activations, FP32
// accumulation on the MFMA units of gfx950.
//
// Network per patch of n x n cells: input (rho, u, v, p) normalised, with a
// halo of 3 cells, [n+6]^2 pixels x 4 channels; three valid 3x3
// convolutions 4 -> 16 -> 16 -> 1 with bias, ReLU after the first two;
// output logits on the n x n interior.  Activations are stored pixel-major
// with the channels innermost (HWC), so that the 4 consecutive channels an
// MFMA lane needs are one 8-byte load.
//
// MFMA operand layout: see cnn_device.hpp.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "amr_internal.hpp"
#include "cnn_device.hpp"
#include "cnn_internal.hpp"

namespace amr {
namespace {

using namespace cnnd;

constexpr int NG = kNG;

// ---------------------------------------------------------------------------
// gather: normalised BF16 input tiles from the FP64 state (ghosts filled)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_cnn_gather(DevMesh m, const double* __restrict__ U,
                                                    const int* __restrict__ pids, int count,
                                                    int n, CnnNorm norm,
                                                    unsigned short* __restrict__ X) {
#pragma clang fp contract(off)
  const int w = n + 6;
  const int P0 = w * w;
  const long long total = (long long)count * P0;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
       t += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(t / P0);
    const int p = (int)(t - (long long)b * P0);
    const int pid = pids[b];
    const int l = m.level[pid];
    const LevelC& L = m.lv[l];
    const int y = p / w - 3, x = p % w - 3;
    const double* P = U + L.pool_off + (long long)(pid - L.pid_base) * L.stride;
    const long long vs = (long long)L.full * L.full;
    const long long off = (long long)(y + NG) * L.full + (x + NG);
    const double rho = P[off], mx = P[vs + off], my = P[2 * vs + off], E = P[3 * vs + off];
    const double ux = mx / rho, uy = my / rho;
    double ke = mx * ux;
    ke = ke + my * uy;
    ke = 0.5 * ke;
    const double pr = m.gm1 * (E - ke);
    const double f[4] = {rho, ux, uy, pr};
    unsigned short* o = X + ((long long)b * P0 + p) * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double z = (f[c] - (double)norm.mean[c]) * (double)norm.istd[c];
      o[c] = f2bf((float)z);
    }
  }
}

// ---------------------------------------------------------------------------
// fused forward of one patch per block; activations in LDS
// ---------------------------------------------------------------------------
// A block per patch: more waves shorten its latency while a plane has blocks of
// 16 pixels for them (25 and 21 of them at edge 16, 9 and 7 at edge 8).
// With 4 waves, weights gathered by every wave from global memory and 16-wide K
// chunks: 256 patches of edge 16 12.2 us, 4096 70; 7.2 and 40 now.
constexpr int FWD_THREADS = 1024;
static int fwd_threads(int n) { return n > 8 ? FWD_THREADS : 512; }

// p / w for the pixel indices of a plane of edge w <= 38 (p < w^2) by one
// product: m = ceil(2^16 / w) exceeds 2^16 / w by less than 1, so the product
// exceeds 2^16 p / w by less than p < 1444, below the 2^16 / w >= 1724 that
// would change the quotient.  p m fits 32 bits.
struct PixelDiv {
  unsigned m;
  __device__ __forceinline__ explicit PixelDiv(int w) : m(65535u / (unsigned)w + 1u) {}
  __device__ __forceinline__ int operator()(int p) const { return (int)(((unsigned)p * m) >> 16); }
};

// layer-1 B operand (weights) for k-chunk kc: k = (tap, channel), tap = 4 kc +
// kq; read in any case (no branch around the loads), zero past the last tap
__device__ __forceinline__ s4 w1_operand(const unsigned short* __restrict__ W, int j, int kq, int kc) {
  const int tap = 4 * kc + kq;
  const unsigned short* w = W + j * 36 + (tap < 9 ? tap : 8);  // W1 layout [o][c][tap], o = j
  const s4 r = pack4((short)w[0], (short)w[9], (short)w[18], (short)w[27]);
  return tap < 9 ? r : zero4();
}

// Layer 2 takes K chunks of 32: 2 taps x 16 channels, a lane's 8 values being
// channels 8 (kq % 2) .. of the pixel at tap 2 kc + kq / 2 (one 16-byte read).
// Its weights in LDS as B operands: [10 taps][16 columns][16 K channels], tap 9
// zero.
constexpr int KC2 = 5;
constexpr int OPS2 = 2 * KC2 * 16 * 16;

// column j, K channel k and tap t from w[(j SJ + k SK) 9 + t], by the block
template <int SJ, int SK>
__device__ __forceinline__ void stage_operands(unsigned short* ops, const unsigned short* w) {
  for (int t = threadIdx.x; t < OPS2; t += blockDim.x) {
    const int k = t & 15, j = (t >> 4) & 15, tap = t >> 8;
    ops[t] = tap < 9 ? w[(j * SJ + k * SK) * 9 + tap] : (unsigned short)0;
  }
}

// One 16-pixel block of layer 2 (or, FLIP, of its data gradient): `pixel` is
// this lane's pixel at tap 0 in a plane of width wi; FLIP reads backwards.
template <bool FLIP>
struct Conv2 {
  u4 w[KC2];
  int off[KC2];
  bool last;  // the lane has a tap in the last chunk
  __device__ __forceinline__ Conv2(const unsigned short* ops, int wi, int j, int kq)
      : last(kq < 2) {
#pragma unroll
    for (int kc = 0; kc < KC2; ++kc) {
      const int tap = 2 * kc + (kq >> 1), t = min(tap, 8);
      w[kc] = reinterpret_cast<const u4*>(ops)[(tap * 16 + j) * 2 + (kq & 1)];
      const int o = ((t / 3) * wi + t % 3) * 16;
      off[kc] = (FLIP ? -o : o) + 8 * (kq & 1);
    }
  }
  __device__ __forceinline__ f4 operator()(const unsigned short* pixel) const {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KC2; ++kc) {
      u4 a = *reinterpret_cast<const u4*>(pixel + off[kc]);
      if (kc == KC2 - 1 && !last) a = u4{0u, 0u, 0u, 0u};
      acc = mfma32(a, w[kc], acc);
    }
    return acc;
  }
};

// conv 3x3 valid, 16 output channels, from an HWC LDS input of width wi and
// CI channels (4 or 16) to an HWC LDS output of width wo = wi - 2 (bias, ReLU,
// BF16); rows of 16 output pixels per MFMA tile.  W: layer 1 as stored, layer 2
// as staged operands.
template <int CI>
__device__ __forceinline__ void conv16(const unsigned short* __restrict__ in, int wi,
                                       unsigned short* __restrict__ out,
                                       const unsigned short* __restrict__ W,
                                       const float* __restrict__ bias) {
  const int wo = wi - 2;
  const PixelDiv dv(wo);
  const int P = wo * wo;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  const int i = lane & 15, kq = lane >> 4;
  const float bcol = bias[i];  // D column j = lane % 16
  const int nblk = (P + 15) / 16;
  // D[i'][j]: j = lane % 16, i' = 4 kq + e -> pixel 16 blk + 4 kq + e
  auto store = [&](int blk, const f4& acc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = 16 * blk + 4 * kq + e;
      if (q < P) {
        float v = acc[e] + bcol;
        v = v > 0.f ? v : 0.f;
        out[q * 16 + i] = f2bf_hw(v);
      }
    }
  };
  // A rows: output pixel p = 16 blk + i (clamped for the tail), at tap 0
  auto pixel = [&](int blk) {
    const int p = 16 * blk + i, pc = p < P ? p : P - 1;
    const int py = dv(pc);
    return in + (py * wi + pc - py * wo) * CI;
  };
  if constexpr (CI == 4) {
    s4 bop[3];  // 3 chunks of 16: 4 taps x 4 channels
    int off[3];
#pragma unroll
    for (int kc = 0; kc < 3; ++kc) {
      const int t = min(4 * kc + kq, 8);
      bop[kc] = w1_operand(W, i, kq, kc);
      off[kc] = ((t / 3) * wi + t % 3) * 4;
    }
    for (int blk = wave; blk < nblk; blk += nw) {
      const unsigned short* at = pixel(blk);
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 3; ++kc) {
        s4 a = load4(at + off[kc]);
        if (4 * kc + kq >= 9) a = zero4();
        acc = mfma(a, bop[kc], acc);
      }
      store(blk, acc);
    }
  } else {
    const Conv2<false> conv(W, wi, i, kq);
    for (int blk = wave; blk < nblk; blk += nw) store(blk, conv(pixel(blk)));
  }
}

// LDS of the forward kernel (bytes)
struct FwdLds {
  int a1, a2, w1, w2, w3, total;
  __host__ __device__ explicit FwdLds(int n) {
    const int P0 = (n + 6) * (n + 6), P1 = (n + 4) * (n + 4), P2 = (n + 2) * (n + 2);
    a1 = (P0 * 4 * 2 + 15) / 16 * 16;
    a2 = a1 + P1 * 16 * 2;
    w1 = a2 + P2 * 16 * 2;
    w2 = w1 + 16 * 4 * 9 * 2;
    w3 = w2 + OPS2 * 2;
    total = w3 + 144 * 4;
  }
};

__global__ __launch_bounds__(FWD_THREADS) void k_cnn_fwd(int count, int n,
                                                         const unsigned short* __restrict__ X,
                                                         const unsigned short* __restrict__ Wb,
                                                         const float* __restrict__ params,
                                                         float* __restrict__ Z) {
  extern __shared__ __align__(16) unsigned char fwd_smem[];
  const int b = blockIdx.x;
  if (b >= count) return;
  const FwdLds S(n);
  const int w0 = n + 6, w1 = n + 4, w2 = n + 2;
  const int P0 = w0 * w0;
  unsigned short* sx = (unsigned short*)fwd_smem;           // P0 x 4
  unsigned short* s1 = (unsigned short*)(fwd_smem + S.a1);  // P1 x 16
  unsigned short* s2 = (unsigned short*)(fwd_smem + S.a2);  // P2 x 16
  unsigned short* W1 = (unsigned short*)(fwd_smem + S.w1);
  unsigned short* W2 = (unsigned short*)(fwd_smem + S.w2);
  float* W3 = (float*)(fwd_smem + S.w3);                    // 9 taps x 16
  const unsigned short* xg = X + (long long)b * P0 * 4;
  for (int t = threadIdx.x; t < P0; t += blockDim.x)
    *reinterpret_cast<uint2*>(sx + 4 * t) = *reinterpret_cast<const uint2*>(xg + 4 * t);
  for (int t = threadIdx.x; t < 576; t += blockDim.x) W1[t] = Wb[CNN_W1 + t];
  stage_operands<16, 1>(W2, Wb + CNN_W2);
  for (int t = threadIdx.x; t < 144; t += blockDim.x) W3[(t % 9) * 16 + t / 9] = bf2f(Wb[CNN_W3 + t]);
  __syncthreads();
  conv16<4>(sx, w0, s1, W1, params + CNN_B1);
  __syncthreads();
  conv16<16>(s1, w1, s2, W2, params + CNN_B2);
  __syncthreads();
  // layer 3 (16 -> 1) on the VALU
  const int P3 = n * n;
  const PixelDiv div3(n);
  const float b3 = params[CNN_B3];
  for (int p = threadIdx.x; p < P3; p += blockDim.x) {
    const int py = div3(p), px = p - py * n;
    float acc = 0.f;
#pragma unroll 1  // all 9 taps' weights do not fit the registers
    for (int tap = 0; tap < 9; ++tap) {
      const unsigned short* at = s2 + ((py + tap / 3) * w2 + px + tap % 3) * 16;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u4 a = *reinterpret_cast<const u4*>(at + 8 * h);
        const float4 wa = *reinterpret_cast<const float4*>(W3 + tap * 16 + 8 * h);
        const float4 wb = *reinterpret_cast<const float4*>(W3 + tap * 16 + 8 * h + 4);
        const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
        for (int c = 0; c < 8; ++c)
          acc += bf2f((unsigned short)(a[c >> 1] >> (16 * (c & 1)))) * w[c];
      }
    }
    Z[(long long)b * P3 + p] = acc + b3;
  }
}

// ---------------------------------------------------------------------------
// training: forward, loss and backward of one patch per block, the per-patch
// parameter gradients and loss to global memory
// ---------------------------------------------------------------------------
// A batch is tens of patches, so a launch is one patch's latency: 16 waves per
// patch, every activation and gradient of it in LDS from the input to the
// gradients (no activation goes through memory), the reductions spread over
// the waves as MFMA chains.  It replaces a forward, a loss and a backward
// launch (with 8 waves and serial per-parameter loops): 11.5 + 4.5 + 68.9 us
// for 64 patches of edge 16; 20.4 us with 16-wide K chunks, 18.5
// with a fixed share of dz1 per wave, 17.9 now.
constexpr int TRAIN_THREADS = 1024;
constexpr int TRAIN_WAVES = TRAIN_THREADS / 64;

// LDS of the training kernel (bytes).  dz1 (whole blocks of 16 pixels) takes
// the place of the second activation, the logit gradients and the FP32 copy of
// W3, which are read before it is written; dz2 is stored with a border of two
// zero pixels, so that the data gradient reads it without bounds checks.
struct TrainLds {
  int x, a1, a2, g, w3, dz1, dz2, red, w1, w2, w2f, next, total;
  __host__ __device__ explicit TrainLds(int n) {
    const int P0 = (n + 6) * (n + 6), P1 = (n + 4) * (n + 4), P2 = (n + 2) * (n + 2), P3 = n * n;
    x = 0;
    a1 = x + (P0 * 4 * 2 + 15) / 16 * 16;
    a2 = dz1 = a1 + P1 * 16 * 2;
    g = a2 + P2 * 16 * 2;
    w3 = g + P3 * 4;
    const int after_a = w3 + 144 * 4, after_b = dz1 + (P1 + 15) / 16 * 16 * 32;
    dz2 = ((after_a > after_b ? after_a : after_b) + 15) / 16 * 16;
    red = dz2 + P1Z(n) * 16 * 2;
    w2 = dz2;  // until layer 2 is done
    w1 = red + 12 * 256 * 4;
    w2f = w1 + 16 * 4 * 9 * 2;
    next = w2f + OPS2 * 2;  // block counter of dz1
    total = next + 16;
  }
  static __host__ __device__ int P1Z(int n) { return (n + 6) * (n + 6); }  // dz2 with its border
};

__device__ __forceinline__ float softplus_tail(float z) { return log1pf(expf(-fabsf(z))); }

__global__ __launch_bounds__(TRAIN_THREADS) void k_cnn_train(
    int count, int n, const unsigned short* __restrict__ X, const uint8_t* __restrict__ Y,
    const unsigned short* __restrict__ Wg, const float* __restrict__ params, float pos_weight,
    float inv_total, float* __restrict__ partials, float* __restrict__ loss_part) {
  extern __shared__ __align__(16) unsigned char train_smem[];
  const int b = blockIdx.x;
  if (b >= count) return;
  const TrainLds S(n);
  unsigned short* x = (unsigned short*)(train_smem + S.x);      // P0 x 4
  unsigned short* a1 = (unsigned short*)(train_smem + S.a1);    // P1 x 16
  unsigned short* a2 = (unsigned short*)(train_smem + S.a2);    // P2 x 16
  float* g = (float*)(train_smem + S.g);                        // P3
  float* w3 = (float*)(train_smem + S.w3);                      // 9 taps x 16
  unsigned short* dz1 = (unsigned short*)(train_smem + S.dz1);  // P1 x 16
  unsigned short* dz2 = (unsigned short*)(train_smem + S.dz2);  // (w2 + 4)^2 x 16
  float* red = (float*)(train_smem + S.red);
  unsigned short* W1 = (unsigned short*)(train_smem + S.w1);
  unsigned short* W2 = (unsigned short*)(train_smem + S.w2);
  unsigned short* W2f = (unsigned short*)(train_smem + S.w2f);
  int* next = (int*)(train_smem + S.next);
  const int w0 = n + 6, w1 = n + 4, w2 = n + 2, wz = n + 6;
  const int P0 = w0 * w0, P1 = w1 * w1, P2 = w2 * w2, P3 = n * n;
  const PixelDiv div1(w1), div2(w2), div3(n);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, kq = lane >> 4;
  float* part = partials + (long long)b * CNN_NPARAM;

  {
    const uint2* gx = reinterpret_cast<const uint2*>(X + (long long)b * P0 * 4);
    for (int t = tid; t < P0; t += TRAIN_THREADS) reinterpret_cast<uint2*>(x)[t] = gx[t];
    for (int t = tid; t < 576; t += TRAIN_THREADS) W1[t] = Wg[CNN_W1 + t];
    stage_operands<16, 1>(W2, Wg + CNN_W2);
    stage_operands<1, 16>(W2f, Wg + CNN_W2);
    if (tid == 0) next[0] = 0;
    if (tid < 144) w3[(tid % 9) * 16 + tid / 9] = bf2f(Wg[CNN_W3 + tid]);
  }
  __syncthreads();
  conv16<4>(x, w0, a1, W1, params + CNN_B1);
  __syncthreads();
  conv16<16>(a1, w1, a2, W2, params + CNN_B2);
  __syncthreads();
  for (int t = tid; t < wz * wz * 2; t += TRAIN_THREADS)
    reinterpret_cast<uint4*>(dz2)[t] = uint4{0u, 0u, 0u, 0u};

  // --- layer 3 and the loss: 4 lanes per pixel, 4 channels each; the logit
  // gradient of the mean over all cells
  {
    const float b3 = params[CNN_B3];
    const uint8_t* y = Y + (long long)b * P3;
    const int cq = 4 * (lane & 3);
    float loss = 0.f;
    for (int t = tid; t < 4 * P3; t += TRAIN_THREADS) {
      const int p = t >> 2, py = div3(p), px = p - py * n;
      float acc = 0.f;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const s4 a = load4(a2 + ((py + tap / 3) * w2 + px + tap % 3) * 16 + cq);
        const float4 w = *reinterpret_cast<const float4*>(w3 + tap * 16 + cq);
        acc += bf2f((unsigned short)a.x) * w.x;
        acc += bf2f((unsigned short)a.y) * w.y;
        acc += bf2f((unsigned short)a.z) * w.z;
        acc += bf2f((unsigned short)a.w) * w.w;
      }
      acc += __shfl_xor(acc, 1);
      acc += __shfl_xor(acc, 2);
      if ((lane & 3) == 0) {
        const float z = acc + b3;
        const float yv = y[p] ? 1.f : 0.f;
        const float tail = softplus_tail(z);
        loss += pos_weight * yv * (fmaxf(-z, 0.f) + tail) + (1.f - yv) * (fmaxf(z, 0.f) + tail);
        const float s = 1.f / (1.f + expf(-z));
        g[p] = (pos_weight * yv * (s - 1.f) + (1.f - yv) * s) * inv_total;
      }
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
  // every 16th pixel, a lane one tap and 4 channels (36 lanes; lane 36 sums
  // g); partial sums per wave into red
  if (lane <= 36) {
    const int tap = lane >> 2, cq = 4 * (lane & 3);
    const int shift = lane < 36 ? ((tap / 3) * w2 + tap % 3) * 16 + cq : 0;
    float acc[4] = {0.f, 0.f, 0.f, 0.f}, gs = 0.f;
#pragma unroll 4
    for (int p = wave; p < P3; p += TRAIN_WAVES) {
      const int py = div3(p), px = p - py * n;
      const float gv = g[p];
      const s4 a = load4(a2 + (py * w2 + px) * 16 + shift);
      gs += gv;
      acc[0] += bf2f((unsigned short)a.x) * gv;
      acc[1] += bf2f((unsigned short)a.y) * gv;
      acc[2] += bf2f((unsigned short)a.z) * gv;
      acc[3] += bf2f((unsigned short)a.w) * gv;
    }
    if (lane < 36) {
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave * 145 + (cq + e) * 9 + tap] = acc[e];
    } else {
      red[wave * 145 + 144] = gs;
    }
  }
  // --- dz2 = relu'(z2) * (W3 (x) g) on the P2 grid, 4 channels per item
  for (int t = tid; t < 4 * P2; t += TRAIN_THREADS) {
    const int q = t >> 2, cq = 4 * (t & 3);
    const int qy = div2(q), qx = q - qy * w2;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      // read in any case (no branch around the loads), zero outside
      const int py = qy - tap / 3, px = qx - tap % 3;
      const bool in = (unsigned)py < (unsigned)n && (unsigned)px < (unsigned)n;
      const float gr = g[in ? py * n + px : 0];
      const float gv = in ? gr : 0.f;
      const float4 w = *reinterpret_cast<const float4*>(w3 + tap * 16 + cq);
      acc[0] += w.x * gv;
      acc[1] += w.y * gv;
      acc[2] += w.z * gv;
      acc[3] += w.w * gv;
    }
    const s4 on = load4(a2 + q * 16 + cq);  // a2 = relu(z2) in BF16: nonzero iff z2 > 0
    uint2 o;
    o.x = f2bf_hw(on.x ? acc[0] : 0.f) | ((unsigned)f2bf_hw(on.y ? acc[1] : 0.f) << 16);
    o.y = f2bf_hw(on.z ? acc[2] : 0.f) | ((unsigned)f2bf_hw(on.w ? acc[3] : 0.f) << 16);
    *reinterpret_cast<uint2*>(dz2 + ((qy + 2) * wz + qx + 2) * 16 + cq) = o;
  }
  __syncthreads();

  if (tid < 145) {
    float s = 0.f;
    for (int k = 0; k < TRAIN_WAVES; ++k) s += red[k * 145 + tid];
    part[CNN_W3 + tid] = s;  // db3 follows W3
  }
  // --- dW2[o][c][tap] = sum_p dz2[p][o] a1[p + tap][c]: D[i = o][j = c], K =
  // pixels, a tap per wave; db2 by the wave after them
  static_assert(CNN_B3 == CNN_W3 + 144 && TRAIN_WAVES >= 10, "a wave per tap and one for db2");
  // this lane's row (of the 4 of its K group) and 4 columns in transposed reads
  const int row = 4 * kq + (i16 >> 2), col = 4 * (i16 & 3);
  if (wave < 9) {
    const int shift = ((wave / 3) * w1 + wave % 3) * 16 + col;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < P2; p0 += 32) {
      s4 a[2], bb[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int p = p0 + 16 * h + row;
        // past the last pixel: a border pixel of dz2 (zero)
        const bool in = p < P2;
        const int py = div2(in ? p : 0), px = (in ? p : 0) - py * w2;
        a[h] = load4_tr(dz2 + (in ? ((py + 2) * wz + px + 2) * 16 : 0) + col);
        bb[h] = load4_tr(a1 + (py * w1 + px) * 16 + shift);
      }
      acc = mfma32(join(a[0], a[1]), join(bb[0], bb[1]), acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      part[CNN_W2 + ((4 * kq + e) * 16 + i16) * 9 + wave] = acc[e];
  } else if (wave == 9) {
    float s = 0.f;
#pragma unroll 4
    for (int p = kq; p < P2; p += 4) {
      const int py = div2(p), px = p - py * w2;
      s += bf2f(dz2[((py + 2) * wz + px + 2) * 16 + i16]);
    }
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (kq == 0) part[CNN_B2 + i16] = s;
  }
  // --- dz1[q][c] = relu'(z1) sum_tap sum_o W2[o][c][tap] dz2[q - tap][o]:
  // D[i = pixel][j = c], stored like the activations in whole blocks of 16 pixels
  {
    const Conv2<true> conv(W2f, wz, i16, kq);
    const int nblk = (P1 + 15) / 16;
    // blocks as the waves come: those with a tap above arrive last
    for (int blk = take(next); blk < nblk; blk = take(next)) {
      const int p = 16 * blk + i16;
      const int pc = p < P1 ? p : P1 - 1;
      const int qy = div1(pc), qx = pc - qy * w1;
      const f4 acc = conv(dz2 + ((qy + 2) * wz + qx + 2) * 16);
      // the rows past the last pixel of the last block are zero
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = 16 * blk + 4 * kq + e;
        const bool on = q < P1 && a1[q * 16 + i16] != 0;
        dz1[q * 16 + i16] = f2bf_hw(on ? acc[e] : 0.f);
      }
    }
  }
  __syncthreads();

  // --- dW1[o][c][tap] = sum_p dz1[p][o] x[p + tap][c]: D[i = o][j = k'] with
  // k' = 4 tap' + c over 3 chunks (taps 4 kc .. 4 kc + 3), the pixels in 4
  // parts (12 waves); db1 by the wave after them
  if (wave < 12) {
    const int kc = wave % 3, quarter = wave / 3;
    const int tap = 4 * kc + (i16 & 3);  // taps 9 .. 11 do not exist: columns not used
    const int shift = tap < 9 ? ((tap / 3) * w0 + tap % 3) * 4 : 0;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    auto step = [&](int p0, s4& a, s4& v) {
      const int p = p0 + row, pc = p < P1 ? p : 0;
      const int py = div1(pc), px = pc - py * w1;
      a = load4_tr(dz1 + p * 16 + col);
      v = load4_tr(x + (py * w0 + px) * 4 + shift);
    };
    int p0 = 16 * quarter;
    s4 a, v, a2, v2;
    for (; p0 + 64 < P1; p0 += 128) {
      step(p0, a, v);
      step(p0 + 64, a2, v2);
      acc = mfma32(join(a, a2), join(v, v2), acc);
    }
    if (p0 < P1) {
      step(p0, a, v);
      acc = mfma(a, v, acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave * 256 + (4 * kq + e) * 16 + i16] = acc[e];
  } else if (wave == 12) {
    float s = 0.f;
#pragma unroll 4
    for (int q = kq; q < P1; q += 4) s += bf2f(dz1[q * 16 + i16]);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (kq == 0) part[CNN_B1 + i16] = s;
  }
  __syncthreads();
  if (tid < 576) {
    // parameter (o, c, tap) is element (o, 4 tap + c) of the chunk matrices
    const int o = tid / 36, c = (tid / 9) % 4, tap = tid % 9;
    const int kp = 4 * tap + c, at = (kp >> 4) * 256 + o * 16 + (kp & 15);
    part[CNN_W1 + tid] = ((red[at] + red[at + 768]) + red[at + 1536]) + red[at + 2304];
  }
}

// ---------------------------------------------------------------------------
// parameter update: the sum of the per-tile gradients (fixed order: a wave
// takes every 16th tile, the 16 sums are added in wave order), then Adam on
// the FP32 master weights and the BF16 copy (round to nearest even).  One
// block per 64 parameters; the block after them sums the loss.
// ---------------------------------------------------------------------------
// With one thread per parameter walking all tiles, a loss kernel of one
// serial thread, a gradient copy and a separate Adam launch the update took
// 15.9 + 13.1 + 5.3 + 4.7 us for 64 tiles; one 4.7 us launch now.
constexpr int UPDATE_THREADS = 1024;

__global__ __launch_bounds__(UPDATE_THREADS) void k_cnn_update(
    const float* __restrict__ partials, const float* __restrict__ loss_part, int count, int np,
    float* __restrict__ grads, float* __restrict__ loss, int adam, float* __restrict__ params,
    float* __restrict__ m, float* __restrict__ v, float lr, float c1, float c2,
    unsigned short* __restrict__ Wb) {
  __shared__ float red[UPDATE_THREADS];
  constexpr int NW = UPDATE_THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == gridDim.x - 1) {
    float s = 0.f;
    for (int b = tid; b < count; b += UPDATE_THREADS) s += loss_part[b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
      for (int k = 0; k < NW; ++k) t += red[k];
      loss[0] = t;
    }
    return;
  }
  const int k = blockIdx.x * 64 + lane;
  float s = 0.f;
  if (k < np) {
#pragma unroll 4
    for (int b = wave; b < count; b += NW) s += partials[(long long)b * np + k];
  }
  red[tid] = s;
  __syncthreads();
  if (wave > 0 || k >= np) return;
  float g = red[lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) g += red[64 * w + lane];
  if (grads) grads[k] = g;
  if (!adam) return;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mk = b1 * m[k] + (1.f - b1) * g;
  const float vk = b2 * v[k] + (1.f - b2) * g * g;
  m[k] = mk;
  v[k] = vk;
  const float mh = mk / c1, vh = vk / c2;
  const float p = params[k] - lr * mh / (sqrtf(vh) + eps);
  params[k] = p;
  Wb[k] = f2bf(p);
}

__global__ void k_cnn_to_bf16(const float* __restrict__ params, int np, unsigned short* __restrict__ Wb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < np) Wb[k] = f2bf(params[k]);
}

// per-patch refine request: any logit above the threshold
__global__ __launch_bounds__(256) void k_cnn_requests(int count, int n, const float* __restrict__ Z,
                                                      const int* __restrict__ pids, float zt,
                                                      uint8_t* __restrict__ flag) {
  const int b = blockIdx.x;
  if (b >= count) return;
  int any = 0;
  for (int p = threadIdx.x; p < n * n; p += blockDim.x) any |= Z[(long long)b * n * n + p] > zt;
  any = __syncthreads_or(any);
  if (threadIdx.x == 0) flag[pids[b]] = any ? 1 : 0;
}

// MFMA lane-layout check: D = A B for 16x16 BF16 matrices (row-major inputs)
__global__ void k_mfma_selftest(const unsigned short* __restrict__ A, const unsigned short* __restrict__ B,
                                float* __restrict__ D) {
  const int l = threadIdx.x;
  const int i = l & 15, kq = l >> 4;
  s4 a, b;
  a.x = (short)A[i * 16 + 4 * kq + 0];
  a.y = (short)A[i * 16 + 4 * kq + 1];
  a.z = (short)A[i * 16 + 4 * kq + 2];
  a.w = (short)A[i * 16 + 4 * kq + 3];
  b.x = (short)B[(4 * kq + 0) * 16 + i];
  b.y = (short)B[(4 * kq + 1) * 16 + i];
  b.z = (short)B[(4 * kq + 2) * 16 + i];
  b.w = (short)B[(4 * kq + 3) * 16 + i];
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  acc = mfma(a, b, acc);
  for (int e = 0; e < 4; ++e) D[(4 * kq + e) * 16 + i] = acc[e];
}

}  // namespace

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
size_t Cnn::fwd_lds(int n) { return FwdLds(n).total; }

void Cnn::gather(const DevMesh& m, const double* U, const int* pids, int count, int n,
                 const CnnNorm& norm, unsigned short* X, hipStream_t s) {
  if (count <= 0) return;
  const long long total = (long long)count * (n + 6) * (n + 6);
  const int blocks = (int)std::min<long long>((total + 255) / 256, 65535);
  hipLaunchKernelGGL(k_cnn_gather, dim3(blocks), dim3(256), 0, s, m, U, pids, count, n, norm, X);
}

static void allow_large_lds() {
  static bool done = false;
  if (done) return;
  done = true;
  (void)hipFuncSetAttribute((const void*)k_cnn_fwd, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
  (void)hipFuncSetAttribute((const void*)k_cnn_train, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
}

void Cnn::forward(int count, int n, const unsigned short* X, const unsigned short* Wb,
                  const float* params, float* Z, hipStream_t s) {
  if (count <= 0) return;
  allow_large_lds();
  hipLaunchKernelGGL(k_cnn_fwd, dim3(count), dim3(fwd_threads(n)), fwd_lds(n), s, count, n, X, Wb,
                     params, Z);
}

void Cnn::train(int count, int n, const unsigned short* X, const uint8_t* Y,
                const unsigned short* Wb, const float* params, float pos_weight, float* partials,
                float* loss_part, hipStream_t s) {
  if (count <= 0) return;
  allow_large_lds();
  const float inv_total = 1.0f / (float)((long long)count * n * n);
  hipLaunchKernelGGL(k_cnn_train, dim3(count), dim3(TRAIN_THREADS), TrainLds(n).total, s, count, n,
                     X, Y, Wb, params, pos_weight, inv_total, partials, loss_part);
}

void Cnn::update(const float* partials, const float* loss_part, int count, int np, float* grads,
                 float* loss, float* params, float* m, float* v, float lr, int t,
                 unsigned short* Wb, hipStream_t s) {
  const int adam = lr > 0.f ? 1 : 0;
  const float c1 = adam ? 1.f - powf(0.9f, (float)t) : 1.f;
  const float c2 = adam ? 1.f - powf(0.999f, (float)t) : 1.f;
  hipLaunchKernelGGL(k_cnn_update, dim3((np + 63) / 64 + 1), dim3(UPDATE_THREADS), 0, s, partials,
                     loss_part, count, np, grads, loss, adam, params, m, v, lr, c1, c2, Wb);
}

void Cnn::to_bf16(const float* params, int np, unsigned short* Wb, hipStream_t s) {
  hipLaunchKernelGGL(k_cnn_to_bf16, dim3((np + 255) / 256), dim3(256), 0, s, params, np, Wb);
}

void Cnn::requests(int count, int n, const float* Z, const int* pids, float zt, uint8_t* flag,
                   hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_cnn_requests, dim3(count), dim3(256), 0, s, count, n, Z, pids, zt, flag);
}

void Cnn::mfma_selftest(const unsigned short* A, const unsigned short* B, float* D, hipStream_t s) {
  hipLaunchKernelGGL(k_mfma_selftest, dim3(1), dim3(64), 0, s, A, B, D);
}

}  // namespace amr

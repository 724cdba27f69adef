// Kernels of the learned initial guess (see bs_mlp.hpp for the layouts).
#pragma once
#include <type_traits>

#include "bs_mlp.hpp"

namespace bs {
namespace mlp {

constexpr int kLdZ = 192 + kPad;   // Z tile row stride (features padded to 192 at most)
constexpr int kLdH = kH + kPad;    // hidden tile row stride
constexpr int kLdY = 64 + kPad;    // output-gradient tile row stride
constexpr int kNetWG = 512;        // eight waves: wave w owns hidden columns 32w .. 32w+31

// B fragments of a layer for CB column blocks from column c0, all KS k-steps
// (K of them used), straight from global memory into registers.
template <int KS, int CB>
__device__ __forceinline__ void load_w(bf16x8 (&b)[KS][CB], const uint16_t* __restrict__ Bt, int ldb,
                                       int c0, int K) {
  const int l = threadIdx.x & 63, r16 = l & 15, q = l >> 4;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    if (32 * ks < K) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        b[ks][cb] = frag(Bt + (size_t)(c0 + 16 * cb + r16) * ldb + 32 * ks + 8 * q);
    }
}

// acc[rb][cb] += A[16 rb .. +16][0..K) * b: A in LDS, row-major, stride lda, the
// k-steps in increasing order.  A k-step's reads are issued ahead of the
// products of the one before it, and no further ahead (the empty asm): all of
// them at once push the weights out of the registers.
template <int RB, int KS, int CB>
__device__ __forceinline__ void gemm_reg(floatx4 (&acc)[RB][CB], const uint16_t* A, int lda,
                                         const bf16x8 (&b)[KS][CB], int K) {
  const int l = threadIdx.x & 63, r16 = l & 15, q = l >> 4;
  const uint16_t* at = A + r16 * lda + 8 * q;
  bf16x8 a[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) a[rb] = frag(at + 16 * rb * lda);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    if (32 * ks < K) {
      bf16x8 next[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        next[rb] = ks + 1 < KS && 32 * (ks + 1) < K ? frag(at + 16 * rb * lda + 32 * (ks + 1)) : a[rb];
      __asm__ volatile("" ::: "memory");
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], b[ks][cb], acc[rb][cb], 0, 0, 0);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) a[rb] = next[rb];
    }
}

// H = relu(acc + bias) of a hidden layer into LDS, rounded to BF16; h keeps the
// lane's own values ([rb][cb][i] for row 16 rb + 4 q + i).
template <int RB>
__device__ __forceinline__ void relu_out(uint16_t (&h)[RB][2][4], const floatx4 (&acc)[RB][2],
                                         const float (&bias)[2], uint16_t* H, int c0) {
  const int l = threadIdx.x & 63, r16 = l & 15, q = l >> 4;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h[rb][cb][i] = to_bf16(fmaxf(acc[rb][cb][i] + bias[cb], 0.f));
        H[(16 * rb + 4 * q + i) * kLdH + c0 + 16 * cb + r16] = h[rb][cb][i];
      }
}

// Row blocks of the output layer that a wave takes beside its column block
// 16 (w & 3): the eight waves split a tile's row blocks in two halves.
template <int RB>
constexpr int kOutRB = RB >= 2 ? RB / 2 : 1;

// Inference (kInfer: features from the batch itself, x0 out) and forward
// (kForward: raw FP32 features, network outputs out).  Eight waves, one
// workgroup per compute unit, walk over tiles of 16 RB systems with the
// weights held on chip: W1 and W2 as B fragments in registers (28 fragments,
// 112 registers a lane), W3 in LDS.  Reading the weights from L2 for every tile
// (240 KB per 64 systems) and waiting for the inputs of a tile before its
// products left the matrix cores idle 95 % of the time: 2^16 systems of 54 rows
// took 93 us with their diagonals given, 164 with the diagonals gathered from
// the values; now 48 and 116.  A tile's inputs are loaded into registers while
// the tile before it is computed.  The gather touches every line of the values
// (0.55 GB, 5 TB/s with the rest, the rate of a large copy).
enum Mode { kInfer = 0, kForward = 1 };

template <int MODE, int RB>
__global__ __launch_bounds__(kNetWG) __attribute__((amdgpu_waves_per_eu(2)))
void k_mlp_forward(const Net net, const Src src, float* y_out, int64_t M, int64_t tiles) {
  constexpr int T = 16 * RB, ROWS = T / 8, ORB = kOutRB<RB>;
  __shared__ __align__(16) uint16_t sZ[T * kLdZ], sH1[T * kLdH], sH2[T * kLdH], sW3[64 * kLdH];
  __shared__ double sMu[192], sSd[192];  // feature means, spreads (kInfer: their reciprocals)
  const int tid = threadIdx.x, l = tid & 63, r16 = l & 15, q = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // rows and columns of a wave: scalar
  const int n = net.n, F = net.F, Fp = net.Fp, O = net.O, Op = net.Op;

  // this wave's rows of the first tile, and its inputs: lane l takes unknown l
  // (kInfer) or features l, l+64, l+128 (kForward)
  using In = typename std::conditional<MODE == kInfer, double, float>::type;
  In in[3][ROWS];
  const bool jok = l < n;
  const int dpos = (MODE == kInfer && !src.diag && jok) ? src.diag_pos[l] : -1;
  auto load = [&](int64_t tile) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int64_t m = tile * T + ROWS * w + i;
#pragma unroll
      for (int t = 0; t < 3; ++t) in[t][i] = 0;
      if (m < M) {
        if constexpr (MODE == kInfer) {
          if (jok) {
            if (src.diag) in[0][i] = src.diag[m * n + l];
            else if (dpos >= 0) in[0][i] = src.values[m * src.nnz + dpos];
            in[1][i] = src.b[m * n + l];
            in[2][i] = src.x_prev[m * n + l];
          }
        } else {
          const int64_t s = src.rows ? (int64_t)src.rows[m] : m;
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (l + 64 * t < F) in[t][i] = src.feat[s * F + l + 64 * t];
        }
      }
    }
  };
  load(blockIdx.x);

  bf16x8 w1[6][2], w2[8][2];
  load_w(w1, net.w1t, Fp, 32 * w, Fp);
  load_w(w2, net.w2t, kH, 32 * w, kH);
  for (int e = tid; e < Op * (kH / 8); e += kNetWG) {
    const int r = e / (kH / 8), c = e - r * (kH / 8);
    *reinterpret_cast<uint4*>(sW3 + r * kLdH + 8 * c) =
        *reinterpret_cast<const uint4*>(net.w3t + (size_t)r * kH + 8 * c);
  }
  // columns past the features stay zero
  for (int e = tid; e < T * kLdZ / 8; e += kNetWG) reinterpret_cast<uint4*>(sZ)[e] = uint4{0, 0, 0, 0};
  if (tid < F) {
    sMu[tid] = net.mu_f[tid];
    sSd[tid] = MODE == kInfer ? 1.0 / net.sd_f[tid] : net.sd_f[tid];
  }
  float bias1[2], bias2[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    bias1[cb] = net.b1[32 * w + 16 * cb + r16];
    bias2[cb] = net.b2[32 * w + 16 * cb + r16];
  }
  const int c3 = 16 * (w & 3), ocol = c3 + r16, orb = ORB * (w >> 2);
  const bool out = c3 < Op && orb < RB, cok = out && ocol < O;
  const float bias3 = cok ? net.b3[ocol] : 0.f;
  const double sdd = (MODE == kInfer && cok) ? net.sd_d[ocol] : 0.0;
  __syncthreads();

  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t m0 = tile * T;
    // ---- normalised features -> BF16: feature t of this lane in each row
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int f = MODE == kInfer ? t * n + l : 64 * t + l;
      if (MODE == kInfer ? jok : f < F) {
        const double mu = sMu[f], sd = sSd[f];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
          const int row = ROWS * w + i;
          float z;
          if constexpr (MODE == kInfer) {
            const double v = t == 1 ? in[1][i] - in[2][i] : in[t][i];
            z = (float)((v - mu) * sd);
          } else {
            z = (float)(((double)in[t][i] - mu) / sd);
          }
          sZ[row * kLdZ + f] = to_bf16(m0 + row < M ? z : 0.f);
        }
      }
    }
    __syncthreads();
    if (tile + gridDim.x < tiles) load(tile + gridDim.x);
    uint16_t h[RB][2][4];
    // ---- layer 1: H1 = relu(Z W1 + b1)
    {
      floatx4 acc[RB][2];
      zero(acc);
      gemm_reg(acc, sZ, kLdZ, w1, Fp);
      relu_out<RB>(h, acc, bias1, sH1, 32 * w);
    }
    __syncthreads();
    // ---- layer 2: H2 = relu(H1 W2 + b2)
    {
      floatx4 acc[RB][2];
      zero(acc);
      gemm_reg(acc, sH1, kLdH, w2, kH);
      relu_out<RB>(h, acc, bias2, sH2, 32 * w);
    }
    __syncthreads();
    // ---- layer 3: Y = H2 W3 + b3
    if (out) {
      floatx4 acc[ORB][1];
      zero(acc);
#pragma unroll 2
      for (int ks = 0; ks < kH / 32; ++ks) {
        const bf16x8 b = frag(sW3 + (c3 + r16) * kLdH + 32 * ks + 8 * q);
#pragma unroll
        for (int rb = 0; rb < ORB; ++rb) {
          const bf16x8 a = frag(sH2 + (16 * (orb + rb) + r16) * kLdH + 32 * ks + 8 * q);
          acc[rb][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[rb][0], 0, 0, 0);
        }
      }
#pragma unroll
      for (int rb = 0; rb < ORB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t m = m0 + 16 * (orb + rb) + 4 * q + i;
          const float y = acc[rb][0][i] + bias3;
          if (cok && m < M) {
            if constexpr (MODE == kInfer) src.x0[m * n + ocol] = src.x_prev[m * n + ocol] + sdd * (double)y;
            else y_out[m * O + ocol] = y;
          }
        }
    }
  }
}

// Training: forward and backward of one tile of 16 RB samples per workgroup
// (RB = 4 when that fills the card, else 2 or 1), activations and their
// gradients written feature-major for the weight gradients.  A tile's phases
// follow one another, so its time is their latency: each layer's weights are
// loaded into registers while the layer before it runs, and a lane's column of
// a row-block pair covers eight consecutive samples (row r of block h of the
// pair is sample 8 (r / 4) + 4 h + r % 4), one 16-byte store.  64-sample tiles on
// four waves, weights read a k-step ahead and 8-byte stores took 73 us for
// 8192 samples of 54 rows (128 workgroups on 256 compute units); now 28.
template <int RB>
__device__ __forceinline__ int sample_of(int p) {  // of tile row p
  if constexpr (RB == 1) return p;
  else return (p & ~31) | (p & 12) << 1 | (p & 16) >> 2 | (p & 3);
}

// The lane's values of one column (rows 4 q + i of the row blocks rb0 ..) into a
// feature-major [column][Mp] array at the tile's first sample.
template <int RB, int NB>
__device__ __forceinline__ void store_col(uint16_t* dst, int rb0, const uint16_t (&h)[NB][4]) {
  const int q = (threadIdx.x & 63) >> 4;
  auto word = [&](int b, int i) { return (uint32_t)h[b][i] | ((uint32_t)h[b][i + 1] << 16); };
  if constexpr (RB >= 2 && NB >= 2) {
#pragma unroll
    for (int b = 0; b < NB; b += 2)
      *reinterpret_cast<uint4*>(dst + 16 * (rb0 + b) + 8 * q) =
          uint4{word(b, 0), word(b, 2), word(b + 1, 0), word(b + 1, 2)};
  } else {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      *reinterpret_cast<uint2*>(dst + sample_of<RB>(16 * (rb0 + b) + 4 * q)) = uint2{word(b, 0), word(b, 2)};
  }
}

template <int RB>
__global__ __launch_bounds__(kNetWG) __attribute__((amdgpu_waves_per_eu(2)))
void k_mlp_train(const Net net, const Src src, const Train tr, int64_t M) {
  constexpr int T = 16 * RB, ROWS = T / 8, ORB = kOutRB<RB>;
  __shared__ __align__(16) uint16_t sZ[T * kLdZ], sH1[T * kLdH], sH2[T * kLdH], sD[T * kLdH], sDY[T * kLdY];
  __shared__ float s_loss[kNetWG / 64];
  const int tid = threadIdx.x, l = tid & 63, r16 = l & 15, q = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // rows and columns of a wave: scalar
  const int64_t m0 = (int64_t)blockIdx.x * T;
  const int F = net.F, Fp = net.Fp, O = net.O, Op = net.Op;
  const int c0 = 32 * w, c3 = 16 * (w & 3), ocol = c3 + r16, orb = ORB * (w >> 2);

  bf16x8 w1[6][2], w2[8][2];
  load_w(w1, net.w1t, Fp, c0, Fp);

  // ---- raw FP32 features of the (listed) samples, normalised -> BF16
  float v[3][ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int64_t m = m0 + sample_of<RB>(ROWS * w + i);
    const int64_t s = m < M ? (src.rows ? (int64_t)src.rows[m] : m) : 0;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      v[t][i] = 0.f;
      if (m < M && l + 64 * t < F) v[t][i] = src.feat[s * F + l + 64 * t];
    }
  }
  load_w(w2, net.w2t, kH, c0, kH);
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int f = l + 64 * t;
    if (f >= Fp) continue;
    const double mu = f < F ? net.mu_f[f] : 0.0, sd = f < F ? net.sd_f[f] : 1.0;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int row = ROWS * w + i;
      const bool ok = f < F && m0 + sample_of<RB>(row) < M;
      sZ[row * kLdZ + f] = to_bf16(ok ? (float)(((double)v[t][i] - mu) / sd) : 0.f);
    }
  }
  __syncthreads();
  // Z feature-major for the first layer's weight gradient: eight samples of a
  // feature per lane and step
  for (int e = tid; e < Fp * (T / 8); e += kNetWG) {
    const int f = e / (T / 8), j = e - f * (T / 8);
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // tile rows of samples 8j+2k, 8j+2k+1
      const int b = 2 * k;
      const int p = RB == 1 ? 8 * j + b : (32 * (j >> 2) + 4 * (j & 3)) + ((b & 4) << 2) + (b & 3);
      u[k] = (uint32_t)sZ[p * kLdZ + f] | ((uint32_t)sZ[(p + 1) * kLdZ + f] << 16);
    }
    *reinterpret_cast<uint4*>(tr.zT + (size_t)f * tr.Mp + m0 + 8 * j) = uint4{u[0], u[1], u[2], u[3]};
  }

  uint16_t h[RB][2][4];
  auto store_hidden = [&](uint16_t* dstT) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      uint16_t c[RB][4];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[rb][i] = h[rb][cb][i];
      store_col<RB, RB>(dstT + (size_t)(c0 + 16 * cb + r16) * tr.Mp + m0, 0, c);
    }
  };
  // ---- layer 1: H1 = relu(Z W1 + b1)
  {
    const float bias[2] = {net.b1[c0 + r16], net.b1[c0 + 16 + r16]};
    floatx4 acc[RB][2];
    zero(acc);
    gemm_reg(acc, sZ, kLdZ, w1, Fp);
    relu_out<RB>(h, acc, bias, sH1, c0);
  }
  bf16x8 w3t[8][1], w3[2][2];
  if (c3 < Op) load_w(w3t, net.w3t, kH, c3, kH);
  load_w(w3, net.w3, Op, c0, Op);
  store_hidden(tr.h1T);
  __syncthreads();

  // ---- layer 2: H2 = relu(H1 W2 + b2)
  {
    const float bias[2] = {net.b2[c0 + r16], net.b2[c0 + 16 + r16]};
    floatx4 acc[RB][2];
    zero(acc);
    gemm_reg(acc, sH1, kLdH, w2, kH);
    relu_out<RB>(h, acc, bias, sH2, c0);
  }
  load_w(w2, net.w2, kH, c0, kH);
  store_hidden(tr.h2T);
  __syncthreads();

  // ---- layer 3: Y = H2 W3 + b3, the loss and its gradient
  float sq = 0.f;
  if (c3 < Op && orb < RB) {
    floatx4 acc[ORB][1];
    zero(acc);
    gemm_reg(acc, sH2 + 16 * orb * kLdH, kLdH, w3t, kH);
    const bool cok = ocol < O;
    const float bias = cok ? net.b3[ocol] : 0.f;
    uint16_t dh[ORB][4];
#pragma unroll
    for (int rb = 0; rb < ORB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * (orb + rb) + 4 * q + i;
        const int64_t m = m0 + sample_of<RB>(row);
        const float y = acc[rb][0][i] + bias;
        float g = 0.f;
        if (cok && m < M) {
          const int64_t s = src.rows ? (int64_t)src.rows[m] : m;
          const float t = (float)((double)src.delta[s * O + ocol] / net.sd_d[ocol]);
          const float e = y - t;
          sq += e * e;
          g = 2.f * e / (float)((double)M * O);
        }
        dh[rb][i] = to_bf16(g);
        sDY[row * kLdY + ocol] = dh[rb][i];
      }
    store_col<RB, ORB>(tr.dyT + (size_t)ocol * tr.Mp + m0, orb, dh);
  }
  // the tile's loss, in a fixed order
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
  if (l == 0) s_loss[w] = sq;
  __syncthreads();
  if (tid == 0)
    tr.loss_part[blockIdx.x] = ((s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3])) +
                               ((s_loss[4] + s_loss[5]) + (s_loss[6] + s_loss[7]));

  // ---- dZ2 = (dY W3^T) * [H2 > 0], dZ1 = (dZ2 W2^T) * [H1 > 0]
  auto masked = [&](const floatx4 (&acc)[RB][2], const uint16_t* H) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool on = from_bf16(H[(16 * rb + 4 * q + i) * kLdH + c0 + 16 * cb + r16]) > 0.f;
          h[rb][cb][i] = to_bf16(on ? acc[rb][cb][i] : 0.f);
        }
  };
  {
    floatx4 acc[RB][2];
    zero(acc);
    gemm_reg(acc, sDY, kLdY, w3, Op);
    masked(acc, sH2);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) sD[(16 * rb + 4 * q + i) * kLdH + c0 + 16 * cb + r16] = h[rb][cb][i];
  }
  __syncthreads();
  store_hidden(tr.dz2T);
  {
    floatx4 acc[RB][2];
    zero(acc);
    gemm_reg(acc, sD, kLdH, w2, kH);
    masked(acc, sH1);
  }
  store_hidden(tr.dz1T);
}

// ---------------------------------------------------------------- weight gradients
// dW_l[k_in][n_out] = sum_m A_l[m][k_in] dZ_l[m][n_out] over one chunk of
// samples per workgroup; tiles of 64 x 64 over the three layers.  FP32 partials
// per chunk, summed in order by k_mlp_apply.
struct WGrad {
  const uint16_t* aT[3];   // Z^T, H1^T, H2^T
  const uint16_t* dT[3];   // dZ1^T, dZ2^T, dY^T
  int kin[3];              // Fp, kH, kH
  int nout[3];             // kH, kH, Op
  int tiles_c[3];          // column tiles per layer
  int tile_start[4];       // first tile of each layer (prefix sums)
  int64_t part_off[3];     // offset of each layer's block in a chunk's partials
  int64_t part_ld;         // floats per chunk
  int64_t Mp;
  int chunk;               // samples per chunk (multiple of 32)
  float* part;
};

// Bias gradients: row sums of dZ^T over all samples, one workgroup per row,
// fixed summation order.  The loss: the tiles' sums in order, one workgroup.
struct BGrad {
  const uint16_t* dT[3];
  int rows[3];             // kH, kH, Op
  int64_t Mp;
  float* out;              // [kH + kH + Op]
  const float* loss_part;  // null: no loss wanted
  int tiles;
  double scale;
  float* loss;
};

// The weight gradients (workgroups 0 .. tiles*chunks-1), the bias gradients
// and the loss of one step in one launch: 19 us for 8192 samples of 54 rows
// where three launches took 25, 10 and 6.  Bound by the operands' way through
// L2 (64 x 64 tiles, a quarter per wave; 64 x 32 took 26 us), four k-steps'
// loads in flight at a time.
__global__ __launch_bounds__(kWG) void k_mlp_wgrad(const WGrad g, const BGrad bg, int chunks) {
  const int wtiles = g.tile_start[3];
  int block = blockIdx.x;
  if (block >= wtiles * chunks) {
    block -= wtiles * chunks;
    __shared__ float red[kWG];
    const int nrow = bg.rows[0] + bg.rows[1] + bg.rows[2];
    if (block == nrow) {  // the loss, when it is wanted
      double s = 0.0;
      for (int t0 = 0; t0 < bg.tiles; t0 += kWG) {
        const int t = t0 + (int)threadIdx.x;
        red[threadIdx.x] = t < bg.tiles ? bg.loss_part[t] : 0.f;
        __syncthreads();
        if (threadIdx.x == 0)
#pragma unroll 8
          for (int i = 0; i < kWG; ++i) s += red[i];
        __syncthreads();
      }
      if (threadIdx.x == 0) *bg.loss = (float)(s * bg.scale);
      return;
    }
    int r = block, layer = 0;
    while (layer < 2 && r >= bg.rows[layer]) r -= bg.rows[layer++];
    const uint16_t* p = bg.dT[layer] + (size_t)r * bg.Mp;
    float s = 0.f;
#pragma unroll 8
    for (int64_t i = threadIdx.x; i < bg.Mp; i += kWG) s += from_bf16(p[i]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
      if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) bg.out[block] = red[0];
    return;
  }
  const int t = block % wtiles, chunk = block / wtiles;
  const int layer = t < g.tile_start[1] ? 0 : (t < g.tile_start[2] ? 1 : 2);
  const int lt = t - g.tile_start[layer];
  const int tr = lt / g.tiles_c[layer], tc = lt - tr * g.tiles_c[layer];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, r16 = l & 15, q = l >> 4;
  // the waves take the quarters of a 64 x 64 tile, 32 x 32 each
  const int r0 = 64 * tr + 32 * (w >> 1), c0 = 64 * tc + 32 * (w & 1);
  if (c0 >= g.nout[layer]) return;
  const int64_t k_begin = (int64_t)chunk * g.chunk;
  const int64_t k_end = min(k_begin + g.chunk, g.Mp);
  const uint16_t *A[2], *D[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    A[h] = g.aT[layer] + (size_t)(r0 + 16 * h + r16) * g.Mp + 8 * q;
    D[h] = g.dT[layer] + (size_t)(c0 + 16 * h + r16) * g.Mp + 8 * q;
  }
  floatx4 acc[2][2];
  zero(acc);
  auto steps = [&](int64_t k0, auto count) {
    constexpr int U = decltype(count)::value;
    bf16x8 a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[u][h] = frag(A[h] + k0 + 32 * u);
        b[u][h] = frag(D[h] + k0 + 32 * u);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][rb], b[u][cb], acc[rb][cb], 0, 0, 0);
  };
  int64_t k0 = k_begin;
  for (; k0 + 128 <= k_end; k0 += 128) steps(k0, std::integral_constant<int, 4>());
  for (; k0 < k_end; k0 += 32) steps(k0, std::integral_constant<int, 1>());
  float* out = g.part + (size_t)chunk * g.part_ld + g.part_off[layer];
  const int ld = g.nout[layer];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out[(size_t)(r0 + 16 * rb + 4 * q + i) * ld + c0 + 16 * cb + r16] = acc[rb][cb][i];
}

// Per parameter (flat order W1, b1, W2, b2, W3, b3): gather the gradient from
// the partials, optionally export it, optionally take an Adam step on the FP32
// master copy, and refresh the BF16 copies the products read.
struct Apply {
  int F, Fp, O, Op;
  int64_t nparam;
  float* master;
  float* m;
  float* v;
  const float* part;       // null: no gradient (refresh the BF16 copies only)
  int64_t part_ld;
  int64_t part_off[3];
  int chunks;
  const float* bgrad;      // [kH + kH + Op]
  float* grad_out;         // optional
  int update;              // take an Adam step
  float lr, c1, c2;        // c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t)
  uint16_t* w1t;
  uint16_t* w2t;
  uint16_t* w3t;
  uint16_t* w2;
  uint16_t* w3;
};

__global__ __launch_bounds__(kWG) void k_mlp_apply(const Apply a) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= a.nparam) return;
  const int64_t nW1 = (int64_t)a.F * kH, nW2 = (int64_t)kH * kH;
  const int64_t o_b1 = nW1, o_W2 = o_b1 + kH, o_b2 = o_W2 + nW2, o_W3 = o_b2 + kH;
  const int64_t o_b3 = o_W3 + (int64_t)kH * a.O;
  int kind;          // 0..5 = W1, b1, W2, b2, W3, b3
  int r = 0, c = 0;  // row / column within a weight matrix (or bias index in c)
  if (i < o_b1) { kind = 0; r = (int)(i / kH); c = (int)(i % kH); }
  else if (i < o_W2) { kind = 1; c = (int)(i - o_b1); }
  else if (i < o_b2) { kind = 2; r = (int)((i - o_W2) / kH); c = (int)((i - o_W2) % kH); }
  else if (i < o_W3) { kind = 3; c = (int)(i - o_b2); }
  else if (i < o_b3) { kind = 4; r = (int)((i - o_W3) / a.O); c = (int)((i - o_W3) % a.O); }
  else { kind = 5; c = (int)(i - o_b3); }

  float theta = a.master[i];
  if (a.part) {
    float g = 0.f;
    if (kind == 1 || kind == 3 || kind == 5) {
      g = a.bgrad[(kind == 1 ? 0 : kind == 3 ? kH : 2 * kH) + c];
    } else {
      const int layer = kind / 2;
      const int ld = layer == 2 ? a.Op : kH;
      const float* p = a.part + a.part_off[layer] + (size_t)r * ld + c;
#pragma unroll 8
      for (int s = 0; s < a.chunks; ++s) g += p[(size_t)s * a.part_ld];
    }
    if (a.grad_out) a.grad_out[i] = g;
    if (a.update) {
      const float mm = 0.9f * a.m[i] + 0.1f * g;
      const float vv = 0.999f * a.v[i] + 0.001f * g * g;
      a.m[i] = mm;
      a.v[i] = vv;
      theta -= a.lr * (mm * a.c1) / (sqrtf(vv * a.c2) + 1e-8f);
      a.master[i] = theta;
    }
  }
  const uint16_t h = to_bf16(theta);
  if (kind == 0) a.w1t[(size_t)c * a.Fp + r] = h;
  else if (kind == 2) { a.w2t[(size_t)c * kH + r] = h; a.w2[(size_t)r * kH + c] = h; }
  else if (kind == 4) { a.w3t[(size_t)c * kH + r] = h; a.w3[(size_t)r * a.Op + c] = h; }
}

// Raw training data: features [diag, b - x_prev, x_prev] (the difference in
// FP64, then rounded) and the change x_next - x_prev.
__global__ __launch_bounds__(kWG) void k_mlp_features(int64_t M, int n, int nnz, const int* diag_pos,
                                                      const double* values, const double* b,
                                                      const double* x_prev, const double* x_next,
                                                      float* feat, float* delta) {
  const int F = 3 * n, C = F + (x_next ? n : 0);
  const int64_t total = M * C;
  for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kWG) {
    const int64_t m = i / C;
    const int c = (int)(i - m * C);
    if (c < n) {
      const int p = diag_pos[c];
      feat[m * F + c] = p >= 0 ? (float)values[m * nnz + p] : 0.f;
    } else if (c < 2 * n) {
      feat[m * F + c] = (float)(b[m * n + c - n] - x_prev[m * n + c - n]);
    } else if (c < F) {
      feat[m * F + c] = (float)x_prev[m * n + c - 2 * n];
    } else {
      const int o = c - F;
      delta[m * n + o] = (float)(x_next[m * n + o] - x_prev[m * n + o]);
    }
  }
}

// Column moments of [feat | delta] (ncol <= kWG): partial sums per chunk of
// rows, of the values (mean == null) or of squared deviations from mean.
__global__ __launch_bounds__(kWG) void k_mlp_moments(int64_t M, int F, int O, const float* feat,
                                                     const float* delta, const double* mean,
                                                     int64_t chunk, double* part) {
  const int c = threadIdx.x, ncol = F + O;
  if (c >= ncol) return;
  const int64_t r0 = (int64_t)blockIdx.x * chunk, r1 = min(r0 + chunk, M);
  double s = 0.0;
  for (int64_t r = r0; r < r1; ++r) {
    const double v = c < F ? (double)feat[r * F + c] : (double)delta[r * O + (c - F)];
    s += mean ? (v - mean[c]) * (v - mean[c]) : v;
  }
  part[(size_t)blockIdx.x * ncol + c] = s;
}

// Sum the chunks in order: the mean (stage 0) or the standard deviation
// (stage 1, zero spread -> 1), written to out[0..ncol).
__global__ void k_mlp_moments_final(int chunks, int ncol, int64_t M, const double* part,
                                    int stage, double* out) {
  const int c = threadIdx.x;
  if (c >= ncol) return;
  double s = 0.0;
  for (int g = 0; g < chunks; ++g) s += part[(size_t)g * ncol + c];
  s /= (double)M;
  if (stage == 1) {
    const double sd = sqrt(s);
    s = sd > 1e-30 ? sd : 1.0;
  }
  out[c] = s;
}

}  // namespace mlp
}  // namespace bs

// Fourier-feature MLP velocity model on gfx950 (the neural-network velocity
// representation of the paper's workflows, Sec. 1): 2-D coordinates -> 64
// random Fourier frequencies (cos, sin: 128 features) -> 4 x 256 ReLU -> 1,
// v = vmin + vscale sigmoid(y). Matrix products run on the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16) with float32 accumulation; features, weights,
// hidden activations and back-propagated pre-activation gradients are stored as
// bfloat16 (round to nearest even), biases and everything else as float32.
//
// MFMA 32x32x16 operand layout (lane l of a wave64): A holds row l%32 and the 8
// reduction indices (l/32)*8 .. +7; B holds column l%32 and the same 8
// reduction indices; the 16 accumulators of lane l are rows 8i + (l/32)*4 + j,
// column l%32 (element 4i + j).
//
// The layers of 128 points stay in one work-group: the activations (backward:
// the pre-activation gradients) of its rows live in LDS from layer to layer, so
// that HBM sees the features once and every stored activation plane once each
// way. The weights are the A operand, read straight from L2 in the order of the
// matrix instructions (the pack), and the points the B operand, so a lane ends
// up with 4 consecutive outputs of one point.
#include "mlp.h"

namespace sweep {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t f2bf(float x) {  // round to nearest, ties to even
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}
// two floats as bf16 (round to nearest, ties to even), the first in the low half
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), b2));
}

// --------------------------------------------------------------------------
// gamma[m] = [cos(2 pi B x_m), sin(2 pi B x_m)], x_m = (i/(nx-1), j/(nz-1))
// --------------------------------------------------------------------------
__global__ void mlp_encode_kernel(const float* B, int nx, int nz, uint16_t* feats) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t M = (size_t)nx * nz;
  if (t >= M * kMlpFreq) return;
  const size_t m = t / kMlpFreq;
  const int f = (int)(t % kMlpFreq);
  const int i = (int)(m % nx), j = (int)(m / nx);
  const double x = nx > 1 ? (double)i / (nx - 1) : 0.0;
  const double z = nz > 1 ? (double)j / (nz - 1) : 0.0;
  const double ph = 2.0 * M_PI * ((double)B[2 * f] * x + (double)B[2 * f + 1] * z);
  feats[m * kMlpFeat + f] = f2bf((float)cos(ph));
  feats[m * kMlpFeat + kMlpFreq + f] = f2bf((float)sin(ph));
}

// bf16 weight pack. A matrix of R inputs and 256 outputs is stored as the A
// operands of its products: for output tile t (32 rows) and reduction step k
// (16 inputs), lane l's 8 values are W[32 t + l % 32][16 k + 8 (l / 32) ..],
// 64 lanes of 16 bytes, steps of a tile following each other. Layers 2..4 are
// also stored transposed (outputs and inputs exchanged) for the backward.
__global__ void mlp_cast_kernel(const float* theta, uint16_t* wp) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int n1 = kMlpWidth * kMlpFeat / 8, n2 = kMlpWidth * kMlpWidth / 8;
  if (t < n1 + 6 * n2) {
    const int q = t < n1 ? 0 : (t - n1) % (3 * n2) / n2;  // hidden matrix (t >= n1)
    const bool tr = t >= n1 + 3 * n2;
    const int e = t < n1 ? t : (t - n1) % n2;
    const int R = t < n1 ? kMlpFeat : kMlpWidth, KS = R / 16;
    const int l = e & 63, k = (e >> 6) % KS, tile = (e >> 6) / KS;
    const int row = 32 * tile + (l & 31), col = 16 * k + 8 * (l >> 5);
    const float* W = theta + (t < n1 ? kTh1 : kThHidden[q]);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = tr ? W[(col + j) * kMlpWidth + row] : W[row * R + col + j];
    uint16_t* dst = wp + (t < n1 ? kWp1 : tr ? kWpHiddenT[q] : kWpHidden[q]);
    reinterpret_cast<uint4*>(dst)[e] =
        make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
  }
  if (t < kMlpWidth) wp[kWp5 + t] = f2bf(theta[kTh5 + t]);
}

// --------------------------------------------------------------------------
// Fused layers. Work-group: 128 points, 4 waves; X holds their rows in LDS
// (256 bf16 and 16 bytes of padding, so that the 32 rows a half wave reads
// fall in different banks). Wave w takes outputs 64 w .. 64 w + 63 of all 128
// points: 2 x 4 accumulator tiles, 8 matrix instructions for every 2 A operands
// from L2 and 4 B operands from LDS. 67.6 KB of LDS and at most 256 registers
// a lane: two work-groups per CU. Bound by HBM (each activation plane once) and
// by the waits at the layers' barriers. 300 000 points: forward 690 MB in 194 us
// (one product per launch, with every plane written and read again: 927 us);
// backward chain 1.23 GB in 379 us (head and three products: 907 us).
// --------------------------------------------------------------------------
constexpr int kPts = 128;             // points of a work-group
constexpr int kXS = kMlpWidth + 8;    // LDS row stride (bf16)
constexpr int kAhead = 3;             // reduction steps of A operands in flight

// acc[t][p] = W[64 w + 32 t ..][:] X[32 p ..][:]^T over R inputs (steps of 16 in
// order).
template <int R>
__device__ __forceinline__ void layer_product(const uint16_t* __restrict__ W,
                                              const uint16_t* X, floatx16 (&acc)[2][4]) {
  constexpr int KS = R / 16;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint16_t* wa = W + ((size_t)(2 * w) * KS * 64 + l) * 8;
  const uint16_t* xb = X + (l & 31) * kXS + 8 * (l >> 5);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int p = 0; p < 4; ++p) acc[t][p] = floatx16{0};
  bf16x8 a[kAhead + 1][2];
#pragma unroll
  for (int k = 0; k < kAhead; ++k)
#pragma unroll
    for (int t = 0; t < 2; ++t) a[k][t] = load8(wa + (t * KS + k) * 512);
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    if (k + kAhead < KS) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        a[(k + kAhead) % (kAhead + 1)][t] = load8(wa + (t * KS + k + kAhead) * 512);
    }
    bf16x8 b[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) b[p] = load8(xb + p * 32 * kXS + 16 * k);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int p = 0; p < 4; ++p)
        acc[t][p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k % (kAhead + 1)][t], b[p],
                                                            acc[t][p], 0, 0, 0);
  }
}

// Rows r0 + 8 i of X (i < 16, r0 = thread / 32; 16 bytes at column 8 c,
// c = thread % 32) to or from rows of a global [M][256] plane.
__device__ __forceinline__ int copy_row(int i) { return (threadIdx.x >> 5) + 8 * i; }
__device__ __forceinline__ void store_rows(const uint16_t* X, uint16_t* out, int m0, int M) {
  const int c = 8 * (threadIdx.x & 31);
#pragma unroll
  for (int i = 0; i < kPts / 8; ++i) {
    const int r = copy_row(i);
    if (m0 + r < M)
      *reinterpret_cast<uint4*>(out + (size_t)(m0 + r) * kMlpWidth + c) =
          *reinterpret_cast<const uint4*>(X + r * kXS + c);
  }
}

// parameters start at any 4-byte address
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// X <- relu(acc + bias) (all waves have read X before).
__device__ __forceinline__ void put_relu(const floatx16 (&acc)[2][4], const float* bias,
                                         uint16_t* X) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = 64 * w + 32 * t + 8 * i + 4 * (l >> 5);
      const f4u b = *reinterpret_cast<const f4u*>(bias + n);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const floatx16& a = acc[t][p];
        const uint2 v = make_uint2(
            pack2(fmaxf(a[4 * i] + b.x, 0.0f), fmaxf(a[4 * i + 1] + b.y, 0.0f)),
            pack2(fmaxf(a[4 * i + 2] + b.z, 0.0f), fmaxf(a[4 * i + 3] + b.w, 0.0f)));
        *reinterpret_cast<uint2*>(X + (32 * p + (l & 31)) * kXS + n) = v;
      }
    }
}

__global__ __launch_bounds__(256, 2) void mlp_forward_kernel(
    const uint16_t* __restrict__ wp, const float* __restrict__ theta,
    const uint16_t* __restrict__ feats, int M, float vmin, float vscale, uint16_t* H, float* y,
    float* v) {
  __shared__ __attribute__((aligned(16))) uint16_t X[kPts * kXS];
  const int tid = threadIdx.x, m0 = blockIdx.x * kPts;
  const size_t plane = (size_t)M * kMlpWidth;
#pragma unroll
  for (int i = 0; i < 8; ++i) {  // rows past M are clamped and not stored
    const int r = (tid >> 4) + 16 * i, c = 8 * (tid & 15);
    *reinterpret_cast<uint4*>(X + r * kXS + c) = *reinterpret_cast<const uint4*>(
        feats + (size_t)min(m0 + r, M - 1) * kMlpFeat + c);
  }
  __syncthreads();
  floatx16 acc[2][4];
  layer_product<kMlpFeat>(wp + kWp1, X, acc);
  __syncthreads();
  put_relu(acc, theta + kThB1, X);
  __syncthreads();
  store_rows(X, H, m0, M);
#pragma unroll 1
  for (int l = 0; l < 3; ++l) {
    layer_product<kMlpWidth>(wp + kWpHidden[l], X, acc);
    __syncthreads();
    put_relu(acc, theta + kThBHidden[l], X);
    __syncthreads();
    store_rows(X, H + (size_t)(l + 1) * plane, m0, M);
  }
  // y_m = h4_m . w5 + b5 (float32, in order), v_m = vmin + vscale sigmoid(y_m)
  if (tid < kPts && m0 + tid < M) {
    const uint16_t* h = X + tid * kXS;
    const uint16_t* w5 = wp + kWp5;
    float s = 0.0f;
#pragma unroll 4
    for (int k = 0; k < kMlpWidth; k += 8) {
      const uint4 q = *reinterpret_cast<const uint4*>(h + k);
      const uint16_t* e = reinterpret_cast<const uint16_t*>(&q);
#pragma unroll
      for (int t = 0; t < 8; ++t) s = fmaf(bf2f(e[t]), bf2f(w5[k + t]), s);
    }
    const float yy = s + theta[kThB5];
    y[m0 + tid] = yy;
    v[m0 + tid] = vmin + vscale / (1.0f + expf(-yy));
  }
}

// Pre-activation gradients of the 4 hidden layers: dy_m = dv_m vscale s (1 - s),
// dZ4 = bf16(dy w5 [h4 > 0]), dZ_{l-1} = bf16((dZ_l W_l) [h_{l-1} > 0]); and for
// each work-group the sums of dy h4 (-> grad w5) and of dy (-> grad b5).
__global__ __launch_bounds__(256, 2) void mlp_backward_kernel(
    const uint16_t* __restrict__ wp, const uint16_t* __restrict__ H, const float* dv,
    const float* y, int M, float vscale, uint16_t* dZ, float* partial) {
  __shared__ __attribute__((aligned(16))) uint16_t X[kPts * kXS];
  __shared__ float sdy[kPts];
  const int tid = threadIdx.x, m0 = blockIdx.x * kPts, l = tid & 63, w = tid >> 6;
  const int c = 8 * (tid & 31), g = tid >> 5;
  const size_t plane = (size_t)M * kMlpWidth;
  constexpr int NI = kPts / 8;
  uint4 h[NI];
  auto load_h = [&](const uint16_t* src) {  // rows past M: 0 (their gradients are 0)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = m0 + copy_row(i);
      h[i] = m < M ? *reinterpret_cast<const uint4*>(src + (size_t)m * kMlpWidth + c)
                   : make_uint4(0, 0, 0, 0);
    }
  };
  load_h(H + 3 * plane);
  if (tid < kPts) {
    float dy = 0.0f;
    if (m0 + tid < M) {
      const float s = 1.0f / (1.0f + expf(-y[m0 + tid]));
      dy = dv[m0 + tid] * vscale * s * (1.0f - s);
    }
    sdy[tid] = dy;
  }
  __syncthreads();
  {
    const uint4 wq = *reinterpret_cast<const uint4*>(wp + kWp5 + c);
    const uint16_t* we = reinterpret_cast<const uint16_t*>(&wq);
    float accw[8], accb = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) accw[t] = 0.0f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = copy_row(i);
      const float dy = sdy[r];
      const uint16_t* he = reinterpret_cast<const uint16_t*>(&h[i]);
      float z[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float hv = bf2f(he[t]);
        accw[t] = fmaf(dy, hv, accw[t]);
        z[t] = hv > 0.0f ? dy * bf2f(we[t]) : 0.0f;
      }
      accb += dy;
      const uint4 q = make_uint4(pack2(z[0], z[1]), pack2(z[2], z[3]), pack2(z[4], z[5]),
                                 pack2(z[6], z[7]));
      *reinterpret_cast<uint4*>(X + r * kXS + c) = q;
      if (m0 + r < M)
        *reinterpret_cast<uint4*>(dZ + 3 * plane + (size_t)(m0 + r) * kMlpWidth + c) = q;
    }
    // the 8 row groups' sums, added in order
    __shared__ float red[8][kMlpWidth + 1];
#pragma unroll
    for (int t = 0; t < 8; ++t) red[g][c + t] = accw[t];
    if ((tid & 31) == 0) red[g][kMlpWidth] = accb;
    __syncthreads();
    float* out = partial + (size_t)blockIdx.x * (kMlpWidth + 1);
    for (int k = tid; k <= kMlpWidth; k += 256) {
      float s = red[0][k];
#pragma unroll
      for (int q = 1; q < 8; ++q) s += red[q][k];
      out[k] = s;
    }
  }
#pragma unroll 1
  for (int q = 2; q >= 0; --q) {
    floatx16 acc[2][4];
    layer_product<kMlpWidth>(wp + kWpHiddenT[q], X, acc);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = 64 * w + 32 * t + 8 * i + 4 * (l >> 5);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const floatx16& a = acc[t][p];
          *reinterpret_cast<uint2*>(X + (32 * p + (l & 31)) * kXS + n) =
              make_uint2(pack2(a[4 * i], a[4 * i + 1]), pack2(a[4 * i + 2], a[4 * i + 3]));
        }
      }
    load_h(H + q * plane);  // the masks
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = copy_row(i);
      uint4 z = *reinterpret_cast<const uint4*>(X + r * kXS + c);
      uint32_t* ze = reinterpret_cast<uint32_t*>(&z);
      const uint32_t* he = reinterpret_cast<const uint32_t*>(&h[i]);
#pragma unroll
      for (int t = 0; t < 4; ++t) {  // h > 0: positive as a 16-bit integer
        const uint32_t lo = (int16_t)(he[t] & 0xffffu) > 0 ? 0xffffu : 0u;
        const uint32_t hi = (int16_t)(he[t] >> 16) > 0 ? 0xffff0000u : 0u;
        ze[t] &= lo | hi;
      }
      *reinterpret_cast<uint4*>(X + r * kXS + c) = z;
      if (m0 + r < M)
        *reinterpret_cast<uint4*>(dZ + q * plane + (size_t)(m0 + r) * kMlpWidth + c) = z;
    }
    __syncthreads();
  }
}

// --------------------------------------------------------------------------
// partial[chunk][n][k] = sum over the chunk's rows m of dZ[m][n] H[m][k], and
// pb[chunk][n] = sum of dZ[m][n]. The reduction runs over the rows of both
// operands, so their tiles (32 rows) are staged in LDS as they lie in memory and
// read back transposed (ds_read_b64_tr_b16: the 16 lanes of a group read 4 rows
// of 16 values, lane i gets column i of the 4 rows). Rows are padded by 64
// bytes: the 4 rows and 2 groups of a read then cover all banks. The loads of
// the next 32 rows are in flight while the matrix instructions run.
// Work-group: BN x BK outputs, 4 waves of BN/2 x BK/2. 128 x 256 outputs read
// each operand nearly once from HBM; 64 x 64 keep more work-groups busy when
// there are few chunks. 300 000 points x 256 x 256: 122 us (307 MB read, 77 MB of
// partials), against 247 us with 2-byte loads down the columns and 28 us more
// for the column sums.
// --------------------------------------------------------------------------
constexpr int kDwRows = 32;
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

// 8 consecutive rows (from row) of the column c0 + lane % 32, of an LDS tile of
// stride S: the MFMA operand of this lane
template <int S>
__device__ __forceinline__ bf16x8 read_tr(const uint16_t* tile, int row, int c0) {
  const int l = threadIdx.x & 63, s = l & 15;
  const uint16_t* p = tile + (row + 8 * (l >> 5) + (s >> 2)) * S + c0 + 16 * ((l >> 4) & 1) +
                      4 * (s & 3);
  typedef __attribute__((address_space(3))) s4 lds_s4;
  const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p);
  const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + 4 * S));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int BN, int BK, int K>
__global__ __launch_bounds__(256, BN == 128 ? 2 : 4) void mlp_dw_kernel(
    const uint16_t* __restrict__ dZ, const uint16_t* __restrict__ H, int M, float* partial,
    float* pb) {
  constexpr int SN = BN + 32, SK = BK + 32;         // LDS row strides
  constexpr int TN = BN / 64, TK = BK / 64;         // accumulator tiles of a wave
  constexpr int LN = kDwRows * BN / 8 / 256, LK = kDwRows * BK / 8 / 256;  // loads a thread
  static_assert(BN / 8 * 8 == BN && 256 % (BN / 8) == 0 && 256 % (BK / 8) == 0, "dw geometry");
  __shared__ __attribute__((aligned(16))) uint16_t sn[2][kDwRows * SN], sk[2][kDwRows * SK];
  __shared__ float red[256 / (BN / 8)][BN];
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const int n0 = blockIdx.x * BN, k0 = blockIdx.y * BK;
  const int m0 = blockIdx.z * kMlpChunk, m1 = min(M, m0 + kMlpChunk);
  const int cn = 8 * (tid % (BN / 8)), rn = tid / (BN / 8);
  const int ck = 8 * (tid % (BK / 8)), rk = tid / (BK / 8);
  uint4 gn[LN], gk[LK];
  float db[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) db[t] = 0.0f;
  auto gload = [&](int m) {  // rows past the chunk: 0
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      const int r = m + rn + i * (256 / (BN / 8));
      gn[i] = r < m1 ? *reinterpret_cast<const uint4*>(dZ + (size_t)r * kMlpWidth + n0 + cn)
                     : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < LK; ++i) {
      const int r = m + rk + i * (256 / (BK / 8));
      gk[i] = r < m1 ? *reinterpret_cast<const uint4*>(H + (size_t)r * K + k0 + ck)
                     : make_uint4(0, 0, 0, 0);
    }
  };
  auto lstore = [&](int u) {
#pragma unroll
    for (int i = 0; i < LN; ++i) {
      *reinterpret_cast<uint4*>(&sn[u][(rn + i * (256 / (BN / 8))) * SN + cn]) = gn[i];
      const uint16_t* e = reinterpret_cast<const uint16_t*>(&gn[i]);
#pragma unroll
      for (int t = 0; t < 8; ++t) db[t] += bf2f(e[t]);
    }
#pragma unroll
    for (int i = 0; i < LK; ++i)
      *reinterpret_cast<uint4*>(&sk[u][(rk + i * (256 / (BK / 8))) * SK + ck]) = gk[i];
  };
  floatx16 acc[TN][TK];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TK; ++j) acc[i][j] = floatx16{0};
  const int wn = (w & 1) * (BN / 2), wk = (w >> 1) * (BK / 2);
  gload(m0);
  lstore(0);
  __syncthreads();
  for (int m = m0, u = 0; m < m1; m += kDwRows, u ^= 1) {
    const bool more = m + kDwRows < m1;
    if (more) gload(m + kDwRows);
#pragma unroll
    for (int s = 0; s < kDwRows; s += 16) {
      bf16x8 a[TN], b[TK];
#pragma unroll
      for (int i = 0; i < TN; ++i) a[i] = read_tr<SN>(sn[u], s, wn + 32 * i);
#pragma unroll
      for (int j = 0; j < TK; ++j) b[j] = read_tr<SK>(sk[u], s, wk + 32 * j);
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TK; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // the other buffer was last read before the previous barrier
    if (more) lstore(u ^ 1);
    __syncthreads();
  }
  float* out = partial + (size_t)blockIdx.z * kMlpWidth * K;
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TK; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int n = n0 + wn + 32 * i + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
        out[(size_t)n * K + k0 + wk + 32 * j + (l & 31)] = acc[i][j][e];
      }
  if (blockIdx.y == 0) {  // the thread groups' column sums, added in order
#pragma unroll
    for (int t = 0; t < 8; ++t) red[rn][cn + t] = db[t];
    __syncthreads();
    if (tid < BN) {
      float s = red[0][tid];
      for (int q = 1; q < 256 / (BN / 8); ++q) s += red[q][tid];
      pb[(size_t)blockIdx.z * kMlpWidth + n0 + tid] = s;
    }
  }
}

// dst[e] = sum over chunks c of partial[c * len + e] (e < len), then dst2[e] =
// sum of partial2[c * len2 + e], in float64: four sums over c mod 4, one for each
// wave of the work-group, added in order. 64 outputs a work-group and 16 loads
// in flight a lane: one thread for all four sums left a 293-chunk reduction of
// 65 792 outputs at 29 us (2.6 TB/s).
__global__ __launch_bounds__(256) void mlp_reduce_kernel(const float* __restrict__ partial,
                                                         int len, float* dst,
                                                         const float* __restrict__ partial2,
                                                         int len2, float* dst2, int nchunk) {
  __shared__ double part[4][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  int e = blockIdx.x * 64 + l;
  const bool in = e < len + len2, second = in && e >= len;
  if (second) e -= len;
  const int stride = second ? len2 : len;
  const float* p = (second ? partial2 : partial) + (in ? e : 0);
  double acc = 0.0;
  int c = w;
  for (; c + 4 * 15 < nchunk; c += 4 * 16) {
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = p[(size_t)(c + 4 * j) * stride];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc += (double)v[j];
  }
  for (; c < nchunk; c += 4) acc += (double)p[(size_t)c * stride];
  part[w][l] = acc;
  __syncthreads();
  if (w == 0 && in)
    (second ? dst2 : dst)[e] = (float)(((part[0][l] + part[1][l]) + part[2][l]) + part[3][l]);
}

// Adam with bias correction: c1 = 1/(1-b1^t), c2 = 1/(1-b2^t)
__global__ void adam_kernel(float* theta, float* m, float* v, const float* g, size_t n,
                            float lr, float b1, float b2, float eps, float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

}  // namespace

size_t mlp_workspace_bytes(int M) {
  const size_t Mz = (size_t)M;
  const int nch = (M + kMlpChunk - 1) / kMlpChunk;
  size_t off = 0;
  off = align_up(off + 4 * Mz * kMlpWidth * 2);  // H1..H4 (bf16)
  off = align_up(off + Mz * 4);                  // y
  off = align_up(off + 4 * Mz * kMlpWidth * 2);  // dZ1..dZ4 (bf16)
  off = align_up(off + (size_t)nch * kMlpWidth * kMlpWidth * 4);  // dW partials
  off = align_up(off + (size_t)nch * (kMlpWidth + 1) * 4);        // head / bias partials
  return off;
}

MlpWork mlp_carve(void* work, int M) {
  MlpWork w;
  const size_t Mz = (size_t)M;
  const int nch = (M + kMlpChunk - 1) / kMlpChunk;
  char* b = static_cast<char*>(work);
  size_t off = 0;
  for (int l = 0; l < 4; ++l) w.H[l] = reinterpret_cast<uint16_t*>(b + off) + (size_t)l * Mz * kMlpWidth;
  off = align_up(off + 4 * Mz * kMlpWidth * 2);
  w.y = reinterpret_cast<float*>(b + off);
  off = align_up(off + Mz * 4);
  for (int l = 0; l < 4; ++l) w.dZ[l] = reinterpret_cast<uint16_t*>(b + off) + (size_t)l * Mz * kMlpWidth;
  off = align_up(off + 4 * Mz * kMlpWidth * 2);
  w.pW = reinterpret_cast<float*>(b + off);
  off = align_up(off + (size_t)nch * kMlpWidth * kMlpWidth * 4);
  w.pB = reinterpret_cast<float*>(b + off);
  w.nchunk = nch;
  return w;
}

int mlp_launch_encode(const float* B, int nx, int nz, uint16_t* feats, hipStream_t s) {
  const size_t n = (size_t)nx * nz * kMlpFreq;
  hipLaunchKernelGGL(mlp_encode_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, nx,
                     nz, feats);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int mlp_launch_cast(const float* theta, uint16_t* wp, hipStream_t s) {
  const int n = kMlpWidth * (kMlpFeat + 6 * kMlpWidth) / 8;
  hipLaunchKernelGGL(mlp_cast_kernel, dim3((n + 255) / 256), dim3(256), 0, s, theta, wp);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int mlp_launch_forward(const uint16_t* wp, const float* theta, const uint16_t* feats, int M,
                       float vmin, float vscale, float* v, const MlpWork& w, hipStream_t s) {
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((M + kPts - 1) / kPts), dim3(256), 0, s, wp, theta,
                     feats, M, vmin, vscale, w.H[0], w.y, v);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

namespace {
// dW and db of a layer: 128 x 256 (128 x 128 for the features) outputs a
// work-group where the chunks alone give two for every CU, else 64 x 64
template <int K>
void launch_dw(const uint16_t* dz, const uint16_t* h, int M, const MlpWork& w, hipStream_t s) {
  constexpr int BK = K < 256 ? K : 256;
  const dim3 t(256);
  if (w.nchunk * (kMlpWidth / 128) >= 256)
    hipLaunchKernelGGL((mlp_dw_kernel<128, BK, K>), dim3(kMlpWidth / 128, K / BK, w.nchunk), t, 0,
                       s, dz, h, M, w.pW, w.pB);
  else
    hipLaunchKernelGGL((mlp_dw_kernel<64, 64, K>), dim3(kMlpWidth / 64, K / 64, w.nchunk), t, 0,
                       s, dz, h, M, w.pW, w.pB);
}
void launch_reduce(const float* p, int len, float* dst, const float* p2, int len2, float* dst2,
                   int n, hipStream_t s) {
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3((len + len2 + 63) / 64), dim3(256), 0, s, p, len,
                     dst, p2, len2, dst2, n);
}
}  // namespace

int mlp_launch_backward(const uint16_t* wp, const uint16_t* feats, int M, float vscale,
                        const float* dv, float* grad, const MlpWork& w, hipStream_t s) {
  // the work-groups' sums for the output layer (257 floats each) take the room
  // of the dW partials, which are written later
  const int ng = (M + kPts - 1) / kPts;
  static_assert((kMlpChunk / kPts) * (kMlpWidth + 1) <= kMlpWidth * kMlpWidth,
                "the dW partials of a chunk hold its work-groups' output-layer sums");
  hipLaunchKernelGGL(mlp_backward_kernel, dim3(ng), dim3(256), 0, s, wp, (const uint16_t*)w.H[0],
                     dv, (const float*)w.y, M, vscale, w.dZ[0], w.pW);
  launch_reduce(w.pW, kMlpWidth + 1, grad + kTh5, nullptr, 0, nullptr, ng, s);
  // hidden layers 4..1: dW = dZ^T H_prev, db = column sums of dZ
  for (int l = 3; l >= 0; --l) {
    if (l > 0)
      launch_dw<kMlpWidth>(w.dZ[l], w.H[l - 1], M, w, s);
    else
      launch_dw<kMlpFeat>(w.dZ[0], feats, M, w, s);
    launch_reduce(w.pW, kMlpWidth * (l == 0 ? kMlpFeat : kMlpWidth),
                  grad + (l == 0 ? kTh1 : kThHidden[l - 1]), w.pB, kMlpWidth,
                  grad + (l == 0 ? kThB1 : kThBHidden[l - 1]), w.nchunk, s);
  }
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

int launch_adam(float* theta, float* m, float* v, const float* g, size_t n, float lr, float b1,
                float b2, float eps, int t, hipStream_t s) {
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)b1, t)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)b2, t)));
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, m, v,
                     g, n, lr, b1, b2, eps, c1, c2);
  SWEEP_HIP(hipGetLastError());
  return SWEEP_OK;
}

}  // namespace sweep

// Warm-start network 4 -> 128 -> 128 -> 64 (SiLU, SiLU, linear) on bf16 MFMA
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
//
// Precision contract (the oracle follows the same steps in FP64): inputs and
// weights are rounded to bf16 (round to nearest even); biases stay FP32;
// hidden activations are rounded to bf16 after SiLU; the output is FP32.  The
// backward pass rounds the three error signals G3, G2, G1 to bf16 before their
// products (standard bf16 mixed precision); weight gradients are FP32 MFMA
// sums over a workgroup's rows (64 at most), then FP64 fixed-order sums over
// workgroups.
//
// One workgroup = up to 4 blocks of 16 batch rows in turn, 4 wavefronts;
// wavefront w owns outputs 32 w .. 32 w + 31 of the hidden layers and 16 w ..
// 16 w + 15 of the last, and keeps its rows of all five weight matrices and its
// gradient tiles in registers (about 100 each) from start to end.  Only
// activations and errors go through LDS.  MFMA lane layout (16x16x32): lane l
// holds A[m = l % 16][k = 8 (l / 16) + i] and B[k = 8 (l / 16) + i][n = l % 16]
// for i < 8, and C[m = 4 (l / 16) + r][n = l % 16] for r < 4.  A 16x16x16
// operand holds k = 4 (l / 16) + i for i < 4: a C tile of errors or activations,
// rounded, is therefore the operand of the weight gradient's product (a
// reduction over the 16 rows) as it stands, and the other waves' tiles are read
// as 8 bytes a lane from a copy with the rows innermost.
//
// Bound by latency at the batch sizes of training: a block is five dependent
// layers of a few MFMA each.  1,024 rows: 16.2 us on 64 workgroups, against 43.6
// on 16 of 64 rows whose wavefronts each read all weights from L2 for 16 rows and
// gathered the gradients' operands element by element.  From about 50,000 rows on
// by the partials (101 KB per 64 rows, written and read once): 100,000 rows with
// the update kernel 0.42 ms, 0.88 before.
#include "mlp_internal.h"

#include <algorithm>

namespace fock {
namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int AS = 136, GS = 72, RS = 20;  // LDS strides in bf16 elements: rows (multiples of 8), columns

// Round to nearest even (add 0x7fff plus the lowest kept bit, truncate).
__device__ __forceinline__ uint16_t to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p) {
  const u16x8 v = *reinterpret_cast<const u16x8 *>(p);
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mma16(i16x4 a, i16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float from_bf16(short h) { return from_bf16((uint16_t)h); }
// Sum over a C tile's 16 rows of this lane's column.
__device__ __forceinline__ float column_sum(i16x4 v) {
  float s = (from_bf16(v[0]) + from_bf16(v[1])) + (from_bf16(v[2]) + from_bf16(v[3]));
  s += __shfl_xor(s, 16, 64);
  return s + __shfl_xor(s, 32, 64);
}

__device__ __forceinline__ float sigm(float z) { return 1.f / (1.f + expf(-z)); }

__device__ __forceinline__ double block_sum(double v, double *red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// Forward for the workgroup's rows; with BWD also the masked-MSE error and
// this workgroup's share of every parameter gradient (partial + blockIdx.x *
// NPAR, parameter order) and of the loss numerator (lossp[blockIdx.x]).
// count: N is summed here, by every workgroup, and stored by the first.
template <bool BWD>
__global__ __launch_bounds__(256) void k_mlp(Weights w, const float *__restrict__ X, const float *__restrict__ T,
                                             const int *__restrict__ nvalid, Count *__restrict__ cnt, int count, int B,
                                             int blocks, float *__restrict__ Y, float *__restrict__ partial,
                                             double *__restrict__ lossp) {
  __shared__ __attribute__((aligned(16))) uint16_t a1s[16 * AS];
  __shared__ __attribute__((aligned(16))) uint16_t a2s[16 * AS];  // A2, later G2
  __shared__ __attribute__((aligned(16))) uint16_t g3s[16 * GS];
  __shared__ __attribute__((aligned(8))) uint16_t a1t[NH * RS], a2t[NH * RS];  // rows innermost
  __shared__ double red[4];
  __shared__ int rsum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int n0 = 32 * wave + lr, n3 = 16 * wave + lr;  // this lane's outputs: n0, n0 + 16 (hidden), n3 (last)

  // weights and biases, once
  bf16x8 w1[2], w2[2][4], w3[4], w3t[2][2], w2t[2][4];
  float b1[2], b2[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int n = n0 + 16 * t;
    w1[t] = ld8(w.w1b + n * KIN + 8 * lq);
    b1[t] = w.params[OB1 + n];
    b2[t] = w.params[OB2 + n];
#pragma unroll
    for (int s = 0; s < 4; ++s) w2[t][s] = ld8(w.w2b + n * NH + 32 * s + 8 * lq);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) w3[s] = ld8(w.w3b + n3 * NH + 32 * s + 8 * lq);
  const float b3 = w.params[OB3 + n3];
  float invN = 0.f;
  if constexpr (BWD) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int n = n0 + 16 * t;
#pragma unroll
      for (int s = 0; s < 2; ++s) w3t[t][s] = ld8(w.w3t + n * NOUT + 32 * s + 8 * lq);
#pragma unroll
      for (int s = 0; s < 4; ++s) w2t[t][s] = ld8(w.w2t + n * NH + 32 * s + 8 * lq);
    }
    if (count) {
      int s = 0;
      for (int b = tid; b < B; b += 256) s += min(max(nvalid[b], 0), NOUT);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (lane == 0) rsum[wave] = s;
      __syncthreads();
      const double N = (double)(rsum[0] + rsum[1] + rsum[2] + rsum[3]);
      invN = N > 0.0 ? (float)(1.0 / N) : 0.f;
      if (blockIdx.x == 0 && tid == 0) {
        cnt->N = N;
        cnt->invN = invN;
      }
    } else {
      invN = cnt->invN;
    }
  }

  f32x4 dw1[2], dw2[2][8], dw3[8];
  float db1[2] = {0.f, 0.f}, db2[2] = {0.f, 0.f}, db3 = 0.f;
  double loss = 0.0;
#pragma unroll
  for (int t = 0; t < 8; ++t) dw3[t] = dw2[0][t] = dw2[1][t] = dw1[t & 1] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int blk = 0; blk < blocks; ++blk) {
    const int row0 = (blockIdx.x * blocks + blk) * 16;
    if (row0 >= B) break;
    const int rq = row0 + 4 * lq;  // this lane's rows in a C tile: rq .. rq + 3
    // inputs: the layer-1 operand (K padded to 32 with zeros), and for the
    // backward pass the same with rows as the reduction, targets and masks
    bf16x8 xa = {};
    if (lq == 0 && row0 + lr < B) {
      const float *v = X + (size_t)(row0 + lr) * NIN;
      u16x8 u = {to_bf16(v[0]), to_bf16(v[1]), to_bf16(v[2]), to_bf16(v[3]), 0, 0, 0, 0};
      xa = __builtin_bit_cast(bf16x8, u);
    }
    i16x4 xt = {0, 0, 0, 0};
    float tv[4];
    int nv[4];
    if constexpr (BWD) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int g = rq + r;
        if (lr < NIN && g < B) xt[r] = (short)to_bf16(X[(size_t)g * NIN + lr]);
        tv[r] = g < B ? T[(size_t)g * NOUT + n3] : 0.f;
        nv[r] = g < B ? nvalid[g] : 0;
      }
    }
    float ds1[2][4], ds2[2][4];  // SiLU'(Z1), SiLU'(Z2)
    // One hidden tile: SiLU, its derivative, the rounded activation to LDS
    auto activate = [&](f32x4 c, float bias, float (&ds)[4], uint16_t *rows, uint16_t *cols, int n) {
      i16x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = c[r] + bias, s = sigm(z);
        const uint16_t h = to_bf16(z * s);
        v[r] = (short)h;
        rows[(4 * lq + r) * AS + n] = h;
        ds[r] = s * (1.f + z * (1.f - s));
      }
      if (BWD) *reinterpret_cast<i16x4 *>(cols + n * RS + 4 * lq) = v;
    };
    auto rows4 = [&](const uint16_t *a, int s) { return ld8(a + lr * AS + 32 * s + 8 * lq); };
    // layer 1: Z1 = Xb W1^T + b1
#pragma unroll
    for (int t = 0; t < 2; ++t)
      activate(mma(xa, w1[t], f32x4{0.f, 0.f, 0.f, 0.f}), b1[t], ds1[t], a1s, a1t, n0 + 16 * t);
    __syncthreads();
    // layer 2: Z2 = A1 W2^T + b2
    {
      f32x4 c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bf16x8 a = rows4(a1s, s);
        c[0] = mma(a, w2[0][s], c[0]);
        c[1] = mma(a, w2[1][s], c[1]);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) activate(c[t], b2[t], ds2[t], a2s, a2t, n0 + 16 * t);
    }
    __syncthreads();
    // layer 3: Y = A2 W3^T + b3
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) y = mma(rows4(a2s, s), w3[s], y);
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] += b3;
    if (Y) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (rq + r < B) Y[(size_t)(rq + r) * NOUT + n3] = y[r];
    }
    if constexpr (BWD) {
      auto tile = [&](const uint16_t *cols, int t) {
        return *reinterpret_cast<const i16x4 *>(cols + (16 * t + lr) * RS + 4 * lq);
      };
      // G3 = bf16(2 M (Y - T) / N) and the loss numerator
      i16x4 g3;
      float lsum = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float gv = 0.f;
        if (n3 < nv[r]) {
          const float dl = y[r] - tv[r];
          lsum = fmaf(dl, dl, lsum);
          gv = 2.f * dl * invN;
        }
        const uint16_t h = to_bf16(gv);
        g3[r] = (short)h;
        g3s[(4 * lq + r) * GS + n3] = h;
      }
      loss += (double)lsum;
      // dW3[out][in] = sum_rows G3[row][out] A2[row][in]
#pragma unroll
      for (int t = 0; t < 8; ++t) dw3[t] = mma16(g3, tile(a2t, t), dw3[t]);
      db3 += column_sum(g3);
      __syncthreads();
      // G2 = bf16((G3 W3) * SiLU'(Z2)), written over A2
      i16x4 g2[2];
      {
        f32x4 c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const bf16x8 a = ld8(g3s + lr * GS + 32 * s + 8 * lq);
          c[0] = mma(a, w3t[0][s], c[0]);
          c[1] = mma(a, w3t[1][s], c[1]);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint16_t h = to_bf16(c[t][r] * ds2[t][r]);
            g2[t][r] = (short)h;
            a2s[(4 * lq + r) * AS + n0 + 16 * t] = h;
          }
      }
      // dW2 = G2^T A1
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const i16x4 a = tile(a1t, t);
        dw2[0][t] = mma16(g2[0], a, dw2[0][t]);
        dw2[1][t] = mma16(g2[1], a, dw2[1][t]);
      }
      db2[0] += column_sum(g2[0]);
      db2[1] += column_sum(g2[1]);
      __syncthreads();
      // G1 = bf16((G2 W2) * SiLU'(Z1)); dW1 = G1^T Xb
      f32x4 c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bf16x8 a = rows4(a2s, s);
        c[0] = mma(a, w2t[0][s], c[0]);
        c[1] = mma(a, w2t[1][s], c[1]);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        i16x4 g1;
#pragma unroll
        for (int r = 0; r < 4; ++r) g1[r] = (short)to_bf16(c[t][r] * ds1[t][r]);
        dw1[t] = mma16(g1, xt, dw1[t]);
        db1[t] += column_sum(g1);
      }
    }
  }
  if constexpr (BWD) {
    float *P = partial + (size_t)blockIdx.x * NPAR;
    const int m0 = 32 * wave + 4 * lq, m3 = 16 * wave + 4 * lq;  // first output of this lane's gradient tiles
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        P[OW3 + (m3 + r) * NH + 16 * t + lr] = dw3[t][r];
        P[OW2 + (m0 + r) * NH + 16 * t + lr] = dw2[0][t][r];
        P[OW2 + (m0 + 16 + r) * NH + 16 * t + lr] = dw2[1][t][r];
      }
      if (lr < NIN) {
        P[OW1 + (m0 + r) * NIN + lr] = dw1[0][r];
        P[OW1 + (m0 + 16 + r) * NIN + lr] = dw1[1][r];
      }
    }
    if (lq == 0) {
      P[OB3 + n3] = db3;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        P[OB2 + n0 + 16 * t] = db2[t];
        P[OB1 + n0 + 16 * t] = db1[t];
      }
    }
    const double ls = block_sum(loss, red);
    if (tid == 0) lossp[blockIdx.x] = ls;
  }
}

// N = sum_b min(max(n_b, 0), 64) and 1 / N (one workgroup; batches over kCountInline).
__global__ __launch_bounds__(256) void k_mlp_count(const int *__restrict__ nvalid, int B, Count *__restrict__ cnt) {
  __shared__ double red[4];
  double s = 0.0;
  for (int b = threadIdx.x; b < B; b += 256) s += (double)min(max(nvalid[b], 0), NOUT);
  s = block_sum(s, red);
  if (threadIdx.x == 0) {
    cnt->N = s;
    cnt->invN = s > 0.0 ? (float)(1.0 / s) : 0.f;
  }
}

// Workgroup b < ceil(NPAR / 64): the gradient of 64 parameters, a fixed-order
// FP64 sum of the workgroup partials in four strided shares (nwg may be 0: no
// gradient), optional Adam update of the FP32 master value (Kingma & Ba,
// Algorithm 1; bc1 = 1 - beta1^t, bc2 = 1 - beta2^t), and, where the master
// values are new, the bf16 copies the forward and backward kernels read.  The
// last workgroup: loss = sum of the numerators / N.  grad and loss may be host
// memory.  4.5 us at 64 partials, the gradient in host memory; with one thread a
// parameter, a loss launch and copies of both results 5.2 us at 16, 4.7 and two
// copies.
__global__ __launch_bounds__(256) void k_mlp_update(const float *__restrict__ partial, int nwg, float *__restrict__ grad,
                                                    float *__restrict__ params, float *__restrict__ m,
                                                    float *__restrict__ v, AdamArgs ad, uint16_t *__restrict__ wb,
                                                    const double *__restrict__ lossp, const Count *__restrict__ cnt,
                                                    double *__restrict__ loss) {
  __shared__ double red[256];
  if (blockIdx.x == (NPAR + 63) / 64) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nwg; b += 256) s += lossp[b];
    s = block_sum(s, red);
    if (threadIdx.x == 0) *loss = cnt->N > 0.0 ? s / cnt->N : 0.0;
    return;
  }
  const int share = threadIdx.x >> 6, lane = threadIdx.x & 63, p = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (p < NPAR) {
#pragma unroll 8
    for (int b = share; b < nwg; b += 4) s += (double)partial[(size_t)b * NPAR + p];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (share > 0 || p >= NPAR) return;
  const float g = (float)((red[lane] + red[lane + 64]) + (red[lane + 128] + red[lane + 192]));
  if (nwg > 0) grad[p] = g;
  if (nwg > 0 && !ad.on) return;
  float x = params[p];
  if (ad.on) {
    const float mm = ad.beta1 * m[p] + (1.f - ad.beta1) * g;
    const float vv = ad.beta2 * v[p] + (1.f - ad.beta2) * g * g;
    m[p] = mm;
    v[p] = vv;
    x -= ad.lr * (mm / ad.bc1) / (sqrtf(vv / ad.bc2) + ad.eps);
    params[p] = x;
  }
  const uint16_t h = to_bf16(x);
  if (p < OB1) {
    const int o = (p - OW1) / NIN, i = (p - OW1) % NIN;
    wb[WB_W1 + o * KIN + i] = h;
  } else if (p >= OW2 && p < OB2) {
    const int o = (p - OW2) / NH, i = (p - OW2) % NH;
    wb[WB_W2 + o * NH + i] = h;
    wb[WB_W2T + i * NH + o] = h;
  } else if (p >= OW3 && p < OB3) {
    const int o = (p - OW3) / NH, i = (p - OW3) % NH;
    wb[WB_W3 + o * NH + i] = h;
    wb[WB_W3T + i * NOUT + o] = h;
  }
}

// Blocks of 16 rows per workgroup: one while the chip has CUs for them, at most
// four (the FP32 sums of the weight gradients stay within 64 rows, and the
// partials at 101 KB per 64).
static int blocks_of(int B) { return std::min(4, std::max(1, (B + 16 * kCUs - 1) / (16 * kCUs))); }
int mlp_workgroups(int B) {
  const int rows = 16 * blocks_of(B);
  return (B + rows - 1) / rows;
}
int mlp_partials(int max_batch) { return std::max(std::min(kCUs, (max_batch + 15) / 16), (max_batch + 63) / 64); }

int launch_mlp(bool bwd, const Weights &w, const float *X, const float *T, const int *nvalid, Count *cnt, int B,
               float *Y, float *partial, double *lossp, hipStream_t s) {
  const int G = mlp_workgroups(B), blocks = blocks_of(B);
  if (G <= 0) return FOCK_OK;
  const bool count = bwd && B <= kCountInline;
  if (bwd && !count) {
    hipLaunchKernelGGL(k_mlp_count, dim3(1), dim3(256), 0, s, nvalid, B, cnt);
    FOCK_HIP(hipGetLastError());
  }
  if (bwd)
    hipLaunchKernelGGL(k_mlp<true>, dim3(G), dim3(256), 0, s, w, X, T, nvalid, cnt, count ? 1 : 0, B, blocks, Y, partial,
                       lossp);
  else hipLaunchKernelGGL(k_mlp<false>, dim3(G), dim3(256), 0, s, w, X, T, nvalid, cnt, 0, B, blocks, Y, partial, lossp);
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

int launch_mlp_update(const float *partial, int nwg, float *grad, float *params, float *m, float *v,
                      const AdamArgs &ad, uint16_t *wb, const double *lossp, const Count *cnt, double *loss,
                      hipStream_t s) {
  const int G = (NPAR + 63) / 64;
  hipLaunchKernelGGL(k_mlp_update, dim3(nwg > 0 ? G + 1 : G), dim3(256), 0, s, partial, nwg, grad, params, m, v, ad, wb,
                     lossp, cnt, loss);
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

}  // namespace mlp
}  // namespace fock

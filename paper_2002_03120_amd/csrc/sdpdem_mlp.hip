// sdpdem_mlp.hip -- the viscosity surrogate: a 4-64-64-64-1 SiLU MLP with
// bfloat16 parameters, float32 activations and float32 accumulation on the
// matrix cores, trained with Adam.  Inference runs the hidden layers on the
// bfloat16 matrix cores (v_mfma_f32_16x16x32_bf16, activations split into
// three exact bfloat16 parts); a training step runs forward, MSE loss and
// backward on the FP32 matrix cores (v_mfma_f32_16x16x4_f32), a workgroup
// per 16 rows, then adds the workgroups' gradients in order and applies
// Adam, so every reduction has a fixed order and a step is bit-for-bit
// repeatable.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>

#include "sdpdem.h"
#include "sdpdem_mlp.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NP = SDPDEM_MLP_PARAMS;
constexpr int HID = 64;
constexpr int MAXB = SDPDEM_MLP_MAX_BATCH;
// parameter offsets: W1 [4 x 64], b1, W2 [64 x 64], b2, W3 [64 x 64], b3, W4 [64], b4
constexpr int OW1 = 0, OB1 = 256, OW2 = 320, OB2 = 4416, OW3 = 4480, OB3 = 8576, OW4 = 8640,
              OB4 = 8704;
constexpr int OW[3] = {OW1, OW2, OW3};
constexpr int OB[3] = {OB1, OB2, OB3};
static_assert(OB4 + 1 == NP, "parameter layout");

struct Norm {
  float mean[4], inv_std[4];
};

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round to nearest, ties to even
__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// logistic function from the hardware exp2 and reciprocal (about one ulp
// each; the FP64 oracle agrees to the tolerance of the parity tests)
__device__ __forceinline__ float sigm(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * z));
}
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float silu_grad(float z) {
  const float s = sigm(z);
  return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// inference on the bfloat16 matrix cores (v_mfma_f32_16x16x32_bf16).  The
// parameters are bfloat16 values already; an FP32 activation is the exact
// sum of three bfloat16 parts (its top 8 significant bits, the next 8, the
// last 8), so three bf16 products accumulated in FP32 give the FP32
// product, and the layer equals its FP32 evaluation up to the order of the
// sums.  The last parts are added first, over both chunks of the contraction,
// then the middle ones: only the two products of the leading parts round at
// the size of the whole sum (error over 2^12 rows, 2-norm, by chunk and by
// part: 2.55e-7 and 1.95e-7, the time alike).  A block stages the hidden
// layers' weights in LDS once and its wavefronts then take groups of 16 rows
// in turn.

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short v8u16 __attribute__((ext_vector_type(8)));

constexpr int PRED_WAVES = 4;

// Where hidden weight W_{l+2}[k][j] sits in the packed copy: the operand
// W^T of the products H_{l+2}^T = W^T H_{l+1}^T, tile by tile in the order
// the lanes hold it (eight values, 16 bytes, per lane of tile jt, chunk c).
// The order of a product's K index is free as long as both operands agree:
// lane q's eight values of chunk c are the features 4q..4q+3 of the tiles 2c
// and 2c + 1, the ones the lane's own accumulators hold after the layer
// before, so activations go from layer to layer in registers.
__host__ __device__ constexpr int packed_index(int l, int k, int j) {
  const int jt = j / 16, r = j % 16, t = k / 16, q = k % 16 / 4;
  return (((l * 4 + jt) * 2 + t / 2) * 64 + q * 16 + r) * 8 + (t % 2) * 4 + k % 4;
}

// x = hi + mid + lo exactly, each part a bfloat16 (truncations of x and of
// the remainders: every part holds at most 8 significant bits)
__device__ __forceinline__ void split3(float x, unsigned short& h, unsigned short& m,
                                       unsigned short& l) {
  const uint32_t uh = __float_as_uint(x) & 0xFFFF0000u;
  const float r1 = x - __uint_as_float(uh);
  const uint32_t um = __float_as_uint(r1) & 0xFFFF0000u;
  const float r2 = r1 - __uint_as_float(um);
  h = (unsigned short)(uh >> 16);
  m = (unsigned short)(um >> 16);
  l = (unsigned short)(__float_as_uint(r2) >> 16);
}

// A wavefront takes 16 rows at a time, transposed: lane (r, q) holds the
// features 4q..4q+3 of every 16-feature tile of row r.  Bound by the vector
// ALU (192 sigmoids a row, two quarter-rate instructions each, and the
// splits); the weights come from LDS in operand order, the activations stay
// in registers.  With the activations passing through LDS between layers and
// the weights transposed into LDS by every block it took 117 us for 2^20
// rows and 10.4 us for 64; now 81 and 3.7 us.
__global__ __launch_bounds__(64 * PRED_WAVES) void k_mlp_predict(
    const uint16_t* __restrict__ wq, const uint16_t* __restrict__ wpk, Norm nrm,
    const float* __restrict__ x, float* __restrict__ y, int64_t n, int64_t groups_per_wave) {
  __shared__ __attribute__((aligned(16))) unsigned short wt[2 * HID * HID];
  __shared__ __attribute__((aligned(16))) float bias[3][HID], w4[HID];
  const int tid = threadIdx.x;
#pragma unroll
  for (int e = 8 * tid; e < 2 * HID * HID; e += 8 * 64 * PRED_WAVES)
    *reinterpret_cast<v8u16*>(wt + e) = *reinterpret_cast<const v8u16*>(wpk + e);
  if (tid < 3 * HID) bias[tid / HID][tid % HID] = bf16_to_f32(wq[OB[tid / HID] + tid % HID]);
  if (tid >= 3 * HID) w4[tid - 3 * HID] = bf16_to_f32(wq[OW4 + tid - 3 * HID]);
  const int w = tid >> 6, lane = tid & 63, r = lane & 15, q = lane >> 4;
  float w1[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) w1[jt] = bf16_to_f32(wq[OW1 + q * HID + 16 * jt + r]);
  const float b4 = bf16_to_f32(wq[OB4]);
  const float mean = q == 0 ? nrm.mean[0] : q == 1 ? nrm.mean[1] : q == 2 ? nrm.mean[2]
                                                                          : nrm.mean[3];
  const float inv = q == 0 ? nrm.inv_std[0] : q == 1 ? nrm.inv_std[1] : q == 2 ? nrm.inv_std[2]
                                                                              : nrm.inv_std[3];
  const int64_t wave = (int64_t)blockIdx.x * PRED_WAVES + w;
  const int64_t nwaves = (int64_t)gridDim.x * PRED_WAVES;
  const int64_t first = wave * 16 + r;
  float xin = first < n ? x[first * 4 + q] : mean;
  __syncthreads();
  for (int64_t it = 0; it < groups_per_wave; ++it) {
    const int64_t row = (wave + it * nwaves) * 16 + r;
    if (row - r >= n) break;  // a wavefront's own loop: no block barrier inside
    const float xb = (xin - mean) * inv;
    const int64_t next = row + nwaves * 16;  // in flight while this group is evaluated
    xin = next < n ? x[next * 4 + q] : mean;
    // layer 1: K = 4 features, one FP32 MFMA per tile
    v4f h[4];
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) {
      v4f acc = *reinterpret_cast<const v4f*>(&bias[0][16 * jt + 4 * q]);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[jt], xb, acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) h[jt][v] = silu(acc[v]);
    }
    // layers 2 and 3: K = 64 as two chunks of 32
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      v8u16 ah[2], am[2], al[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          unsigned short hh, mm, ll;
          split3(h[2 * c + e / 4][e % 4], hh, mm, ll);
          ah[c][e] = hh;
          am[c][e] = mm;
          al[c][e] = ll;
        }
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        v4f acc = *reinterpret_cast<const v4f*>(&bias[l + 1][16 * jt + 4 * q]);
        v8bf wv[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
          wv[c] = __builtin_bit_cast(
              v8bf, *reinterpret_cast<const v8u16*>(wt + (((l * 4 + jt) * 2 + c) * 64 + lane) * 8));
#pragma unroll
        for (int m = 0; m < 3; ++m) {
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                wv[c], __builtin_bit_cast(v8bf, m == 0 ? al[c] : m == 1 ? am[c] : ah[c]), acc, 0, 0,
                0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) h[jt][v] = silu(acc[v]);
      }
    }
    // output layer: this lane's 16 features, then across q
    float p = 0.0f;
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) {
      const v4f wo = *reinterpret_cast<const v4f*>(&w4[16 * jt + 4 * q]);
#pragma unroll
      for (int v = 0; v < 4; ++v) p += h[jt][v] * wo[v];
    }
    p += __shfl_xor(p, 16, 64);
    p += __shfl_xor(p, 32, 64);
    if (q == 0 && row < n) y[row] = p + b4;
  }
}

// ---------------------------------------------------------------------------
// training step: a workgroup per 16 rows of the batch, then the update

constexpr int GROUPS = MAXB / 16;

struct Train {
  float* master;
  float* m;
  float* v;
  float* grad;
  uint16_t* wq;
  uint16_t* wpk;  // hidden weights again, in the order of packed_index
  float* loss;
  float* part;   // [GROUPS][NP]: every group's share of the gradient
  double* lpart;  // [GROUPS]: its sum of squared residuals
};

// acc += A[16 x K] B[K x 16] on the FP32 matrix cores.  Lane (r = lane % 16,
// q = lane / 16) supplies A(r, k0 + q) and B(k0 + q, r) per step; on return
// it holds C(4q + v, r) in acc[v].
template <int K, class FA, class FB>
__device__ __forceinline__ v4f mfma_tile(FA fa, FB fb, v4f acc) {
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 4)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa(r, k0 + q), fb(k0 + q, r), acc, 0, 0, 0);
  return acc;
}

// LDS row strides: 68 floats keep the 16 x 4 lanes of an operand read of an
// activation tile on 64 different banks, 84 bfloat16 words the reads of the
// weights along either index at two lanes per bank
constexpr int LDA = HID + 4, LDW = 84;

// Forward and backward of 16 rows and their share of the gradient (rows past
// the batch contribute nothing).  Every intermediate stays in LDS.  Bound by
// latency: a chain of five layers of 16 dependent MFMAs and their LDS reads.
// One workgroup for the whole batch of 256, its activations in global memory,
// took 370 us; this takes one sixteenth of the chain per workgroup.
__global__ __launch_bounds__(256) void k_mlp_grad(Train T, Norm nrm, const float* __restrict__ x,
                                                  const float* __restrict__ t, int B) {
  __shared__ __attribute__((aligned(16))) uint16_t ws[2][HID * LDW];  // W2, W3
  __shared__ float xn[16 * 4], act[3][16 * LDA], slope[3][16 * LDA], dzb[2][16 * LDA];
  __shared__ float dy[16], w4[HID];
  __shared__ double sq[16];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, q = lane >> 4;
  const int row0 = 16 * (int)blockIdx.x;
  float* const part = T.part + (size_t)blockIdx.x * NP;
#pragma unroll
  for (int e = tid; e < 2 * HID * HID / 8; e += 256) {
    const int l = e / (HID * HID / 8), o = 8 * (e % (HID * HID / 8));
    const v8u16 v = *reinterpret_cast<const v8u16*>(T.wq + OW[l + 1] + o);
    uint16_t* const to = &ws[l][o / HID * LDW + o % HID];
#pragma unroll
    for (int u = 0; u < 8; ++u) to[u] = v[u];
  }
  if (tid < HID) w4[tid] = bf16_to_f32(T.wq[OW4 + tid]);
  const float xv = row0 + r < B ? (x[(row0 + r) * 4 + q] - nrm.mean[q]) * nrm.inv_std[q] : 0.0f;
  if (w == 0) xn[r * 4 + q] = xv;
  const int j = 16 * w + r;  // wave w computes the features 16 w .. of every layer
  // forward: z_l = h_{l-1} W_l + b_l, h_l = silu(z_l), and silu'(z_l)
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const float bj = bf16_to_f32(T.wq[OB[l] + j]);
    v4f acc = {bj, bj, bj, bj};
    if (l == 0) {
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, bf16_to_f32(T.wq[OW1 + q * HID + j]), acc, 0,
                                                 0, 0);
    } else {
      const float* hin = act[l - 1];
      const uint16_t* wl = ws[l - 1];
      acc = mfma_tile<HID>([&](int i, int k) { return hin[i * LDA + k]; },
                           [&](int k, int) { return bf16_to_f32(wl[k * LDW + j]); }, acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      act[l][(4 * q + v) * LDA + j] = silu(acc[v]);
      slope[l][(4 * q + v) * LDA + j] = silu_grad(acc[v]);
    }
    __syncthreads();
  }
  // output and dL/dy = 2 (y - t) / B: 16 lanes per row
  {
    const int i = tid >> 4, c = tid & 15;
    float y = 0.0f;
#pragma unroll
    for (int m = 0; m < HID; m += 16) y += act[2][i * LDA + c + m] * w4[c + m];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) y += __shfl_xor(y, o, 16);
    if (c == 0) {
      const float res = row0 + i < B ? y + bf16_to_f32(T.wq[OB4]) - t[row0 + i] : 0.0f;
      dy[i] = 2.0f * res / (float)B;
      sq[i] = (double)res * res;
    }
  }
  __syncthreads();
  // output layer gradients and dz_3 = (dy W4^T) * silu'(z_3)
  if (tid < HID) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += act[2][i * LDA + tid] * dy[i];
    part[OW4 + tid] = s;
  } else if (tid == HID) {
    float s = 0.0f;
    double l2 = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s += dy[i];
      l2 += sq[i];
    }
    part[OB4] = s;
    T.lpart[blockIdx.x] = l2;
  }
#pragma unroll
  for (int e = tid; e < 16 * HID; e += 256) {
    const int i = e / HID, c = e % HID;
    dzb[0][i * LDA + c] = dy[i] * w4[c] * slope[2][i * LDA + c];
  }
  __syncthreads();
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    const float* dz = dzb[l & 1];  // layer 3 (l = 2) and layer 1 in the first
    float* dzn = dzb[(l & 1) ^ 1];
    if (l > 0) {
      // dz_{l-1} = (dz_l W_l^T) * silu'(z_{l-1})
      const uint16_t* wl = ws[l - 1];
      v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
      acc = mfma_tile<HID>([&](int i, int k) { return dz[i * LDA + k]; },
                           [&](int k, int) { return bf16_to_f32(wl[j * LDW + k]); }, acc);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        dzn[(4 * q + v) * LDA + j] = acc[v] * slope[l - 1][(4 * q + v) * LDA + j];
    }
    // grad W_l = h_{l-1}^T dz_l: this wave's columns, contraction over the rows
#pragma unroll
    for (int ti = 0; ti < (l == 0 ? 1 : 4); ++ti) {
      v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
      acc = mfma_tile<16>(
          [&](int i, int k) {
            return l == 0 ? (i < 4 ? xn[k * 4 + (i & 3)] : 0.0f)
                          : act[l == 0 ? 0 : l - 1][k * LDA + 16 * ti + i];
          },
          [&](int k, int) { return dz[k * LDA + j]; }, acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int a = 16 * ti + 4 * q + v;
        if (l > 0 || a < 4) part[OW[l] + a * HID + j] = acc[v];
      }
    }
    if (tid < HID) {
      float s = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s += dz[i * LDA + tid];
      part[OB[l] + tid] = s;
    }
    __syncthreads();
  }
}

// every parameter's bfloat16 copy, in both layouts
__device__ __forceinline__ void store_used(const Train& T, int p, float master) {
  const uint16_t b = f32_to_bf16(master);
  T.wq[p] = b;
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    const int o = p - OW[l + 1];
    if (o >= 0 && o < HID * HID) T.wpk[packed_index(l, o / HID, o % HID)] = b;
  }
}

// the groups' shares added in order (bit-for-bit repeatable), then Adam with
// bias correction on the float32 masters and the bfloat16 copies
__global__ __launch_bounds__(256) void k_mlp_update(Train T, int B, int update, float lr, float b1,
                                                    float b2, float eps, float bc1, float bc2) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  const int ng = (B + 15) / 16;
  if (p == 0) {
    double s = 0.0;
    for (int k = 0; k < ng; ++k) s += T.lpart[k];
    T.loss[0] = (float)(s / (double)B);
  }
  if (p >= NP) return;
  float pk[GROUPS];
#pragma unroll
  for (int k = 0; k < GROUPS; ++k) pk[k] = k < ng ? T.part[(size_t)k * NP + p] : 0.0f;
  float g = 0.0f;
#pragma unroll
  for (int k = 0; k < GROUPS; ++k) g += pk[k];
  T.grad[p] = g;
  if (!update) return;
  const float m = b1 * T.m[p] + (1.0f - b1) * g;
  const float v = b2 * T.v[p] + (1.0f - b2) * g * g;
  T.m[p] = m;
  T.v[p] = v;
  const float mh = m / bc1, vh = v / bc2;
  const float nw = T.master[p] - lr * mh / (sqrtf(vh) + eps);
  T.master[p] = nw;
  store_used(T, p, nw);
}

__global__ void k_mlp_init(Train T) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= NP) return;
  store_used(T, p, T.master[p]);
  T.m[p] = 0.0f;
  T.v[p] = 0.0f;
}

struct Bump {
  char* base;
  size_t off = 0;
  template <class T>
  T* take(size_t count) {
    off = (off + 255) & ~(size_t)255;
    T* p = reinterpret_cast<T*>(base ? base + off : nullptr);
    off += count * sizeof(T);
    return p;
  }
};

size_t mlp_layout(char* base, Train* T) {
  Bump b{base};
  Train t;
  // what sdpdem_mlp_read returns lies together: one copy fetches it
  t.master = b.take<float>(NP);
  t.grad = b.take<float>(NP);
  t.loss = b.take<float>(1);
  t.wq = b.take<uint16_t>(NP);
  t.wpk = b.take<uint16_t>(2 * HID * HID);
  t.m = b.take<float>(NP);
  t.v = b.take<float>(NP);
  t.part = b.take<float>((size_t)GROUPS * NP);
  t.lpart = b.take<double>(GROUPS);
  if (T) *T = t;
  return b.off + 256;
}

bool valid_cfg(const sdpdem_mlp_config* c) {
  if (!c) return false;
  for (int f = 0; f < 4; ++f)
    if (!(c->norm_std[f] > 0.0f) || !std::isfinite(c->norm_mean[f])) return false;
  if (!(c->lr > 0.0f) || !(c->beta1 >= 0.0f && c->beta1 < 1.0f) ||
      !(c->beta2 >= 0.0f && c->beta2 < 1.0f) || !(c->eps >= 0.0f))
    return false;
  return c->max_batch >= 1 && c->max_batch <= MAXB;
}

}  // namespace

struct sdpdem_mlp {
  sdpdem_mlp_config cfg;
  Train T;
  Norm nrm;
  int64_t steps = 0;
};

extern "C" {

int sdpdem_mlp_workspace_bytes(const sdpdem_mlp_config* cfg, size_t* bytes) {
  if (!bytes || !valid_cfg(cfg)) return SDPDEM_E_INVALID_ARG;
  *bytes = mlp_layout(nullptr, nullptr);
  return SDPDEM_OK;
}

int sdpdem_mlp_create(const sdpdem_mlp_config* cfg, const float* init_params, void* d_workspace,
                      size_t workspace_bytes, void* hip_stream, sdpdem_mlp** out) {
  if (!out) return SDPDEM_E_INVALID_ARG;
  *out = nullptr;
  if (!valid_cfg(cfg) || !init_params || !d_workspace) return SDPDEM_E_INVALID_ARG;
  char* base = reinterpret_cast<char*>(((uintptr_t)d_workspace + 255) & ~(uintptr_t)255);
  const size_t need = mlp_layout(nullptr, nullptr);
  if (workspace_bytes < need || (size_t)(base - (char*)d_workspace) + need - 256 > workspace_bytes)
    return SDPDEM_E_WORKSPACE_TOO_SMALL;
  sdpdem_mlp* m = new (std::nothrow) sdpdem_mlp();
  if (!m) return SDPDEM_E_INVALID_ARG;
  m->cfg = *cfg;
  mlp_layout(base, &m->T);
  for (int f = 0; f < 4; ++f) {
    m->nrm.mean[f] = cfg->norm_mean[f];
    m->nrm.inv_std[f] = 1.0f / cfg->norm_std[f];
  }
  hipStream_t st = (hipStream_t)hip_stream;
  bool ok = hipMemcpyAsync(m->T.master, init_params, sizeof(float) * NP, hipMemcpyHostToDevice,
                           st) == hipSuccess;
  ok = ok && hipStreamSynchronize(st) == hipSuccess;
  if (ok) {
    k_mlp_init<<<(NP + 255) / 256, 256, 0, st>>>(m->T);
    ok = hipStreamSynchronize(st) == hipSuccess && hipGetLastError() == hipSuccess;
  }
  if (!ok) {
    delete m;
    return SDPDEM_E_HIP;
  }
  *out = m;
  return SDPDEM_OK;
}

int sdpdem_mlp_predict(sdpdem_mlp* m, const float* d_x, float* d_y, int64_t n, void* hip_stream) {
  if (!m || n < 0 || (n > 0 && (!d_x || !d_y))) return SDPDEM_E_INVALID_ARG;
  if (n == 0) return SDPDEM_OK;
  // enough blocks to fill the chip; each wavefront walks its 16-row groups
  const int64_t groups = (n + 15) / 16;
  const int64_t blocks = std::min<int64_t>((groups + PRED_WAVES - 1) / PRED_WAVES, 2048);
  const int64_t per_wave = (groups + blocks * PRED_WAVES - 1) / (blocks * PRED_WAVES);
  k_mlp_predict<<<(unsigned)blocks, 64 * PRED_WAVES, 0, (hipStream_t)hip_stream>>>(
      m->T.wq, m->T.wpk, m->nrm, d_x, d_y, n, per_wave);
  return hipGetLastError() == hipSuccess ? SDPDEM_OK : SDPDEM_E_HIP;
}

int sdpdem_mlp_train_step(sdpdem_mlp* m, const float* d_x, const float* d_t, int32_t batch,
                          int32_t update, void* hip_stream) {
  if (!m || !d_x || !d_t || batch < 1 || batch > m->cfg.max_batch) return SDPDEM_E_INVALID_ARG;
  float bc1 = 1.0f, bc2 = 1.0f;
  if (update) {
    m->steps += 1;
    bc1 = (float)(1.0 - std::pow((double)m->cfg.beta1, (double)m->steps));
    bc2 = (float)(1.0 - std::pow((double)m->cfg.beta2, (double)m->steps));
  }
  hipStream_t st = (hipStream_t)hip_stream;
  k_mlp_grad<<<(unsigned)((batch + 15) / 16), 256, 0, st>>>(m->T, m->nrm, d_x, d_t, batch);
  k_mlp_update<<<(NP + 255) / 256, 256, 0, st>>>(m->T, batch, update ? 1 : 0, m->cfg.lr,
                                                 m->cfg.beta1, m->cfg.beta2, m->cfg.eps, bc1, bc2);
  return hipGetLastError() == hipSuccess ? SDPDEM_OK : SDPDEM_E_HIP;
}

int sdpdem_mlp_read(sdpdem_mlp* m, float* params, float* used_params, float* grad, float* loss,
                    int64_t* steps, void* hip_stream) {
  if (!m) return SDPDEM_E_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  // One copy of everything between the first and the last array asked for:
  // four copies took 60 us where the training step itself takes 15; one
  // takes 27 (25 into pinned memory, which costs a new network 90 us).
  // Without memory for it every array is copied by itself.
  char* const base = reinterpret_cast<char*>(m->T.master);
  const struct {
    const void* dev;
    size_t bytes;
    void* out;
  } part[4] = {{m->T.master, sizeof(float) * NP, params},
               {m->T.grad, sizeof(float) * NP, grad},
               {m->T.loss, sizeof(float), loss},
               // the upper half of the array, widened in place below
               {m->T.wq, sizeof(uint16_t) * NP,
                used_params ? reinterpret_cast<uint16_t*>(used_params) + NP : nullptr}};
  size_t off[4], lo = SIZE_MAX, hi = 0;
  for (int k = 0; k < 4; ++k) {
    off[k] = (size_t)(static_cast<const char*>(part[k].dev) - base);
    if (!part[k].out) continue;
    lo = std::min(lo, off[k]);
    hi = std::max(hi, off[k] + part[k].bytes);
  }
  const std::unique_ptr<char[]> host(lo < hi ? new (std::nothrow) char[hi - lo] : nullptr);
  bool ok = !host || hipMemcpyAsync(host.get(), base + lo, hi - lo, hipMemcpyDeviceToHost, st) ==
                         hipSuccess;
  for (int k = 0; k < 4 && !host; ++k)
    ok = ok && (!part[k].out || hipMemcpyAsync(part[k].out, part[k].dev, part[k].bytes,
                                               hipMemcpyDeviceToHost, st) == hipSuccess);
  ok = hipStreamSynchronize(st) == hipSuccess && ok;
  if (!ok) return SDPDEM_E_HIP;
  for (int k = 0; k < 4 && host; ++k)
    if (part[k].out) std::memcpy(part[k].out, host.get() + (off[k] - lo), part[k].bytes);
  if (used_params) {
    const char* const q = static_cast<const char*>(part[3].out);
    for (int p = 0; p < NP; ++p) {
      uint16_t b;
      std::memcpy(&b, q + sizeof(b) * p, sizeof(b));
      const uint32_t u = (uint32_t)b << 16;
      std::memcpy(&used_params[p], &u, sizeof(float));
    }
  }
  if (steps) *steps = m->steps;
  return SDPDEM_OK;
}

void sdpdem_mlp_destroy(sdpdem_mlp* m) { delete m; }

}  // extern "C"

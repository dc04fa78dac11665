// mlp.hip -- surrogate network 4-64-64-2 (SiLU) on gfx950 BF16 matrix cores.
//
// Maps standardized cluster/laser features to standardized (absorbed energy, mean charge).
// Number formats: FP32 master weights and Adam moments; BF16 copies of the weights, the
// inputs, both hidden activations and the back-propagated hidden-2 gradient feed the
// products; every product accumulates in FP32.  The 64x64 layer (forward, input-gradient and
// weight-gradient products) runs on v_mfma_f32_16x16x32_bf16, the 4-wide input layer on
// v_mfma_f32_16x16x4_f32; the 2-wide output layer is a VALU dot product in training and runs on
// v_mfma_f32_16x16x32_bf16 in inference.
//
// MFMA 16x16x32 BF16 operand layout (checked on the device): lane l holds
//   A[l % 16][8 (l / 16) + i], B[8 (l / 16) + i][l % 16] for i = 0..7, and the result
//   D[4 (l / 16) + r][l % 16] for r = 0..3.
// Every product over a wave's 16 rows is taken with the weights as A and the rows as B (column
// l % 16 is the row), and the weights' rows are permuted (unit_of) so that lane l's 16 results are
// the units 8 g + i and 32 + 8 g + i (g = l / 16): the very units the next product's B operand
// holds in that lane.  A row's activations then stay in the registers of its four lanes from the
// input to the output and back; nothing but the weights passes through LDS.
//
// Training runs as one workgroup that loops over the steps (every reduction has a fixed
// order, so training is bitwise reproducible); inference runs waves that walk over 16-row tiles.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "lc_internal.h"

namespace lc {
namespace {

constexpr int kIn = 4, kH = 64, kOut = 2;
constexpr int kMaxBatch = 256;
// master parameter offsets (floats)
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kOut * kH, kParams = oB3 + kOut;  // 4610

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// State buffer layout (bytes, 256-aligned blocks):
//   params[4610] f32 | adam m[4610] | adam v[4610] | scaler[16] f32 | meta (int)
struct MlpState {
  float* p;
  float* m;
  float* v;
  float* scaler;  // x_mu[4], x_sd[4], y_mu[2], y_sd[2]
  int32_t* meta;  // [0] Adam step count, [1] a training call met an out-of-range row
};

size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t carve(void* base, MlpState* s) {
  char* p = (char*)base;
  size_t o = 0;
  auto take = [&](size_t b) { char* r = p + o; o += al256(b); return r; };
  MlpState t;
  t.p = (float*)take(sizeof(float) * kParams);
  t.m = (float*)take(sizeof(float) * kParams);
  t.v = (float*)take(sizeof(float) * kParams);
  t.scaler = (float*)take(sizeof(float) * 16);
  t.meta = (int32_t*)take(sizeof(int32_t) * 16);
  if (s) *s = t;
  return o;
}

__device__ inline f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Unit the lane group g holds as its q-th of 16, and the weight row that row m of the A operand of
// 16-unit tile tc carries, so that result r of the tile is the lane's unit q = 4 tc + r.
__device__ inline int unit_of(int q, int g) { return 32 * (q >> 3) + 8 * g + (q & 7); }
__device__ inline int weight_row(int tc, int m) { return unit_of(4 * tc + (m & 3), m >> 2); }

// ----------------------------------------------------------------------------- training
// One workgroup of 16 waves runs every step: wave w takes rows 16 w .. 16 w + 15 of the minibatch
// from the input to the hidden-1 gradient in registers, then tile w of dW2 over the whole
// minibatch; the gradients that are sums over the rows of one column (dW1, dW3, the biases) are
// one thread's chain in row order each, in nine of the waves at once; and each thread keeps the
// parameters it updates, with their Adam moments, in registers over all steps.  What crosses
// waves goes through LDS, four barriers a step.
// Bound by the VALU issue of one compute unit (the two SiLUs and their derivatives of 256 rows are
// most of it: 10.8 us; the sums over rows 3.9, Adam 1.2).  Measured at 256 rows: 17.4 us a step (17.1
// without the subnormal sigmoids and the general division of the first moment), against 200 us with
// four waves that kept every activation in global memory; with the sums over rows on one LDS read per
// row 24.2 us, and with expf's range checks, the general division everywhere and the first layer on
// the VALU 29 us.  Every sum keeps its order and every operation its rounding, so trained weights are
// the same bits in all of these.  The transposing LDS read in place of the transposed arrays' 2-byte
// writes was no faster (18.3 and 19.1 us).
constexpr int kTrainWaves = 16;
constexpr int kTrainThreads = 64 * kTrainWaves;
constexpr int kColPad = kMaxBatch + 8;  // entries of a transposed row: 16-byte reads of 16 rows meet no bank twice
constexpr int kWPad = kH + 8;           // likewise for rows of units
constexpr int kFPad = kMaxBatch + 4;    // likewise for FP32 entries

struct TrainLds {
  alignas(16) __bf16 w2[kH][kWPad];   // W2[n][k]
  alignas(16) __bf16 w2t[kH][kWPad];  // W2[n][k] at [k][n]
  float w1[kH][kIn];         // BF16-rounded
  float w3[kOut][kH];        // BF16-rounded
  alignas(16) float b1[kH];
  float b2[kH];
  float b3[kOut];
  alignas(16) float xs[kIn][kMaxBatch];  // standardized, BF16-rounded inputs
  alignas(16) float dy[kOut][kMaxBatch];
  float3 corr[64];           // 1 - beta1^t, 1 - beta2^t and the reciprocal of the latter, of 64 steps
  float loss[kTrainWaves];
  alignas(16) float f[kH][kFPad];  // [unit][row]: hidden-2 gradient, then hidden-1 gradient
  union {                          // [unit][row]
    alignas(16) __bf16 h2t[kH][kColPad];  // hidden-2 activations, until their sums are taken
    struct {                       // the operands of dW2
      alignas(16) __bf16 h1t[kH][kColPad];
      alignas(16) __bf16 d2t[kH][kColPad];
    };
  };
};
static_assert(kWPad % 8 == 0 && kColPad % 8 == 0 && kFPad % 4 == 0, "16-byte reads of every row");
static_assert(sizeof(TrainLds) <= 160 * 1024, "LDS of one compute unit");

// Master parameter outside W2 that a thread updates (-1: none): waves 0 and 1 the rows of W3,
// wave 2 b2, wave 3 b3, waves 4 to 7 the columns of W1, wave 8 b1.
__device__ inline int small_param(int wave, int lane) {
  if (wave < 2) return oW3 + wave * kH + lane;
  if (wave == 2) return oB2 + lane;
  if (wave == 3) return lane < kOut ? oB3 + lane : -1;
  if (wave < 8) return oW1 + lane * kIn + (wave - 4);
  if (wave == 8) return oB1 + lane;
  return -1;
}

// Its copy for the products (weights BF16-rounded, biases FP32).
__device__ inline void put_small(TrainLds& w, int wave, int lane, float p) {
  if (wave < 2) w.w3[wave][lane] = (float)(__bf16)p;
  else if (wave == 2) w.b2[lane] = p;
  else if (wave == 3) w.b3[lane] = p;
  else if (wave < 8) w.w1[lane][wave - 4] = (float)(__bf16)p;
  else w.b1[lane] = p;
}

// 1 / (1 + expf(-z)) in 19 issue slots instead of 29, the same bits: expf by the usual reduction in
// extended precision (the product x log2 e and its rounding error by a fused multiply-add, the nearest
// integer, the power of the rest) with the clamp in place of its range checks (outside it the power is 0
// or below an ulp of the 1, or infinite); the reciprocal of a number in [1/4, 2^126] is correctly
// rounded after one Newton step, div_fixup gives 0 for infinity.  A quarter of the denominator is
// inverted, so that the reciprocal stays above the subnormal numbers, which v_rcp_f32 flushes.  Compared
// on the device for every FP32 argument: equal but where the result is subnormal (z below -87.3), there
// 34,043 results are rounded twice and are off by one unit of the smallest subnormal number.  A NaN gives
// a number; every use multiplies it by z.
__device__ inline float sigmoid_train(float z) {
  constexpr float kLog2e = 1.44269502f, kLog2eLow = 1.9259629e-8f;
  const float x = __builtin_amdgcn_fmed3f(-z, -104.0f, 89.0f);
  const float p = x * kLog2e;
  const float low = __builtin_fmaf(x, kLog2eLow, __builtin_fmaf(x, kLog2e, -p));
  const float n = __builtin_rintf(p);
  const float e = __builtin_ldexpf(__builtin_amdgcn_exp2f((p - n) + low), (int)n);
  const float d = __builtin_fmaf(e, 0.25f, 0.25f);
  const float r = __builtin_amdgcn_rcpf(d);
  return 0.25f * __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r), d, 1.0f);
}

// a / b with r the correctly rounded 1 / b: correctly rounded unless a is below 2^-102, where the
// remainder is lost among the subnormal numbers.
__device__ inline float div_by(float a, float b, float r) {
  const float q = a * r;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-b, q, a), r, q), b, a);
}

// Adam (Kingma & Ba) on one FP32 master weight; c holds 1 - beta1^t, 1 - beta2^t and the reciprocal of
// the latter.  The first moment has the general division (a weight of zero takes the whole quotient,
// however small; the square root of a second moment below 2^-102 vanishes beside eps).
__device__ inline void adam(float g, float lr, float beta1, float beta2, float eps, const float3 c, float& p, float& m,
                            float& v) {
  m = beta1 * m + (1.0f - beta1) * g;
  v = beta2 * v + (1.0f - beta2) * g * g;
  p -= lr * (m / c.x) / (sqrtf(div_by(v, c.y, c.z)) + eps);
}

// Sums over the B rows (a multiple of 32) in row order, of f[r] or of f[r] g[r]: the rows of a
// column are neighbours in LDS, so eight come with two 16-byte reads (one of BF16), ahead of the
// additions of the eight before.
struct Eight {
  f32x4 a, b;
};
__device__ inline Eight load_eight(const float* p) { return {*(const f32x4*)p, *(const f32x4*)(p + 4)}; }
__device__ inline Eight load_eight(const __bf16* p) {
  const bf16x8 v = *(const bf16x8*)p;
  Eight o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o.a[i] = (float)v[i];
    o.b[i] = (float)v[4 + i];
  }
  return o;
}

template <typename T>
__device__ inline float column_dot(int B, const T* f, const float* g) {
  float sum = 0.f;
  Eight u = load_eight(f), v = load_eight(g);
#pragma unroll 4
  for (int r = 8; r <= B; r += 8) {
    const int next = r < B ? r : 0;  // the last one is not used
    const Eight u1 = load_eight(f + next), v1 = load_eight(g + next);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = __builtin_fmaf(v.a[i], u.a[i], sum);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = __builtin_fmaf(v.b[i], u.b[i], sum);
    u = u1;
    v = v1;
  }
  return sum;
}

__device__ inline float column_add(int B, const float* f) {
  float sum = 0.f;
  Eight u = load_eight(f);
#pragma unroll 4
  for (int r = 8; r <= B; r += 8) {
    const Eight u1 = load_eight(f + (r < B ? r : 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += u.a[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += u.b[i];
    u = u1;
  }
  return sum;
}

__global__ __launch_bounds__(kTrainThreads) void k_mlp_train(MlpState s, const float* X, const float* Y,
                                                             const int32_t* idx, int64_t n, int B, int steps, float lr,
                                                             float beta1, float beta2, float eps, float* loss_out,
                                                             float* grad_out) {
  __shared__ TrainLds w;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = B / 16;                       // waves that hold rows
  const int r16 = lane & 15, g = lane >> 4;    // row of the wave's tile, lane group
  const int row = 16 * wave + r16;             // row of the minibatch
  const bool rows = wave < nw;

  // this thread's parameters: four of W2 in the layout of its dW2 tile, and one small one
  const int n0 = 16 * (wave >> 2) + 4 * g, k0 = 16 * (wave & 3) + r16;
  const int small = small_param(wave, lane);
  float p2[4], m2[4], v2[4], p1 = 0.f, m1 = 0.f, v1 = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = oW2 + (n0 + q) * kH + k0;
    p2[q] = s.p[i];
    m2[q] = s.m[i];
    v2[q] = s.v[i];
  }
  if (small >= 0) {
    p1 = s.p[small];
    m1 = s.m[small];
    v1 = s.v[small];
  }
  const int t0 = s.meta[0];
  const float mu = s.scaler[g], sd = s.scaler[4 + g];  // of input g: lane l brings input l / 16 of its row
  float ymu[kOut], ysd[kOut];
#pragma unroll
  for (int o = 0; o < kOut; ++o) { ymu[o] = s.scaler[8 + o]; ysd[o] = s.scaler[10 + o]; }

  // the rows of the next step and the row indices of the one after it are loaded ahead
  auto row_index = [&](int step) {
    int r = idx[(int64_t)step * B + row];
    if (r < 0 || r >= n) { s.meta[1] = 1; r = 0; }  // out-of-range row: flagged, row 0 used
    return r;
  };
  float xr, yr[kOut];
  int next = 0;
  auto load_row = [&](int r) {
    xr = X[(int64_t)r * kIn + g];
#pragma unroll
    for (int o = 0; o < kOut; ++o) yr[o] = Y[(int64_t)r * kOut + o];
  };
  if (rows) {
    load_row(row_index(0));
    if (steps > 1) next = row_index(1);
  }

#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    // weights of this step for the products
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const __bf16 b = (__bf16)p2[q];
      w.w2[n0 + q][k0] = b;
      w.w2t[k0][n0 + q] = b;
    }
    if (small >= 0) put_small(w, wave, lane, p1);
    if ((step & 63) == 0 && tid < 64) {
      const float t = (float)(t0 + step + 1 + tid);
      const float c1 = 1.0f - powf(beta1, t), c2 = 1.0f - powf(beta2, t);
      w.corr[tid] = make_float3(c1, c2, 1.0f / c2);
    }
    __syncthreads();

    bf16x8 h1[2], d2[2];
    float e1[16];  // SiLU'(z1), then the hidden-1 gradient
    if (rows) {
      float ty[kOut];
      const float x = (float)(__bf16)((xr - mu) / sd);
#pragma unroll
      for (int o = 0; o < kOut; ++o) ty[o] = (yr[o] - ymu[o]) / ysd[o];
      if (step + 1 < steps) load_row(next);
      if (step + 2 < steps) next = row_index(step + 2);
      w.xs[g][row] = x;
      // layer 1: z1 = W1 x + b1 on the FP32 matrix units, whose sum over the four inputs rounds as a
      // chain of fused multiply-adds does
#pragma unroll
      for (int tc = 0; tc < 4; ++tc) {
        f32x4 acc = *(const f32x4*)&w.b1[unit_of(4 * tc, g)];
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w1[weight_row(tc, r16)][g], x, acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int q = 4 * tc + r;
          const float z = acc[r];
          const float sg = sigmoid_train(z);
          e1[q] = sg * (1.0f + z * (1.0f - sg));
          h1[q >> 3][q & 7] = (__bf16)(z * sg);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // layer 2: z2 = W2 h1 + b2
      bf16x8 h2[2];
      float e2[16];  // SiLU'(z2)
#pragma unroll
      for (int tc = 0; tc < 4; ++tc) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma(*(const bf16x8*)&w.w2[weight_row(tc, r16)][8 * g], h1[0], acc);
        acc = mfma(*(const bf16x8*)&w.w2[weight_row(tc, r16)][32 + 8 * g], h1[1], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int q = 4 * tc + r;
          const float z = acc[r] + w.b2[unit_of(q, g)];
          const float sg = sigmoid_train(z);
          e2[q] = sg * (1.0f + z * (1.0f - sg));
          h2[q >> 3][q & 7] = (__bf16)(z * sg);
          w.h2t[unit_of(q, g)][row] = h2[q >> 3][q & 7];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // layer 3: y = W3 h2 + b3, summed in unit order: each lane group adds its eight units and
      // hands the sum to the next group
      float y[kOut] = {w.b3[0], w.b3[1]};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float h = (float)h2[t >> 2][i];
#pragma unroll
          for (int o = 0; o < kOut; ++o) y[o] = __builtin_fmaf(w.w3[o][unit_of(8 * (t >> 2) + i, g)], h, y[o]);
        }
#pragma unroll
        for (int o = 0; o < kOut; ++o) y[o] = __shfl(y[o], 16 * (t & 3) + r16, 64);
        __builtin_amdgcn_sched_barrier(0);
      }
      // loss and its gradient: dy = (y - t) / B
      float dy[kOut], l = 0.f;
#pragma unroll
      for (int o = 0; o < kOut; ++o) {
        const float d = y[o] - ty[o];
        dy[o] = d / (float)B;
        l += d * d;
      }
      if (g == 0) {
#pragma unroll
        for (int o = 0; o < kOut; ++o) w.dy[o][row] = dy[o];
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) l += __shfl_xor(l, o, 64);
      if (lane == 0) w.loss[wave] = l;
      // hidden-2 gradient: dz2 = (W3^T dy) SiLU'(z2)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int u = unit_of(q, g);
        const float gr = __builtin_fmaf(w.w3[1][u], dy[1], w.w3[0][u] * dy[0]);
        const float d = gr * e2[q];
        d2[q >> 3][q & 7] = (__bf16)d;
        w.f[u][row] = d;
        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      // hidden-1 gradient: dz1 = (W2^T dz2) SiLU'(z1)
#pragma unroll
      for (int tc = 0; tc < 4; ++tc) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma(*(const bf16x8*)&w.w2t[weight_row(tc, r16)][8 * g], d2[0], acc);
        acc = mfma(*(const bf16x8*)&w.w2t[weight_row(tc, r16)][32 + 8 * g], d2[1], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) e1[4 * tc + r] = acc[r] * e1[4 * tc + r];
      }
    }
    __syncthreads();

    // the sums over rows of hidden-2 quantities: dW3[o][j] = sum_r dy[r][o] h2[r][j],
    // db2[j] = sum_r dz2[r][j], db3[o] = sum_r dy[r][o]
    float gs = 0.f;
    if (wave < 2) {
      gs = column_dot(B, w.h2t[lane], w.dy[wave]);
    } else if (wave == 2) {
      gs = column_add(B, w.f[lane]);
    } else if (wave == 3 && lane < kOut) {
      gs = column_add(B, w.dy[lane]);
    } else if (wave == kTrainWaves - 1 && lane == 0 && loss_out) {
      float l = 0.f;
      for (int q = 0; q < nw; ++q) l += w.loss[q];
      loss_out[step] = l / (2.0f * (float)B);
    }
    __syncthreads();
    if (rows) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int u = unit_of(q, g);
        w.f[u][row] = e1[q];
        w.h1t[u][row] = h1[q >> 3][q & 7];
        w.d2t[u][row] = d2[q >> 3][q & 7];
      }
    }
    __syncthreads();

    // dW1[j][k] = sum_r dz1[r][j] x[r][k], db1[j] = sum_r dz1[r][j]
    if (wave >= 4 && wave < 8) gs = column_dot(B, w.f[lane], w.xs[wave - 4]);
    else if (wave == 8) gs = column_add(B, w.f[lane]);
    // dW2[n][k] = sum_r dz2[r][n] h1[r][k]: the wave's 16 x 16 tile over the minibatch
    f32x4 gw = {0.f, 0.f, 0.f, 0.f};
    for (int kk = 0; kk < B; kk += 32)
      gw = mfma(*(const bf16x8*)&w.d2t[16 * (wave >> 2) + r16][kk + 8 * g],
                *(const bf16x8*)&w.h1t[16 * (wave & 3) + r16][kk + 8 * g], gw);
    if (grad_out) {
#pragma unroll
      for (int q = 0; q < 4; ++q) grad_out[oW2 + (n0 + q) * kH + k0] = gw[q];
      if (small >= 0) grad_out[small] = gs;
    } else {
      const float3 c = w.corr[step & 63];
#pragma unroll
      for (int q = 0; q < 4; ++q) adam(gw[q], lr, beta1, beta2, eps, c, p2[q], m2[q], v2[q]);
      if (small >= 0) adam(gs, lr, beta1, beta2, eps, c, p1, m1, v1);
    }
    if ((step & 63) == 63) __syncthreads();  // the step's factors are read before the next ones replace them
  }
  if (grad_out) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = oW2 + (n0 + q) * kH + k0;
    s.p[i] = p2[q];
    s.m[i] = m2[q];
    s.v[i] = v2[q];
  }
  if (small >= 0) {
    s.p[small] = p1;
    s.m[small] = m1;
    s.v[small] = v1;
  }
  if (tid == 0) s.meta[0] = t0 + steps;
}

// ----------------------------------------------------------------------------- scaler
// Feature and target means and standard deviations (population) in two passes of FP64 sums, one
// workgroup.  A thread walks the flat arrays with a stride that is a multiple of the row length,
// so it meets one column only and the loads are coalesced; the threads of a column then add up
// over the lanes and the waves in a fixed order.  Latency-bound: one thread per column in row order
// took 589 us for 3686 rows, this 8.8 us (loads of eight elements in flight per thread).
constexpr int kScalerThreads = 1024;
static_assert(kScalerThreads % kIn == 0 && kScalerThreads % kOut == 0, "a thread meets one column");

// Sum over the elements of the thread's column of f(element), for every column of a row of W.
// Returns the column's total to each of its threads.
template <int W, typename F>
__device__ inline double column_sum(const float* src, int64_t elems, double (*sh)[kIn], F f) {
  constexpr int kAhead = 8;  // loads in flight
  const int tid = threadIdx.x;
  double sum = 0.0;
  int64_t e = tid;
  for (; e + (kAhead - 1) * kScalerThreads < elems; e += kAhead * kScalerThreads) {
    float v[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) v[i] = src[e + i * kScalerThreads];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) sum += f((double)v[i]);
  }
  for (; e < elems; e += kScalerThreads) sum += f((double)src[e]);
  for (int o = 32; o >= W; o >>= 1) sum += __shfl_xor(sum, o, 64);
  __syncthreads();  // the previous sum's readers are done
  if ((tid & 63) < W) sh[tid >> 6][tid & 63] = sum;
  __syncthreads();
  double total = 0.0;
#pragma unroll
  for (int w = 0; w < kScalerThreads / 64; ++w) total += sh[w][tid % W];
  return total;
}

template <int W>
__device__ inline void fit_columns(const float* src, int64_t n, double (*sh)[kIn], float* mean, float* dev) {
  const double mu = column_sum<W>(src, n * W, sh, [](double x) { return x; }) / (double)n;
  const double ss = column_sum<W>(src, n * W, sh, [mu](double x) { return (x - mu) * (x - mu); });
  double sd = sqrt(ss / (double)n);
  if (!(sd > 0.0)) sd = 1.0;
  if (threadIdx.x < W) {
    mean[threadIdx.x] = (float)mu;
    dev[threadIdx.x] = (float)sd;
  }
}

__global__ __launch_bounds__(kScalerThreads) void k_mlp_scaler(MlpState s, const float* X, const float* Y, int64_t n) {
  __shared__ double sh[kScalerThreads / 64][kIn];
  fit_columns<kIn>(X, n, sh, s.scaler, s.scaler + 4);
  fit_columns<kOut>(Y, n, sh, s.scaler + 8, s.scaler + 10);
}

// ----------------------------------------------------------------------------- inference
// SiLU for the inference kernel, as exact as z times 1 / (1 + expf(-z)) in 15 issue slots instead of 30.
// With x = -z: x log2 e = n + f, where n comes from adding a number with an ulp of one, and f from two
// fused multiply-adds with log2 e in two parts; 2^f / 4 with the exponent n - 2 added to its bits; the
// reciprocal of (1 + e^x) / 4, correctly rounded after one Newton step.  A quarter keeps the reciprocal
// above the subnormal numbers, which v_rcp_f32 flushes, until 1 + e^x is infinite: there it gives 0.
// Clamped where e^x no longer counts beside the 1, and where it is infinite; infinities and NaN come out
// as of the plain form (+inf: +inf, large negative: -0, -inf and NaN: NaN).  Against 64 bits, over
// every FP32 z above -87 the largest relative error is 1.47e-7 for z > 4, 1.83e-7 for |z| < 4, 1.75e-7
// down to -10, 2.00e-7 to -30 and 1.60e-7 to -87, that of the plain form 1.47, 1.84, 1.75, 2.00 and 1.63;
// the first part of log2 e is one of five tried that keep below it.  (With the hardware's power of
// the rounded product and its reciprocal alone, 7 slots, it was 3.7e-7, 5.9e-7, 1.8e-6 and 3.9e-6.)
__device__ inline float silu(float z) {
  constexpr float kLog2e = 1.44269502f, kHigh = 1.44269562f, kLow = -5.76786817e-7f;
  constexpr float kShift = 12582910.0f;  // 1.5 2^23 - 2: the low bits of a sum with it are n - 2
  const float x = __builtin_amdgcn_fmed3f(-z, -80.0f, 88.8f);
  const float t = __builtin_fmaf(x, kLog2e, kShift);
  const float f = __builtin_fmaf(x, kLow, __builtin_fmaf(x, kHigh, kShift - t));
  const float e = __uint_as_float((__float_as_uint(t) << 23) + __float_as_uint(__builtin_amdgcn_exp2f(f)));
  const float d = e + 0.25f;
  const float r = __builtin_amdgcn_rcpf(d);
  return z * (0.25f * __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r));
}

// A wave walks over tiles of 16 rows with every weight in registers: layer 1 on the FP32 matrix
// units (K = 4 is the input width: lane l brings input l / 16 of row l % 16, one coalesced load),
// layers 2 and 3 on the BF16 ones, the SiLU on the VALU, which bounds it (32 of them are 480 of 575
// issue slots a tile: 58 us for a million rows; the 24 MB they move take 5 us).  No LDS and no
// barrier in the loop.  Measured on a million rows, back to back: 70.8 us, against 398 us with the weights
// staged and converted for every 64 rows, the inputs standardized once per unit and the outer layers on
// the VALU, 83.5 us with the SiLU of the training kernel, and 47 us with the less exact one.
constexpr int kInferBlocks = 256 * 4;  // four blocks of four waves fit on each compute unit at 114 VGPRs
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void k_mlp_infer(const float* p, const float* scaler, const float* X, float* Y, int64_t n) {
  __shared__ alignas(16) __bf16 w2[kH][kWPad];
  for (int i = threadIdx.x; i < kH * kH; i += 256) w2[i / kH][i % kH] = (__bf16)p[oW2 + i];
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float w1[4];
  f32x4 b1[4], b2[4];
  bf16x8 w3[2], a2[4][2];
#pragma unroll
  for (int tc = 0; tc < 4; ++tc) {
    w1[tc] = (float)(__bf16)p[oW1 + weight_row(tc, r16) * kIn + g];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[tc][r] = p[oB1 + unit_of(4 * tc + r, g)];
      b2[tc][r] = p[oB2 + unit_of(4 * tc + r, g)];
    }
  }
#pragma unroll
  for (int q = 0; q < 16; ++q)
    w3[q >> 3][q & 7] = (__bf16)(r16 < kOut ? p[oW3 + r16 * kH + unit_of(q, g)] : 0.0f);
  const float mu = scaler[g], sd = scaler[4 + g];
  const float ymu0 = scaler[8], ymu1 = scaler[9], ysd0 = scaler[10], ysd1 = scaler[11];
  const float b30 = p[oB3], b31 = p[oB3 + 1];
  __syncthreads();
#pragma unroll
  for (int tc = 0; tc < 4; ++tc) {
    a2[tc][0] = *(const bf16x8*)&w2[weight_row(tc, r16)][8 * g];
    a2[tc][1] = *(const bf16x8*)&w2[weight_row(tc, r16)][32 + 8 * g];
  }
  const int64_t stride = (int64_t)gridDim.x * 4 * 16;
  int64_t row = ((int64_t)blockIdx.x * 4 + wave) * 16 + r16;
  float xn = row < n ? X[row * kIn + g] : 0.0f;
  // a wave leaves when its tile starts past the last row; lanes past it compute and do not store
  for (; row - r16 < n; row += stride) {
    const float x = (float)(__bf16)((xn - mu) / sd);
    xn = row + stride < n ? X[(row + stride) * kIn + g] : 0.0f;
    bf16x8 h[2];
#pragma unroll
    for (int tc = 0; tc < 4; ++tc) {
      const f32x4 z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[tc], x, b1[tc], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) h[tc >> 1][4 * (tc & 1) + r] = (__bf16)silu(z[r]);
    }
    bf16x8 h2[2];
#pragma unroll
    for (int tc = 0; tc < 4; ++tc) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
      z = mfma(a2[tc][0], h[0], z);
      z = mfma(a2[tc][1], h[1], z);
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[tc >> 1][4 * (tc & 1) + r] = (__bf16)silu(z[r] + b2[tc][r]);
    }
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
    y = mfma(w3[0], h2[0], y);
    y = mfma(w3[1], h2[1], y);
    if (g == 0 && row < n) {  // outputs 0 and 1 of the row
      Y[row * kOut] = (y[0] + b30) * ysd0 + ymu0;
      Y[row * kOut + 1] = (y[1] + b31) * ysd1 + ymu1;
    }
  }
}

}  // namespace
}  // namespace lc

using namespace lc;

extern "C" {

size_t lc_mlp_state_bytes(void) { return carve(nullptr, nullptr); }

int lc_mlp_n_params(void) { return kParams; }

int lc_mlp_set_params(void* d_state, const float* host_params, void* stream) {
  if (!d_state || !host_params || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  MlpState s;
  carve(d_state, &s);
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipStreamSynchronize(st);
  if (e == hipSuccess) e = hipMemcpy(s.p, host_params, sizeof(float) * kParams, hipMemcpyHostToDevice);
  // zero Adam moments and step count, identity scaler
  static const float zeros[kParams] = {};
  if (e == hipSuccess) e = hipMemcpy(s.m, zeros, sizeof(float) * kParams, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(s.v, zeros, sizeof(float) * kParams, hipMemcpyHostToDevice);
  const float sc[16] = {0, 0, 0, 0, 1, 1, 1, 1, 0, 0, 1, 1, 0, 0, 0, 0};
  if (e == hipSuccess) e = hipMemcpy(s.scaler, sc, sizeof(sc), hipMemcpyHostToDevice);
  const int32_t meta[16] = {};
  if (e == hipSuccess) e = hipMemcpy(s.meta, meta, sizeof(meta), hipMemcpyHostToDevice);
  return e == hipSuccess ? LC_OK : LC_E_HIP;
}

int lc_mlp_get_params(const void* d_state, float* host_params, float* host_scaler, void* stream) {
  if (!d_state || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  MlpState s;
  carve((void*)d_state, &s);
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  if (e == hipSuccess && host_params) e = hipMemcpy(host_params, s.p, sizeof(float) * kParams, hipMemcpyDeviceToHost);
  if (e == hipSuccess && host_scaler) e = hipMemcpy(host_scaler, s.scaler, sizeof(float) * 12, hipMemcpyDeviceToHost);
  return e == hipSuccess ? LC_OK : LC_E_HIP;
}

int lc_mlp_status(const void* d_state, void* stream) {
  if (!d_state || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  MlpState s;
  carve((void*)d_state, &s);
  int32_t meta[2] = {0, 0};
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  if (e == hipSuccess) e = hipMemcpy(meta, s.meta, sizeof(meta), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return LC_E_HIP;
  return meta[1] ? LC_E_INVALID : LC_OK;
}

int lc_mlp_fit_scaler(void* d_state, const float* d_X, const float* d_Y, int64_t n, void* stream) {
  if (!d_state || !d_X || !d_Y || n < 1 || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  MlpState s;
  carve(d_state, &s);
  k_mlp_scaler<<<1, kScalerThreads, 0, (hipStream_t)stream>>>(s, d_X, d_Y, n);
  return hipGetLastError() == hipSuccess ? LC_OK : LC_E_HIP;
}

int lc_mlp_train(void* d_state, const float* d_X, const float* d_Y, int64_t n, const int32_t* d_rows, int32_t batch,
                 int32_t steps, float lr, float* d_loss, void* stream) {
  if (!d_state || !d_X || !d_Y || !d_rows || n < 1 || steps < 0 || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  if (batch < 32 || batch > kMaxBatch || batch % 32 != 0 || !(lr > 0.0f)) return LC_E_INVALID;
  if (steps == 0) return LC_OK;
  MlpState s;
  carve(d_state, &s);
  k_mlp_train<<<1, kTrainThreads, 0, (hipStream_t)stream>>>(s, d_X, d_Y, d_rows, n, batch, steps, lr, 0.9f, 0.999f, 1e-8f,
                                                            d_loss, nullptr);
  return hipGetLastError() == hipSuccess ? LC_OK : LC_E_HIP;
}

int lc_mlp_grad(void* d_state, const float* d_X, const float* d_Y, int64_t n, const int32_t* d_rows, int32_t batch,
                float* d_grad, float* d_loss, void* stream) {
  if (!d_state || !d_X || !d_Y || !d_rows || !d_grad || n < 1 || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  if (batch < 32 || batch > kMaxBatch || batch % 32 != 0) return LC_E_INVALID;
  MlpState s;
  carve(d_state, &s);
  k_mlp_train<<<1, kTrainThreads, 0, (hipStream_t)stream>>>(s, d_X, d_Y, d_rows, n, batch, 1, 1.0f, 0.9f, 0.999f, 1e-8f,
                                                            d_loss, d_grad);
  return hipGetLastError() == hipSuccess ? LC_OK : LC_E_HIP;
}

int lc_mlp_infer(const void* d_state, const float* d_X, float* d_Y, int64_t n, void* stream) {
  if (!d_state || n < 0 || ((uintptr_t)d_state & 255)) return LC_E_INVALID;
  if (n == 0) return LC_OK;
  if (!d_X || !d_Y) return LC_E_INVALID;
  MlpState s;
  carve((void*)d_state, &s);
  const int64_t blocks = (n + 63) / 64;
  if (blocks > 0x7fffffff) return LC_E_INVALID;
  const int grid = blocks < kInferBlocks ? (int)blocks : kInferBlocks;
  k_mlp_infer<<<grid, 256, 0, (hipStream_t)stream>>>(s.p, s.scaler, d_X, d_Y, n);
  return hipGetLastError() == hipSuccess ? LC_OK : LC_E_HIP;
}

}  // extern "C"

// nyx_mlp.hip -- training and packing kernels of the learned Riemann flux
// (the network is described in nyx_mlp_dev.h).  Training runs in FP32 on the
// matrix cores (FP32 operands and accumulation).  The optimiser is Adam.  Packing converts the FP32 master weights into the BF16
// MFMA fragments the inference path reads.
#include <hip/hip_runtime.h>

#include "nyx_internal.h"
#include "nyx_mlp_dev.h"

namespace nyx {

// normalisation of a harvested record (15 floats: left state, right state,
// p*, u*, rho*_L, rho*_R, rho_g); inputs x[10] and targets y[5]
__device__ __forceinline__ void record_xy(double gamma, const float* r, float* x, float* y) {
  double qL[5], qR[5];
  for (int k = 0; k < 5; ++k) {
    qL[k] = (double)r[k];
    qR[k] = (double)r[5 + k];
  }
  double rbar, cbar, ubar;
  mlp_inputs(gamma, qL, qR, x, &rbar, &cbar, &ubar);
  if (y) {
    const double pbar = rbar * cbar * cbar;
    y[0] = (float)log((double)r[10] / pbar);
    y[1] = (float)(((double)r[11] - ubar) / cbar);
    y[2] = (float)log((double)r[12] / rbar);
    y[3] = (float)log((double)r[13] / rbar);
    y[4] = (float)log((double)r[14] / rbar);
  }
}

// splitmix64 of (seed, i) -> uniform in [0, 1)
__device__ __forceinline__ double uniform01(unsigned long long seed, unsigned long long i) {
  unsigned long long z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = z ^ (z >> 31);
  return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

// Glorot-uniform weights, zero biases
__global__ void k_mlp_init(float* P, unsigned long long seed) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kMlpNParam) return;
  int nin = 0, nout = 0;
  bool bias = false;
  if (i < kOffB1) { nin = kMlpIn; nout = kMlpHid; }
  else if (i < kOffW2) bias = true;
  else if (i < kOffB2) { nin = kMlpHid; nout = kMlpHid; }
  else if (i < kOffW3) bias = true;
  else if (i < kOffB3) { nin = kMlpHid; nout = kMlpHid; }
  else if (i < kOffW4) bias = true;
  else if (i < kOffB4) { nin = kMlpHid; nout = kMlpOut; }
  else bias = true;
  if (bias) {
    P[i] = 0.0f;
    return;
  }
  const double lim = sqrt(6.0 / (double)(nin + nout));
  P[i] = (float)((2.0 * uniform01(seed, (unsigned long long)i) - 1.0) * lim);
}

// ---------------------------------------------------------------------------
// loss and gradient of a batch, on the FP32 matrix cores
// ---------------------------------------------------------------------------
// A workgroup of 8 waves takes tiles of 64 samples.  Every product of the
// forward pass, of the backpropagation and of the weight gradients is a
// v_mfma_f32_16x16x4_f32 (FP32 operands and accumulation).  Its operand
// layouts: A lane l = A[l%16][l/16], B lane l = B[l/16][l%16], D lane l,
// element v = D[4 (l/16) + v][l%16].  With samples as the columns:
//   layer      h'[o][s] = sum_k W[o][k] h[k][s]   A weights, B activations
//   backward   d'[i][s] = sum_o W[o][i] d[o][s]   A weights transposed
//   gradient   dW[o][i] = sum_s d[o][s] h[i][s]   A deltas, B activations
// The weights a wave needs stay in its registers (one 16-row tile of each
// matrix and of its transpose), activations and deltas live in LDS as
// [sample][feature] rows of kRow floats: a lane's four elements of D are four
// neighbouring places (one 16-byte store), and the sums over features read
// four neighbouring places per 16-byte load; with kRow = 68 neither these
// nor the gradients' reads, which walk the samples, meet in a bank.  Place p
// of a row holds feature feat(p): the four steps that use one 16-byte load then
// take the features 4 apart that make every sum run through its features in
// order, from the bias on, as a plain loop does; a hidden unit near zero is
// then on or off as it is there.  The
// gradients accumulate in registers over all tiles of a workgroup and are
// added to memory once at its end, 9349 atomics per workgroup.
// What bounds it: up to one tile per CU the latency of a tile's nine
// dependent products (17 us) and the atomics (14 us with 256 workgroups, each
// starting at a parameter of its own; 38 us when all start at the first);
// beyond, the products.  Measured: 64 samples 34 us, 16384 samples 48 us (with
// 128 workgroups 58, with 64 87; 4530 us with one lane per sample and a wave
// reduction per weight), 2^20 samples 1.15 ms, 50 TFLOP/s of FP32.
constexpr int kGradWaves = 8, kGradThreads = 64 * kGradWaves;
constexpr int kTile = 64;        // samples per tile
constexpr int kRow = 68;         // floats per activation row
constexpr int kXRow = 20;        // floats per input / output-delta row
constexpr int kGradChunk = 512;  // samples whose inputs a workgroup prepares at once
constexpr int kGradBlocks = 256;  // one per CU (its 146 KB of LDS allow no second)
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct GradLds {
  float x[kGradChunk * kXRow];   // inputs, 10 features, then 1 (the bias), zeros
  float y[kGradChunk * 8];       // targets, then 1 for a sample in the loss, else 0
  float h[3][kTile * kRow];      // activations
  float d[2][kTile * kRow];      // deltas (two layers at a time)
  float d4[kTile * kXRow];       // output deltas, padded to 16
  float loss[kGradWaves];
};

// feature at place p of a row: each block of 16 as a transposed 4 x 4
__device__ __forceinline__ int feat(int p) { return (p & ~15) + 4 * (p & 3) + (p >> 2 & 3); }

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// acc[t] += sum over 64 features of A (this wave's rows; element 4 q + r is
// place 16 q + 4 (l/16) + r) and the rows of samples s0 + 16 t of `rows`
__device__ __forceinline__ void mm64(const f32x4* a, const float* rows, int s0, f32x4* acc) {
  const int l = threadIdx.x & 63, g = l >> 4, c = l & 15;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 b0 = *(const f32x4*)(rows + (s0 + c) * kRow + 16 * q + 4 * g);
    const f32x4 b1 = *(const f32x4*)(rows + (s0 + 16 + c) * kRow + 16 * q + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[0] = mfma4(a[q][r], b0[r], acc[0]);
      acc[1] = mfma4(a[q][r], b1[r], acc[1]);
    }
  }
}

// sample of step t for lane group g in the gradients' sums over a tile: a
// wave half reads samples 4 apart, whose rows are 16 banks apart
__device__ __forceinline__ int grad_sample(int t, int g) { return 16 * (t >> 2) + 4 * g + (t & 3); }

// dw[t] += sum_s da[s][o] hb[s][i0 + 16 t]; db += sum_s da[s][o]
__device__ __forceinline__ void grad64(const float* da, int arow, int o0, const float* hb, int brow,
                                       int i0, int ntile, f32x4* dw, f32x4* db) {
  const int l = threadIdx.x & 63, g = l >> 4, c = l & 15;
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int s = grad_sample(t, g);
    const float a = da[s * arow + o0 + c];
#pragma unroll
    for (int n = 0; n < ntile; ++n) dw[n] = mfma4(a, hb[s * brow + i0 + 16 * n + c], dw[n]);
    if (db) *db = mfma4(a, 1.0f, *db);
  }
}

__device__ __forceinline__ f32x4 relu4(f32x4 z) {
  f32x4 r;
  for (int v = 0; v < 4; ++v) r[v] = z[v] > 0.0f ? z[v] : 0.0f;
  return r;
}
__device__ __forceinline__ f32x4 mask4(f32x4 d, f32x4 h) {
  f32x4 r;
  for (int v = 0; v < 4; ++v) r[v] = h[v] > 0.0f ? d[v] : 0.0f;
  return r;
}

// grad and loss are accumulated (the caller zeroes them); `inv_n` = 1 /
// (samples in the whole batch); `tpb` tiles per workgroup
__global__ __launch_bounds__(kGradThreads) void k_mlp_loss_grad(const float* __restrict__ P,
                                                                const float* __restrict__ rec,
                                                                long long n, double gamma,
                                                                float inv_n, long long tpb,
                                                                float* __restrict__ grad,
                                                                float* __restrict__ loss) {
  __shared__ __align__(16) GradLds S;
  const int tid = (int)threadIdx.x, l = tid & 63, w = tid >> 6;
  const int g = l >> 4, c = l & 15;
  const int ot = 16 * (w & 3);    // this wave's 16 rows
  const int s0 = 32 * (w >> 2);   // and its 32 samples of a tile
  const int it0 = 32 * (w >> 2);  // its two tiles of gradient columns
  // weights of this wave's rows: forward (row ot + c) and transposed
  f32x4 a1, a2[4], a3[4], a4[4], t2[4], t3[4];
  float t4[2];
  const int fc = ot + feat(c);
  for (int r = 0; r < 4; ++r) {
    const int k = feat(4 * g + r);
    a1[r] = k < kMlpIn ? P[kOffW1 + fc * kMlpIn + k] : 0.0f;
  }
  for (int q = 0; q < 4; ++q)
    for (int r = 0; r < 4; ++r) {
      const int k = feat(16 * q + 4 * g + r);
      a2[q][r] = P[kOffW2 + fc * kMlpHid + k];
      a3[q][r] = P[kOffW3 + fc * kMlpHid + k];
      a4[q][r] = c < kMlpOut ? P[kOffW4 + c * kMlpHid + k] : 0.0f;
      t2[q][r] = P[kOffW2 + k * kMlpHid + fc];
      t3[q][r] = P[kOffW3 + k * kMlpHid + fc];
    }
  for (int t = 0; t < 2; ++t) t4[t] = 4 * t + g < kMlpOut ? P[kOffW4 + (4 * t + g) * kMlpHid + fc] : 0.0f;
  f32x4 bias1, bias2, bias3, bias4;
  for (int v = 0; v < 4; ++v) {
    bias1[v] = P[kOffB1 + feat(ot + 4 * g + v)];
    bias2[v] = P[kOffB2 + feat(ot + 4 * g + v)];
    bias3[v] = P[kOffB3 + feat(ot + 4 * g + v)];
    bias4[v] = 4 * g + v < kMlpOut ? P[kOffB4 + 4 * g + v] : 0.0f;
  }
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 dw3[2] = {zero, zero}, dw2[2] = {zero, zero}, db = zero, dw14 = zero, db4 = zero;
  float lsum = 0.0f;

  const long long first = (long long)blockIdx.x * tpb * kTile;
  long long last = first + tpb * kTile;
  last = last < n ? last : n;
  for (long long c0 = first; c0 < last; c0 += kGradChunk) {
    // inputs and targets of up to kGradChunk samples, one per thread
    const long long s = c0 + tid;
    float x[kMlpIn], y[kMlpOut];
    bool valid = s < last;
    if (valid) {
      record_xy(gamma, rec + 15 * s, x, y);
      // only samples inside the training domain enter the loss
      for (int k = 0; k < kMlpIn; ++k) valid = valid && fabsf(x[k]) <= kMlpDomain;
      for (int k = 0; k < kMlpOut; ++k) valid = valid && fabsf(y[k]) <= kMlpDomain;
    }
    for (int k = 0; k < 16; ++k)
      S.x[tid * kXRow + feat(k)] = k < kMlpIn ? (valid ? x[k] : 0.0f) : (k == kMlpIn ? 1.0f : 0.0f);
    for (int k = 0; k < kMlpOut; ++k) S.y[tid * 8 + k] = valid ? y[k] : 0.0f;
    S.y[tid * 8 + kMlpOut] = valid ? 1.0f : 0.0f;
    __syncthreads();
    const int ntile = (int)(((last - c0 < kGradChunk ? last - c0 : kGradChunk) + kTile - 1) / kTile);
    for (int tile = 0; tile < ntile; ++tile) {
      const float* X = S.x + tile * kTile * kXRow;
      const float* Y = S.y + tile * kTile * 8;
      f32x4 acc[2];
      // forward
      for (int t = 0; t < 2; ++t) {
        const f32x4 b = *(const f32x4*)(X + (s0 + 16 * t + c) * kXRow + 4 * g);
        acc[t] = bias1;
        for (int r = 0; r < 4; ++r) acc[t] = mfma4(a1[r], b[r], acc[t]);
        *(f32x4*)(S.h[0] + (s0 + 16 * t + c) * kRow + ot + 4 * g) = relu4(acc[t]);
      }
      __syncthreads();
      acc[0] = acc[1] = bias2;
      mm64(a2, S.h[0], s0, acc);
      for (int t = 0; t < 2; ++t)
        *(f32x4*)(S.h[1] + (s0 + 16 * t + c) * kRow + ot + 4 * g) = relu4(acc[t]);
      __syncthreads();
      acc[0] = acc[1] = bias3;
      mm64(a3, S.h[1], s0, acc);
      for (int t = 0; t < 2; ++t)
        *(f32x4*)(S.h[2] + (s0 + 16 * t + c) * kRow + ot + 4 * g) = relu4(acc[t]);
      __syncthreads();
      // outputs (rows 0..4 of one 16-row tile), the loss and its derivative:
      // waves 0-3, 16 samples each
      if (w < 4) {
        const int sw = 16 * w + c;
        f32x4 o = bias4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 b = *(const f32x4*)(S.h[2] + sw * kRow + 16 * q + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) o = mfma4(a4[q][r], b[r], o);
        }
        const bool in = Y[sw * 8 + kMlpOut] != 0.0f;
        f32x4 d4;
        for (int v = 0; v < 4; ++v) {
          const int k = 4 * g + v;
          const float e = in && k < kMlpOut ? o[v] - Y[sw * 8 + (k < kMlpOut ? k : 0)] : 0.0f;
          lsum += e * e;
          d4[v] = 2.0f * e * inv_n;
        }
        *(f32x4*)(S.d4 + sw * kXRow + 4 * g) = d4;
      }
      __syncthreads();
      // backward through the output layer, and its gradient
      for (int t = 0; t < 2; ++t) {
        const int sl = s0 + 16 * t + c;
        acc[t] = mfma4(t4[0], S.d4[sl * kXRow + g], zero);
        acc[t] = mfma4(t4[1], S.d4[sl * kXRow + 4 + g], acc[t]);
        const f32x4 h = *(const f32x4*)(S.h[2] + sl * kRow + ot + 4 * g);
        *(f32x4*)(S.d[0] + sl * kRow + ot + 4 * g) = mask4(acc[t], h);
      }
      if (w >= 4) grad64(S.d4, kXRow, 0, S.h[2], kRow, ot, 1, &dw14, w == 4 ? &db4 : nullptr);
      __syncthreads();
      acc[0] = acc[1] = zero;
      mm64(t3, S.d[0], s0, acc);
      for (int t = 0; t < 2; ++t) {
        const int sl = s0 + 16 * t + c;
        const f32x4 h = *(const f32x4*)(S.h[1] + sl * kRow + ot + 4 * g);
        *(f32x4*)(S.d[1] + sl * kRow + ot + 4 * g) = mask4(acc[t], h);
      }
      grad64(S.d[0], kRow, ot, S.h[1], kRow, it0, 2, dw3, w < 4 ? &db : nullptr);
      __syncthreads();
      acc[0] = acc[1] = zero;
      mm64(t2, S.d[1], s0, acc);
      for (int t = 0; t < 2; ++t) {
        const int sl = s0 + 16 * t + c;
        const f32x4 h = *(const f32x4*)(S.h[0] + sl * kRow + ot + 4 * g);
        *(f32x4*)(S.d[0] + sl * kRow + ot + 4 * g) = mask4(acc[t], h);
      }
      grad64(S.d[1], kRow, ot, S.h[0], kRow, it0, 2, dw2, w >= 4 ? &db : nullptr);
      __syncthreads();
      // input layer: features 0..9 its weights' gradient, feature 10 the bias's
      if (w < 4) grad64(S.d[0], kRow, ot, X, kXRow, 0, 1, &dw14, nullptr);
      __syncthreads();
    }
  }
  // this workgroup's sums, gathered in parameter order in LDS and added to
  // memory from a starting point of its own: workgroups that end together
  // then add to different lines
  float* G = S.x;  // the inputs are no longer needed (the loop ends with a barrier)
  static_assert(kGradChunk * kXRow >= kMlpNParam, "gradient fits the input area");
  for (int v = 0; v < 4; ++v) {
    const int o = feat(ot + 4 * g + v), ci = feat(c);  // gradient row and column of this lane
    for (int t = 0; t < 2; ++t) {
      G[kOffW3 + o * kMlpHid + it0 + 16 * t + ci] = dw3[t][v];
      G[kOffW2 + o * kMlpHid + it0 + 16 * t + ci] = dw2[t][v];
    }
    if (w < 4) {
      if (ci < kMlpIn) G[kOffW1 + o * kMlpIn + ci] = dw14[v];
      else if (ci == kMlpIn) G[kOffB1 + o] = dw14[v];
      if (c == 0) G[kOffB3 + o] = db[v];
    } else {
      const int k = 4 * g + v;
      if (k < kMlpOut) G[kOffW4 + k * kMlpHid + fc] = dw14[v];
      if (c == 0) G[kOffB2 + o] = db[v];
      if (w == 4 && c == 0 && k < kMlpOut) G[kOffB4 + k] = db4[v];
    }
  }
  __syncthreads();
  const int rot = (int)((blockIdx.x * 2654435761u >> 16) % (kMlpNParam / 64)) * 64;
  for (int i = tid; i < kMlpNParam; i += kGradThreads) {
    int k = i + rot;
    k = k < kMlpNParam ? k : k - kMlpNParam;
    atomicAdd(grad + k, G[k]);
  }
  for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
  if (l == 0) S.loss[w] = lsum;
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    for (int i = 0; i < 4; ++i) t += S.loss[i];
    atomicAdd(loss, t * inv_n);
  }
}

__global__ void k_mlp_adam(float* P, float* m, float* v, const float* g, float lr, float b1,
                           float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kMlpNParam) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  P[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// FP32 master weights -> BF16 MFMA fragments + FP32 (padded) biases
__global__ void k_mlp_pack(const float* P, unsigned char* packed) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < kMlpFrags * 64 * 8) {
    const int f = t / 512, l = (t / 8) % 64, e = t % 8;
    int layer, m, s;
    if (f < 2) { layer = 0; m = f; s = 0; }
    else if (f < 10) { layer = 1; m = (f - 2) / 4; s = (f - 2) % 4; }
    else if (f < 18) { layer = 2; m = (f - 10) / 4; s = (f - 10) % 4; }
    else { layer = 3; m = 0; s = f - 18; }
    const int row = 32 * m + (l & 31), k = 16 * s + 8 * (l >> 5) + e;
    const int nin = layer == 0 ? kMlpIn : kMlpHid;
    const int nout = layer == 3 ? kMlpOut : kMlpHid;
    const int woff = layer == 0 ? kOffW1 : (layer == 1 ? kOffW2 : (layer == 2 ? kOffW3 : kOffW4));
    const float w = (row < nout && k < nin) ? P[woff + row * nin + k] : 0.0f;
    ((__bf16*)packed)[t] = (__bf16)w;
  } else if (t < kMlpFrags * 64 * 8 + 224) {
    const int j = t - kMlpFrags * 64 * 8;
    float b;
    if (j < 64) b = P[kOffB1 + j];
    else if (j < 128) b = P[kOffB2 + j - 64];
    else if (j < 192) b = P[kOffB3 + j - 128];
    else b = (j - 192) < kMlpOut ? P[kOffB4 + j - 192] : 0.0f;
    ((float*)(packed + kMlpBiasOff))[j] = b;
  }
}

// inference on harvested records (BF16 MFMA path): out[n][5]
__global__ __launch_bounds__(256) void k_mlp_predict(const void* packed, const float* rec,
                                                      long long n, double gamma, float* out) {
  __shared__ __bf16 lds[4 * kMlpWaveLds];
  const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
  float x[kMlpIn];
  if (s < n) {
    record_xy(gamma, rec + 15 * s, x, nullptr);
  } else {
    for (int k = 0; k < kMlpIn; ++k) x[k] = 1.0f;
  }
  float y[kMlpOut];
  mlp_wave_forward(packed, x, lds + (threadIdx.x >> 6) * kMlpWaveLds, y);
  if (s < n)
    for (int k = 0; k < kMlpOut; ++k) out[5 * s + k] = y[k];
}

// ---- launchers ----
hipError_t launch_mlp_init(float* P, unsigned long long seed, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_init, dim3((kMlpNParam + 255) / 256), dim3(256), 0, st, P, seed);
  return hipGetLastError();
}
hipError_t launch_mlp_loss_grad(const float* P, const float* rec, long long n, double gamma,
                                float inv_n, float* grad, float* loss, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const long long tiles = (n + kTile - 1) / kTile;
  const long long tpb = (tiles + kGradBlocks - 1) / kGradBlocks;
  const unsigned blocks = (unsigned)((tiles + tpb - 1) / tpb);
  hipLaunchKernelGGL(k_mlp_loss_grad, dim3(blocks), dim3(kGradThreads), 0, st, P, rec,
                     n, gamma, inv_n, tpb, grad, loss);
  return hipGetLastError();
}
hipError_t launch_mlp_adam(float* P, float* m, float* v, const float* g, int t, float lr, float b1,
                           float b2, float eps, hipStream_t st) {
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpNParam + 255) / 256), dim3(256), 0, st, P, m, v, g, lr,
                     b1, b2, eps, c1, c2);
  return hipGetLastError();
}
hipError_t launch_mlp_pack(const float* P, void* packed, hipStream_t st) {
  const int n = kMlpFrags * 64 * 8 + 224;
  hipLaunchKernelGGL(k_mlp_pack, dim3((n + 255) / 256), dim3(256), 0, st, P,
                     (unsigned char*)packed);
  return hipGetLastError();
}
hipError_t launch_mlp_predict(const void* packed, const float* rec, long long n, double gamma,
                              float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_predict, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, packed,
                     rec, n, gamma, out);
  return hipGetLastError();
}

}  // namespace nyx

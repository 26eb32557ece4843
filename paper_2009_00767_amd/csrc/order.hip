// order.hip -- learned expansion order per level (2D).
//
// A small multilayer perceptron predicts, for one system and one level k, the
// truncation error that level's far field would carry at each order of a grid
// p = 4..24; the smallest order whose predicted error fits the level's share of
// the tolerance is used.  Features of a (system, level):
//   f0 = k / 10,  f1 = log2(non-empty boxes at level k) / 20,  f2 = log10 ||q||_2.
// Network: 3 -> 64 ReLU -> 64 ReLU -> 21 linear (predicted log10 errors).
// Parameters, one FP32 array (row-major, output index major):
//   W1[64][3], b1[64], W2[64][64], b2[64], W3[21][64], b3[21].
// Training minimises the mean squared error over the 21 outputs with Adam
// (Kingma and Ba 2015, Algorithm 1); every kernel here is deterministic
// (fixed-order reductions, no floating-point atomics).
//
// The order selection evaluates one sample at a time by a wavefront, lane j
// owning hidden unit j (64 hidden units = 64 lanes), with the weights staged in
// LDS in rows padded to 65 floats so that both row and column walks are free of
// bank conflicts; batches of samples run on the matrix cores (below).
#include "device_common.h"

namespace sffmm {

constexpr int kNI = 3, kNH = 64, kNO = 21;
// Order selection keeps a margin below each level's budget for the network's
// own error of fit: 0.3 in log10 units (a factor of 2), about the RMS error of
// the packaged model's predictions on its training labels (mean squared loss
// 0.10 in log10^2 units).
constexpr float kOrderMargin = 0.3f;
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kNH * kNI, kOffW2 = kOffB1 + kNH,
              kOffB2 = kOffW2 + kNH * kNH, kOffW3 = kOffB2 + kNH, kOffB3 = kOffW3 + kNO * kNH,
              kNParam = kOffB3 + kNO;
static_assert(kNParam == FMM_MLP_NPARAM, "parameter count");
constexpr int kRow = 65;  // padded LDS row

struct MlpLds {
  float w1[kNH * kNI], b1[kNH], w2[kNH * kRow], b2[kNH], w3[kNO * kRow], b3[kNO];
};

__device__ void stage_weights(const float* __restrict__ w, MlpLds& s) {
  for (int e = threadIdx.x; e < kNParam; e += blockDim.x) {
    const float v = w[e];
    if (e < kOffB1) {
      s.w1[e] = v;
    } else if (e < kOffW2) {
      s.b1[e - kOffB1] = v;
    } else if (e < kOffB2) {
      const int r = (e - kOffW2) / kNH, c = (e - kOffW2) % kNH;
      s.w2[r * kRow + c] = v;
    } else if (e < kOffW3) {
      s.b2[e - kOffB2] = v;
    } else if (e < kOffB3) {
      const int r = (e - kOffW3) / kNH, c = (e - kOffW3) % kNH;
      s.w3[r * kRow + c] = v;
    } else {
      s.b3[e - kOffB3] = v;
    }
  }
}

// Orders the LDS writes of a wave before its later LDS reads of other lanes'
// values (all lanes of the wave pass it together).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Forward pass of one sample by one wave (lane = hidden unit).  h1s / h2s are
// the wave's LDS vectors.  Returns output `lane` (valid for lanes < 21).
__device__ __forceinline__ float wave_forward(const MlpLds& s, float x0, float x1, float x2,
                                              float* h1s, float* h2s, float& z1, float& h1,
                                              float& z2, float& h2) {
  const int j = threadIdx.x & 63;
  z1 = s.b1[j] + s.w1[j * 3] * x0 + s.w1[j * 3 + 1] * x1 + s.w1[j * 3 + 2] * x2;
  h1 = z1 > 0.f ? z1 : 0.f;
  h1s[j] = h1;
  wave_sync();
  float a = s.b2[j];
#pragma unroll 16
  for (int i = 0; i < kNH; ++i) a += s.w2[j * kRow + i] * h1s[i];
  z2 = a;
  h2 = z2 > 0.f ? z2 : 0.f;
  h2s[j] = h2;
  wave_sync();
  float y = 0.f;
  if (j < kNO) {
    y = s.b3[j];
#pragma unroll 16
    for (int i = 0; i < kNH; ++i) y += s.w3[j * kRow + i] * h2s[i];
  }
  return y;
}

// ---------------------------------------------------------------------------
// Batches: 16 samples at a time by a workgroup of four waves, every layer and
// every weight gradient a dense product on v_mfma_f32_16x16x4f32 (FP32 inputs
// and accumulation).  Lane l of a wave holds A[l % 16][l / 16] and B[l / 16][l %
// 16] of a step and rows 4 (l / 16) + r, column l % 16 of the result.  The LDS
// row of 68 floats puts the 16 rows of one step on distinct banks.
// Bound by latency (2003 samples are 126 workgroups and 68 Mflop): one wave per
// sample, lane by hidden unit, had 64 + 64 serial LDS products a sample.
// Measured at 2003 samples: the gradient 67 -> 13 us, its reduction 35 -> 4.5
// us, the forward pass 7.9 -> 6.3 us.
// ---------------------------------------------------------------------------
typedef float mlpx4 __attribute__((ext_vector_type(4)));
constexpr int kTile = 16;    // samples
constexpr int kStride = 68;  // LDS row
constexpr int kNO2 = 32;     // output rows padded to two blocks of 16

struct MlpTile {
  float w2[kNH * kStride], w3[kNO2 * kStride];
  float w1[kNH * kNI], b1[kNH], b2[kNH], b3[kNO2];
  float x[kTile][kNI];
  float h1[kTile * kStride], h2[kTile * kStride];
};

__device__ __forceinline__ void stage_tile_weights(const float* __restrict__ w, MlpTile& s) {
  for (int e = threadIdx.x; e < kNH * kNH; e += 256)
    s.w2[(e / kNH) * kStride + e % kNH] = w[kOffW2 + e];
  for (int e = threadIdx.x; e < kNO2 * kNH; e += 256)
    s.w3[(e / kNH) * kStride + e % kNH] = e < kNO * kNH ? w[kOffW3 + e] : 0.f;
  if (threadIdx.x < kNH * kNI) s.w1[threadIdx.x] = w[kOffW1 + threadIdx.x];
  if (threadIdx.x < kNH) {
    s.b1[threadIdx.x] = w[kOffB1 + threadIdx.x];
    s.b2[threadIdx.x] = w[kOffB2 + threadIdx.x];
  }
  if (threadIdx.x < kNO2) s.b3[threadIdx.x] = threadIdx.x < kNO ? w[kOffB3 + threadIdx.x] : 0.f;
}

// C += A B over K = 4 steps: a(i, k), b(k, j) give the operands of row i and column j.
template <int STEPS, class FA, class FB>
__device__ __forceinline__ mlpx4 mlp_product(mlpx4 c, FA&& a, FB&& b) {
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int st = 0; st < STEPS; ++st)
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a(i, 4 * st + g), b(4 * st + g, i), c, 0, 0, 0);
  return c;
}

// Hidden layers of the tile's samples s0.. into h1 and h2, then the outputs:
// result rows of output block `wave` (waves 0 and 1 only).  Past m the first
// hidden layer is zero, so that no padding sample overflows where the samples do
// not (its zero output error times infinity would reach the gradient).
// Ends with the tile's h1 and h2 visible to the workgroup.
__device__ __forceinline__ mlpx4 tile_forward(const float* __restrict__ x, int64_t m, int64_t s0,
                                              MlpTile& s) {
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, col = lane & 15, g = lane >> 4;
  if (t < kTile * kNI) {
    const int64_t e = kNI * s0 + t;
    s.x[t / kNI][t % kNI] = e < kNI * m ? x[e] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kTile / 4; ++u) {
    const int i = 4 * u + wave;
    const float z = s.b1[lane] + s.w1[lane * 3] * s.x[i][0] + s.w1[lane * 3 + 1] * s.x[i][1] +
                    s.w1[lane * 3 + 2] * s.x[i][2];
    s.h1[i * kStride + lane] = z > 0.f && s0 + i < m ? z : 0.f;
  }
  __syncthreads();
  {
    const int n0 = 16 * wave;
    const float b = s.b2[n0 + col];
    const mlpx4 z = mlp_product<kNH / 4>(
        mlpx4{b, b, b, b}, [&](int i, int k) { return s.h1[i * kStride + k]; },
        [&](int k, int j) { return s.w2[(n0 + j) * kStride + k]; });
#pragma unroll
    for (int r = 0; r < 4; ++r) s.h2[(4 * g + r) * kStride + n0 + col] = z[r] > 0.f ? z[r] : 0.f;
  }
  __syncthreads();
  mlpx4 y = {0.f, 0.f, 0.f, 0.f};
  if (wave < 2) {
    const int n0 = 16 * wave;
    const float b = s.b3[n0 + col];
    y = mlp_product<kNH / 4>(
        mlpx4{b, b, b, b}, [&](int i, int k) { return s.h2[i * kStride + k]; },
        [&](int k, int j) { return s.w3[(n0 + j) * kStride + k]; });
  }
  return y;
}

__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ w,
                                                     const float* __restrict__ x, int64_t m,
                                                     float* __restrict__ y) {
  __shared__ MlpTile s;
  stage_tile_weights(w, s);
  const int lane = threadIdx.x & 63, o = 16 * (threadIdx.x >> 6) + (lane & 15), g = lane >> 4;
  for (int64_t s0 = (int64_t)blockIdx.x * kTile; s0 < m; s0 += (int64_t)gridDim.x * kTile) {
    const mlpx4 v = tile_forward(x, m, s0, s);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t smp = s0 + 4 * g + r;
      if (o < kNO && smp < m) y[kNO * smp + o] = v[r];
    }
    __syncthreads();  // the next tile overwrites h1 and h2
  }
}

// Loss gradient: a workgroup takes tiles blockIdx, blockIdx + grid, ...  Matrix
// accumulators and FP32 sums hold the gradient of one tile's 16 samples; it is
// added to FP64 sums before the next tile, so that no FP32 chain grows with the
// batch.  Each workgroup writes one partial vector, and a second kernel adds
// those in a fixed order in FP64.  At most kGradBlocks workgroups, so the partials
// are bounded whatever the batch.  Partials and sums are of type P: float where a
// workgroup has one tile, whose FP32 gradient is its partial (gradient and
// predictions of 2003 samples: 41.9 us, 42.9 with FP64 partials), else double
// (gradient of 8000 samples 42 us, of 10^6 1.37 ms; 37 and 1.27 with an FP32 chain
// over all of a workgroup's tiles, which loses what cancels).
constexpr int kGradBlocks = 256;
static __device__ double g_mlp_part[(size_t)kGradBlocks * kNParam];
static __device__ double g_mlp_part_loss[kGradBlocks];

// part == NULL: the partials go to the device's own array (one user at a time).
template <typename P>
__global__ __launch_bounds__(256) void k_mlp_grad_partial(const float* __restrict__ w,
                                                          const float* __restrict__ x,
                                                          const float* __restrict__ t, int64_t m,
                                                          float scale, P* part,
                                                          double* part_loss) {
  __shared__ MlpTile s;
  __shared__ float dys[kTile * 36], dz2[kTile * kStride], dz1[kTile * kStride];
  __shared__ double lsum[2];
  if (!part) {
    part = reinterpret_cast<P*>(g_mlp_part);
    part_loss = g_mlp_part_loss;
  }
  stage_tile_weights(w, s);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, g = lane >> 4;
  const int n0 = 16 * wave;
  // rows n0.. of dW2 by four blocks of columns; dW3, columns n0..
  P g2[4][4] = {}, g3[2][4] = {};
  // wave 0: db1, wave 1..3: columns of dW1; db2 (wave 0) and db3 (wave 1) beside them
  P gv = 0, gb = 0;
  double loss = 0.0;
  for (int64_t s0 = (int64_t)blockIdx.x * kTile; s0 < m; s0 += (int64_t)gridDim.x * kTile) {
    const mlpx4 y = tile_forward(x, m, s0, s);
    if (wave < 2) {
      const int o = n0 + col;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t smp = s0 + 4 * g + r;
        float dy = 0.f;
        if (o < kNO && smp < m) {
          const float e = y[r] - t[kNO * smp + o];
          loss += (double)e * (double)e;
          dy = 2.f * e * scale;
        }
        dys[(4 * g + r) * 36 + o] = dy;
      }
    }
    __syncthreads();
    {  // dh2 = dY W3, through the rectifier
      const mlpx4 d = mlp_product<6>(
          mlpx4{0.f, 0.f, 0.f, 0.f}, [&](int i, int k) { return dys[i * 36 + k]; },
          [&](int k, int j) { return s.w3[k * kStride + n0 + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = (4 * g + r) * kStride + n0 + col;
        dz2[e] = s.h2[e] > 0.f ? d[r] : 0.f;
      }
    }
    __syncthreads();
    {  // dh1 = dZ2 W2, through the rectifier
      const mlpx4 d = mlp_product<kNH / 4>(
          mlpx4{0.f, 0.f, 0.f, 0.f}, [&](int i, int k) { return dz2[i * kStride + k]; },
          [&](int k, int j) { return s.w2[k * kStride + n0 + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = (4 * g + r) * kStride + n0 + col;
        dz1[e] = s.h1[e] > 0.f ? d[r] : 0.f;
      }
    }
    // dW2[r][k] += dZ2^T H1, dW3[o][k] += dY^T H2
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const mlpx4 d = mlp_product<kTile / 4>(
          mlpx4{0.f, 0.f, 0.f, 0.f}, [&](int i, int k) { return dz2[k * kStride + n0 + i]; },
          [&](int k, int j) { return s.h1[k * kStride + 16 * b + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) g2[b][r] += (P)d[r];
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const mlpx4 d = mlp_product<kTile / 4>(
          mlpx4{0.f, 0.f, 0.f, 0.f}, [&](int i, int k) { return dys[k * 36 + 16 * b + i]; },
          [&](int k, int j) { return s.h2[k * kStride + n0 + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) g3[b][r] += (P)d[r];
    }
    __syncthreads();
    float tv = 0.f, tb = 0.f;
#pragma unroll
    for (int i = 0; i < kTile; ++i) {
      const float d = dz1[i * kStride + lane];
      tv += wave == 0 ? d : d * s.x[i][wave - 1];
      if (wave == 0) tb += dz2[i * kStride + lane];
      if (wave == 1 && lane < kNO) tb += dys[i * 36 + lane];
    }
    gv += (P)tv;
    gb += (P)tb;
    __syncthreads();
  }
  P* pp = part + (int64_t)blockIdx.x * kNParam;
  if (wave == 0) {
    pp[kOffB1 + lane] = gv;
    pp[kOffB2 + lane] = gb;
  } else {
    pp[kOffW1 + lane * kNI + wave - 1] = gv;
    if (wave == 1 && lane < kNO) pp[kOffB3 + lane] = gb;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int b = 0; b < 4; ++b) pp[kOffW2 + (n0 + 4 * g + r) * kNH + 16 * b + col] = g2[b][r];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int o = 16 * b + 4 * g + r;
      if (o < kNO) pp[kOffW3 + o * kNH + n0 + col] = g3[b][r];
    }
  }
  // waves 0 and 1 hold the squared errors of their outputs
  for (int d = 32; d >= 1; d >>= 1) loss += __shfl_xor(loss, d, 64);
  if (wave < 2 && lane == 0) lsum[wave] = loss;
  __syncthreads();
  if (tid == 0) part_loss[blockIdx.x] = lsum[0] + lsum[1];
}

// 32 parameters by a workgroup, eight threads each: thread u adds partials u, u
// + 8, ... in FP64, and the eight sums are added in order.
template <typename P>
__global__ __launch_bounds__(256) void k_mlp_grad_reduce(const P* part, const double* part_loss,
                                                         int64_t nb, float scale,
                                                         float* __restrict__ grad,
                                                         float* __restrict__ loss) {
  __shared__ double red[8][32];
  if (!part) {
    part = reinterpret_cast<P*>(g_mlp_part);
    part_loss = g_mlp_part_loss;
  }
  const int c = threadIdx.x & 31, u = threadIdx.x >> 5, e = blockIdx.x * 32 + c;
  double a = 0.0;
  if (e < kNParam) {
#pragma unroll 8
    for (int64_t r = u; r < nb; r += 8) a += (double)part[r * kNParam + e];
  }
  red[u][c] = a;
  __syncthreads();
  if (u == 0 && e < kNParam) {
#pragma unroll
    for (int v = 1; v < 8; ++v) a += red[v][c];
    grad[e] = (float)a;
  }
  if (blockIdx.x == 0 && loss) {
    __syncthreads();
    double l = 0.0;
    if (threadIdx.x < 64)
      for (int64_t r = threadIdx.x; r < nb; r += 64) l += part_loss[r];
    for (int d = 32; d >= 1; d >>= 1) l += __shfl_xor(l, d, 64);
    if (threadIdx.x == 0) *loss = (float)(l * (double)scale);
  }
}

// omb1 / omb2 are 1 - beta1 / 1 - beta2 formed in FP64 and rounded once (in FP32
// 1 - 0.999f is 1.3e-5 away from 0.001).
__global__ void k_mlp_adam(float* __restrict__ w, const float* __restrict__ g,
                           float* __restrict__ m1, float* __restrict__ m2, float lr, float beta1,
                           float beta2, float omb1, float omb2, float eps, float c1, float c2) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kNParam) return;
  const float gi = g[e];
  const float a = beta1 * m1[e] + omb1 * gi;
  const float b = beta2 * m2[e] + omb2 * gi * gi;
  m1[e] = a;
  m2[e] = b;
  w[e] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

int64_t mlp_grad_blocks(int64_t m) {
  return std::min<int64_t>((m + kTile - 1) / kTile, kGradBlocks);
}

void launch_mlp_forward(const float* w, const float* x, int64_t m, float* y, hipStream_t st) {
  if (m <= 0) return;
  const int64_t blocks = std::min<int64_t>((m + kTile - 1) / kTile, 1024);
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(256), 0, st, w, x, m, y);
}

template <typename P>
static void mlp_grad(const float* w, const float* x, const float* t, int64_t m, P* part,
                     double* part_loss, float* grad, float* loss, hipStream_t st) {
  const float scale = 1.f / (float)(kNO * (m > 0 ? m : 1));
  const int64_t nb = mlp_grad_blocks(m);
  if (nb > 0)
    hipLaunchKernelGGL(k_mlp_grad_partial<P>, dim3((unsigned)nb), dim3(256), 0, st, w, x, t, m,
                       scale, part, part_loss);
  hipLaunchKernelGGL(k_mlp_grad_reduce<P>, dim3((kNParam + 31) / 32), dim3(256), 0, st, part,
                     part_loss, nb, scale, grad, loss);
}

void launch_mlp_grad(const float* w, const float* x, const float* t, int64_t m, double* part,
                     double* part_loss, float* grad, float* loss, hipStream_t st) {
  if (m <= (int64_t)kGradBlocks * kTile)
    mlp_grad(w, x, t, m, reinterpret_cast<float*>(part), part_loss, grad, loss, st);
  else
    mlp_grad(w, x, t, m, part, part_loss, grad, loss, st);
}

void launch_mlp_adam(float* w, const float* g, float* m1, float* m2, int step, float lr,
                     hipStream_t st) {
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - std::pow(b1, (double)step));
  const float c2 = (float)(1.0 - std::pow(b2, (double)step));
  hipLaunchKernelGGL(k_mlp_adam, dim3((kNParam + 255) / 256), dim3(256), 0, st, w, g, m1, m2, lr,
                     (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f, c1, c2);
}

// ---------------------------------------------------------------------------
// Order selection inside an evaluation.
//   k_order_partials: block b of system s covers sorted positions
//     [start_s + c * kChunk, ...) with c = b - blk0_s; it counts, for every
//     level, the positions whose level-k box differs from the previous
//     position's (the first position of a system counts too) and sums q^2 in
//     FP64 (fixed order).
//   k_order_select: one block per system sums its chunks in order, forms the
//     features of every level 2..L_s, runs the network (one wave per level) and
//     raises the order of the system's depth group at that level to its choice.
// ---------------------------------------------------------------------------
constexpr int kChunk = 4096;

__global__ __launch_bounds__(256) void k_order_partials(const OrderSys* __restrict__ sys, int nsys,
                                                        const uint32_t* __restrict__ keys,
                                                        const int32_t* __restrict__ perm,
                                                        const double* __restrict__ q, int kbits,
                                                        double* __restrict__ pq,
                                                        int32_t* __restrict__ pcnt,
                                                        const BatchIo* __restrict__ io) {
  if (io) q = io->q;
  // system of this block: last s with blk0 <= blockIdx.x
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sys[mid].blk0 <= (int)blockIdx.x)
      lo = mid;
    else
      hi = mid - 1;
  }
  const OrderSys sy = sys[lo];
  const int c = (int)blockIdx.x - sy.blk0;
  const int64_t a = (int64_t)sy.start + (int64_t)c * kChunk;
  const int64_t end = (int64_t)sy.start + sy.n;
  const int64_t e = a + kChunk < end ? a + kChunk : end;
  int cnt[kMaxLevels2D + 1];
#pragma unroll
  for (int k = 0; k <= kMaxLevels2D; ++k) cnt[k] = 0;
  double s2 = 0.0;
  for (int64_t j = a + threadIdx.x; j < e; j += 256) {
    const double qq = q[perm[j]];
    s2 += qq * qq;
    const uint32_t kj = keys[j];
    const bool first = j == sy.start;
    const uint32_t kp = first ? 0u : keys[j - 1];
#pragma unroll
    for (int k = 0; k <= kMaxLevels2D; ++k) {
      if (k <= sy.L) {
        const int sh = 2 * (kbits - k);
        cnt[k] += (first || (kj >> sh) != (kp >> sh)) ? 1 : 0;
      }
    }
  }
  __shared__ double rs[256];
  __shared__ int rc[256];
  rs[threadIdx.x] = s2;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) rs[threadIdx.x] += rs[threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) pq[blockIdx.x] = rs[0];
  for (int k = 0; k <= kMaxLevels2D; ++k) {
    __syncthreads();
    rc[threadIdx.x] = cnt[k];
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
      if ((int)threadIdx.x < d) rc[threadIdx.x] += rc[threadIdx.x + d];
      __syncthreads();
    }
    if (threadIdx.x == 0) pcnt[(int64_t)blockIdx.x * (kMaxLevels2D + 1) + k] = rc[0];
  }
}

__global__ __launch_bounds__(256) void k_order_select(const OrderSys* __restrict__ sys,
                                                      const float* __restrict__ w,
                                                      const double* __restrict__ pq,
                                                      const int32_t* __restrict__ pcnt,
                                                      float log10_budget, int32_t* __restrict__ ord,
                                                      int ord_cols, float* __restrict__ feat_out) {
  __shared__ MlpLds s;
  __shared__ float hs[4][2][kNH];
  __shared__ double qsum;
  __shared__ int boxes[kMaxLevels2D + 1];
  stage_weights(w, s);
  const OrderSys sy = sys[blockIdx.x];
  if (threadIdx.x == 0) {
    double a = 0.0;
    for (int c = 0; c < sy.nblk; ++c) a += pq[sy.blk0 + c];
    qsum = a;
  }
  if ((int)threadIdx.x <= kMaxLevels2D) {
    int b = 0;
    for (int c = 0; c < sy.nblk; ++c) b += pcnt[(int64_t)(sy.blk0 + c) * (kMaxLevels2D + 1) + threadIdx.x];
    boxes[threadIdx.x] = b;
  }
  __syncthreads();
  if (sy.L < 2 || sy.n == 0) return;
  const int wv = threadIdx.x >> 6, j = threadIdx.x & 63;
  const float qn = (float)log10(fmax(sqrt(qsum), 1e-30));
  // the error budget of one level: tol / (number of levels with a far field),
  // less kOrderMargin for the network's own error of fit
  const float thr = log10_budget - log10f((float)(sy.L - 1)) - kOrderMargin;
  for (int k = 2 + wv; k <= sy.L; k += 4) {
    const float f0 = (float)k / 10.f;
    const float f1 = log2f((float)max(boxes[k], 1)) / 20.f;
    float z1, h1, z2, h2;
    const float y = wave_forward(s, f0, f1, qn, hs[wv][0], hs[wv][1], z1, h1, z2, h2);
    const bool ok = j < kNO && y <= thr;
    const uint64_t mask = __ballot(ok);
    if (j == 0) {
      const int p = mask ? 4 + __builtin_ctzll(mask) : 4 + kNO - 1;
      atomicMax(&ord[sy.group * ord_cols + k], p);
      if (feat_out) {
        float* fo = feat_out + ((int64_t)sy.id * (kMaxLevels2D + 1) + k) * 3;
        fo[0] = f0;
        fo[1] = f1;
        fo[2] = qn;
      }
    }
    wave_sync();
  }
}

void launch_order_select(const OrderSys* sys, int nsys, int total_blocks, const uint32_t* keys,
                         const int32_t* perm, const double* q, int kbits, const float* w,
                         double* pq, int32_t* pcnt, float log10_budget, int32_t* ord, int ord_cols,
                         float* feat_out, hipStream_t st, const BatchIo* io) {
  if (nsys <= 0) return;
  if (total_blocks > 0)
    hipLaunchKernelGGL(k_order_partials, dim3(total_blocks), dim3(256), 0, st, sys, nsys, keys,
                       perm, q, kbits, pq, pcnt, io);
  hipLaunchKernelGGL(k_order_select, dim3(nsys), dim3(256), 0, st, sys, w, pq, pcnt, log10_budget,
                     ord, ord_cols, feat_out);
}

int order_chunk() { return kChunk; }

__global__ void k_set_ordsys(OrderSys* dst, OrderSys v) { *dst = v; }

void launch_set_ordsys(OrderSys* dst, const OrderSys& v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_ordsys, dim3(1), dim3(1), 0, st, dst, v);
}

// ---------------------------------------------------------------------------
// Judge: the relative L2 difference of the potentials from the fixed-order
// result over every particle of each system (one workgroup per system, its
// range of the concatenated arrays), and the largest over the systems; if that
// is above tol, flag[1] = tag and the outputs are replaced by the fixed-order
// result.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_judge_sys(const double* __restrict__ pot,
                                                   const double* __restrict__ ref,
                                                   const int64_t* __restrict__ sys_off, int64_t n,
                                                   double* __restrict__ err_sys) {
  __shared__ double a[256], b[256];
  const int64_t i0 = sys_off ? sys_off[blockIdx.x] : 0;
  const int64_t i1 = sys_off ? sys_off[blockIdx.x + 1] : n;
  double num = 0.0, den = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const double d = pot[i] - ref[i];
    num += d * d;
    den += ref[i] * ref[i];
  }
  a[threadIdx.x] = num;
  b[threadIdx.x] = den;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) {
      a[threadIdx.x] += a[threadIdx.x + d];
      b[threadIdx.x] += b[threadIdx.x + d];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0)
    err_sys[blockIdx.x] = b[0] > 0 ? sqrt(a[0] / b[0]) : (a[0] > 0 ? INFINITY : 0.0);
}

__global__ __launch_bounds__(256) void k_judge_max(const double* __restrict__ err_sys, int nsys,
                                                   double tol, int32_t* flag, int32_t tag,
                                                   double* __restrict__ err_out) {
  __shared__ double m[256];
  __shared__ int reject;
  if (threadIdx.x == 0) reject = 0;
  __syncthreads();
  double e = 0.0;
  bool bad = false;
  for (int s = threadIdx.x; s < nsys; s += 256) {
    const double v = err_sys[s];
    bad = bad || !(v <= tol);  // NaN rejects too
    e = fmax(e, v);
  }
  if (bad) atomicOr(&reject, 1);
  m[threadIdx.x] = e;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) m[threadIdx.x] = fmax(m[threadIdx.x], m[threadIdx.x + d]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    err_out[0] = m[0];
    if (reject) flag[1] = tag;
  }
}

__global__ void k_judge_apply(double* __restrict__ pot, double* __restrict__ field,
                              const double* __restrict__ rpot, const double* __restrict__ rfield,
                              int64_t n, int dim, const int32_t* flag, int32_t tag) {
  if (flag[1] != tag) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  pot[i] = rpot[i];
  if (field)
    for (int d = 0; d < dim; ++d) field[dim * i + d] = rfield[dim * i + d];
}

void launch_judge(double* pot, double* field, const double* rpot, const double* rfield, int64_t n,
                  int dim, const int64_t* sys_off, int nsys, double tol, int32_t* flag,
                  int32_t tag, double* err_out, hipStream_t st) {
  if (n <= 0 || nsys <= 0) return;
  hipLaunchKernelGGL(k_judge_sys, dim3((unsigned)nsys), dim3(256), 0, st, pot, rpot, sys_off, n,
                     err_out + 1);
  hipLaunchKernelGGL(k_judge_max, dim3(1), dim3(256), 0, st, err_out + 1, nsys, tol, flag, tag,
                     err_out);
  hipLaunchKernelGGL(k_judge_apply, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pot,
                     field, rpot, rfield, n, dim, flag, tag);
}

}  // namespace sffmm

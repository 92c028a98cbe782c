// Learned EOS seed: a 2 -> 64 -> 64 -> 1 ReLU network predicting normalised
// log T from normalised (log rho, log e), used to seed the table inversion.
// bf16 operands, fp32 accumulation.  The 64x64 hidden layer runs on the
// matrix cores (v_mfma_f32_16x16x32_bf16); the 2-wide input layer and the
// 1-wide output layer are plain vector arithmetic.
//
// MFMA 16x16x32 lane layout (lane l, e = 0..7, r = 0..3):
//   A (16 x 32, rows M):  row l%16, k = 8*(l/16) + e
//   B (32 x 16, cols N):  col l%16, k = 8*(l/16) + e
//   D (16 x 16):          col l%16, row 4*(l/16) + r
// A wave handles 64 samples: M/N tiles mt, nt in 0..3, K tiles kt in 0..1.
//
// Parameter vector (fp32 master copy, 4417 values): W1[64][2], b1[64],
// W2[64 out][64 in], b2[64], W3[64], b3.
#include "tdh_mlp_dev.hpp"

namespace tdh {

// ---------------------------------------------------------------------------
// inference over n queries (raw log10 rho, log10 e) -> log10 T
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mlp_forward_kernel(MlpDev w, Seed s, const double *in, double *out,
                                                          long long n) {
  const long long nw = ((n + 63) / 64);
  const long long wave0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / 64;
  const long long wstride = ((long long)gridDim.x * blockDim.x) / 64;
  const int l = threadIdx.x & 63;
  for (long long wv = wave0; wv < nw; wv += wstride) {  // wave-uniform loop
    const long long q = wv * 64 + l;
    const bool ok = q < n;
    const float x0 = ok ? norm01(in[2 * q], s.lr_lo, s.lr_hi) : 0.0f;
    const float x1 = ok ? norm01(in[2 * q + 1], s.le_lo, s.le_hi) : 0.0f;
    const float y = mlp_wave_forward_fast(w, x0, x1, l);
    if (ok) out[q] = s.lt_lo + 0.5 * ((double)y + 1.0) * (s.lt_hi - s.lt_lo);
  }
}

// ---------------------------------------------------------------------------
// training: forward + backward of 64 samples per workgroup (four waves)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// One 64-sample share of the batch, the four waves of a workgroup taking a
// quarter of each product: wave t the samples 16 t .. of the input and output
// layers, the units 16 t .. of the hidden layer's pre-activations and of every
// gradient.  A sum runs in one wave in a fixed order (samples in tile and row
// order), so the gradients do not depend on the split.  What bounds it: the
// latency of the chain of layers, each a few instructions per wave (one wave for
// all of it took 16 us per step for a batch of 4096).
//   part: per-workgroup gradient partials [gridDim.x][NPARAM]; loss_part[gridDim.x].
constexpr int HP = H + 8;  // padded LDS row of 64 bf16 values (16-byte reads of 16 rows spread over the banks)
__global__ __launch_bounds__(256) void mlp_fwd_bwd_kernel(MlpDev w, Seed s, const double *in, const double *tgt,
                                                          long long n, int batch, uint64_t seed, int step,
                                                          int random_batch, float *part, float *loss_part) {
  __shared__ __align__(16) short h1[H * HP];    // [q][k]
  __shared__ __align__(16) short h1t[H * HP];   // [k][q]
  __shared__ __align__(16) short dz2[H * HP];   // [q][o]
  __shared__ __align__(16) short dz2t[H * HP];  // [o][q]
  __shared__ float term[4][4][4][64];           // output-layer products [hidden tile][sample tile][row][lane]
  __shared__ float ys[H];
  const int l = threadIdx.x & 63, t = threadIdx.x >> 6, c = l & 15, g = l >> 4;
  const long long slot = (long long)blockIdx.x * 64 + l;
  long long q;
  if (random_batch)
    q = (long long)(splitmix64(seed ^ ((uint64_t)step << 32) ^ (uint64_t)slot) % (uint64_t)n);
  else
    q = slot;
  // this wave's weights
  const int o = 16 * t + c;  // its hidden unit (layer 2 output, or the layer 1 unit of the gradients)
  bf16x8 w2[2], w2t[2];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    w2[kt] = *(const bf16x8 *)(w.w2b + o * H + 32 * kt + 8 * g);
    w2t[kt] = *(const bf16x8 *)(w.w2tb + o * H + 32 * kt + 8 * g);
  }
  const float b2 = w.b2[o], w3 = from_bf16(w.w3b[o]);
  const float b1 = w.b1[o], w10 = from_bf16(w.w1b[2 * o]), w11 = from_bf16(w.w1b[2 * o + 1]);
  const float x0 = norm01(in[2 * q], s.lr_lo, s.lr_hi);
  const float x1 = norm01(in[2 * q + 1], s.le_lo, s.le_hi);
  const float tg = norm01(tgt[q], s.lt_lo, s.lt_hi);
  const float xb0 = round_bf16(x0), xb1 = round_bf16(x1);
  // layer 1 of the wave's sample tile
  {
    const int qq = 16 * t + c;
    const float a0 = __shfl(xb0, qq, 64), a1 = __shfl(xb1, qq, 64);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      bf16x8 a;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 32 * kt + 8 * g + e;
        float z = w.b1[k];
        z += from_bf16(w.w1b[2 * k]) * a0;
        z += from_bf16(w.w1b[2 * k + 1]) * a1;
        a[e] = to_bf16(fmaxf(z, 0.0f));
        h1t[k * HP + qq] = a[e];
      }
      *(bf16x8 *)(h1 + qq * HP + 32 * kt + 8 * g) = a;
    }
  }
  __syncthreads();
  // layer 2: the wave's 16 units for all samples; the output layer's products
  f32x4 acc[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
      z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8 *)(h1 + (16 * mt + c) * HP + 32 * kt + 8 * g), w2[kt],
                                                  z, 0, 0, 0);
    acc[mt] = z;
#pragma unroll
    for (int r = 0; r < 4; ++r) term[t][mt][r][l] = w3 * round_bf16(fmaxf(z[r] + b2, 0.0f));
  }
  __syncthreads();
  // layer 3 of the wave's sample tile: over the four unit tiles in order, then
  // over the 16 units of a tile
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = 0.0f;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) v += term[nt][t][r][l];
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    if (c == 0) ys[16 * t + 4 * g + r] = v + w.b3[0];
  }
  __syncthreads();
  const float y = ys[l];
  const float dy = 2.0f * (y - tg) / (float)batch;
  // output-layer and hidden-layer gradients of the wave's units
  float gW3 = 0.0f, gB2 = 0.0f;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qq = 16 * mt + 4 * g + r;
      const float dyq = __shfl(dy, qq, 64);
      const float z = acc[mt][r] + b2;
      gW3 += dyq * round_bf16(fmaxf(z, 0.0f));
      const float dz = z > 0.0f ? dyq * w3 : 0.0f;
      gB2 += dz;
      const short db = to_bf16(dz);
      dz2[qq * HP + o] = db;
      dz2t[o * HP + qq] = db;
    }
  __syncthreads();
  // dW2 = dz2^T h1: M = o (the wave's tile), N = k, K = q
  float *P = part + (long long)blockIdx.x * NPARAM;
  bf16x8 dA[2];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) dA[kt] = *(const bf16x8 *)(dz2t + o * HP + 32 * kt + 8 * g);
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
      d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dA[kt], *(const bf16x8 *)(h1t + (16 * nt + c) * HP + 32 * kt + 8 * g),
                                                  d, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) P[OFF_W2 + (16 * t + 4 * g + r) * H + 16 * nt + c] = d[r];
  }
  // dH1 = dz2 W2: M = q, N = k (the wave's tile), K = o; then the input layer
  float gB1 = 0.0f, gW10 = 0.0f, gW11 = 0.0f;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
      d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8 *)(dz2 + (16 * mt + c) * HP + 32 * kt + 8 * g), w2t[kt],
                                                  d, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qq = 16 * mt + 4 * g + r;
      const float xq0 = __shfl(xb0, qq, 64), xq1 = __shfl(xb1, qq, 64);
      float z1 = b1;
      z1 += w10 * xq0;
      z1 += w11 * xq1;
      const float dz1 = z1 > 0.0f ? d[r] : 0.0f;
      gB1 += dz1;
      gW10 += dz1 * xq0;
      gW11 += dz1 * xq1;
    }
  }
  // sum the per-lane partials over the four row groups (lanes with equal l%16)
  float v[5] = {gW3, gB2, gB1, gW10, gW11};
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    v[i] += __shfl_xor(v[i], 16, 64);
    v[i] += __shfl_xor(v[i], 32, 64);
  }
  if (l < 16) {
    P[OFF_W3 + o] = v[0];
    P[OFF_B2 + o] = v[1];
    P[OFF_B1 + o] = v[2];
    P[OFF_W1 + 2 * o] = v[3];
    P[OFF_W1 + 2 * o + 1] = v[4];
  }
  if (t == 0) {
    float gb3 = dy, loss = (y - tg) * (y - tg);
    for (int k = 32; k > 0; k >>= 1) {
      gb3 += __shfl_xor(gb3, k, 64);
      loss += __shfl_xor(loss, k, 64);
    }
    if (l == 0) {
      P[OFF_B3] = gb3;
      loss_part[blockIdx.x] = loss;
    }
  }
}

__device__ __forceinline__ void pack_param(int i, float x, short *w1b, short *w2b, short *w2tb, short *w3b, float *b1,
                                           float *b2, float *b3) {
  if (i < OFF_B1) {
    w1b[i] = to_bf16(x);
  } else if (i < OFF_W2) {
    b1[i - OFF_B1] = x;
  } else if (i < OFF_B2) {
    const int j = i - OFF_W2, o = j / H, k = j % H;
    w2b[o * H + k] = to_bf16(x);
    w2tb[k * H + o] = to_bf16(x);
  } else if (i < OFF_W3) {
    b2[i - OFF_B2] = x;
  } else if (i < OFF_B3) {
    w3b[i - OFF_W3] = to_bf16(x);
  } else {
    b3[0] = x;
  }
}

// Sum of the workgroup partials in their order, one parameter per thread, and
// with `a.apply` the Adam step on the fp32 master weights and the refresh of the
// copies the kernels read.  The last workgroup sums the loss.  One wave per
// workgroup, so the parameters spread over 70 compute units, and sixteen
// partials in flight per thread (as three kernels, the first with the loss as one
// thread's serial loop: 26 us per step for a batch of 4096).
struct AdamArgs {
  int apply;
  float lr, b1, b2, eps, c1, c2;
};
constexpr int kUpdateThreads = 64;
__global__ __launch_bounds__(kUpdateThreads) void mlp_update_kernel(const float *part, int nparts, float *grad,
                                                                    const float *loss_part, float *loss, int batch,
                                                                    AdamArgs a, float *wm, float *m, float *v,
                                                                    short *w1b, short *w2b, short *w2tb, short *w3b,
                                                                    float *b1, float *b2, float *b3) {
  if (blockIdx.x == gridDim.x - 1) {
    if (!loss) return;
    float s = 0.0f;
    for (int p0 = 0; p0 < nparts; p0 += 64) {
      const int p = p0 + (int)threadIdx.x;
      const float x = p < nparts ? loss_part[p] : 0.0f;
      const int most = nparts - p0 < 64 ? nparts - p0 : 64;
      for (int k = 0; k < most; ++k) s += __shfl(x, k, 64);
    }
    if (threadIdx.x == 0) *loss = s / (float)batch;
    return;
  }
  const int i = blockIdx.x * kUpdateThreads + threadIdx.x;
  if (i >= NPARAM) return;
  float s = 0.0f;
  int p = 0;
  for (; p + 16 <= nparts; p += 16) {
    float x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = part[(long long)(p + k) * NPARAM + i];
#pragma unroll
    for (int k = 0; k < 16; ++k) s += x[k];
  }
  for (; p < nparts; ++p) s += part[(long long)p * NPARAM + i];
  if (grad) grad[i] = s;
  if (!a.apply) return;
  const float mi = a.b1 * m[i] + (1.0f - a.b1) * s;
  const float vi = a.b2 * v[i] + (1.0f - a.b2) * s * s;
  m[i] = mi;
  v[i] = vi;
  const float x = wm[i] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  wm[i] = x;
  pack_param(i, x, w1b, w2b, w2tb, w3b, b1, b2, b3);
}

__global__ void mlp_pack_kernel(const float *wm, short *w1b, short *w2b, short *w2tb, short *w3b, float *b1, float *b2,
                                float *b3) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < NPARAM; i += gridDim.x * blockDim.x)
    pack_param(i, wm[i], w1b, w2b, w2tb, w3b, b1, b2, b3);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t mlp_launch_forward(const MlpDev &w, const Seed &s, const double *in, double *out, int64_t n,
                              hipStream_t st) {
  const long long waves = (n + 63) / 64;
  const long long blocks = (waves + 3) / 4;
  const int grid = blocks < 8192 ? (int)blocks : 8192;
  if (grid <= 0) return hipSuccess;
  hipLaunchKernelGGL(mlp_forward_kernel, dim3(grid), dim3(256), 0, st, w, s, in, out, (long long)n);
  return hipGetLastError();
}

hipError_t mlp_launch_fwd_bwd(const MlpDev &w, const Seed &s, const double *in, const double *tgt, int64_t n,
                              int batch, uint64_t seed, int step, int random_batch, float *part, float *loss_part,
                              hipStream_t st) {
  hipLaunchKernelGGL(mlp_fwd_bwd_kernel, dim3(batch / 64), dim3(256), 0, st, w, s, in, tgt, (long long)n, batch, seed,
                     step, random_batch, part, loss_part);
  return hipGetLastError();
}

static hipError_t launch_update(const float *part, int nparts, float *grad, const float *loss_part, float *loss,
                                int batch, const AdamArgs &a, float *wm, float *m, float *v, const MlpDev &w,
                                hipStream_t st) {
  hipLaunchKernelGGL(mlp_update_kernel, dim3((NPARAM + kUpdateThreads - 1) / kUpdateThreads + 1), dim3(kUpdateThreads),
                     0, st, part, nparts, grad, loss_part, loss, batch, a, wm, m, v, (short *)w.w1b, (short *)w.w2b,
                     (short *)w.w2tb, (short *)w.w3b, (float *)w.b1, (float *)w.b2, (float *)w.b3);
  return hipGetLastError();
}

hipError_t mlp_launch_reduce(const float *part, int nparts, float *grad, const float *loss_part, float *loss, int batch,
                             const MlpDev &w, hipStream_t st) {
  return launch_update(part, nparts, grad, loss_part, loss, batch, AdamArgs{}, nullptr, nullptr, nullptr, w, st);
}

hipError_t mlp_launch_adam(const float *part, int nparts, const float *loss_part, float *loss, int batch, float *wm,
                           float *m, float *v, float lr, float b1, float b2, float eps, float c1, float c2,
                           const MlpDev &w, hipStream_t st) {
  return launch_update(part, nparts, nullptr, loss_part, loss, batch, AdamArgs{1, lr, b1, b2, eps, c1, c2}, wm, m, v,
                       w, st);
}

hipError_t mlp_launch_pack(const float *wm, short *w1b, short *w2b, short *w2tb, short *w3b, float *b1, float *b2,
                           float *b3, hipStream_t st) {
  hipLaunchKernelGGL(mlp_pack_kernel, dim3((NPARAM + 255) / 256), dim3(256), 0, st, wm, w1b, w2b, w2tb, w3b, b1, b2,
                     b3);
  return hipGetLastError();
}

}  // namespace tdh

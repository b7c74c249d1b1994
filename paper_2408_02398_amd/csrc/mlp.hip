// mlp.hip -- training of the learned start on the GPU (BF16 matrix cores, FP32
// accumulation and FP32 master weights with Adam), and packing of the
// inference parameters.
//
// One training step on a batch of B (tensor, target direction) pairs, for the
// network of kin = 32 (K <= 32) or 48 (K <= 48) inputs and d' outputs:
//   X  = features(C)                         B x kin
//   Z1 = X W1 + b1,  H1 = bf16(relu Z1)      B x 64
//   Z2 = H1 W2 + b2, H2 = bf16(relu Z2)      B x 64
//   Y  = H2 W3 + b3                          B x 16 (d' used)
//   L  = mean_b 1 - (y_b . t_b / |y_b||t_b|)^2
//   dY, then dW3 = H2^T dY, dZ2 = (dY W3^T) * [Z2 > 0], dW2 = H1^T dZ2,
//   dZ1 = (dZ2 W2^T) * [Z1 > 0], dW1 = X^T dZ1, bias gradients = column sums,
//   Adam on the FP32 masters, then the BF16 fragment-ordered inference copy.
// Two kernels: k_train takes a part of the batch through the whole forward and
// backward pass and writes its share of the gradients, k_train_update adds the
// shares in order and updates.  Every product runs on BF16 matrix-core tiles
// (operands rounded to BF16, FP32 accumulation).
#include <algorithm>

#include "internal.hpp"
#include "mlp_core.hpp"
#include "sym_tables.hpp"

namespace ttm {

namespace {

// Samples a workgroup takes at a time: 16 for each of its wavefronts.  A batch
// is dealt out over at most kTrainGroups workgroups (their gradient shares are
// 29 KB each and are read again by the update): one for every CU.  With 128 / 256, a
// step of degree 6 takes 22 / 22 us for 8192 samples, 28 / 23 for 8193, 28 / 26 for
// 16384, 34 / 29 for 16385, 64 / 44 for 65 536 and 245 / 134 for 262 144.
constexpr int kTrainWaves = 4;
constexpr int kTrainBlock = 16 * kTrainWaves;
constexpr int kTrainGroups = 256;

__host__ __device__ inline int train_rows(int B) {   // samples per workgroup
  return ((B + kTrainBlock * kTrainGroups - 1) / (kTrainBlock * kTrainGroups)) * kTrainBlock;
}
__host__ __device__ inline int train_groups(int B) { return (B + train_rows(B) - 1) / train_rows(B); }

__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d) {
  bf16x4 r;
  r[0] = (short)bf16_bits(a);
  r[1] = (short)bf16_bits(b);
  r[2] = (short)bf16_bits(c);
  r[3] = (short)bf16_bits(d);
  return r;
}
__device__ __forceinline__ bf16x4 pack4(const f32x4& v) { return pack4(v[0], v[1], v[2], v[3]); }

// One wavefront's 16 x 64 tile of BF16 values in LDS.  A product's result
// fragment holds rows (samples) 4 (L/16) + j of column (unit) L % 16; stored by
// put, it is read back by get as the left operand of the next product, row
// L % 16, columns 16 s + 4 (L/16) + j.
struct Turn {
  static constexpr int kPitch = 68;
  unsigned short* t;
  __device__ __forceinline__ void put(int lane, int nt, const bf16x4& v) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) t[(4 * (lane >> 4) + j) * kPitch + 16 * nt + (lane & 15)] = (unsigned short)v[j];
  }
  __device__ __forceinline__ bf16x4 get(int lane, int s) const {
    const uint2 q = *reinterpret_cast<const uint2*>(t + (lane & 15) * kPitch + 16 * s + 4 * (lane >> 4));
    bf16x4 r;
    r[0] = (short)(q.x & 0xffffu);
    r[1] = (short)(q.x >> 16);
    r[2] = (short)(q.y & 0xffffu);
    r[3] = (short)(q.y >> 16);
    return r;
  }
};

// Forward and backward pass of train_rows(B) samples; the workgroup's gradient
// share goes to part[blockIdx.x * params ...] and its loss sum to
// loss_part[blockIdx.x].  A wavefront takes 16 samples through all layers: the
// activations stay in its registers (and a 2 KB turning buffer in LDS), and so
// do its shares of dW1, dW2 and dW3 (28 tiles of 16 x 16).  With each layer's
// product, column sum and split reduction a launch of its own (20 launches), a
// step of 8192 samples took 212 us, most of it in short kernels that each waited
// for one dependent load after another; now 22 us.
template <int N, int DP, int KT>
__global__ __launch_bounds__(64 * kTrainWaves) void k_train(const float* __restrict__ Cin,
                                                           const float* __restrict__ T, int B,
                                                           const float* __restrict__ params,
                                                           float* __restrict__ part,
                                                           float* __restrict__ loss_part) {
  using Lay = MlpLayout<KT>;
  constexpr int K = DP == 3 ? ncomp3(N) : ncomp4(N), NT = 64 * kTrainWaves;
  // weights as right operands, W[16 s + 4 (L/16) + j][16 n + L % 16]: W1, W2, W3;
  // and of the transposes, W[16 n + L % 16][16 s + 4 (L/16) + j]: W3^T, W2^T
  constexpr int F2 = 4 * KT, F3 = F2 + 16, F3T = F3 + 4, F2T = F3T + 4, FN = F2T + 16;
  struct Work {
    bf16x4 frag[FN][64];
    unsigned short turn[kTrainWaves][16 * Turn::kPitch];
    float c[kTrainWaves][16][K | 1];
  };
  constexpr size_t kGrad = (size_t)Lay::params * 4 * kTrainWaves;
  __shared__ __align__(16) unsigned char smem[sizeof(Work) > kGrad ? sizeof(Work) : kGrad];
  __shared__ float smu[16 * KT];      // sqrt(mu), 0 past K
  __shared__ float lsum[kTrainWaves];
  Work& w = *reinterpret_cast<Work*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, q = lane >> 4;
  for (int e = tid; e < FN * 64; e += NT) {
    const int f = e >> 6, l = e & 63, c16 = l & 15, k4 = 4 * (l >> 4);
    const float* W;
    int ld, row, col, dr, dc;
    if (f < F3) {               // W1, W2
      W = params + (f < F2 ? Lay::off_w1 : Lay::off_w2);
      const int g = f < F2 ? f : f - F2;
      ld = kMlpHid; row = 16 * (g >> 2) + k4; col = 16 * (g & 3) + c16; dr = 1; dc = 0;
    } else if (f < F3T) {       // W3
      W = params + Lay::off_w3;
      ld = kMlpOut; row = 16 * (f - F3) + k4; col = c16; dr = 1; dc = 0;
    } else if (f < F2T) {       // W3^T
      W = params + Lay::off_w3;
      ld = kMlpOut; row = 16 * (f - F3T) + c16; col = k4; dr = 0; dc = 1;
    } else {                    // W2^T
      W = params + Lay::off_w2;
      const int g = f - F2T;
      ld = kMlpHid; row = 16 * (g & 3) + c16; col = 16 * (g >> 2) + k4; dr = 0; dc = 1;
    }
    const float* e0 = W + row * ld + col;
    const int st = dr * ld + dc;
    w.frag[f][l] = pack4(e0[0], e0[st], e0[2 * st], e0[3 * st]);
  }
#pragma unroll
  for (int k = 0; k < 16 * KT; ++k) {
    float m = 0.0f;
    if constexpr (DP == 3) {
      constexpr Sym3<N> sy{};
      if (k < K) m = sqrtf(sy.mu[k < K ? k : 0]);
    } else {
      constexpr Sym4<N> sy{};
      if (k < K) m = sqrtf(sy.mu[k < K ? k : 0]);
    }
    if (tid == 0) smu[k] = m;
  }
  __syncthreads();
  float b1[4], b2[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    b1[n] = params[Lay::off_b1 + 16 * n + r16];
    b2[n] = params[Lay::off_b2 + 16 * n + r16];
  }
  const float b3 = params[Lay::off_b3 + r16];
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 dw1[KT][4], dw2[4][4], dw3[4];
  float db1[4] = {0.f, 0.f, 0.f, 0.f}, db2[4] = {0.f, 0.f, 0.f, 0.f}, db3 = 0.0f, loss = 0.0f;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    dw3[m] = zero;
#pragma unroll
    for (int n = 0; n < 4; ++n) dw2[m][n] = zero;
  }
#pragma unroll
  for (int m = 0; m < KT; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) dw1[m][n] = zero;
  const Turn turn{w.turn[wave]};
  float (&cs)[16][K | 1] = w.c[wave];
  const int rows = train_rows(B);
  for (int i0 = 0; i0 < rows; i0 += kTrainBlock) {
    const int s0 = blockIdx.x * rows + i0 + 16 * wave;   // this wavefront's first sample
    if (s0 >= B) break;
    // features sqrt(mu) C / ||C||_F, 0 past the batch
    const int ns = min(16, B - s0);
    for (int e = lane; e < 16 * K; e += 64) {
      const int i = e / K, k = e - i * K;
      cs[i][k] = i < ns ? Cin[(size_t)s0 * K + e] : 0.0f;
    }
    wave_lds_sync();
    float f2 = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float c = cs[r16][k] * smu[k];
      f2 = fmaf(c, c, f2);
    }
    const float inv = f2 > 0.0f ? 1.0f / sqrtf(f2) : 0.0f;   // of sample r16
    float invr[4];                                           // of samples 4 q + j
#pragma unroll
    for (int j = 0; j < 4; ++j) invr[j] = __shfl(inv, 4 * q + j);
    bf16x4 xa[KT], xt[KT];   // X as a left operand, and X^T (rows: features)
#pragma unroll
    for (int s = 0; s < KT; ++s) {
      float v[4], u[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 16 * s + 4 * q + j, kt = 16 * s + r16;
        v[j] = k < K ? cs[r16][k < K ? k : 0] * smu[k] * inv : 0.0f;
        u[j] = kt < K ? cs[4 * q + j][kt < K ? kt : 0] * smu[kt] * invr[j] : 0.0f;
      }
      xa[s] = pack4(v[0], v[1], v[2], v[3]);
      xt[s] = pack4(u[0], u[1], u[2], u[3]);
    }
    // forward; h1t, h2t: the activations as left operands of the weight
    // gradients (rows: units), which is how a product leaves them
    bf16x4 h1t[4], h2t[4];
    unsigned on1 = 0, on2 = 0;   // bit 4 n + j: Z > 0
    wave_lds_sync();
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = zero;
#pragma unroll
      for (int s = 0; s < KT; ++s) z = mfma16(xa[s], w.frag[4 * s + n][lane], z);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        z[j] += b1[n];
        on1 |= (z[j] > 0.0f ? 1u : 0u) << (4 * n + j);
        z[j] = fmaxf(z[j], 0.0f);
      }
      h1t[n] = pack4(z);
      turn.put(lane, n, h1t[n]);
    }
    wave_lds_sync();
    bf16x4 a[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = turn.get(lane, s);
    wave_lds_sync();
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = zero;
#pragma unroll
      for (int s = 0; s < 4; ++s) z = mfma16(a[s], w.frag[F2 + 4 * s + n][lane], z);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        z[j] += b2[n];
        on2 |= (z[j] > 0.0f ? 1u : 0u) << (4 * n + j);
        z[j] = fmaxf(z[j], 0.0f);
      }
      h2t[n] = pack4(z);
      turn.put(lane, n, h2t[n]);
    }
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = turn.get(lane, s);
    wave_lds_sync();
    f32x4 y = zero;
#pragma unroll
    for (int s = 0; s < 4; ++s) y = mfma16(a[s], w.frag[F3 + s][lane], y);
    // dL/dY for L = mean 1 - (u.t)^2, u = y/|y| over the first DP outputs:
    // dY = -2 c (t - c u) / (|y| B); lane: samples 4 q + j, output r16
    f32x4 dy = zero;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float yj = y[j] + b3;
      const int b = s0 + 4 * q + j;
      float yv[4], t[4], tt = 0.0f, yy = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        yv[i] = __shfl(yj, 16 * q + i);
        if (i >= DP) yv[i] = 0.0f;
        t[i] = i < DP ? T[(size_t)DP * min(b, B - 1) + i] : 0.0f;
        tt = fmaf(t[i], t[i], tt);
        yy = fmaf(yv[i], yv[i], yy);
      }
      const float tn = 1.0f / sqrtf(tt);
      const float ny = sqrtf(yy);
      const float iy = ny > 0.0f ? 1.0f / ny : 0.0f;
      float u[4], c = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t[i] *= tn;
        u[i] = yv[i] * iy;
        c = fmaf(u[i], t[i], c);
      }
      const float sc = -2.0f * c * iy / (float)B;
      if (b < B) {
#pragma unroll
        for (int i = 0; i < DP; ++i)
          if (r16 == i) dy[j] = sc * (t[i] - c * u[i]);
        if (r16 == 0) loss += 1.0f - c * c;
      }
    }
    // backward
    const bf16x4 dyt = pack4(dy);
    db3 += (dy[0] + dy[1]) + (dy[2] + dy[3]);
    turn.put(lane, 0, dyt);
    wave_lds_sync();
    const bf16x4 ady = turn.get(lane, 0);
    wave_lds_sync();
    bf16x4 dzt[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) dw3[m] = mfma16(h2t[m], dyt, dw3[m]);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = mfma16(ady, w.frag[F3T + n][lane], zero);
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = (on2 >> (4 * n + j)) & 1u ? z[j] : 0.0f;
      db2[n] += (z[0] + z[1]) + (z[2] + z[3]);
      dzt[n] = pack4(z);
      turn.put(lane, n, dzt[n]);
    }
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = turn.get(lane, s);
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n) dw2[m][n] = mfma16(h1t[m], dzt[n], dw2[m][n]);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = zero;
#pragma unroll
      for (int s = 0; s < 4; ++s) z = mfma16(a[s], w.frag[F2T + 4 * s + n][lane], z);
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = (on1 >> (4 * n + j)) & 1u ? z[j] : 0.0f;
      db1[n] += (z[0] + z[1]) + (z[2] + z[3]);
      const bf16x4 zt = pack4(z);
#pragma unroll
      for (int m = 0; m < KT; ++m) dw1[m][n] = mfma16(xt[m], zt, dw1[m][n]);
    }
    wave_lds_sync();
  }
  // sums over the samples that other lanes hold
  for (int off = 16; off < 64; off <<= 1) {
    db3 += __shfl_xor(db3, off);
    loss += __shfl_xor(loss, off);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      db1[n] += __shfl_xor(db1[n], off);
      db2[n] += __shfl_xor(db2[n], off);
    }
  }
  __syncthreads();   // the operands in LDS are done with
  float* g = reinterpret_cast<float*>(smem) + wave * Lay::params;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = 16 * n + r16;
#pragma unroll
      for (int m = 0; m < KT; ++m) g[Lay::off_w1 + (16 * m + 4 * q + j) * kMlpHid + col] = dw1[m][n][j];
#pragma unroll
      for (int m = 0; m < 4; ++m) g[Lay::off_w2 + (16 * m + 4 * q + j) * kMlpHid + col] = dw2[m][n][j];
      g[Lay::off_w3 + (16 * n + 4 * q + j) * kMlpOut + r16] = dw3[n][j];
    }
  if (q == 0) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      g[Lay::off_b1 + 16 * n + r16] = db1[n];
      g[Lay::off_b2 + 16 * n + r16] = db2[n];
    }
    g[Lay::off_b3 + r16] = db3;
  }
  if (lane == 0) lsum[wave] = loss;
  __syncthreads();
  const float* all = reinterpret_cast<const float*>(smem);
  for (int i = tid; i < Lay::params; i += NT) {
    float v = all[i];
#pragma unroll
    for (int x = 1; x < kTrainWaves; ++x) v += all[x * Lay::params + i];
    part[(size_t)blockIdx.x * Lay::params + i] = v;
  }
  if (tid == 0) {
    float l = lsum[0];
    for (int x = 1; x < kTrainWaves; ++x) l += lsum[x];
    loss_part[blockIdx.x] = l;
  }
}

// Place of master parameter i in the packed inference copy: a BF16 value of a
// weight fragment, or (bias) an FP32 value.
__device__ __forceinline__ void pack_param(const MlpRt& r, int i, float p, unsigned char* out) {
  int off = -1, base = 0, ld = kMlpHid;
  if (i < r.off_b1) { base = i; off = 0; }
  else if (i >= r.off_w2 && i < r.off_b2) { base = i - r.off_w2; off = r.pk_w2; }
  else if (i >= r.off_w3 && i < r.off_b3) { base = i - r.off_w3; off = r.pk_w3; ld = kMlpOut; }
  if (off >= 0) {
    const int row = base / ld, col = base % ld;
    const int frag = ld == kMlpOut ? row / 16 : (row / 16) * 4 + col / 16;
    const int lane = ((row % 16) / 4) * 16 + col % 16;
    reinterpret_cast<unsigned short*>(out + off)[(frag * 64 + lane) * 4 + row % 4] = bf16_bits(p);
  } else if (i < r.off_w2) {
    reinterpret_cast<float*>(out + r.pk_b1)[i - r.off_b1] = p;
  } else if (i < r.off_w3) {
    reinterpret_cast<float*>(out + r.pk_b2)[i - r.off_b2] = p;
  } else {
    reinterpret_cast<float*>(out + r.pk_b3)[i - r.off_b3] = p;
  }
}

// Adds the gradient shares (four threads per parameter, each a run of the
// shares in order, then the runs in order), hands the gradients out, and takes
// Adam's step with bias correction on the FP32 masters (padded rows / columns
// stay 0) and on the inference copy.
__global__ __launch_bounds__(256) void k_train_update(const float* __restrict__ part, int ng,
                                                      const float* __restrict__ loss_part, float inv_b,
                                                      float* __restrict__ loss_out, float* __restrict__ grads,
                                                      float* __restrict__ p, float* __restrict__ m,
                                                      float* __restrict__ v, MlpRt r, int adam, float lr,
                                                      float b1, float b2, float eps, float bc1, float bc2,
                                                      int K, int dout, unsigned char* __restrict__ packed) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane, per = (ng + 3) / 4;
  float s = 0.0f;
  if (i < r.params) {
#pragma unroll 8
    for (int g = sub * per; g < min(ng, (sub + 1) * per); ++g) s += part[(size_t)g * r.params + i];
  }
  red[sub][lane] = s;
  __syncthreads();
  if (sub == 1 && blockIdx.x == 0) {     // the loss, in order, on one wavefront
    float l = 0.0f;
    for (int g = lane; g < ng; g += 64) l += loss_part[g];
    for (int off = 32; off > 0; off >>= 1) l += __shfl_down(l, off);
    if (lane == 0) loss_out[0] = l * inv_b;
  }
  if (sub != 0 || i >= r.params) return;
  const float gi = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
  if (grads) grads[i] = gi;
  float pi = p[i];
  if (adam) {
    bool pad = false;
    if (i < r.off_b1) pad = (i / kMlpHid) >= K;                               // W1 rows >= K
    else if (i >= r.off_w3 && i < r.off_b3) pad = ((i - r.off_w3) % kMlpOut) >= dout;
    else if (i >= r.off_b3) pad = (i - r.off_b3) >= dout;
    float mi = 0.0f, vi = 0.0f;
    if (pad) {
      pi = 0.0f;
    } else {
      mi = b1 * m[i] + (1.0f - b1) * gi;
      vi = b2 * v[i] + (1.0f - b2) * gi * gi;
      pi -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    }
    m[i] = mi;
    v[i] = vi;
    p[i] = pi;
  }
  if (packed) pack_param(r, i, pi, packed);
}

// FP32 masters -> BF16 fragment-ordered weights + FP32 biases.
__global__ void k_pack(const float* __restrict__ p, MlpRt r, unsigned char* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < r.params) pack_param(r, i, p[i], out);
}

}  // namespace

size_t mlp_train_workspace(int B) {
  // gradient shares and loss sums of the workgroups: as many as any batch of up to B
  // samples has (a batch just over a multiple of kTrainBlock * kTrainGroups has fewer
  // than one just under it)
  const size_t most = std::min((size_t)kTrainGroups, ((size_t)B + kTrainBlock - 1) / kTrainBlock);
  return most * (MlpLayout<3>::params + 1) * 4;
}

int mlp_train_step(int degree, int dprime, const float* Cin, const float* T, int B, float* params,
                   float* adam_m, float* adam_v, int step, float lr, unsigned char* packed,
                   float* loss_out, float* grads_out, void* ws, hipStream_t s) {
  const int K = dprime == 3 ? ncomp3(degree) : ncomp4(degree);
  const MlpRt r = mlp_rt_for(K);
  const int ng = train_groups(B);
  float* part = static_cast<float*>(ws);
  float* lpart = part + (size_t)ng * r.params;
  const dim3 grid(ng), block(64 * kTrainWaves);
  switch (dprime * 10 + degree) {
    case 32: hipLaunchKernelGGL((k_train<2, 3, 2>), grid, block, 0, s, Cin, T, B, params, part, lpart); break;
    case 34: hipLaunchKernelGGL((k_train<4, 3, 2>), grid, block, 0, s, Cin, T, B, params, part, lpart); break;
    case 36: hipLaunchKernelGGL((k_train<6, 3, 2>), grid, block, 0, s, Cin, T, B, params, part, lpart); break;
    case 42: hipLaunchKernelGGL((k_train<2, 4, 2>), grid, block, 0, s, Cin, T, B, params, part, lpart); break;
    case 44: hipLaunchKernelGGL((k_train<4, 4, 3>), grid, block, 0, s, Cin, T, B, params, part, lpart); break;
    default: set_error("mlp: degree %d not built for d'=%d", degree, dprime); return -4;
  }
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float bc1 = 1.0f - powf(b1, (float)step), bc2 = 1.0f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_train_update, dim3((r.params + 63) / 64), dim3(256), 0, s, part, ng, lpart,
                     1.0f / (float)B, loss_out, grads_out, params, adam_m, adam_v, r, lr > 0.0f ? 1 : 0,
                     lr, b1, b2, eps, bc1, bc2, K, dprime, packed);
  TTM_HIP(hipGetLastError());
  return 0;
}

int mlp_pack(int K, const float* params, unsigned char* packed, hipStream_t s) {
  const MlpRt r = mlp_rt_for(K);
  hipLaunchKernelGGL(k_pack, dim3((r.params + 255) / 256), dim3(256), 0, s, params, r, packed);
  TTM_HIP(hipGetLastError());
  return 0;
}

}  // namespace ttm

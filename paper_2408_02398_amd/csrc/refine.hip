// refine.hip -- position refinement TTM-ref (Sec. 3.3, Alg. 3) and the tensor
// field at listed voxels by real-space sums (gfx950).
//
// For each peak x^i of the score map the search visits the sphere of voxels
// |x - x^i| <= r_s (the peak first, then the other offsets in lexicographic
// (dz, dy, dx) order, skipping voxels outside the valid region), takes at
// each voxel the optimal rotation of its tensor C(x) (the dominant
// eigenvector on S^3, d' = 4, Sec. 3.1) and the LNCC at that single rotation,
//   c(x, R) = w(x) sum_p g(x + p - c) t'(c + R^T (p - c))      (Eq. lncc),
// computed in real space from the template window, and keeps the voxel with
// the largest LNCC (a later voxel only on a strictly larger value, so ties
// keep the earlier one and the peak itself stays unless beaten).
//
// Kernels: k_offsets (the sphere's offsets), k_candidates (peak x offset ->
// voxel, or invalid), k_field_pack and k_field_at (C at every candidate, a product of the template
// components with the candidates' windows of g on the matrix cores), the d' = 4 multistart extraction (extract4.hip) on those
// tensors, k_ball and k_lncc (a wavefront per candidate, only the template voxels
// within r + 2 of the centre, where the rotated t' can be non-zero), k_best (one
// thread per peak).
#include "internal.hpp"
#include "mlp_core.hpp"

namespace ttm {

namespace {

constexpr int kFieldWaves = 4;
constexpr int field_mt(int K) { return (K + 15) / 16; }   // tiles of 16 components
constexpr int kMaxRefineRadius = 8;

struct RefineWs {
  int4* offs;       // sphere offsets (dz, dy, dx, 0), the zero offset first
  int* n_offs;
  int4* cand;       // candidate voxel (z, y, x, valid)
  unsigned* ball;   // template voxels the LNCC visits, x | y << 8 | z << 16
  int* n_ball;
  float* pack;      // template components in the order k_field_at reads them
  float* C;         // K x (n_peaks * V) tensors
  float* lam;       // n_peaks * V
  float* quat;      // n_peaks * V x 4
  float* lncc;      // n_peaks * V
  void* ext;        // d' = 4 extraction workspace
};

__host__ __device__ inline size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

// Offsets of the sphere of radius r_s as the device kernels enumerate them.
int sphere_count(float rs) {
  const int R = (int)floorf(rs);
  int n = 0;
  for (int dz = -R; dz <= R; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx)
        if ((float)(dz * dz + dy * dy + dx * dx) <= rs * rs) ++n;
  return n;
}

namespace {

constexpr size_t kOffsetBytes =
    (size_t)(2 * kMaxRefineRadius + 1) * (2 * kMaxRefineRadius + 1) * (2 * kMaxRefineRadius + 1) * 16;
constexpr size_t kBallBytes = (size_t)64 * 64 * 64 * 4;   // template edges are at most 64

// Blocks of 16 voxels of the template, each within one row.
__host__ __device__ inline int field_blocks(int L) { return L * L * ((L + 15) / 16); }

size_t refine_bytes(int K, int L, int n_peaks, int V, void* base, RefineWs* out) {
  const size_t n_cand = (size_t)n_peaks * V;
  char* p = static_cast<char*>(base);
  RefineWs w;
  auto take = [&](size_t bytes) {
    char* at = p;
    p += a256(bytes);
    return at;
  };
  w.offs = reinterpret_cast<int4*>(take(kOffsetBytes));
  w.n_offs = reinterpret_cast<int*>(take(256));
  w.n_ball = w.n_offs + 1;
  w.cand = reinterpret_cast<int4*>(take(n_cand * 16));
  w.ball = reinterpret_cast<unsigned*>(take(kBallBytes));
  w.pack = reinterpret_cast<float*>(take((size_t)field_blocks(L) * field_mt(K) * 256 * 4));
  w.C = reinterpret_cast<float*>(take((size_t)K * n_cand * 4));
  w.lam = reinterpret_cast<float*>(take(n_cand * 4));
  w.quat = reinterpret_cast<float*>(take(n_cand * 16));
  w.lncc = reinterpret_cast<float*>(take(n_cand * 4));
  w.ext = p;
  if (out) *out = w;
  return (size_t)(p - static_cast<char*>(base));
}

__global__ void k_offsets(float rs, int4* offs, int* n_offs) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int R = (int)floorf(rs);
  int n = 0;
  offs[n++] = make_int4(0, 0, 0, 0);
  for (int dz = -R; dz <= R; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx)
        if ((dz | dy | dx) != 0 && (float)(dz * dz + dy * dy + dx * dx) <= rs * rs)
          offs[n++] = make_int4(dz, dy, dx, 0);
  *n_offs = n;
}

// Candidate i * V + j = peak i + offset j, valid when its template window lies
// inside the volume (lo <= voxel <= hi on every axis).
__global__ void k_candidates(const int32_t* __restrict__ peaks, int n_peaks, const int4* __restrict__ offs,
                             int V, int4 lo, int4 hi, int4* __restrict__ cand) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (size_t)n_peaks * V) return;
  const int i = (int)(k / V), j = (int)(k % V);
  const int4 o = offs[j];
  const int z = peaks[3 * i] + o.x, y = peaks[3 * i + 1] + o.y, x = peaks[3 * i + 2] + o.z;
  const bool ok = z >= lo.x && z <= hi.x && y >= lo.y && y <= hi.y && x >= lo.z && x <= hi.z;
  cand[k] = make_int4(z, y, x, ok ? 1 : 0);
}

// x[4 g + j] in register j of lane group g (16 lanes) to x[4 s + g] in register s.
__device__ __forceinline__ void turn4(float (&v)[4]) {
  unsigned u[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) u[j] = __float_as_uint(v[j]);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const auto p = __builtin_amdgcn_permlane32_swap(u[j], u[j + 2], false, false);
    u[j] = p[0];
    u[j + 2] = p[1];
  }
#pragma unroll
  for (int j = 0; j < 4; j += 2) {
    const auto p = __builtin_amdgcn_permlane16_swap(u[j], u[j + 1], false, false);
    u[j] = p[0];
    u[j + 1] = p[1];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(u[j]);
}

// Block u of 16 template voxels of component tile m, 0 past the row's end and past
// the last component, in the order of k_field_at's loads: element
// ((u MT + m) 16 + a) 16 + 4 g + s holds voxel 4 s + g of component 16 m + a.
// (Read where they lie, the components are L^3 floats apart: at L = 32 every load
// of 16 of them met one memory channel, 2.4 ms against 0.85 ms for k_field_at.)
__global__ __launch_bounds__(256) void k_field_pack(const float* __restrict__ T, int K, int MT, int L,
                                                    float* __restrict__ pack) {
  const int e = threadIdx.x, m = blockIdx.y, u = blockIdx.x, ns = (L + 15) / 16;
  const int a = 16 * m + (e >> 4), x = 16 * (u % ns) + 4 * (e & 3) + ((e >> 2) & 3);
  pack[((size_t)u * MT + m) * 256 + e] =
      a < K && x < L ? T[(size_t)a * L * L * L + (size_t)(u / ns) * L + x] : 0.0f;
}

// C_a(x) = w(x) sum_p g(x + p - c) T_a(p) at every candidate x (Eq. tcc at single
// voxels): workgroup (peak, block of kFieldWaves tiles of 16 candidates, MW tiles
// of 16 components), one candidate tile per wavefront.
//
// A product T [a][p] x windows [p][x] on FP32 matrix-core tiles of 16
// components x 16 candidates x 4 template voxels.  A tile adds its four products
// one after the other like fmaf, and one accumulator takes all template voxels in
// order, so the sums are those of a plain loop over p, bit for bit: a candidate's
// best start is decided among runs whose lambda differ in the last bits, and
// another order of summation picks another of them (rotations 5e-3 apart).
// Lane l loads four voxels of window l % 16 at once, from 4 (l / 16) on, and turn4
// puts them into the order of the four steps.  Blocks of kFieldAhead x 16 voxels
// are loaded one ahead.  Bound by the matrix cores (three tiles for K = 35, a
// chain of products each) and the windows' scattered loads.  125 peaks x 123
// voxels, L = 32, K = 35: 0.85 ms, against 9.8 ms with a candidate per lane,
// whose K broadcast reads per voxel and 250 wavefronts left the chip idle.
constexpr int kFieldAhead = 4;
constexpr long kFieldSplitBelow = 128;   // workgroups

template <int K, int MW>
__global__ __launch_bounds__(64 * kFieldWaves) void k_field_at(
    const float* __restrict__ g, const float* __restrict__ w, int ny, int nx, const float* __restrict__ pack, int L,
    const int4* __restrict__ cand, int V, size_t n_cand, float* __restrict__ C) {
  constexpr int D = kFieldAhead, MT = field_mt(K);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, q4 = 4 * (lane >> 4);
  const int j0 = (blockIdx.y * kFieldWaves + wave) * 16, m0 = blockIdx.z * MW;
  if (j0 >= V) return;            // uniform per wavefront, and there is no barrier
  const int c = L / 2;
  const size_t k = (size_t)blockIdx.x * V + min(j0 + r16, V - 1);
  const int4 cv = cand[k];
  // an invalid candidate's sums are not used: it reads the volume's first window
  const float* win = g + (cv.w ? ((size_t)(cv.x - c) * ny + (cv.y - c)) * nx + (cv.z - c) : 0);
  const float* tp = pack + m0 * 256 + r16 * 16 + q4;
  // 16 voxels of a window row, from x on: this lane's four start at x + q4, moved
  // back where they would pass the row's end (then `last` turns them into the
  // voxels before the end and zeros)
  const int ns = (L + 15) / 16, U = L * L * ns, xl = 16 * (ns - 1) + q4;
  const int over = min(xl + 4 - L, 4);            // of the lane's four, in a row's last block: past the end
  auto load4 = [&](const float* row, int x, float (&v)[4]) {
    if (L >= 4) {
      __builtin_memcpy(v, row + min(x + q4, L - 4), 16);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = row[min(x + q4 + j, L - 1)];
    }
  };
  auto last = [&](float (&v)[4]) {
    const float o[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float s = o[j];
      if (L >= 4) {
        if (over == 1 && j < 3) s = o[j < 3 ? j + 1 : 3];
        if (over == 2 && j < 2) s = o[j < 2 ? j + 2 : 3];
        if (over == 3 && j < 1) s = o[3];
      }
      v[j] = xl + j < L ? s : 0.0f;
    }
  };
  int row = 0, t = 0, uf = 0;                     // of the block that is loaded next
  size_t go = 0;
  float an[D][MW][4], bn[D][4];
  auto fetch = [&]() {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      load4(win + go, 16 * t, bn[d]);
#pragma unroll
      for (int m = 0; m < MW; ++m) {
        const float4 q = *reinterpret_cast<const float4*>(tp + ((size_t)uf * MT + m) * 256);
        an[d][m][0] = q.x; an[d][m][1] = q.y; an[d][m][2] = q.z; an[d][m][3] = q.w;
      }
      if (uf + 1 < U) {                           // past the last block: loaded again, not used
        ++uf;
        if (++t == ns) {
          t = 0;
          ++row;
          go = ((size_t)(row / L) * ny + row % L) * nx;
        }
      }
    }
  };
  f32x4 acc[MW];
#pragma unroll
  for (int m = 0; m < MW; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
  fetch();
  int tc = 0;
  for (int u = 0; u < U; u += D) {
    float a[D][MW][4], b[D][4];
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        b[d][j] = bn[d][j];
#pragma unroll
        for (int m = 0; m < MW; ++m) a[d][m][j] = an[d][m][j];
      }
    }
    if (u + D < U) fetch();
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (u + d >= U) break;                      // uniform
      if (++tc == ns) {
        tc = 0;
        if (L % 16) last(b[d]);
      }
      turn4(b[d]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MW; ++m)
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][m][s], b[d][s], acc[m], 0, 0, 0);
    }
  }
  if (j0 + r16 >= V) return;
  const float wv = cv.w ? w[((size_t)cv.x * ny + cv.y) * nx + cv.z] : 0.0f;
#pragma unroll
  for (int m = 0; m < MW; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = 16 * (m0 + m) + q4 + i;       // lane: candidate r16, components 4 (l / 16) + i
      if (a < K) C[(size_t)a * n_cand + k] = cv.w ? wv * acc[m][i] : 0.0f;
    }
}

// The template voxels within r + 2 of the centre, in box order (one workgroup;
// a thread takes rows in turn).
__global__ __launch_bounds__(1024) void k_ball(int L, float r, unsigned* __restrict__ ball, int* __restrict__ n_ball) {
  __shared__ int at[64 * 64 + 1];
  const int c = L / 2, rows = L * L;
  const float lim = (r + 2.0f) * (r + 2.0f);
  auto half = [&](int i) {       // row i holds x in [c - h, c + h], h = -1: none
    const int dz = i / L - c, dy = i % L - c;
    int h = -1;
    while (h < L && (float)((h + 1) * (h + 1)) + (float)(dy * dy) + (float)(dz * dz) <= lim) ++h;
    return h;
  };
  for (int i = threadIdx.x; i < rows; i += 1024) {
    const int h = half(i);
    at[i] = h < 0 ? 0 : min(L - 1, c + h) - max(0, c - h) + 1;
  }
  __syncthreads();
  if (threadIdx.x < 64) {        // exclusive scan by one wavefront, a run of rows per lane
    const int per = (rows + 63) / 64, lo = min(rows, (int)threadIdx.x * per), hi = min(rows, lo + per);
    int own = 0;
    for (int i = lo; i < hi; ++i) own += at[i];
    int run = own;
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(run, off);
      if ((int)threadIdx.x >= off) run += v;
    }
    if (threadIdx.x == 63) *n_ball = run;
    run -= own;
    for (int i = lo; i < hi; ++i) {
      const int v = at[i];
      at[i] = run;
      run += v;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < rows; i += 1024) {
    const int h = half(i);
    if (h < 0) continue;
    unsigned* out = ball + at[i];
    for (int x = max(0, c - h); x <= min(L - 1, c + h); ++x)
      *out++ = (unsigned)x | (unsigned)(i % L) << 8 | (unsigned)(i / L) << 16;
  }
}

// LNCC of every candidate at its own rotation (Eq. lncc), in real space: one
// wavefront per candidate, persistent workgroups.  With BOX, t' sits in LDS
// (edges up to kBoxEdge); each sample reads its eight cells as four pairs along
// x, clamped into the box, with hat weights that are 0 for a cell not next to
// the point.  125 peaks x 123 voxels, L = 32, r = 14: 0.74 ms, against 3.6 ms
// with a workgroup per candidate and eight bounds-checked gathers from L2.
constexpr int kBoxEdge = 34;
constexpr int kLnccWaves = 16;

template <bool BOX>
__global__ __launch_bounds__(64 * kLnccWaves) void k_lncc(const float* __restrict__ g, const float* __restrict__ w,
                                                         int ny, int nx, const float* __restrict__ tn, int L,
                                                         const unsigned* __restrict__ ball,
                                                         const int* __restrict__ n_ball,
                                                         const int4* __restrict__ cand,
                                                         const float* __restrict__ quat, size_t n_cand,
                                                         float* __restrict__ lncc) {
  // odd row and slice pitches: a rotated row of samples can run along any axis
  constexpr int kPitch = kBoxEdge | 1;
  __shared__ float box[BOX ? kBoxEdge * ((kPitch * kBoxEdge) | 1) : 1];
  const int rp = BOX ? L | 1 : L, sp = BOX ? (rp * L) | 1 : L * L;
  if constexpr (BOX) {
    for (int i = threadIdx.x; i < L * L * L; i += 64 * kLnccWaves)
      box[i / (L * L) * sp + (i / L) % L * rp + i % L] = tn[i];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int c = L / 2, nb = *n_ball;
  const float cf = (float)c, top = (float)(L - 2);
  const size_t stride = (size_t)gridDim.x * kLnccWaves;
  for (size_t k = (size_t)blockIdx.x * kLnccWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); k < n_cand;
       k += stride) {
    const int4 cv = cand[k];
    if (cv.w == 0) {
      if (lane == 0) lncc[k] = -INFINITY;
      continue;
    }
    float qw = quat[4 * k], qx = quat[4 * k + 1], qy = quat[4 * k + 2], qz = quat[4 * k + 3];
    const float qn = sqrtf(qw * qw + qx * qx + qy * qy + qz * qz);
    if (!(qn > 0.0f)) {     // zero tensor: no rotation, the identity stands in
      qw = 1.0f; qx = qy = qz = 0.0f;
    } else {
      qw /= qn; qx /= qn; qy /= qn; qz /= qn;
    }
    const float R[9] = {1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                        2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                        2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)};
    const float* win = g + ((size_t)(cv.x - c) * ny + (cv.y - c)) * nx + (cv.z - c);
    float acc = 0.0f;
#pragma unroll 2
    for (int p = lane; p < nb; p += 64) {
      const unsigned v = ball[p];
      const int ix = v & 255, iy = (v >> 8) & 255, iz = v >> 16;
      const float gv = win[((size_t)iz * ny + iy) * nx + ix];
      const float dx = (float)(ix - c), dy = (float)(iy - c), dz = (float)(iz - c);
      // source point c + R^T (p - c), (x, y, z)
      const float sx = cf + R[0] * dx + R[3] * dy + R[6] * dz;
      const float sy = cf + R[1] * dx + R[4] * dy + R[7] * dz;
      const float sz = cf + R[2] * dx + R[5] * dy + R[8] * dz;
      const float fx = fminf(fmaxf(floorf(sx), 0.0f), top), fy = fminf(fmaxf(floorf(sy), 0.0f), top),
                  fz = fminf(fmaxf(floorf(sz), 0.0f), top);
      const float tx = sx - fx, ty = sy - fy, tz = sz - fz;
      const float wx0 = fmaxf(1.0f - fabsf(tx), 0.0f), wx1 = fmaxf(1.0f - fabsf(1.0f - tx), 0.0f);
      const float wy0 = fmaxf(1.0f - fabsf(ty), 0.0f), wy1 = fmaxf(1.0f - fabsf(1.0f - ty), 0.0f);
      const float wz0 = fmaxf(1.0f - fabsf(tz), 0.0f), wz1 = fmaxf(1.0f - fabsf(1.0f - tz), 0.0f);
      const int o = (int)fz * sp + (int)fy * rp + (int)fx;
      const float* t = BOX ? box + o : tn + o;
      float2 p00, p01, p10, p11;     // (x, x + 1) pairs, 4-byte aligned
      if constexpr (BOX) {
        p00 = make_float2(t[0], t[1]);
        p01 = make_float2(t[rp], t[rp + 1]);
        p10 = make_float2(t[sp], t[sp + 1]);
        p11 = make_float2(t[sp + rp], t[sp + rp + 1]);
      } else {
        __builtin_memcpy(&p00, t, 8);
        __builtin_memcpy(&p01, t + L, 8);
        __builtin_memcpy(&p10, t + L * L, 8);
        __builtin_memcpy(&p11, t + L * L + L, 8);
      }
      const float v0 = wy0 * (wx0 * p00.x + wx1 * p00.y) + wy1 * (wx0 * p01.x + wx1 * p01.y);
      const float v1 = wy0 * (wx0 * p10.x + wx1 * p10.y) + wy1 * (wx0 * p11.x + wx1 * p11.y);
      acc = fmaf(wz0 * v0 + wz1 * v1, gv, acc);
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
    if (lane == 0) lncc[k] = w[((size_t)cv.x * ny + cv.y) * nx + cv.z] * acc;
  }
}

// Per peak: the candidate with the largest LNCC, the peak itself first and a
// later candidate only on a strictly larger value.
__global__ void k_best(const int4* __restrict__ cand, const float* __restrict__ quat,
                       const float* __restrict__ lncc, int n_peaks, int V, int32_t* __restrict__ pos_out,
                       float* __restrict__ quat_out, float* __restrict__ lncc_out,
                       float* __restrict__ quat_peak, float* __restrict__ lncc_peak) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_peaks) return;
  const size_t k0 = (size_t)i * V;
  size_t best = k0;
  float bv = lncc[k0];
  for (int j = 1; j < V; ++j) {
    const float v = lncc[k0 + j];
    if (v > bv) {
      bv = v;
      best = k0 + j;
    }
  }
  pos_out[3 * i] = cand[best].x;
  pos_out[3 * i + 1] = cand[best].y;
  pos_out[3 * i + 2] = cand[best].z;
  lncc_out[i] = bv;
#pragma unroll
  for (int d = 0; d < 4; ++d) quat_out[4 * i + d] = quat[4 * best + d];
  if (quat_peak) {
#pragma unroll
    for (int d = 0; d < 4; ++d) quat_peak[4 * i + d] = quat[4 * k0 + d];
  }
  if (lncc_peak) lncc_peak[i] = lncc[k0];
}

template <int K>
void launch_field(const float* g, const float* w, int ny, int nx, const float* T, int L, const RefineWs& rw,
                  int n_peaks, int V, hipStream_t s) {
  constexpr int MT = field_mt(K);
  const int vb = (V + 16 * kFieldWaves - 1) / (16 * kFieldWaves);
  // One wavefront per candidate tile shares its windows among all component
  // tiles (125 peaks: 0.85 ms, 1.64 ms with a wavefront per component tile); with
  // fewer workgroups than half the CUs each component tile gets a wavefront of
  // its own, as the time is then that of one wavefront's chain of products.
  hipLaunchKernelGGL(k_field_pack, dim3(field_blocks(L), MT), dim3(256), 0, s, T, K, MT, L, rw.pack);
  const bool split = (long)n_peaks * vb < kFieldSplitBelow;
  hipLaunchKernelGGL(split ? (k_field_at<K, 1>) : (k_field_at<K, MT>), dim3(n_peaks, vb, split ? MT : 1),
                     dim3(64 * kFieldWaves), 0, s, g, w, ny, nx, rw.pack, L, rw.cand, V, (size_t)n_peaks * V, rw.C);
}

}  // namespace

size_t refine_workspace(int K, int L, int n_peaks, float rs) {
  const int V = sphere_count(rs);
  return refine_bytes(K, L, n_peaks, V, nullptr, nullptr) + extract_workspace4((size_t)n_peaks * V);
}

int max_refine_radius() { return kMaxRefineRadius; }

int refine(int degree, int K, const float* g, const float* w, int nz, int ny, int nx, const float* T,
           const float* tn, int L, float r, const int32_t* peaks, int n_peaks, float rs,
           const ExtractArgs& opts, int32_t* pos_out, float* quat_out, float* lncc_out,
           float* quat_peak, float* lncc_peak, void* ws, hipStream_t s) {
  const int V = sphere_count(rs);
  const size_t n_cand = (size_t)n_peaks * V;
  RefineWs rw;
  refine_bytes(K, L, n_peaks, V, ws, &rw);
  hipLaunchKernelGGL(k_offsets, dim3(1), dim3(64), 0, s, rs, rw.offs, rw.n_offs);
  const int c = L / 2;
  const int4 lo = make_int4(c, c, c, 0), hi = make_int4(nz - L + c, ny - L + c, nx - L + c, 0);
  hipLaunchKernelGGL(k_candidates, dim3((unsigned)((n_cand + 255) / 256)), dim3(256), 0, s, peaks,
                     n_peaks, rw.offs, V, lo, hi, rw.cand);
  switch (K) {
    case 10: launch_field<10>(g, w, ny, nx, T, L, rw, n_peaks, V, s); break;
    case 35: launch_field<35>(g, w, ny, nx, T, L, rw, n_peaks, V, s); break;
    case 84: launch_field<84>(g, w, ny, nx, T, L, rw, n_peaks, V, s); break;
    default: set_error("field at listed voxels: %d components not built", K); return -4;
  }
  ExtractArgs a = opts;
  a.items = nullptr;
  a.n_items = 0;
  a.C = rw.C;
  a.in_dtype = 0;
  a.plane = n_cand;
  a.by = 1;
  a.bx = (int)n_cand;
  a.score = nullptr;
  a.lam = rw.lam;
  a.dir = rw.quat;
  a.oz = a.oy = a.ox = 0;
  a.dy = 1;
  a.dx = (int)n_cand;
  a.mode = 2;
  a.ws = rw.ext;
  const int rc = launch_extract4(degree, a, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_ball, dim3(1), dim3(1024), 0, s, L, r, rw.ball, rw.n_ball);
  const size_t groups = (n_cand + kLnccWaves - 1) / kLnccWaves;
  // the box in LDS leaves room for one workgroup per CU
  const size_t most = L <= kBoxEdge ? 256 : 512;
  hipLaunchKernelGGL(L <= kBoxEdge ? k_lncc<true> : k_lncc<false>, dim3((unsigned)(groups < most ? groups : most)),
                     dim3(64 * kLnccWaves), 0, s, g, w, ny, nx, tn, L, rw.ball, rw.n_ball, rw.cand, rw.quat, n_cand,
                     rw.lncc);
  hipLaunchKernelGGL(k_best, dim3((n_peaks + 63) / 64), dim3(64), 0, s, rw.cand, rw.quat, rw.lncc,
                     n_peaks, V, pos_out, quat_out, lncc_out, quat_peak, lncc_peak);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "refine launch");
}

}  // namespace ttm

// fft.hip -- batched 3D real FFTs for the tensor-field correlations (gfx950).
//
// Spectrum layout: [kz][kx][ky], ky fastest, kx in 0..N/2 (the R2C half).
// Forward = X pass (two real rows packed as one complex row, R2C split on
// the way out, transposed store so ky becomes contiguous), Y pass (contiguous
// rows), Z pass (strided columns, 16 columns per workgroup so every global
// access is a 128-byte segment).  Templates, which are nonzero only in their
// first L z planes, stop after the Y pass and keep just those planes.
// Inverse = Z pass with the spectral product fused in (one read of G per tile
// for all components from 192 on, for parts of them below; each template column's z
// transform formed in registers from its L stored values), Y pass, X pass with the
// C2R merge, 1/N^3 scale, weight map, crop and dtype conversion fused into the store
// (k_c2c_rows and k_c2r_x; up to 160 both in k_c2r_plane, a plane in LDS).  The inverse
// of the two local sums forms w in its X pass from 192 on.
#include <algorithm>

#include "internal.hpp"

namespace ttm {

namespace {

constexpr int kRowsX = 16;  // real rows per workgroup in the X passes (packed in pairs)
constexpr int kRowsV = 16;  // rows of an inverse X workgroup that forms w: 8 of each local sum

// Tile element (z, y, x) of batch b, read at the nearest source voxel: the
// address is always in bounds, so a thread's loads need no branch and are in
// flight together (behind a bounds branch each load waited for the one before:
// 14 us for a 96^3 tile's X pass, 9 us without).  src_value then puts 0 where
// the element lies outside the source, centres it and squares it.
__device__ __forceinline__ float load_src(const RealSrc& s, int b, int z, int y, int x) {
  const int gz = min(max(s.oz + z, 0), s.dz - 1), gy = min(max(s.oy + y, 0), s.dy - 1),
            gx = min(max(s.ox + x, 0), s.dx - 1);
  return s.p[b * s.batch_stride + ((size_t)gz * s.dy + gy) * s.dx + gx];
}
__device__ __forceinline__ float src_value(const RealSrc& s, int b, int z, int y, int x, float v,
                                           double center) {
  const int gz = s.oz + z, gy = s.oy + y, gx = s.ox + x;
  if (s.center) v = (float)((double)v - center);
  if (s.square || (s.square_odd && (b & 1))) v = v * v;
  return gz < 0 || gz >= s.dz || gy < 0 || gy >= s.dy || gx < 0 || gx >= s.dx ? 0.0f : v;
}

// Workgroups go to the 8 XCDs in turn (workgroup i to XCD i mod 8), and each
// XCD has its own L2.  This renumbering hands every XCD one contiguous range
// of work items, so neighbouring items -- the two halves of a 128-byte line,
// the components that share a crop's weight-map rows -- meet in one L2.
__device__ __forceinline__ unsigned xcd_item(unsigned bid, unsigned n) {
  constexpr unsigned kXcd = 8;
  return n % kXcd ? bid : (bid % kXcd) * (n / kXcd) + bid / kXcd;
}

__device__ __forceinline__ unsigned short f32_to_bf16(float f) {
  unsigned int u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (unsigned short)(u >> 16);
}

// ---------------------------------------------------------------- X forward
template <int N>
__global__ __launch_bounds__(kRowsX / 2 * Plan<N>::T) void k_r2c_x(RealSrc src, cf* __restrict__ spec,
                                                          size_t spec_stride,
                                                          const cf* __restrict__ tw) {
  constexpr int T = Plan<N>::T, E = N / T, NP = kRowsX / 2, NH = N / 2 + 1;
  constexpr int S = lds_stride<N>();
  constexpr int RS = N + 8;  // padded real row
  constexpr int BYTES_A = kRowsX * RS * 4, BYTES_B = NP * S * 8;
  __shared__ __align__(16) unsigned char smem[BYTES_A > BYTES_B ? BYTES_A : BYTES_B];
  float* rows = reinterpret_cast<float*>(smem);
  cf* xl = reinterpret_cast<cf*>(smem);
  const int tid = threadIdx.x;
  const int y0 = blockIdx.x * kRowsX, z = blockIdx.y, b = blockIdx.z;
  const int p = tid / T, t = tid % T;
  FftTw<N> twr;
  twr.load(tw, t);
  {
    constexpr int NTH = NP * T, IT = kRowsX * N / NTH;
    static_assert(kRowsX * N % NTH == 0, "tile rows");
    const double center = src.center ? src.center[0] : 0.0;
    if constexpr (IT <= 32) {
      float ld[IT];  // all loads in flight, then the LDS stores
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int e = tid + i * NTH;
        ld[i] = load_src(src, b, z, y0 + e / N, e % N);
      }
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int e = tid + i * NTH;
        rows[(e / N) * RS + e % N] = src_value(src, b, z, y0 + e / N, e % N, ld[i], center);
      }
    } else {
      // edge 160: 40 loads at once with their index arithmetic take every register
      // and leave one wavefront on a SIMD (41 us a tile and its square; 28 in parts)
      constexpr int PL = IT / 4;
      static_assert(IT % PL == 0, "whole parts");
#pragma unroll 1
      for (int e0 = tid; e0 < kRowsX * N; e0 += PL * NTH) {
        float ld[PL];
#pragma unroll
        for (int i = 0; i < PL; ++i) {
          const int e = e0 + i * NTH;
          ld[i] = load_src(src, b, z, y0 + e / N, e % N);
        }
#pragma unroll
        for (int i = 0; i < PL; ++i) {
          const int e = e0 + i * NTH;
          rows[(e / N) * RS + e % N] = src_value(src, b, z, y0 + e / N, e % N, ld[i], center);
        }
      }
    }
  }
  __syncthreads();
  cf v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int n = t + T * j;
    v[j] = cf{rows[(2 * p) * RS + n], rows[(2 * p + 1) * RS + n]};
  }
  __syncthreads();  // rows and xl share memory
  fft_1d<N, false, true>(v, xl + p * S, twr, t);  // each pair's transform lies in one wavefront
#pragma unroll
  for (int j = 0; j < E; ++j) xl[p * S + lds_idx(t + T * j)] = v[j];
  __syncthreads();
  cf* out = spec + b * spec_stride + (size_t)z * NH * N + y0;
  for (int e = tid; e < NH * kRowsX; e += NP * T) {
    const int r = e % kRowsX, kx = e / kRowsX, pp = r >> 1;
    const cf zk = xl[pp * S + lds_idx(kx)];
    const cf zn = cconj(xl[pp * S + lds_idx((N - kx) % N)]);
    cf o;
    if ((r & 1) == 0) {
      o = cscale(cadd(zk, zn), 0.5f);              // (Z[k] + conj Z[N-k]) / 2
    } else {
      const cf d = csub(zk, zn);                   // (Z[k] - conj Z[N-k]) / 2i
      o = cf{0.5f * d.y, -0.5f * d.x};
    }
    out[(size_t)kx * N + r] = o;
  }
}

// ---------------------------------------------------------------- Y (rows)
template <int N, bool INV>
__global__ __launch_bounds__((128 / Plan<N>::T > 0 ? 128 / Plan<N>::T : 1) * Plan<N>::T) void
k_c2c_rows(cf* __restrict__ data, size_t batch_stride, int row_limit, int out_limit,
           const cf* __restrict__ tw) {
  constexpr int T = Plan<N>::T, E = N / T, RB = (128 / T > 0 ? 128 / T : 1);
  constexpr int S = lds_stride<N>();
  __shared__ cf xl[RB * S];
  const int tid = threadIdx.x;
  const int r = tid / T, t = tid % T;
  const int row = blockIdx.x * RB + r;
  FftTw<N> twr;
  twr.load(tw, t);
  // rows are (z, kx): z = row / (N/2+1); rows with z >= row_limit are not
  // needed and may lie past the end of the buffer, so they are not touched.
  // Only the first out_limit outputs of a row are stored (the inverse pass
  // keeps the crop's rows; the X pass reads no others).
  if ((int)(blockIdx.x * RB) / (N / 2 + 1) >= row_limit) return;  // uniform per workgroup
  const bool live = row / (N / 2 + 1) < row_limit;
  cf* base = data + blockIdx.y * batch_stride + (size_t)row * N;
  cf v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) v[j] = live ? base[t + T * j] : cf{0.0f, 0.0f};
  fft_1d<N, INV, true>(v, xl + r * S, twr, t);  // each row's transform lies in one wavefront
  if (live) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if (t + T * j < out_limit) base[t + T * j] = v[j];
    }
  }
}

// ---------------------------------------------------------------- Z (columns)
template <int N> struct ColBlock { static constexpr int CB = 16; };
// Columns per Z-inverse workgroup: 16 (128-byte row segments), 8 at N = 512
// with more than 2 plane slots (templates over 128 planes, beyond the edge
// the descriptor accepts today), where 16 would not fit the LDS.
template <int N, int JP> struct ZinvBlock { static constexpr int CB = (N >= 512 && JP > 2) ? 8 : 16; };

template <int N, bool INV>
__global__ __launch_bounds__(ColBlock<N>::CB * Plan<N>::T) void k_c2c_cols(
    cf* __restrict__ data, size_t batch_stride, const cf* __restrict__ tw) {
  constexpr int T = Plan<N>::T, E = N / T, CB = ColBlock<N>::CB, NC = (N / 2 + 1) * N;
  constexpr int S = lds_stride_cols<N>();
  __shared__ cf xl[CB * S];
  const int tid = threadIdx.x;
  const int c = tid % CB, t = tid / CB;
  const int col = blockIdx.x * CB + c;
  FftTw<N> twr;
  twr.load(tw, t);
  cf* base = data + blockIdx.y * batch_stride + col;
  cf v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) v[j] = base[(size_t)(t + T * j) * NC];
  fft_1d<N, INV>(v, xl + c * S, twr, t);
#pragma unroll
  for (int j = 0; j < E; ++j) base[(size_t)(t + T * j) * NC] = v[j];
}

// Element at byte offset `off` from `base`.  A 32-bit offset from a pointer
// that is the same for the whole workgroup lets the compiler address through
// a scalar base and one 32-bit register per access.
__device__ __forceinline__ const cf& at_byte(const cf* base, unsigned off) {
  return *reinterpret_cast<const cf*>(reinterpret_cast<const char*>(base) + off);
}

// Raw buffer accesses (a resource of `bytes` bytes from its base; the
// offset is in bytes).  kBufferWord3 is the gfx9 resource word that selects
// 32-bit elements, the format raw byte-offset accesses take.
constexpr int kBufferWord3 = 0x00020000;
typedef int int2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ cf buffer_load_cf(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(cf, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
__device__ __forceinline__ void buffer_store_cf(cf v, __amdgpu_buffer_rsrc_t r, unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(int2v, v), r, (int)off, 0, 0);
}

// Inverse Z pass with the spectral product: out_a = Z^-1( G conj(S_a) ).
// P holds only the sp nonzero z planes of each template after its X and Y
// passes; each column of S_a is their z transform, formed here in registers,
// which reads sp/N of the bytes a stored S_a would cost.  JP >= ceil(sp / T)
// plane slots per thread are kept (JP = 0: no template, G itself is
// inverted).  Each column's transforms run on T consecutive threads, inside
// one wavefront, so their exchanges need no workgroup barrier; global
// accesses go through LDS in the other order (column fastest), so that a
// wavefront reads and writes CB neighbouring columns of a z row together.
// Two workgroup barriers per component: after its planes are staged, and
// after its transformed columns are.  The planes of component a + 1 load
// while component a is transformed.  Grid y picks one of several G spectra
// (g_stride apart) for a one-component product: its output is work
// spectrum blockIdx.y.  Grid z splits the components: workgroup z takes
// components z * ac .. z * ac + ac - 1 (see inverse_n).
template <int N, int JP>
__global__ __launch_bounds__((ZinvBlock<N, JP>::CB * Plan<N>::T)) void k_zinv_mul(
    const cf* __restrict__ G, const cf* __restrict__ P, size_t p_stride, int sp, int A,
    const double* __restrict__ center, cf* __restrict__ out, size_t out_stride, int z_limit,
    const cf* __restrict__ tw, size_t g_stride, int ac) {
  constexpr int T = Plan<N>::T, E = N / T, CB = ZinvBlock<N, JP>::CB, NC = (N / 2 + 1) * N;
  G += blockIdx.y * g_stride;
  out += (blockIdx.y + (size_t)blockIdx.z * ac) * out_stride;
  P += blockIdx.z * ac * p_stride;
  A = min(ac, A - (int)blockIdx.z * ac);
  constexpr int S = lds_stride<N>();
  constexpr int SB = CB + 1;                // staging row: CB columns, one pad element
  constexpr int ZP = JP > 0 ? JP * T : 1;   // staged template planes
  // byte offsets inside one [z][kx][ky] spectrum stay below 2^32 for N <= 512
  constexpr unsigned ZSTEP = (unsigned)T * NC * 8u;
  static_assert((unsigned long long)N * NC * 8ull < (1ull << 32), "32-bit offsets");
  __shared__ cf xl[CB * S];
  __shared__ cf sb[N * SB];
  __shared__ cf pb[ZP * SB];
  const int tid = threadIdx.x;
  const int c = tid / T, t = tid % T;       // transforms: column c, element t + T j
  const int cc = tid % CB, tt = tid / CB;   // global accesses: column cc, z = tt + T k
  const unsigned col0 = xcd_item(blockIdx.x, gridDim.x) * CB;
  const unsigned offc = ((unsigned)tt * NC + col0 + cc) * 8u;
  FftTw<N> twr;
  twr.load(tw, t);
  {
    cf gl[E];
#pragma unroll
    for (int k = 0; k < E; ++k) gl[k] = at_byte(G, offc + k * ZSTEP);
#pragma unroll
    for (int k = 0; k < E; ++k) sb[(tt + T * k) * SB + cc] = gl[k];
  }
  // The template planes are read and the columns written through buffer
  // resources whose size ends at the sp stored planes and at the crop's
  // z_limit rows: the hardware returns 0 for a read past the end and drops a
  // write past it, so no lane needs a branch or a select for its row.
  cf qn[JP > 0 ? JP : 1];  // planes of the next component, global-access order
  auto load_planes = [&](int a) {
    const auto rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<cf*>(P + (size_t)a * p_stride), (short)0,
                                                      sp * NC * 8, kBufferWord3);
#pragma unroll
    for (int k = 0; k < JP; ++k) qn[k] = buffer_load_cf(rp, offc + k * ZSTEP);
  };
  if constexpr (JP > 0) load_planes(0);
  __syncthreads();  // G staged
  cf g[E];
#pragma unroll
  for (int j = 0; j < E; ++j) g[j] = sb[(t + T * j) * SB + c];
  // DC bin (kz = kx = ky = 0) is element j = 0 of thread t = 0 in column 0:
  // restore the mean removed before the forward transform.
  if (JP > 0 && center && col0 + c == 0 && t == 0) {
    g[0].x += (float)(center[0] * (double)N * (double)N * (double)N);
  }
  if constexpr (JP > 0) {
#pragma unroll
    for (int k = 0; k < JP; ++k) pb[(tt + T * k) * SB + cc] = qn[k];
  }
  // Component a: its planes are in pb; the planes of a + 1 load during its
  // transforms and are staged right after its columns are, before its
  // stores are issued.  Waiting for a load also waits for every earlier
  // store (one counter covers both), so staging the planes there waits only
  // for stores issued a whole component earlier, which have drained, and
  // this component's stores drain during the next one's transforms.
  for (int a = 0; a < A; ++a) {
    cf v[E];
    __syncthreads();  // component a's planes staged; the previous columns read from sb
    if constexpr (JP > 0) {
#pragma unroll
      for (int j = 0; j < E; ++j) v[j] = j < JP ? pb[(t + T * j) * SB + c] : cf{0.0f, 0.0f};
      if (a + 1 < A) load_planes(a + 1);
      fft_1d<N, false, true>(v, xl + c * S, twr, t);  // S_a along this column
#pragma unroll
      for (int j = 0; j < E; ++j) v[j] = cmulc(g[j], v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < E; ++j) v[j] = g[j];
    }
    fft_1d<N, true, true>(v, xl + c * S, twr, t);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if (t + T * j < z_limit) sb[(t + T * j) * SB + c] = v[j];
    }
    __syncthreads();  // columns staged; every wave has read component a's planes
    if constexpr (JP > 0) {
      if (a + 1 < A) {
#pragma unroll
        for (int k = 0; k < JP; ++k) pb[(tt + T * k) * SB + cc] = qn[k];
      }
    }
    const auto ro = __builtin_amdgcn_make_buffer_rsrc(out + (size_t)a * out_stride, (short)0,
                                                      z_limit * NC * 8, kBufferWord3);
#pragma unroll
    for (int k = 0; k < E; ++k) buffer_store_cf(sb[(tt + T * k) * SB + cc], ro, offc + k * ZSTEP);
  }
}

// ------------------------------------------------- Y and X inverse of a plane
// For N <= 160 one workgroup takes a whole (kx, ky) plane of one work spectrum
// -- contiguous in memory -- through the inverse Y transforms of its N/2 + 1
// rows and the inverse X transforms of its row pairs, so the plane is read once
// and only the cropped, scaled real rows are written: 2 N (N/2 + 1) * 8 bytes per
// plane less than a Y pass and an X pass of their own move.  Bound by its own
// latency (load, transforms and stores of one plane follow each other, and the
// LDS holds one to three planes per CU): K = 28, 96^3 64 -> 47 us, 128^3 (97^3
// crop) 140 -> 101 us.  Between the two transforms the
// plane sits in LDS as [kx][y].  PITCH (elements per kx row) holds a row's
// exchange area (N + N/16) and is 4 or 12 mod 32, so the 16-byte reads of a
// row pair (y, y + 1) by T consecutive kx fall on different banks.
// The same one-dimensional transforms run as in the separate passes: same bits.
template <int N> struct PlaneWg {
  static constexpr int NTH = ((N / 2 + 1) * Plan<N>::T + 63) / 64 * 64;       // every row at once
  static constexpr int EU = N <= 64 ? 4 : N <= 128 ? 5 : 3;                  // wavefronts per SIMD
};
template <int N> __host__ __device__ constexpr int plane_pitch() { return N == 32 ? 36 : N + 12; }
constexpr int kOutPad = 4;   // floats added to an output row in LDS

// Packed spectrum A + iB of the pair of real rows (2p, 2p + 1) at index n, from
// the plane in LDS (only kx <= N/2 is stored).
template <int N, int PITCH>
__device__ __forceinline__ cf pair_bin(const cf* plane, int p, int n) {
  const int m = n <= N / 2 ? n : N - n;
  const float4 q = *reinterpret_cast<const float4*>(plane + m * PITCH + 2 * p);
  cf a = cf{q.x, q.y}, b = cf{q.z, q.w};
  if (m == 0 || m == N / 2) {  // spectra of real rows: these bins are real
    a.y = 0.0f;
    b.y = 0.0f;
  }
  if (n > N / 2) {
    a = cconj(a);
    b = cconj(b);
  }
  return cf{a.x - b.y, a.y + b.x};  // A + iB
}

// Output rows 0 .. dst.sy - 1 of plane z, batch b, from LDS rows of N + kOutPad
// floats: scaled, weighted, converted.  Short rows (N <= 96) are dealt out voxel
// by voxel, UN weight-map loads in flight per thread; from 128 on a wavefront
// takes every NW-th row, 64 columns of all its rows at a time, so the row bases
// stay in scalar registers (a short row would leave half the lanes idle: whole
// 96^3 tile 172 us against 166, 128^3 tiles 1763 us against 1712 the other way).
template <int N, int NTH>
__device__ __forceinline__ void store_rows(const float* orow, const RealDst& dst, int b, int z, int tid) {
  constexpr int RS = N + kOutPad, NW = NTH / 64;
  const int nr = dst.sy, sx = dst.sx;
  const float* wr = dst.w ? dst.w + ((size_t)(dst.woz + z) * dst.wy + dst.woy) * dst.wx + dst.wox : nullptr;
  const size_t o0 = b * dst.batch_stride + ((size_t)(dst.vz0 + z) * dst.by + dst.vy0) * dst.bx + dst.vx0;
  auto put = [&](size_t row, int x, float v) {
    if (dst.dtype == 1) {
      (reinterpret_cast<unsigned short*>(dst.p) + o0 + row)[(unsigned)x] = f32_to_bf16(v);
    } else {
      (reinterpret_cast<float*>(dst.p) + o0 + row)[(unsigned)x] = v;
    }
  };
  if constexpr (N <= 96) {
    constexpr int UN = 6;
    const int total = nr * sx, dr = NTH / sx, dx = NTH - dr * sx;
    int r = tid / sx, x = tid - r * sx;
    for (int i0 = tid; i0 < total; i0 += UN * NTH) {
      float val[UN], wv[UN];
      int rr[UN], xx[UN];
#pragma unroll
      for (int k = 0; k < UN; ++k) {
        rr[k] = min(r, nr - 1);    // past the end: a row that exists, not stored
        xx[k] = x;
        wv[k] = wr ? wr[(size_t)rr[k] * dst.wx + x] : 1.0f;
        val[k] = orow[rr[k] * RS + x] * dst.scale;
        r += dr;
        x += dx;
        if (x >= sx) {
          x -= sx;
          ++r;
        }
      }
#pragma unroll
      for (int k = 0; k < UN; ++k)
        if (i0 + k * NTH < total) put((size_t)rr[k] * dst.bx, xx[k], wr ? val[k] * wv[k] : val[k]);
    }
  } else {
    constexpr int UN = (N + NW - 1) / NW;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int x = tid & 63; x < sx; x += 64) {
      float wv[UN];
      if (wr) {
#pragma unroll
        for (int k = 0; k < UN; ++k)   // rows past the end: the last one, not stored
          wv[k] = (wr + (size_t)min(wave + k * NW, nr - 1) * dst.wx)[(unsigned)x];
      }
#pragma unroll
      for (int k = 0; k < UN; ++k) {
        const int r = wave + k * NW;
        if (r >= nr) break;
        const float v = orow[r * RS + x] * dst.scale;
        put((size_t)r * dst.bx, x, wr ? v * wv[k] : v);
      }
    }
  }
}

// The whole plane in LDS (111 KB at 160).
template <int N>
__global__ __launch_bounds__(PlaneWg<N>::NTH) __attribute__((amdgpu_waves_per_eu(PlaneWg<N>::EU))) void k_c2r_plane(const cf* __restrict__ spec,
                                                               size_t spec_stride, int A, RealDst dst,
                                                               const cf* __restrict__ tw) {
  constexpr int T = Plan<N>::T, E = N / T, NH = N / 2 + 1, NTH = PlaneWg<N>::NTH, PITCH = plane_pitch<N>();
  constexpr int S = lds_stride<N>(), RS = N + kOutPad;
  constexpr int B1 = NH * PITCH * 8, B2 = N / 2 * S * 8, B3 = N * RS * 4;
  constexpr int BYTES = B1 > B2 ? (B1 > B3 ? B1 : B3) : (B2 > B3 ? B2 : B3);
  static_assert(64 % T == 0 && PITCH % 2 == 0 && PITCH >= N + N / 16 && BYTES <= 160 * 1024, "plane layout");
  __shared__ __align__(16) unsigned char smem[BYTES];
  cf* plane = reinterpret_cast<cf*>(smem);
  cf* xl = reinterpret_cast<cf*>(smem);
  float* orow = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x, q = tid / T, t = tid % T;
  // component fastest: the workgroups that share a plane's weight-map rows run
  // together in one XCD
  const int item = (int)xcd_item(blockIdx.x, gridDim.x);
  const int b = item % A, z = item / A;
  const cf* in = spec + b * spec_stride + (size_t)z * NH * N;
  FftTw<N> twr;
  cf v[E];
  const int row = min(q, NH - 1);                   // the last wavefront's spare lanes read a row that exists
#pragma unroll
  for (int j = 0; j < E; ++j) v[j] = at_byte(in, (unsigned)(row * N + t + T * j) * 8u);
  twr.load(tw, t);
  if (q < NH) {
    cf* mine = plane + q * PITCH;                   // each row's transform lies in one wavefront
    fft_1d<N, true, true>(v, mine, twr, t);
#pragma unroll
    for (int j = 0; j < E; ++j) mine[t + T * j] = v[j];
    // the row paired with the last kept one in one complex transform is zero
    if ((dst.sy & 1) && t == dst.sy % T) mine[dst.sy] = cf{0.0f, 0.0f};
  }
  __syncthreads();
  const bool live = 2 * q < dst.sy;                 // pair q holds a kept row
  if (live) {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = pair_bin<N, PITCH>(plane, q, t + T * j);
  }
  __syncthreads();  // exchange areas overlap the plane
  if (live) fft_1d<N, true, true>(v, xl + q * S, twr, t);
  __syncthreads();  // the rows overlap other pairs' exchange areas
  if (live) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      orow[(2 * q) * RS + t + T * j] = v[j].x;
      orow[(2 * q + 1) * RS + t + T * j] = v[j].y;
    }
  }
  __syncthreads();
  store_rows<N, NTH>(orow, dst, b, z, tid);
}

// ---------------------------------------------------------------- X inverse
// RC output rows of a component in a workgroup (see inverse_n).
// VAR: the two local sums' spectra (spec_stride apart), RC / 2 rows of each, and
// w formed from them in place of two stores, two loads and a launch (512^3 tile:
// 901 -> 529 us for the sums and w, 256^3: 107 -> 77).  Rows are packed in pairs of one sum:
// packed across the sums, each would carry rounding on the other's scale.
template <int N, int RC, bool VAR>
__global__ __launch_bounds__(RC / 2 * Plan<N>::T) __attribute__((amdgpu_waves_per_eu(N == 512 ? 8 : 1))) void k_c2r_x(const cf* __restrict__ spec,
                                                          size_t spec_stride, int A, RealDst dst,
                                                          VarDst var, const cf* __restrict__ tw) {
  constexpr int T = Plan<N>::T, E = N / T, NP = RC / 2, NH = N / 2 + 1;
  constexpr int S = lds_stride<N>();
  constexpr int SPS = NH + 1;  // padded spectrum row
  constexpr int BYTES_A = RC * SPS * 8, BYTES_B = NP * S * 8, BYTES_C = RC * (N + 4) * 4;
  constexpr int BYTES = BYTES_A > BYTES_B ? (BYTES_A > BYTES_C ? BYTES_A : BYTES_C)
                                          : (BYTES_B > BYTES_C ? BYTES_B : BYTES_C);
  __shared__ __align__(16) unsigned char smem[BYTES];
  cf* sp = reinterpret_cast<cf*>(smem);
  cf* xl = reinterpret_cast<cf*>(smem);
  float* orow = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x;
  // work items: component fastest, then row block, then z plane, so the
  // workgroups that share a crop's weight-map rows run together in one XCD
  constexpr int RW = VAR ? RC / 2 : RC;   // output rows
  constexpr int NYB = N / RW;
  const int item = (int)xcd_item(blockIdx.x, gridDim.x);
  if constexpr (VAR) A = 1;
  const int b = item % A, y0 = (item / A) % NYB * RW, z = item / A / NYB;
  if (z >= dst.sz || y0 >= dst.sy) return;  // uniform: nothing of this block is kept
  const int p = tid / T, t = tid % T;
  constexpr int NTH = NP * T, NIN = NH * RC, IT = (NIN + NTH - 1) / NTH;
  const cf* in = spec + b * spec_stride + (size_t)z * NH * N + y0;
  {
    // all loads first (indices clamped, so every one is in bounds), then the
    // LDS stores: the loads are in flight together.  Rows past the crop were
    // not stored by the Y pass; they are read as zeros (each is paired with a
    // kept row in one complex transform, so it must be finite).
    const int nrows_in = min(RW, dst.sy - y0);
    cf ld[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int e = min(tid + i * NTH, NIN - 1);
      const unsigned half = VAR && e % RC >= RW ? (unsigned)spec_stride : 0u;
      ld[i] = e % RW < nrows_in ? at_byte(in, (half + (unsigned)((e / RC) * N + e % RW)) * 8u) : cf{0.0f, 0.0f};
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int e = tid + i * NTH;
      if (e < NIN) sp[(e % RC) * SPS + e / RC] = ld[i];
    }
  }
  FftTw<N> twr;  // in flight across the barrier
  twr.load(tw, t);
  __syncthreads();
  cf v[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int n = t + T * j;
    cf a, bb;
    if (n <= N / 2) {
      a = sp[(2 * p) * SPS + n];
      bb = sp[(2 * p + 1) * SPS + n];
      if (n == 0 || n == N / 2) {  // spectra of real rows: these bins are real
        a.y = 0.0f;
        bb.y = 0.0f;
      }
    } else {
      a = cconj(sp[(2 * p) * SPS + (N - n)]);
      bb = cconj(sp[(2 * p + 1) * SPS + (N - n)]);
    }
    v[j] = cf{a.x - bb.y, a.y + bb.x};  // A + iB
  }
  __syncthreads();
  fft_1d<N, true, true>(v, xl + p * S, twr, t);  // each pair's transform lies in one wavefront
  __syncthreads();  // the row buffer overlaps other pairs' exchange areas
  constexpr int RS = N + 4;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int n = t + T * j;
    orow[(2 * p) * RS + n] = v[j].x;
    orow[(2 * p + 1) * RS + n] = v[j].y;
  }
  __syncthreads();
  const int nrows = min(RW, dst.sy - y0);
  const int sx = dst.sx;
  if constexpr (VAR) {
    const double thr = var.eps * var.M * var.stats[1];
    float* out = var.w + ((size_t)(var.oz + z) * var.ny + (var.oy + y0)) * var.nx + var.ox;
    for (int i = tid; i < nrows * sx; i += NTH) {
      const int r = i / sx, x = i - r * sx;
      out[(size_t)r * var.nx + x] = inverse_deviation(orow[r * RS + x] * dst.scale, orow[(r + RW) * RS + x] * dst.scale,
                                                      var.M, thr);
    }
    return;
  }
  // row bases are the same for the whole workgroup, so each access takes a
  // scalar base and the lane's 32-bit byte offset
  const size_t o0 = b * dst.batch_stride +
                    ((size_t)(dst.vz0 + z) * dst.by + (dst.vy0 + y0)) * dst.bx + dst.vx0;
  const float* wr = dst.w ? dst.w + ((size_t)(dst.woz + z) * dst.wy + (dst.woy + y0)) * dst.wx + dst.wox
                          : nullptr;
  // one output column x of one group of RH rows per thread and pass: the
  // group's weight-map loads (row indices clamped into the crop) are in flight
  // together
  constexpr int RH = 16, NG = RC / RH;
  for (int i = tid; i < sx * NG; i += NTH) {
    const int g = i / sx, x = i - g * sx, r0 = g * RH;
    float val[RH];
#pragma unroll
    for (int r = 0; r < RH; ++r) val[r] = orow[(r0 + r) * RS + x] * dst.scale;
    if (wr) {
      float wv[RH];
#pragma unroll
      for (int r = 0; r < RH; ++r) {
        const float* row = wr + (size_t)min(r0 + r, nrows - 1) * dst.wx;
        wv[r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + 4u * (unsigned)x);
      }
#pragma unroll
      for (int r = 0; r < RH; ++r) val[r] *= wv[r];
    }
    if (dst.dtype == 1) {
      unsigned short* out = reinterpret_cast<unsigned short*>(dst.p) + o0;
#pragma unroll
      for (int r = 0; r < RH; ++r) {
        if (r0 + r < nrows) {
          char* row = reinterpret_cast<char*>(out + (size_t)(r0 + r) * dst.bx);
          *reinterpret_cast<unsigned short*>(row + 2u * (unsigned)x) = f32_to_bf16(val[r]);
        }
      }
    } else {
      float* out = reinterpret_cast<float*>(dst.p) + o0;
#pragma unroll
      for (int r = 0; r < RH; ++r) {
        if (r0 + r < nrows) {
          char* row = reinterpret_cast<char*>(out + (size_t)(r0 + r) * dst.bx);
          *reinterpret_cast<float*>(row + 4u * (unsigned)x) = val[r];
        }
      }
    }
  }
}

__global__ void k_twiddles(cf* tw_all) {
  const int sizes[8] = {32, 64, 128, 256, 512, 96, 160, 192};
  int off = 0;
  for (int s = 0; s < 8; ++s) {
    const int N = sizes[s];
    for (int e = threadIdx.x; e < N; e += blockDim.x) {
      double sv, cv;
      sincospi(-2.0 * (double)e / (double)N, &sv, &cv);
      tw_all[off + e] = cf{(float)cv, (float)sv};
    }
    off += N;
  }
}

template <int N>
int forward_n(const RealSrc& src, int batch, cf* spec, size_t spec_stride, const cf* tw,
              hipStream_t s) {
  constexpr int T = Plan<N>::T;
  hipLaunchKernelGGL(k_r2c_x<N>, dim3(N / kRowsX, N, batch), dim3(kRowsX / 2 * T), 0, s, src, spec,
                     spec_stride, tw);
  constexpr int RB = (128 / T > 0 ? 128 / T : 1);
  constexpr int NROWS = N * (N / 2 + 1);
  hipLaunchKernelGGL((k_c2c_rows<N, false>), dim3(NROWS / RB, batch), dim3(RB * T), 0, s, spec,
                     spec_stride, N, N, tw);
  constexpr int CB = ColBlock<N>::CB;
  hipLaunchKernelGGL((k_c2c_cols<N, false>), dim3(NROWS / CB, batch), dim3(CB * T), 0, s, spec,
                     spec_stride, tw);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "fft forward launch");
}

template <int N>
int forward_planes_n(const RealSrc& src, int batch, int planes, cf* out, size_t out_stride,
                     const cf* tw, hipStream_t s) {
  constexpr int T = Plan<N>::T;
  hipLaunchKernelGGL(k_r2c_x<N>, dim3(N / kRowsX, planes, batch), dim3(kRowsX / 2 * T), 0, s, src,
                     out, out_stride, tw);
  constexpr int RB = (128 / T > 0 ? 128 / T : 1);
  const int rows = planes * (N / 2 + 1);
  hipLaunchKernelGGL((k_c2c_rows<N, false>), dim3((rows + RB - 1) / RB, batch), dim3(RB * T), 0, s,
                     out, out_stride, planes, N, tw);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "fft forward launch");
}

template <int N>
int inverse_n(const cf* G, const cf* Sp, size_t s_stride, int s_planes, int A, const double* center,
              cf* work, size_t work_stride, const RealDst& dst, const cf* tw, hipStream_t s,
              int gb, size_t g_stride, const VarDst* var) {
  constexpr int T = Plan<N>::T;
  constexpr int NROWS = N * (N / 2 + 1);
  const int zlim = dst.sz;
  constexpr int E = N / T;
  // template slots per thread: the next power of two >= ceil(s_planes / T),
  // and at least 2 at N = 512, whose one-slot variant the compiler keeps in
  // more registers (137 against 123)
  int jp = 0;
  if (Sp) {
    jp = N == 512 ? 2 : 1;
    while (jp < E && jp * T < s_planes) jp *= 2;
  }
  // Few columns (a 96^3 tile has 294 workgroups of two wavefronts) leave the
  // chip idle while every workgroup walks all A components, so up to 160 the
  // components are split until 4096 workgroups are in the grid; at least 4 components
  // stay together (2 where the columns alone do not give each CU a workgroup),
  // because each part reads G again.  K = 28: 96^3 75 -> 45 us, 128^3 75 -> 62 us,
  // 64^3 (K = 15) 19 -> 8.5 us.  From 192 on the read of G counts for more, and the Y
  // pass finds less of its input in the caches: 256^3 in two parts, both passes
  // together, K = 6 227 -> 243 us, K = 28 1223 -> 1228.
  auto launch = [&](auto kern, int cb) {
    const int nblk = NROWS / cb, least = nblk < 256 ? 2 : 4;
    const int parts = N < 192 ? std::max(1, std::min((A + least - 1) / least, 4096 / nblk + (4096 % nblk != 0))) : 1;
    const int ac = (A + parts - 1) / parts;
    hipLaunchKernelGGL(kern, dim3(nblk, gb, (A + ac - 1) / ac), dim3(cb * T), 0, s, G, Sp, s_stride,
                       s_planes, A, center, work, work_stride, zlim, tw, g_stride, ac);
  };
  constexpr int J2 = 2 < E ? 2 : E, J4 = 4 < E ? 4 : E, J8 = 8 < E ? 8 : E;
  switch (jp) {
    case 0: launch(k_zinv_mul<N, 0>, ZinvBlock<N, 0>::CB); break;
    case 1: launch(k_zinv_mul<N, 1>, ZinvBlock<N, 1>::CB); break;
    case 2: launch(k_zinv_mul<N, J2>, ZinvBlock<N, J2>::CB); break;
    case 4: launch(k_zinv_mul<N, J4>, ZinvBlock<N, J4>::CB); break;
    case 8: launch(k_zinv_mul<N, J8>, ZinvBlock<N, J8>::CB); break;
    default: launch(k_zinv_mul<N, E>, ZinvBlock<N, E>::CB); break;
  }
  const int nb = A * gb;  // work spectra written by the Z pass
  if constexpr (N <= 160) {   // at 192 one plane fills the LDS: 1084 us a tile (K = 28) in two passes, 1148 us in one
    hipLaunchKernelGGL(k_c2r_plane<N>, dim3(nb * zlim), dim3(PlaneWg<N>::NTH), 0, s, work, work_stride, nb,
                       dst, tw);
  } else {
    constexpr int RB = (128 / T > 0 ? 128 / T : 1);
    hipLaunchKernelGGL((k_c2c_rows<N, true>), dim3(NROWS / RB, nb), dim3(RB * T), 0, s, work,
                       work_stride, zlim, dst.sy, tw);
    static_assert(inverse_fuses_variance(N), "the sums' rows in the X pass");
    auto rows = [&](auto kern, int rc, int items, const VarDst& v) {
      hipLaunchKernelGGL(kern, dim3(items * N), dim3(rc / 2 * T), 0, s, work, work_stride, nb, dst, v, tw);
    };
    // Rows of a workgroup: 16 put more wavefronts on a CU, 32 read the columns in pieces of
    // 256 bytes.  512: 16 (28 components of 473^3 6.63 -> 6.54 ms, bfloat16 5.89 -> 5.57).
    // Below, 32 are 4 to 7 % faster (28 components of 249^3 at 256 866 us against 925,
    // 160^3 at 192 287 against 301; bfloat16 4 %), unless 16 spare half a block of at most
    // 7 (8 for bfloat16): 197^3 at 256 634 us either way, bfloat16 568 -> 548, 35
    // components 614 -> 571.
    const int blocks = (dst.sy + 31) / 32;
    const bool half = (dst.sy - 1) % 32 < 16 && blocks <= (dst.dtype == 1 ? 8 : 7);
    if (var) {
      rows(k_c2r_x<N, kRowsV, true>, kRowsV, N / (kRowsV / 2), *var);
    } else if (N == 512 || half) {
      rows(k_c2r_x<N, 16, false>, 16, nb * (N / 16), VarDst{});
    } else if constexpr (N != 512) {
      rows(k_c2r_x<N, 32, false>, 32, nb * (N / 32), VarDst{});
    }
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "fft inverse launch");
}

}  // namespace

int twiddle_offset(int N) {
  switch (N) {
    case 32: return 0;
    case 64: return 32;
    case 128: return 96;
    case 256: return 224;
    case 512: return 480;
    case 96: return 992;
    case 160: return 1088;
    case 192: return 1248;
    default: return -1;
  }
}

int init_twiddles(cf* tw_all, hipStream_t s) {
  hipLaunchKernelGGL(k_twiddles, dim3(1), dim3(256), 0, s, tw_all);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "twiddle init");
}

int fft3d_forward(int N, const RealSrc& src, int batch, cf* spec, size_t spec_stride,
                  const cf* tw_all, hipStream_t s) {
  const cf* tw = tw_all + twiddle_offset(N);
  switch (N) {
    case 32: return forward_n<32>(src, batch, spec, spec_stride, tw, s);
    case 64: return forward_n<64>(src, batch, spec, spec_stride, tw, s);
    case 128: return forward_n<128>(src, batch, spec, spec_stride, tw, s);
    case 256: return forward_n<256>(src, batch, spec, spec_stride, tw, s);
    case 512: return forward_n<512>(src, batch, spec, spec_stride, tw, s);
    case 96: return forward_n<96>(src, batch, spec, spec_stride, tw, s);
    case 160: return forward_n<160>(src, batch, spec, spec_stride, tw, s);
    case 192: return forward_n<192>(src, batch, spec, spec_stride, tw, s);
    default: set_error("unsupported FFT edge %d", N); return -4;
  }
}

int fft3d_forward_planes(int N, const RealSrc& src, int batch, int planes, cf* out,
                         size_t out_stride, const cf* tw_all, hipStream_t s) {
  const cf* tw = tw_all + twiddle_offset(N);
  switch (N) {
    case 32: return forward_planes_n<32>(src, batch, planes, out, out_stride, tw, s);
    case 64: return forward_planes_n<64>(src, batch, planes, out, out_stride, tw, s);
    case 128: return forward_planes_n<128>(src, batch, planes, out, out_stride, tw, s);
    case 256: return forward_planes_n<256>(src, batch, planes, out, out_stride, tw, s);
    case 512: return forward_planes_n<512>(src, batch, planes, out, out_stride, tw, s);
    case 96: return forward_planes_n<96>(src, batch, planes, out, out_stride, tw, s);
    case 160: return forward_planes_n<160>(src, batch, planes, out, out_stride, tw, s);
    case 192: return forward_planes_n<192>(src, batch, planes, out, out_stride, tw, s);
    default: set_error("unsupported FFT edge %d", N); return -4;
  }
}

int fft3d_inverse_mul(int N, const cf* G, const cf* Sp, size_t s_stride, int s_planes, int A,
                      const double* center, cf* work, size_t work_stride, const RealDst& dst,
                      const cf* tw_all, hipStream_t s, int gb, size_t g_stride, const VarDst* var) {
  if (gb < 1 || (gb > 1 && A != 1)) {
    set_error("fft inverse: a batch of %d G spectra needs one component (A = %d)", gb, A);
    return -1;
  }
  if (var && gb != 2) {
    set_error("fft inverse: w needs the two local sums, not %d spectra", gb);
    return -1;
  }
  const cf* tw = tw_all + twiddle_offset(N);
  switch (N) {
    case 32: return inverse_n<32>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 64: return inverse_n<64>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 128: return inverse_n<128>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 256: return inverse_n<256>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 512: return inverse_n<512>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 96: return inverse_n<96>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 160: return inverse_n<160>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    case 192: return inverse_n<192>(G, Sp, s_stride, s_planes, A, center, work, work_stride, dst, tw, s, gb, g_stride, var);
    default: set_error("unsupported FFT edge %d", N); return -4;
  }
}

}  // namespace ttm

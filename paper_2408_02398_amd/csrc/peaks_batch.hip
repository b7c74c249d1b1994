// peaks_batch.hip -- exact greedy Find Peaks for many score maps in one
// launch (gfx950), for batches of subtomograms that each want few peaks.
//
// The rule (Sec. 3.4) keeps, again and again, the first voxel in visiting
// order (descending score, ties by ascending linear index z*ny*nx + y*nx + x)
// that lies at least D from every peak kept so far, until P peaks are kept or
// none is left.  With the 64-bit key (~score_bits << 32 | linear index) the
// visiting order is ascending key order, so each step takes the smallest key
// among the voxels not yet excluded; after a peak is kept, the voxels of its
// exclusion ball (distance < D) are excluded.  That is the greedy result
// itself, with no sort of the map:
//   k_block_keys  the smallest key of every 8^3 block of every item's valid
//                 region (one workgroup per block)
//   k_nms         one workgroup per item: P times, the smallest block key is
//                 the next peak (or none is left); the ball's voxels are set
//                 in the item's exclusion bitmask, and the blocks the ball
//                 touches are updated: emptied when they lie inside it,
//                 rescanned without the excluded voxels when their smallest
//                 key's voxel was excluded, and otherwise left as they are.
//   k_nms_lds     the same for items of few peaks whose block keys fit LDS, a
//                 block rescanned only once its key comes up (below).
// Every item's work is independent, so one launch serves the whole batch.
#include "../../include/ttm.h"
#include "internal.hpp"

namespace ttm {

namespace {

constexpr int kBlk = 8;                 // block edge (voxels)
constexpr int kNmsThreads = 1024;
constexpr int kMaxBatchPeaks = 4096;

__device__ __forceinline__ unsigned sbits(float s) { return (s > 0.0f) ? __float_as_uint(s) : 0u; }

struct ItemGeo {
  int vz, vy, vx;       // valid box extent
  int bz, by, bx;       // blocks per axis
  size_t words;         // bitmask words
};

__host__ __device__ inline ItemGeo geo(const int32_t lo[3], const int32_t hi[3]) {
  ItemGeo g;
  g.vz = hi[0] - lo[0] + 1;
  g.vy = hi[1] - lo[1] + 1;
  g.vx = hi[2] - lo[2] + 1;
  g.bz = (g.vz + kBlk - 1) / kBlk;
  g.by = (g.vy + kBlk - 1) / kBlk;
  g.bx = (g.vx + kBlk - 1) / kBlk;
  g.words = ((size_t)g.vz * g.vy * g.vx + 31) / 32;
  return g;
}

__host__ __device__ inline size_t a256b(size_t b) { return (b + 255) & ~(size_t)255; }

// An item the kernels can serve: its valid box inside its map, at least one
// peak wanted, a map of fewer than 2^32 voxels (linear indices fit the key).
__device__ __forceinline__ bool item_ok(const ttm_peak_item& it) {
  for (int a = 0; a < 3; ++a)
    if (it.valid_lo[a] < 0 || it.valid_hi[a] >= it.dims[a] || it.valid_lo[a] > it.valid_hi[a]) return false;
  return it.top_p >= 1 && it.top_p <= kMaxBatchPeaks && it.min_dist >= 0.0f && it.score && it.peaks && it.vals && it.n_found &&
         it.scratch && (unsigned long long)it.dims[0] * it.dims[1] * it.dims[2] < (1ull << 32);
}

// scratch of one item: block keys, then the exclusion bitmask (one bit per
// valid voxel, x fastest)
__host__ __device__ inline void scratch_layout(void* base, const ItemGeo& g,
                                               unsigned long long** keys, unsigned** bits) {
  char* p = static_cast<char*>(base);
  *keys = reinterpret_cast<unsigned long long*>(p);
  *bits = reinterpret_cast<unsigned*>(p + a256b((size_t)g.bz * g.by * g.bx * 8));
}

__device__ __forceinline__ unsigned long long voxel_key(const ttm_peak_item& it, const ItemGeo& g,
                                                        const unsigned* bits, int vz, int vy, int vx) {
  const size_t vi = ((size_t)vz * g.vy + vy) * g.vx + vx;
  if (bits && ((bits[vi >> 5] >> (vi & 31)) & 1u)) return ~0ull;
  const int z = it.valid_lo[0] + vz, y = it.valid_lo[1] + vy, x = it.valid_lo[2] + vx;
  const size_t lin = ((size_t)z * it.dims[1] + y) * it.dims[2] + x;
  return ((unsigned long long)(~sbits(it.score[lin])) << 32) | (unsigned long long)lin;
}

__device__ __forceinline__ unsigned long long wave_min(unsigned long long v) {
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(v, off);
    v = o < v ? o : v;
  }
  return v;
}

// Smallest key of one 8^3 block (512 threads, one voxel each), or ~0 when
// every voxel of the block is excluded or outside the valid box.
__device__ __forceinline__ unsigned long long block_min(const ttm_peak_item& it, const ItemGeo& g,
                                                        const unsigned* bits, int b, int t,
                                                        int nthreads) {
  const int bxx = b % g.bx, byy = (b / g.bx) % g.by, bzz = b / (g.bx * g.by);
  unsigned long long m = ~0ull;
  for (int i = t; i < kBlk * kBlk * kBlk; i += nthreads) {
    const int vx = bxx * kBlk + i % kBlk, vy = byy * kBlk + (i / kBlk) % kBlk,
              vz = bzz * kBlk + i / (kBlk * kBlk);
    if (vx < g.vx && vy < g.vy && vz < g.vz) {
      const unsigned long long k = voxel_key(it, g, bits, vz, vy, vx);
      m = k < m ? k : m;
    }
  }
  return m;
}

__global__ __launch_bounds__(512) void k_block_keys(const ttm_peak_item* __restrict__ items) {
  __shared__ unsigned long long red[8];
  const ttm_peak_item it = items[blockIdx.y];
  if (!item_ok(it)) return;
  const ItemGeo g = geo(it.valid_lo, it.valid_hi);
  const int b = blockIdx.x;
  if (b >= g.bz * g.by * g.bx) return;            // uniform per workgroup
  unsigned long long* keys;
  unsigned* bits;
  scratch_layout(it.scratch, g, &keys, &bits);
  unsigned long long m = block_min(it, g, nullptr, b, threadIdx.x, 512);   // nothing excluded yet
  m = wave_min(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long r = red[0];
    for (int i = 1; i < 8; ++i) r = red[i] < r ? red[i] : r;
    keys[b] = r;
  }
}

// Items of k_nms_lds: at most kLdsPeaks peaks (each check of a voxel looks at all
// kept ones, a lane each) and `cap` blocks, the launch's LDS.
constexpr int kLdsPeaks = 512;
constexpr int kLdsBlocks = 18432;       // 144 KB of keys: 211^3 voxels
__device__ __forceinline__ bool in_lds(const ttm_peak_item& it, const ItemGeo& g, int cap) {
  return it.top_p <= kLdsPeaks && (long long)g.bz * g.by * g.bx <= cap;
}

// A workgroup per item, its block keys in LDS.  A key is a lower bound once
// exclusion has removed its voxel, and a block whose key never comes up is never
// rescanned.  In each step every wavefront takes the smallest key of its own
// blocks and tests that voxel against the kept peaks (no bitmask); when it is
// excluded the wavefront rescans the block.  The smallest of the wavefronts' keys
// is the next peak when its voxel was not excluded.  Then blocks inside the
// peak's ball are emptied.  Each step keeps a peak or raises a key, so it ends.
// One workgroup per item, so a chain of latencies: rescanning every touched block
// at once (some 300 of a ball of radius 28, by 16 wavefronts) and the bitmask's
// atomics took 33 us a peak on 160^3 voxels, this 4.5 us.
__global__ __launch_bounds__(kNmsThreads) void k_nms_lds(const ttm_peak_item* __restrict__ items, int cap) {
  constexpr int W = kNmsThreads / 64;
  extern __shared__ unsigned long long keys[];
  __shared__ ushort4 kept[kLdsPeaks];             // z, y, x in the valid box
  __shared__ unsigned long long red_k[2][W];
  __shared__ int red_out[2][W];
  const ttm_peak_item it = items[blockIdx.x];
  if (!item_ok(it)) return;
  const ItemGeo g = geo(it.valid_lo, it.valid_hi);
  if (!in_lds(it, g, cap)) return;
  unsigned long long* gkeys;
  unsigned* bits;
  scratch_layout(it.scratch, g, &gkeys, &bits);
  const int nb = g.bz * g.by * g.bx;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const unsigned ny = (unsigned)it.dims[1], nx = (unsigned)it.dims[2];
  const float D2 = it.min_dist * it.min_dist;
  const int R = (int)ceilf(it.min_dist);
  // Block b is wavefront b % W's, whose keys lie together: the blocks around a peak are
  // spread over the wavefronts, which rescan them side by side (in runs of 64 blocks, 100
  // peaks of equal scores in 96^3: 1287 us, 684 now).
  const int per = (nb + W - 1) / W;
  auto slot = [&](int b) { return b % W * per + b / W; };
  for (int b = threadIdx.x; b < per * W; b += kNmsThreads) keys[slot(b)] = b < nb ? gkeys[b] : ~0ull;
  __syncthreads();
  int found = 0, par = 0;
  while (found < it.top_p) {
    unsigned long long m = ~0ull;
    for (int i = lane; i < per; i += 64) m = keys[wave * per + i] < m ? keys[wave * per + i] : m;
    m = wave_min(m);
    bool out = false;
    if (m != ~0ull) {                             // uniform in the wavefront
      const unsigned lin = (unsigned)m, r = lin / nx, z = r / ny;
      const int vz = (int)z - it.valid_lo[0], vy = (int)(r - z * ny) - it.valid_lo[1],
                vx = (int)(lin - r * nx) - it.valid_lo[2];
      for (int k = lane; k - lane < found && !out; k += 64) {
        bool hit = false;
        if (k < found) {
          const int dz = vz - kept[k].x, dy = vy - kept[k].y, dx = vx - kept[k].z;
          const int d = dz * dz + dy * dy + dx * dx;
          hit = d == 0 || (float)d < D2;
        }
        out = __ballot(hit) != 0ull;
      }
      if (out) {
        // the block's smallest key among the voxels left: lane = (y, x), 8 z each
        const int qz = vz / kBlk * kBlk, qy = vy / kBlk * kBlk, qx = vx / kBlk * kBlk;
        const int y = qy + (lane >> 3), x = qx + (lane & 7);
        const size_t row = ((size_t)it.valid_lo[0] * ny + it.valid_lo[1] + min(y, g.vy - 1)) * nx +
                           it.valid_lo[2] + min(x, g.vx - 1);
        float sc[kBlk];
#pragma unroll
        for (int t = 0; t < kBlk; ++t) sc[t] = it.score[row + (size_t)min(qz + t, g.vz - 1) * ny * nx];
        unsigned gone = 0;
        for (int k0 = 0; k0 < found; k0 += 64) {
          bool near = false;
          if (k0 + lane < found) {
            const ushort4 q = kept[k0 + lane];
            const int dz = max(max(qz - q.x, q.x - (qz + kBlk - 1)), 0), dy = max(max(qy - q.y, q.y - (qy + kBlk - 1)), 0),
                      dx = max(max(qx - q.z, q.z - (qx + kBlk - 1)), 0);
            const int d = dz * dz + dy * dy + dx * dx;
            near = d == 0 || (float)d < D2;
          }
          for (unsigned long long bal = __ballot(near); bal; bal &= bal - 1) {
            const ushort4 q = kept[k0 + __ffsll((long long)bal) - 1];
            const int dy = y - q.y, dx = x - q.z, dyx = dy * dy + dx * dx;
#pragma unroll
            for (int t = 0; t < kBlk; ++t) {
              const int dz = qz + t - q.x, d = dz * dz + dyx;
              gone |= (d == 0 || (float)d < D2 ? 1u : 0u) << t;
            }
          }
        }
        unsigned long long mm = ~0ull;
#pragma unroll
        for (int t = 0; t < kBlk; ++t) {
          const unsigned long long k = ((unsigned long long)(~sbits(sc[t])) << 32) |
                                       (unsigned long long)(row + (size_t)(qz + t) * ny * nx);
          if (y < g.vy && x < g.vx && qz + t < g.vz && !(gone >> t & 1u) && k < mm) mm = k;
        }
        mm = wave_min(mm);
        if (lane == 0) keys[slot((qz / kBlk * g.by + qy / kBlk) * g.bx + qx / kBlk)] = mm;
      }
    }
    if (lane == 0) {
      red_k[par][wave] = m;
      red_out[par][wave] = out ? 1 : 0;
    }
    __syncthreads();
    unsigned long long best = red_k[par][0];
    int best_out = red_out[par][0];
    for (int i = 1; i < W; ++i)
      if (red_k[par][i] < best) {
        best = red_k[par][i];
        best_out = red_out[par][i];
      }
    par ^= 1;
    if (best == ~0ull) break;                     // nothing left
    if (best_out) continue;                       // a lower bound only: its block has been rescanned
    const unsigned lin = (unsigned)best, r = lin / nx, z = r / ny, y = r - z * ny, x = lin - r * nx;
    const int vz = (int)z - it.valid_lo[0], vy = (int)y - it.valid_lo[1], vx = (int)x - it.valid_lo[2];
    if (threadIdx.x == 0) {
      it.peaks[3 * found] = (int)z;
      it.peaks[3 * found + 1] = (int)y;
      it.peaks[3 * found + 2] = (int)x;
      it.vals[found] = it.score[lin];
      kept[found] = make_ushort4((unsigned short)vz, (unsigned short)vy, (unsigned short)vx, 0);
    }
    ++found;
    // blocks whose farthest voxel lies in the ball
    const int bz0 = max(vz - R, 0) / kBlk, nbz = min(vz + R, g.vz - 1) / kBlk - bz0 + 1;
    const int by0 = max(vy - R, 0) / kBlk, nby = min(vy + R, g.vy - 1) / kBlk - by0 + 1;
    const int bx0 = max(vx - R, 0) / kBlk, nbx = min(vx + R, g.vx - 1) / kBlk - bx0 + 1;
    for (int q = threadIdx.x; q < nbz * nby * nbx; q += kNmsThreads) {
      const int qz = bz0 + q / (nby * nbx), qy = by0 + (q / nbx) % nby, qx = bx0 + q % nbx;
      const int fz = max(vz - qz * kBlk, min(qz * kBlk + kBlk, g.vz) - 1 - vz),
                fy = max(vy - qy * kBlk, min(qy * kBlk + kBlk, g.vy) - 1 - vy),
                fx = max(vx - qx * kBlk, min(qx * kBlk + kBlk, g.vx) - 1 - vx);
      if ((float)(fz * fz + fy * fy + fx * fx) < D2) keys[slot((qz * g.by + qy) * g.bx + qx)] = ~0ull;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *it.n_found = found;
}

__global__ __launch_bounds__(256) void k_clear_bits(const ttm_peak_item* __restrict__ items, int cap) {
  const ttm_peak_item it = items[blockIdx.y];
  if (!item_ok(it)) return;
  const ItemGeo g = geo(it.valid_lo, it.valid_hi);
  if (in_lds(it, g, cap)) return;
  unsigned long long* keys;
  unsigned* bits;
  scratch_layout(it.scratch, g, &keys, &bits);
  for (size_t w = (size_t)blockIdx.x * 256 + threadIdx.x; w < g.words; w += (size_t)gridDim.x * 256)
    bits[w] = 0u;
}

__global__ __launch_bounds__(kNmsThreads) void k_nms(const ttm_peak_item* __restrict__ items, int cap) {
  __shared__ unsigned long long red_k[kNmsThreads / 64];
  __shared__ unsigned long long s_best;
  const ttm_peak_item it = items[blockIdx.x];
  if (!item_ok(it)) {
    if (threadIdx.x == 0 && it.n_found) *it.n_found = -1;
    return;
  }
  const ItemGeo g = geo(it.valid_lo, it.valid_hi);
  if (in_lds(it, g, cap)) return;
  unsigned long long* keys;
  unsigned* bits;
  scratch_layout(it.scratch, g, &keys, &bits);
  const int nb = g.bz * g.by * g.bx;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float D = it.min_dist, D2 = D * D;
  const int R = (int)ceilf(D);
  const int P = it.top_p < kMaxBatchPeaks ? it.top_p : kMaxBatchPeaks;
  int found = 0;
  for (int p = 0; p < P; ++p) {
    // 1. the smallest block key: the next voxel in visiting order not excluded
    unsigned long long m = ~0ull;
    for (int b = threadIdx.x; b < nb; b += kNmsThreads) {
      const unsigned long long k = keys[b];
      m = k < m ? k : m;
    }
    m = wave_min(m);
    if (lane == 0) red_k[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long r = red_k[0];
      for (int i = 1; i < kNmsThreads / 64; ++i) r = red_k[i] < r ? red_k[i] : r;
      s_best = r;
    }
    __syncthreads();
    const unsigned long long best = s_best;
    if (best == ~0ull) break;                    // uniform: nothing left
    const unsigned lin = (unsigned)(best & 0xFFFFFFFFull);
    const int x = (int)(lin % (unsigned)it.dims[2]);
    const int y = (int)((lin / (unsigned)it.dims[2]) % (unsigned)it.dims[1]);
    const int z = (int)(lin / ((unsigned)it.dims[2] * (unsigned)it.dims[1]));
    if (threadIdx.x == 0) {
      it.peaks[3 * p] = z;
      it.peaks[3 * p + 1] = y;
      it.peaks[3 * p + 2] = x;
      it.vals[p] = it.score[lin];
    }
    ++found;
    // 2. exclude the ball: every (z, y) row of it is an x range of the bitmask
    const int vz0 = z - it.valid_lo[0], vy0 = y - it.valid_lo[1], vx0 = x - it.valid_lo[2];
    const int rows = (2 * R + 1) * (2 * R + 1);
    for (int rr = threadIdx.x; rr < rows; rr += kNmsThreads) {
      const int dz = rr / (2 * R + 1) - R, dy = rr % (2 * R + 1) - R;
      const int vz = vz0 + dz, vy = vy0 + dy;
      if (vz < 0 || vz >= g.vz || vy < 0 || vy >= g.vy) continue;
      const float rem = D2 - (float)(dz * dz + dy * dy);
      if (!(rem > 0.0f)) continue;
      // |dx| with dx^2 < rem
      int h = (int)sqrtf(rem);
      while ((float)(h * h) >= rem) --h;
      while ((float)((h + 1) * (h + 1)) < rem) ++h;
      const int xa = max(vx0 - h, 0), xb = min(vx0 + h, g.vx - 1);
      if (xa > xb) continue;
      const size_t base = ((size_t)vz * g.vy + vy) * g.vx;
      size_t i0 = base + xa;
      const size_t i1 = base + xb;
      while (i0 <= i1) {
        const size_t w = i0 >> 5;
        const unsigned s0 = (unsigned)(i0 & 31);
        const size_t wend = (w << 5) + 31;
        const unsigned s1 = (unsigned)((i1 < wend ? i1 : wend) & 31);
        const unsigned mask = (s1 == 31 ? 0xFFFFFFFFu : ((1u << (s1 + 1)) - 1u)) & ~((1u << s0) - 1u);
        atomicOr(&bits[w], mask);
        i0 = (w << 5) + 32;
      }
    }
    if (threadIdx.x == 0) {                      // the peak itself is visited (D = 0 too)
      const size_t vi = ((size_t)vz0 * g.vy + vy0) * g.vx + vx0;
      atomicOr(&bits[vi >> 5], 1u << (vi & 31));
    }
    __threadfence_block();
    __syncthreads();
    // 3. the keys of the blocks the ball touches, without the excluded voxels.
    // Exclusion only removes voxels, so a block whose smallest key belongs to
    // a voxel outside the ball keeps it; a block inside the ball is emptied;
    // only a block whose smallest-key voxel was just excluded is rescanned.
    const int bz0 = max(vz0 - R, 0) / kBlk, bz1 = min(vz0 + R, g.vz - 1) / kBlk;
    const int by0 = max(vy0 - R, 0) / kBlk, by1 = min(vy0 + R, g.vy - 1) / kBlk;
    const int bx0 = max(vx0 - R, 0) / kBlk, bx1 = min(vx0 + R, g.vx - 1) / kBlk;
    const int nbz = bz1 - bz0 + 1, nby = by1 - by0 + 1, nbx = bx1 - bx0 + 1;
    for (int q = wave; q < nbz * nby * nbx; q += kNmsThreads / 64) {
      const int qz = bz0 + q / (nby * nbx), qy = by0 + (q / nbx) % nby, qx = bx0 + q % nbx;
      const int b = (qz * g.by + qy) * g.bx + qx;
      const unsigned long long kb = keys[b];     // the same value in every lane
      if (kb == ~0ull) continue;                 // already empty
      // farthest corner of the block's valid part from the peak
      const int cz0 = qz * kBlk - vz0, cz1 = min(qz * kBlk + kBlk, g.vz) - 1 - vz0;
      const int cy0 = qy * kBlk - vy0, cy1 = min(qy * kBlk + kBlk, g.vy) - 1 - vy0;
      const int cx0 = qx * kBlk - vx0, cx1 = min(qx * kBlk + kBlk, g.vx) - 1 - vx0;
      const int fz = max(cz0 * cz0, cz1 * cz1), fy = max(cy0 * cy0, cy1 * cy1), fx = max(cx0 * cx0, cx1 * cx1);
      if ((float)(fz + fy + fx) < D2) {
        if (lane == 0) keys[b] = ~0ull;          // every voxel of the block is excluded
        continue;
      }
      const unsigned kl = (unsigned)(kb & 0xFFFFFFFFull);
      const int mx = (int)(kl % (unsigned)it.dims[2]) - x;
      const int my = (int)((kl / (unsigned)it.dims[2]) % (unsigned)it.dims[1]) - y;
      const int mz = (int)(kl / ((unsigned)it.dims[2] * (unsigned)it.dims[1])) - z;
      const bool gone = (mx | my | mz) == 0 || (float)(mx * mx + my * my + mz * mz) < D2;
      if (!gone) continue;                       // its smallest key is still there
      unsigned long long mm = block_min(it, g, bits, b, lane, 64);
      mm = wave_min(mm);
      if (lane == 0) keys[b] = mm;
    }
    __threadfence_block();
    __syncthreads();
  }
  if (threadIdx.x == 0) *it.n_found = found;
}

}  // namespace

size_t peaks_batch_scratch(const int32_t lo[3], const int32_t hi[3]) {
  const ItemGeo g = geo(lo, hi);
  return a256b((size_t)g.bz * g.by * g.bx * 8) + a256b(g.words * 4);
}

int peaks_batch_max_peaks() { return kMaxBatchPeaks; }

int find_peaks_batch(const ttm_peak_item* items, int n_items, const int32_t max_valid[3],
                     hipStream_t s) {
  const int32_t zero[3] = {0, 0, 0};
  const int32_t hi[3] = {max_valid[0] - 1, max_valid[1] - 1, max_valid[2] - 1};
  const ItemGeo g = geo(zero, hi);
  const int max_blocks = g.bz * g.by * g.bx;
  const size_t max_words = g.words;
  constexpr int W = kNmsThreads / 64;
  const int cap = ((max_blocks < kLdsBlocks ? max_blocks : kLdsBlocks) + W - 1) / W * W;   // a share per wavefront
  const unsigned cw = (unsigned)((max_words + 255) / 256);
  hipLaunchKernelGGL(k_clear_bits, dim3(cw < 256 ? cw : 256, n_items), dim3(256), 0, s, items, cap);
  hipLaunchKernelGGL(k_block_keys, dim3(max_blocks, n_items), dim3(512), 0, s, items);
  hipLaunchKernelGGL(k_nms_lds, dim3(n_items), dim3(kNmsThreads), (size_t)cap * 8, s, items, cap);
  hipLaunchKernelGGL(k_nms, dim3(n_items), dim3(kNmsThreads), 0, s, items, cap);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_status(e, "find peaks batch launch");
}

}  // namespace ttm

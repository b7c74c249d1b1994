// extract_items.hpp -- where a voxel of an extraction call reads its tensor
// field and writes its answer, for one box or a batch of boxes, and what the pooled
// runs share (axis-form and quaternion-form extraction kernels).
#pragma once

#include "internal.hpp"

namespace ttm {

// Output-map index of voxel v of a single-box call: the box voxel (z, y, x)
// lands at (oz + z, oy + y, ox + x) of a dz x dy x dx map (only dy, dx enter).
__device__ __forceinline__ size_t box_map_index(const ExtractArgs& a, size_t v) {
  const int vx = (int)(v % a.bx), vy = (int)((v / a.bx) % a.by), vz = (int)(v / ((size_t)a.bx * a.by));
  return ((size_t)(a.oz + vz) * a.dy + (a.oy + vy)) * a.dx + (a.ox + vx);
}

// The single box, or in a batched call the item holding v (the last whose
// first voxel is <= v, by binary search over the items' first voxels), with
// v's place inside it.
struct VoxelRef {
  const void* C;
  size_t stride;     // voxels per component plane
  size_t lv;         // v within the planes
  size_t o;          // index in the output maps
  float* score;
  float* lam;
  float* dir;        // d' floats per map voxel
};

__device__ __forceinline__ VoxelRef voxel_ref(const ExtractArgs& a, size_t v) {
  if (!a.items) return VoxelRef{a.C, a.plane, v, box_map_index(a, v), a.score, a.lam, a.dir};
  int lo = 0, hi = a.n_items - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.items[mid].first <= v) lo = mid; else hi = mid - 1;
  }
  const ExtractItem& it = a.items[lo];
  const size_t lv = v - it.first;
  const int by = it.box[1], bx = it.box[2];
  const int vx = (int)(lv % bx), vy = (int)((lv / bx) % by), vz = (int)(lv / ((size_t)bx * by));
  const size_t o = ((size_t)(it.out_lo[0] + vz) * it.out_dims[1] + (it.out_lo[1] + vy)) * it.out_dims[2] +
                   (it.out_lo[2] + vx);
  return VoxelRef{it.C, (size_t)it.box[0] * by * bx, lv, o, it.score, it.lambda, it.dir};
}

// 1 / sqrt(n2) as rsqrtf gives it; its steps for subnormal n2 are taken only by
// a wavefront that holds one.
__device__ __forceinline__ float rsqrt_wave(float n2) {
  if (__ballot(n2 < 0x1p-126f) != 0ull) return rsqrtf(n2);
  return __builtin_amdgcn_rsqf(n2);
}

// Orders a wavefront's LDS accesses (its own reads and writes reach LDS in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Pooled workgroups that are on the chip from the start, whatever their LDS and registers (half
// as many of the quaternion form's at degree 6).
constexpr unsigned kPoolOwners = 1024;

// Pooled workgroups for so many runs of a tensor of K components.  A run of max_iter
// updates is a serial chain, and it advances at its wavefront's share of the SIMD: few
// runs end soonest with one wavefront per SIMD (a workgroup per CU), many with all that
// fit.  A workgroup also costs 0.1 us, in chunks taken from one counter, which short
// runs (tensors near one direction) do not hide.  Score and orientation of e^3 voxels with
// 256 / 512 / 768 / 1024 / 2048 workgroups, 16 starts:
//   degree 4, field of a tomogram: e = 32 (0.5 million runs) 307 / 267 / 301 / 364 / 609 us,
//     48 (1.8) 708 / 446 / 386 / 396 / 551, 64 (4.2) 1409 / 833 / 699 / 624 / 656,
//     80 (8.2) 2590 / 1539 / 1256 / 1139 / 1062, 97 (15) 4440 / 2537 / 2113 / 2003 / 1889
//   degree 4, one direction and 1 % noise: e = 24 (0.2) 91 / 132 / 131 / 215 / 262,
//     64 286 / 236 / 250 / 292 / 532, 96 (14) 878 / 583 / 489 / 482 / 680
//   degree 6: 64 2094 / 1288 / 1105 / 1041 / 1018 and 512 / 393 / 361 / 381 / 598,
//     97 6407 / 3875 / 3392 / 3236 / 3308 and (96) 1536 / 1045 / 910 / 884 / 933
//   quaternions, degree 4, 1 %: 32 174 / 218 / 247 / 316 / 530, 64 514 / 412 / 381 / 423 / 659,
//     96 (14) 1607 / 1183 / 1059 / 1035 / 1131
// 2048 thus wait for work of 350 million components (14 million runs at degree 6).
__host__ __device__ inline unsigned pool_groups(size_t runs, int K) {
  return runs < 350000 ? 256 : runs < 750000 ? 512 : runs < 2000000 ? 768 : runs * K < 350000000 ? 1024 : 2048;
}

}  // namespace ttm

// peaks.hip -- exact greedy Find Peaks on the GPU (gfx950).
//
// The rule (Sec. 3.4): visit voxels by descending score, ties by ascending
// linear index, keep a voxel when every kept peak is at least D away, stop
// at P.  A voxel's fate depends only on higher-ranked voxels, so the first P
// kept peaks are decided by the voxels ranked above the P-th of them, and any
// threshold that leaves P kept peaks above it gives the answer.  The search with
// a host count therefore runs on the top-ranked candidates only:
//   1. a histogram of the score bit patterns (scores are >= 0, so the bit
//      pattern is monotone in the value) over a sample of the map, in two
//      levels, picks a threshold that about `want` voxels pass,
//   2. the voxels that pass are compacted as 64-bit keys (~score_bits << 32 |
//      linear index), so ascending key order is exactly the visiting order,
//   3. of a short list the smallest key is kept and drops those within D, again and
//      again (k_short); the candidates of a longer one settle in parallel
//      (k_settle): one is kept once every higher-ranked candidate within D is
//      dropped, and dropped once one of them is kept -- the sequential walk's answer,
//   4. the kept ones are ranked among each other and the first P written.
// If fewer than P peaks are found while lower-ranked voxels remain, `want` is
// raised and the search repeats.  Lists that step 3 does not settle in a few rounds,
// second searches, and the search whose count stays on the device take a sorted walk
// instead:
//   * LSD radix sort of the keys (8-bit digits, stable ranks from wavefront
//     ballots),
//   * one workgroup walks the sorted keys in chunks of 1024: every lane
//     tests its candidate against the kept peaks through a spatial hash of
//     cell size D; the survivors, compacted in rank order, are settled 64 at
//     a time by one wavefront (pairwise conflict bitmasks, then a 64-step
//     in-order acceptance on those masks).
#include <algorithm>
#include <climits>

#include "internal.hpp"

namespace ttm {

size_t peaks_workspace(int64_t n_voxels);

namespace {

constexpr int kHistBins = 4096;   // per level: bits [31:20], then [19:8]
constexpr int kSortIPT = 16;           // keys per thread per sort block
constexpr int kSortBlock = 256;        // threads per sort block
constexpr int kSortTile = kSortIPT * kSortBlock;

__device__ __forceinline__ unsigned score_bits(float s) {
  // scores are norms (>= 0); clamp anything else to 0 so the order is monotone
  return (s > 0.0f) ? __float_as_uint(s) : 0u;
}

struct Region {
  int nz, ny, nx;
  int z0, y0, x0, z1, y1, x1;  // inclusive valid box
};

// Histogram of one 12-bit field of the score bit patterns over the region,
// privatised in LDS per workgroup.  level 0: bits [31:20] of every voxel;
// level 1: bits [19:8] of the voxels whose bits [31:20] equal `top`.
// Each workgroup covers kHistRows rows (y) of one z slice, in groups of 8, so
// clearing and flushing its 16 KB of bins is spread over enough voxels.
// Of the (slice, row block) pairs one in `sample` is read.
constexpr int kHistRows = 32;

// What the threshold search leaves on the device.
struct Pick {
  unsigned top;       // coarse bin
  unsigned most;      // the highest coarse bin that is not empty
  unsigned above;     // sampled voxels in the bins over it
  unsigned key_lo;    // candidates: score bits >= key_lo
  unsigned count;     // candidates
  unsigned undecided, kept;
  int n_found;
  unsigned open;              // candidates that k_drop left undecided
  unsigned long long work;    // candidates in the 27 cells around each of those, added up
};

__global__ __launch_bounds__(256) void k_hist(const float* __restrict__ score, Region r, int level,
                                              const Pick* __restrict__ pick, int sample,
                                              unsigned* __restrict__ hist) {
  __shared__ unsigned h[kHistBins];
  if ((blockIdx.y + 5 * blockIdx.z) % sample) return;   // another row block in each slice
  const unsigned top = level ? pick->top : 0u;
  for (int i = threadIdx.x; i < kHistBins; i += 256) h[i] = 0;
  __syncthreads();
  const int z = r.z0 + blockIdx.z;
  const int nxv = r.x1 - r.x0 + 1;
  // scores crowd into few bins: a thread counts a run of equal bins in a
  // register and adds it at once, instead of one contended LDS atomic each.
  // A thread takes one column x of 8 rows at a time, its 8 loads in flight
  // together.
  unsigned cur = 0xFFFFFFFFu, run = 0;
  for (int y8 = r.y0 + (int)blockIdx.y * kHistRows;
       y8 < min(r.y0 + ((int)blockIdx.y + 1) * kHistRows, r.y1 + 1); y8 += 8) {
    const int nyv = min(8, r.y1 - y8 + 1);
    const float* col0 = score + ((size_t)z * r.ny + y8) * r.nx + r.x0;
    for (int x = blockIdx.x * 256 + threadIdx.x; x < nxv; x += 256 * gridDim.x) {
      float v[8];
#pragma unroll
      for (int yy = 0; yy < 8; ++yy) v[yy] = yy < nyv ? col0[(size_t)yy * r.nx + x] : 0.0f;
#pragma unroll
      for (int yy = 0; yy < 8; ++yy) {
        if (yy >= nyv) break;
        const unsigned b = score_bits(v[yy]);
        unsigned bin = 0xFFFFFFFFu;
        if (level == 0) {
          bin = b >> 20;
        } else if ((b >> 20) == top) {
          bin = (b >> 8) & 0xFFFu;
        }
        if (bin == 0xFFFFFFFFu) continue;
        if (bin != cur) {
          if (run) atomicAdd(&h[cur], run);
          cur = bin;
          run = 0;
        }
        ++run;
      }
    }
  }
  if (run) atomicAdd(&h[cur], run);
  __syncthreads();
  for (int i = threadIdx.x; i < kHistBins; i += 256)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// One workgroup: the bin in which the histogram, summed from the top, reaches
// `want` sampled voxels.  Level 0 leaves the coarse bin, the sum over it and the highest bin in use, level 1
// the threshold (key_lo stays 0, every voxel, when all bins together stay below
// `want`).
__global__ __launch_bounds__(1024) void k_pick(const unsigned* __restrict__ hist, int level, unsigned want, Pick* pick) {
  __shared__ unsigned sum[1024];
  const int t = threadIdx.x;
  unsigned v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = hist[kHistBins - 1 - (4 * t + i)];   // from the top down
  const unsigned own = (v[0] + v[1]) + (v[2] + v[3]);
  sum[t] = own;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const unsigned o = t >= off ? sum[t - off] : 0u;
    __syncthreads();
    sum[t] += o;
    __syncthreads();
  }
  const unsigned base = level ? pick->above : 0u, top = level ? pick->top : 0u;
  const bool none = level && top == 0xFFFFFFFFu;
  __syncthreads();
  unsigned run = base + sum[t] - own;
  if (t == 0 && level == 0 && sum[1023] < want) pick->top = 0xFFFFFFFFu;   // key_lo stays 0
  if (none || run >= want) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (level == 0 && run == 0 && v[i]) pick->most = kHistBins - 1 - (4 * t + i);
    if (run < want && run + v[i] >= want) {
      const unsigned bin = kHistBins - 1 - (4 * t + i);
      if (level == 0) {
        pick->top = bin;
        pick->above = run;
      } else {
        pick->key_lo = top << 20 | bin << 8;
      }
    }
    run += v[i];
  }
}

// Keys of the voxels whose score bits are >= key_lo, in any order.  A workgroup
// takes kCompactRows rows of one z slice in pieces of 256 columns, a wavefront four
// pieces at a time, its 16 loads in flight.  The keys gather in LDS (those past
// kCompactList go out by themselves), so a workgroup reserves its slots with one
// atomic: the counter is one address for the whole chip, and an atomic for each 64
// voxels with a key in them bound this at 465 us for 131 000 keys of
// 512 x 928 x 928 (now 280 us, the map read once).
constexpr int kCompactRows = 16, kCompactList = 1024;
__global__ __launch_bounds__(256) void k_compact(const float* __restrict__ score, Region r,
                                                 const unsigned* __restrict__ key_lo_at,
                                                 unsigned long long* __restrict__ keys,
                                                 unsigned* __restrict__ counter) {
  __shared__ unsigned long long list[kCompactList];
  __shared__ unsigned n_list, slot;
  constexpr int PB = 4;   // pieces whose loads are in flight together
  const unsigned key_lo = key_lo_at ? *key_lo_at : 0u;
  const int z = r.z0 + blockIdx.z, y0 = r.y0 + blockIdx.y * kCompactRows;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const int nch = (r.x1 - r.x0 + 256) / 256;
  const int items = min(kCompactRows, r.y1 - y0 + 1) * nch;
  if (threadIdx.x == 0) n_list = 0;
  __syncthreads();
  for (int it = wave; it < items; it += 4 * PB) {
    float v[PB][4];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int c = min(it + 4 * i, items - 1), yy = c / nch;
      const size_t row = ((size_t)z * r.ny + y0 + yy) * r.nx;
      const int xb = r.x0 + (c - yy * nch) * 256 + lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[i][k] = score[row + min(xb + 64 * k, r.x1)];
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int c = it + 4 * i, yy = c / nch;
      if (c >= items) break;  // uniform
      const size_t row = ((size_t)z * r.ny + y0 + yy) * r.nx;
      const int xb = r.x0 + (c - yy * nch) * 256 + lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int x = xb + 64 * k;
        const unsigned bits = score_bits(v[i][k]);
        const bool take = x <= r.x1 && bits >= key_lo;
        const unsigned long long bal = __ballot(take);
        if (bal == 0ull) continue;  // uniform across the wavefront
        const unsigned long long key = ((unsigned long long)(~bits) << 32) |
                                       (unsigned long long)(row + x);
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(&n_list, (unsigned)__popcll(bal));
        at = (unsigned)__shfl((int)at, 0) + __popcll(bal & lt);
        if (take && at < kCompactList) list[at] = key;
        const unsigned long long over = __ballot(take && at >= kCompactList);
        if (over == 0ull) continue;
        unsigned base = 0;
        if (lane == 0) base = atomicAdd(counter, (unsigned)__popcll(over));
        base = (unsigned)__shfl((int)base, 0);
        if (take && at >= kCompactList) keys[base + __popcll(over & lt)] = key;
      }
    }
  }
  __syncthreads();
  const unsigned n = min(n_list, (unsigned)kCompactList);
  if (n == 0) return;  // uniform
  if (threadIdx.x == 0) slot = atomicAdd(counter, n);
  __syncthreads();
  for (unsigned i = threadIdx.x; i < n; i += 256) keys[slot + i] = list[i];
}

__global__ void k_fill(unsigned long long* __restrict__ keys, size_t from, size_t to) {
  const size_t i = from + (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < to) keys[i] = ~0ull;
}

// ---------------------------------------------------------------- radix sort
__global__ __launch_bounds__(kSortBlock) void k_rs_hist(const unsigned long long* __restrict__ keys,
                                                        int shift, unsigned* __restrict__ hist,
                                                        int nblocks) {
  __shared__ unsigned h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const size_t base = (size_t)blockIdx.x * kSortTile;
  for (int i = 0; i < kSortIPT; ++i) {
    const unsigned d = (unsigned)(keys[base + i * kSortBlock + threadIdx.x] >> shift) & 255u;
    atomicAdd(&h[d], 1u);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// exclusive scan of n values by one workgroup of 1024 threads
__global__ __launch_bounds__(1024) void k_scan(unsigned* __restrict__ a, int n) {
  __shared__ unsigned part[1024];
  const int t = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int lo = min(n, t * per), hi = min(n, lo + per);
  // each thread's segment in batches of 8 loads in flight
  unsigned s = 0;
  int i = lo;
  for (; i + 8 <= hi; i += 8) {
    unsigned v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = a[i + k];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  for (; i < hi; ++i) s += a[i];
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    unsigned v = (t >= off) ? part[t - off] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  unsigned run = (t == 0) ? 0u : part[t - 1];
  for (i = lo; i + 8 <= hi; i += 8) {
    unsigned v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = a[i + k];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      a[i + k] = run;
      run += v[k];
    }
  }
  for (; i < hi; ++i) {
    const unsigned v = a[i];
    a[i] = run;
    run += v;
  }
}

__global__ __launch_bounds__(kSortBlock) void k_rs_scatter(
    const unsigned long long* __restrict__ in, unsigned long long* __restrict__ out, int shift,
    const unsigned* __restrict__ offs, int nblocks) {
  constexpr int NW = kSortBlock / 64;
  __shared__ unsigned run[256];
  __shared__ unsigned wcnt[NW][256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  run[tid] = offs[(size_t)tid * nblocks + blockIdx.x];
  const size_t base = (size_t)blockIdx.x * kSortTile;
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int i = 0; i < kSortIPT; ++i) {
#pragma unroll
    for (int w = 0; w < NW; ++w) wcnt[w][tid] = 0;
    __syncthreads();
    const unsigned long long key = in[base + i * kSortBlock + tid];
    const unsigned d = (unsigned)(key >> shift) & 255u;
    unsigned long long same = ~0ull;
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const unsigned long long bal = __ballot((d >> bit) & 1u);
      same &= ((d >> bit) & 1u) ? bal : ~bal;
    }
    const unsigned rank = __popcll(same & lt);
    if (rank == 0) wcnt[wv][d] = __popcll(same);
    __syncthreads();
    unsigned before = 0;
    for (int w = 0; w < wv; ++w) before += wcnt[w][d];
    out[run[d] + before + rank] = key;
    __syncthreads();
    unsigned tot = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += wcnt[w][tid];
    run[tid] += tot;
    __syncthreads();
  }
}

// ---------------------------------------------------------------- settling
// Candidates in the order of the exclusion grid's cells (edge >= D): those within
// D of one lie in the 27 cells around its own, which are nine runs of the list.
constexpr unsigned kSettleMax = 1u << 20;   // candidates
constexpr unsigned kKeptMax = 16384;        // kept ones
constexpr int kSettleRounds = 6;            // between two looks at what is left (random maps take about 8)
constexpr int kSettleLooks = 32;            // then the sorted walk
constexpr unsigned kSettlePer = 16;         // candidates of a wavefront in a round, few of them open

// Whether the rounds (k_settle) pay, with `open` of m candidates left by k_drop: else
// the sorted walk takes over.  They settle in a few rounds what lies on the slopes
// of peaks or is noise (open / m up to 0.35), and one peak a round along a ramp, a
// ridge or a plateau (0.72 to 1.0); and a round reads every candidate in reach of an
// open one, where the walk reads only kept peaks.  The whole search with rounds against
// with the walk: noise 256^3, 2000 peaks 0.98 / 3.1 ms; ridges 200 x 200 x 400, 2000
// peaks 13.8 / 2.7; equal scores 64^3, 2000 peaks 46 / 2.9; maxima of sigma 9 in 192^3, 30
// peaks 2.9 / 0.78, in 256^3, 30 peaks 2.1 / 0.83.
constexpr unsigned kSettleNear = 2048;      // neighbours of an open candidate, on average
constexpr unsigned long long kSettleWork = 1ull << 27;
__host__ __device__ inline bool rounds_pay(const Pick& p, unsigned m) {
  return 2ull * p.open <= m && p.work <= kSettleWork && p.work <= (unsigned long long)kSettleNear * p.open;
}

struct Settle {
  const unsigned long long* in;   // keys as compacted
  unsigned long long* key;        // in cell order
  ushort4* pos;                   // z, y, x
  int* state;                     // 0 undecided, 1 kept, 2 dropped
  unsigned* start;                // first candidate of each cell, ncell + 1
  unsigned* fill;                 // candidates placed per cell
  unsigned long long* best;       // ~(smallest key) of each cell, 0: none
  ushort4* lead;                  // its place and w = 1 where it is kept at once
  unsigned m;
  int ny, nx;
  float d2, cell;
  int gz, gy, gx;
  Pick* pick;
  unsigned long long* kept;       // kKeptMax keys
};

__device__ __forceinline__ ushort4 key_pos(unsigned long long key, int ny, int nx) {
  const unsigned lin = (unsigned)(key & 0xffffffffull), yx = (unsigned)ny * (unsigned)nx;
  const unsigned z = lin / yx, rz = lin - z * yx, y = rz / (unsigned)nx;
  return make_ushort4((unsigned short)z, (unsigned short)y, (unsigned short)(rz - y * (unsigned)nx), 0);
}
__device__ __forceinline__ int cell_of(const Settle& s, const ushort4& p) {
  return ((int)(p.x / s.cell) * s.gy + (int)(p.y / s.cell)) * s.gx + (int)(p.z / s.cell);
}

// Candidates per cell (cleared before), then, with the cells' starts known, the
// candidates in cell order (in any order within a cell).  The list comes in pieces of
// rows, so neighbouring lanes mostly share a cell: a run of them adds with one atomic
// (with one a lane, those of a wavefront queue for one address: 0.4 to 0.8 ms for
// 260 000 to 880 000 candidates of 64^3 and 96^3 maps).
template <bool SCATTER>
__global__ __launch_bounds__(256) void k_cells(Settle s) {
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const unsigned long long key = i < s.m ? s.in[i] : ~0ull;
  const ushort4 p = key_pos(key, s.ny, s.nx);
  const int c = i < s.m ? cell_of(s, p) : -1;
  const int before = __shfl_up(c, 1);
  const bool head = lane == 0 || before != c;
  const unsigned long long heads = __ballot(head);
  const int first = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
  const unsigned long long rest = lane == 63 ? 0ull : heads >> (lane + 1);
  const int next = rest ? lane + __ffsll((long long)rest) : 64;   // this run: lanes first .. next - 1
  if constexpr (!SCATTER) {
    if (head && c >= 0) atomicAdd(&s.start[c], (unsigned)(next - first));
  } else {
    unsigned long long low = key;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned long long o = __shfl_down(low, off);
      if (lane + off < next && o < low) low = o;
    }
    unsigned base = 0;
    if (head && c >= 0) {
      base = s.start[c] + atomicAdd(&s.fill[c], (unsigned)(next - first));
      atomicMax(&s.best[c], ~low);
    }
    const unsigned at = (unsigned)__shfl((int)base, first) + (unsigned)(lane - first);
    if (i >= s.m) return;
    s.key[at] = key;
    s.pos[at] = p;
    s.state[at] = 0;
  }
}

// The cells' best candidates with nothing ranked higher within D: they are kept.
// A wavefront per cell; cells around it whose best ranks lower hold nothing to look
// at, and one with more than kLeadScan candidates to look at is left to the rounds.
constexpr unsigned kLeadScan = 4096;
__global__ __launch_bounds__(256) void k_lead(Settle s) {
  const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (c >= s.gz * s.gy * s.gx) return;             // uniform per wavefront
  const int x = c % s.gx, y = (c / s.gx) % s.gy, z = c / (s.gx * s.gy);
  const unsigned long long own = ~s.best[c];
  ushort4 p = key_pos(own, s.ny, s.nx);
  // lane: one of the 27 cells
  const int z2 = z + lane / 9 - 1, y2 = y + lane / 3 % 3 - 1, x2 = x + lane % 3 - 1;
  unsigned b = 0, n = 0;
  if (lane < 27 && z2 >= 0 && z2 < s.gz && y2 >= 0 && y2 < s.gy && x2 >= 0 && x2 < s.gx) {
    const int c2 = (z2 * s.gy + y2) * s.gx + x2;
    if (~s.best[c2] < own) {
      b = s.start[c2];
      n = s.start[c2 + 1] - b;
    }
  }
  unsigned all = n;
  for (int off = 32; off > 0; off >>= 1) all += (unsigned)__shfl_xor((int)all, off);
  bool lead = own != ~0ull && all <= kLeadScan;
  for (unsigned long long todo = __ballot(n > 0); todo && lead; todo &= todo - 1) {
    const int o = __ffsll((long long)todo) - 1;
    const unsigned b2 = (unsigned)__shfl((int)b, o), e2 = b2 + (unsigned)__shfl((int)n, o);
    for (unsigned j0 = b2; j0 < e2 && lead; j0 += 64) {
      const unsigned j = j0 + lane;
      bool above = false;
      if (j < e2 && s.key[j] < own) {
        const ushort4 q = s.pos[j];
        const float ddz = (float)((int)p.x - (int)q.x), ddy = (float)((int)p.y - (int)q.y),
                    ddx = (float)((int)p.z - (int)q.z);
        above = ddz * ddz + ddy * ddy + ddx * ddx < s.d2;
      }
      lead = __ballot(above) == 0ull;
    }
  }
  p.w = lead ? 1 : 0;
  if (lane == 0) s.lead[c] = p;
}

// A thread per candidate: kept when it leads its cell, dropped within D of a leader.
// Most candidates of a map of peaks are on the slopes of a leader, and this spares
// them the rounds below.  Those it leaves are counted, and the candidates around them.
__global__ __launch_bounds__(256) void k_drop(Settle s) {
  __shared__ unsigned n_open;
  __shared__ unsigned long long n_work;
  if (threadIdx.x == 0) {
    n_open = 0;
    n_work = 0;
  }
  __syncthreads();
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  unsigned work = 0;
  int state = 2;
  if (i < s.m) {
    const ushort4 p = s.pos[i];
    const int hz = (int)(p.x / s.cell), hy = (int)(p.y / s.cell), hx = (int)(p.z / s.cell);
    state = 0;
#pragma unroll
    for (int o = 0; o < 27; ++o) {
      const int z2 = min(max(hz + o / 9 - 1, 0), s.gz - 1), y2 = min(max(hy + o / 3 % 3 - 1, 0), s.gy - 1),
                x2 = min(max(hx + o % 3 - 1, 0), s.gx - 1);
      const ushort4 q = s.lead[(z2 * s.gy + y2) * s.gx + x2];
      const float ddz = (float)((int)p.x - (int)q.x), ddy = (float)((int)p.y - (int)q.y),
                  ddx = (float)((int)p.z - (int)q.z);
      const float d2 = ddz * ddz + ddy * ddy + ddx * ddx;
      if (q.w) state = d2 == 0.0f ? 1 : (d2 < s.d2 ? 2 : state);
    }
    s.state[i] = state;
    if (state == 0) {
      for (int o = 0; o < 9; ++o) {
        const int z2 = hz + o / 3 - 1, y2 = hy + o % 3 - 1;
        if (z2 < 0 || z2 >= s.gz || y2 < 0 || y2 >= s.gy) continue;
        const int row = (z2 * s.gy + y2) * s.gx;
        work += s.start[row + min(hx + 1, s.gx - 1) + 1] - s.start[row + max(hx - 1, 0)];
      }
    }
  }
  const unsigned long long open = __ballot(state == 0);
  if (open) {                                       // uniform per wavefront
    unsigned long long w = work;
    for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off);
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&n_open, (unsigned)__popcll(open));
      atomicAdd(&n_work, w);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && n_open) {
    atomicAdd(&s.pick->open, n_open);
    atomicAdd(&s.pick->work, n_work);
  }
}

// One round, a wavefront for kSettlePer candidates: among the higher-ranked candidates within D, a kept one drops it, else an undecided one makes it wait
// for a later round, else it is kept.  States only ever leave 0, so one read too
// early costs a round and nothing else.  A walk in rank order by one workgroup
// spent 2.4 ms on 131 000 candidates of 2000 peaks, these rounds alone 0.34 ms,
// and after k_drop they take 16 us (all of Find Peaks on 512 x 928 x 928: 3.78 -> 0.56 ms).
__device__ __forceinline__ void settle_one(const Settle& s, unsigned i, unsigned lane) {
  const unsigned long long key = s.key[i];
  const ushort4 p = s.pos[i];
  const int hz = (int)(p.x / s.cell), hy = (int)(p.y / s.cell), hx = (int)(p.z / s.cell);
  bool wait = false;
  for (int o = 0; o < 9; ++o) {
    const int z2 = hz + o / 3 - 1, y2 = hy + o % 3 - 1;
    if (z2 < 0 || z2 >= s.gz || y2 < 0 || y2 >= s.gy) continue;
    const int row = (z2 * s.gy + y2) * s.gx;
    const unsigned b = s.start[row + max(hx - 1, 0)], e = s.start[row + min(hx + 1, s.gx - 1) + 1];
    for (unsigned j0 = b; j0 < e; j0 += 64 * 4) {   // four loads of a lane in flight
      unsigned long long kj[4];
      ushort4 q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned j = min(j0 + 64 * k + lane, e - 1);
        kj[k] = s.key[j];
        q[k] = s.pos[j];
      }
      bool kept = false, undecided = false;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned j = j0 + 64 * k + lane;
        const float ddz = (float)((int)p.x - (int)q[k].x), ddy = (float)((int)p.y - (int)q[k].y),
                    ddx = (float)((int)p.z - (int)q[k].z);
        if (j < e && kj[k] < key && ddz * ddz + ddy * ddy + ddx * ddx < s.d2) {
          const int st = __hip_atomic_load(&s.state[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          kept = kept || st == 1;
          undecided = undecided || st == 0;
        }
      }
      if (__ballot(kept)) {
        if (lane == 0) __hip_atomic_store(&s.state[i], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
      }
      wait = wait || __ballot(undecided) != 0ull;
    }
  }
  if (!wait && lane == 0) __hip_atomic_store(&s.state[i], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_settle(Settle s) {
  const unsigned i0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * kSettlePer;
  const unsigned lane = threadIdx.x & 63;
  if (i0 >= s.m || !rounds_pay(*s.pick, s.m)) return;   // uniform per wavefront
  const bool open = lane < kSettlePer && i0 + lane < s.m && s.state[i0 + lane] == 0;
  for (unsigned long long todo = __ballot(open); todo; todo &= todo - 1)
    settle_one(s, i0 + (unsigned)__ffsll((long long)todo) - 1, lane);
}

// Undecided candidates counted, kept ones gathered (the counters cleared before);
// more than kKeptMax kept ones stand for a list that is not settled here.
__global__ __launch_bounds__(256) void k_gather(Settle s) {
  __shared__ unsigned n_wait, n_keep, base;
  if (threadIdx.x == 0) n_wait = n_keep = 0;
  __syncthreads();
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  const int st = i < s.m ? s.state[i] : 2, lane = threadIdx.x & 63;
  const unsigned long long wait = __ballot(st == 0), keep = __ballot(st == 1);
  unsigned at = 0;
  if (lane == 0 && wait) atomicAdd(&n_wait, (unsigned)__popcll(wait));
  if (lane == 0 && keep) at = atomicAdd(&n_keep, (unsigned)__popcll(keep));
  at = (unsigned)__shfl((int)at, 0) + __popcll(keep & ((1ull << lane) - 1ull));
  __syncthreads();
  if (threadIdx.x == 0) {
    if (n_wait) atomicAdd(&s.pick->undecided, n_wait);
    if (n_keep) base = atomicAdd(&s.pick->kept, n_keep);
  }
  __syncthreads();
  if (st == 1 && base + at < kKeptMax) s.kept[base + at] = s.key[i];
}

// The candidates that are not dropped, in any order: all that the sorted walk needs,
// as a dropped one lies within D of a kept one that ranks higher.
__global__ __launch_bounds__(256) void k_left(Settle s, unsigned long long* __restrict__ keys,
                                              unsigned* __restrict__ counter) {
  __shared__ unsigned n, base;
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool take = i < s.m && s.state[i] != 2;
  const unsigned long long bal = __ballot(take);
  unsigned at = 0;
  if (lane == 0 && bal) at = atomicAdd(&n, (unsigned)__popcll(bal));
  at = (unsigned)__shfl((int)at, 0) + __popcll(bal & ((1ull << lane) - 1ull));
  __syncthreads();
  if (threadIdx.x == 0 && n) base = atomicAdd(counter, n);
  __syncthreads();
  if (take) keys[base + at] = s.key[i];
}

// Rank of each kept key among the kept, and its place in the output.
__global__ __launch_bounds__(256) void k_rank(const unsigned long long* __restrict__ kept, Pick* pick, int ny, int nx,
                                              int top_p, int* __restrict__ peaks, float* __restrict__ vals) {
  __shared__ unsigned long long tile[1024];
  __shared__ int part[4][64];
  const unsigned n = pick->kept;
  if (n > kKeptMax || blockIdx.x * 64 >= n) return;   // uniform
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned i = blockIdx.x * 64 + lane;
  const unsigned long long key = i < n ? kept[i] : ~0ull;
  int rank = 0;
  for (unsigned t0 = 0; t0 < n; t0 += 1024) {
    __syncthreads();
    for (unsigned k = threadIdx.x; k < 1024; k += 256) tile[k] = t0 + k < n ? kept[t0 + k] : ~0ull;
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < 256; ++k) rank += tile[wave * 256 + k] < key ? 1 : 0;
  }
  part[wave][lane] = rank;
  __syncthreads();
  if (wave) return;
  rank += part[1][lane] + part[2][lane] + part[3][lane];
  if (i == 0) pick->n_found = (int)min(n, (unsigned)top_p);
  if (i < n && rank < top_p) {
    const ushort4 p = key_pos(key, ny, nx);
    peaks[3 * rank + 0] = p.x;
    peaks[3 * rank + 1] = p.y;
    peaks[3 * rank + 2] = p.z;
    vals[rank] = __uint_as_float(~(unsigned)(key >> 32));
  }
}

// ---------------------------------------------------------------- short list
// The rule itself on a list of up to kShortList keys in any order, for a few peaks: one
// workgroup, its keys in registers; the smallest is the next peak, and those within D
// of it are gone.  n_found = -1: a longer list.  Bound by vector issue of one CU, 3 us
// a step, one step a peak whatever the map looks like; the settling is 0.1 ms at the
// least.
constexpr int kShortThreads = 1024;
constexpr int kShortEach = 8;
constexpr unsigned kShortList = kShortThreads * kShortEach;
constexpr int kShortPeaks = 16;
constexpr int64_t kShortWant = 5120;   // (a quarter more where sampled)

__global__ __launch_bounds__(kShortThreads) void k_short(const unsigned long long* __restrict__ keys,
                                                         const unsigned* __restrict__ count, int* __restrict__ n_found,
                                                         int ny, int nx, float d2, int top_p, int* __restrict__ peaks,
                                                         float* __restrict__ vals) {
  constexpr int W = kShortThreads / 64;
  __shared__ unsigned long long red[2][W];
  const unsigned m = *count;
  const int tid = threadIdx.x, wave = tid >> 6;
  if (m > kShortList) {                              // uniform
    if (tid == 0) *n_found = -1;
    return;
  }
  unsigned long long key[kShortEach];
  ushort4 pos[kShortEach];
#pragma unroll
  for (int i = 0; i < kShortEach; ++i) {
    const unsigned j = (unsigned)i * kShortThreads + tid;
    key[i] = j < m ? keys[j] : ~0ull;
    pos[i] = key_pos(key[i], ny, nx);
  }
  int found = 0;
  for (; found < top_p; ++found) {
    unsigned long long best = key[0];
#pragma unroll
    for (int i = 1; i < kShortEach; ++i) best = key[i] < best ? key[i] : best;
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long o = __shfl_xor(best, off);
      best = o < best ? o : best;
    }
    unsigned long long* r = red[found & 1];
    if ((tid & 63) == 0) r[wave] = best;
    __syncthreads();
    best = r[0];
#pragma unroll
    for (int i = 1; i < W; ++i) best = r[i] < best ? r[i] : best;
    if (best == ~0ull) break;                        // uniform
    const ushort4 p = key_pos(best, ny, nx);
    if (tid == 0) {
      peaks[3 * found + 0] = p.x;
      peaks[3 * found + 1] = p.y;
      peaks[3 * found + 2] = p.z;
      vals[found] = __uint_as_float(~(unsigned)(best >> 32));
    }
#pragma unroll
    for (int i = 0; i < kShortEach; ++i) {
      const float ddz = (float)((int)p.x - (int)pos[i].x), ddy = (float)((int)p.y - (int)pos[i].y),
                  ddx = (float)((int)p.z - (int)pos[i].z);
      if (key[i] == best || ddz * ddz + ddy * ddy + ddx * ddx < d2) key[i] = ~0ull;
    }
  }
  if (tid == 0) *n_found = found;
}

// ---------------------------------------------------------------- greedy walk
constexpr int kGreedyThreads = 1024;
constexpr int kMaxPeaks = 2048;
constexpr int kMaxCells = 16384;

// The kept peaks' spatial hash as the greedy leaves it in global memory for
// the filter and for the next walk: head[kMaxCells], then next, pz, py, px
// (kMaxPeaks each), all 16-bit.
constexpr int kHashShorts = kMaxCells + 4 * kMaxPeaks;

struct GreedyArgs {
  const unsigned long long* keys;
  int m;                  // number of candidate keys (sorted ascending)
  const int* m_dev;       // if set, the number of keys is read here instead
  int limit;              // walk at most this many keys (a multiple of the chunk)
  int resume;             // 1: continue from the peaks (and hash) already kept
  int nz, ny, nx;
  float d2;               // squared exclusion distance
  float cell;             // hash cell edge (>= exclusion distance)
  int gz, gy, gx;         // hash grid extent
  int top_p;
  int* peaks;             // top_p x 3
  float* vals;
  int* n_found;           // device
  short* hash;            // kHashShorts, device
};

// Candidates per thread and chunk.  More than one lets a thread issue its
// hash lookups together and a chunk's barriers serve more keys, but then more
// keys reach the serial settle before the hash learns of the peaks kept in
// their chunk; with many peaks (thousands at 2r apart) one per thread is
// faster.
constexpr int kGreedyPer = 1;
constexpr int kGreedyChunk = kGreedyThreads * kGreedyPer;

__global__ __launch_bounds__(kGreedyThreads) void k_greedy(GreedyArgs g) {
  constexpr int NW = kGreedyThreads / 64;
  __shared__ short head[kMaxCells];
  __shared__ short next[kMaxPeaks];
  __shared__ short pz[kMaxPeaks], py[kMaxPeaks], px[kMaxPeaks];
  __shared__ short sz[kGreedyChunk], sy[kGreedyChunk], sx[kGreedyChunk];
  __shared__ int srank[kGreedyChunk];   // rank within the chunk of each survivor
  __shared__ int wsum[kGreedyPer * NW];
  __shared__ int nkept, stop, mlen;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int ncell = g.gz * g.gy * g.gx;
  short* gnext = g.hash + kMaxCells;
  short* gpz = gnext + kMaxPeaks;
  short* gpy = gpz + kMaxPeaks;
  short* gpx = gpy + kMaxPeaks;
  if (tid == 0) {
    nkept = g.resume ? *g.n_found : 0;
    stop = nkept >= g.top_p ? 1 : 0;
    mlen = g.m_dev ? *g.m_dev : g.m;
  }
  __syncthreads();
  if (stop) return;  // uniform: the peaks are complete
  if (g.resume) {
    for (int i = tid; i < ncell; i += kGreedyThreads) head[i] = g.hash[i];
    for (int k = tid; k < nkept; k += kGreedyThreads) {
      next[k] = gnext[k];
      pz[k] = gpz[k];
      py[k] = gpy[k];
      px[k] = gpx[k];
    }
  } else {
    for (int i = tid; i < ncell; i += kGreedyThreads) head[i] = (short)-1;
  }
  __syncthreads();
  const int mm = min(mlen, g.limit);
  // linear indices fit the key's low 32 bits and ny * nx < 2^30 (edges are
  // below 2^15), so the decode divides in 32 bits
  const unsigned yx = (unsigned)g.ny * (unsigned)g.nx, nxu = (unsigned)g.nx;
  const unsigned long long lt = (1ull << lane) - 1ull;
  // candidate k of a thread in a chunk has rank k * kGreedyThreads + tid; its
  // key is loaded one chunk ahead
  unsigned long long key_next[kGreedyPer];
#pragma unroll
  for (int k = 0; k < kGreedyPer; ++k) {
    const int i = k * kGreedyThreads + tid;
    key_next[k] = i < mm ? g.keys[i] : 0ull;
  }
  for (int base = 0; base < mm; base += kGreedyChunk) {
    int cz[kGreedyPer], cy[kGreedyPer], cxx[kGreedyPer], hz[kGreedyPer], hy[kGreedyPer],
        hx[kGreedyPer];
    bool alive[kGreedyPer];
#pragma unroll
    for (int k = 0; k < kGreedyPer; ++k) {
      const int idx = base + k * kGreedyThreads + tid;
      alive[k] = idx < mm;
      const unsigned lin = (unsigned)(key_next[k] & 0xffffffffull);
      const unsigned qz = lin / yx, rz = lin - qz * yx, qy = rz / nxu;
      cz[k] = alive[k] ? (int)qz : 0;
      cy[k] = alive[k] ? (int)qy : 0;
      cxx[k] = alive[k] ? (int)(rz - qy * nxu) : 0;
      hz[k] = (int)(cz[k] / g.cell);
      hy[k] = (int)(cy[k] / g.cell);
      hx[k] = (int)(cxx[k] / g.cell);
      if (idx + kGreedyChunk < mm) key_next[k] = g.keys[idx + kGreedyChunk];
    }
    // a candidate dies when a peak kept in an earlier chunk lies within D;
    // such a peak sits in one of the 27 hash cells around the candidate's
    for (int c = 0; c < 27; ++c) {
      bool any = false;
#pragma unroll
      for (int k = 0; k < kGreedyPer; ++k) any = any || alive[k];
      if (!any) break;
      const int dz = c / 9 - 1, dy = (c / 3) % 3 - 1, dx = c % 3 - 1;
      int p[kGreedyPer];
#pragma unroll
      for (int k = 0; k < kGreedyPer; ++k) {
        const int z2 = hz[k] + dz, y2 = hy[k] + dy, x2 = hx[k] + dx;
        const bool in = alive[k] && z2 >= 0 && z2 < g.gz && y2 >= 0 && y2 < g.gy && x2 >= 0 &&
                        x2 < g.gx;
        p[k] = in ? head[(z2 * g.gy + y2) * g.gx + x2] : -1;
      }
#pragma unroll
      for (int k = 0; k < kGreedyPer; ++k) {
        for (int q = p[k]; q >= 0; q = next[q]) {
          const float ddz = (float)(cz[k] - pz[q]), ddy = (float)(cy[k] - py[q]),
                      ddx = (float)(cxx[k] - px[q]);
          if (ddz * ddz + ddy * ddy + ddx * ddx < g.d2) {
            alive[k] = false;
            break;
          }
        }
      }
    }
    // survivors in rank order (k, then thread): wavefront ballots, then the
    // offsets of the sub-chunks and waves ahead
    unsigned long long bal[kGreedyPer];
#pragma unroll
    for (int k = 0; k < kGreedyPer; ++k) {
      bal[k] = __ballot(alive[k]);
      if (lane == 0) wsum[k * NW + wv] = __popcll(bal[k]);
    }
    __syncthreads();
    int ns = 0;
#pragma unroll
    for (int k = 0; k < kGreedyPer; ++k) {
      int before = 0, tot = 0;
      for (int w = 0; w < NW; ++w) {
        const int v = wsum[k * NW + w];
        before += w < wv ? v : 0;
        tot += v;
      }
      if (alive[k]) {
        const int pos = ns + before + __popcll(bal[k] & lt);
        sz[pos] = (short)cz[k];
        sy[pos] = (short)cy[k];
        sx[pos] = (short)cxx[k];
        srank[pos] = k * kGreedyThreads + tid;
      }
      ns += tot;
    }
    __syncthreads();
    // settle the survivors in order, 64 at a time on wavefront 0: a survivor
    // is kept when no peak kept earlier in this chunk and no kept survivor
    // ahead of it in its group lies within D
    if (wv == 0) {
      const int first_new = nkept;
      for (int g0 = 0; g0 < ns; g0 += 64) {
        if (nkept >= g.top_p) break;
        const int i = g0 + lane;
        bool cand = i < ns;
        int z = 0, y = 0, x = 0;
        if (cand) {
          z = sz[i];
          y = sy[i];
          x = sx[i];
          for (int p = first_new; p < nkept && cand; ++p) {
            const float ddz = (float)(z - pz[p]), ddy = (float)(y - py[p]), ddx = (float)(x - px[p]);
            if (ddz * ddz + ddy * ddy + ddx * ddx < g.d2) cand = false;
          }
        }
        // conflicts with the group's survivors ahead of this one, whose
        // coordinates are read from the lanes that hold them (gn and j are
        // the same on every lane, so these are plain lane reads)
        const int gn = min(64, ns - g0);
        unsigned long long conf = 0;
        for (int j = 0; j < gn; ++j) {
          const int zj = __builtin_amdgcn_readlane(z, j), yj = __builtin_amdgcn_readlane(y, j),
                    xj = __builtin_amdgcn_readlane(x, j);
          const float ddz = (float)(z - zj), ddy = (float)(y - yj), ddx = (float)(x - xj);
          if (j < lane && ddz * ddz + ddy * ddy + ddx * ddx < g.d2) conf |= 1ull << j;
        }
        const unsigned long long cands = __ballot(cand);
        const unsigned conf_lo = (unsigned)conf, conf_hi = (unsigned)(conf >> 32);
        unsigned long long kept = 0;
        int room = g.top_p - nkept;
        for (int l = 0; l < gn && room > 0; ++l) {
          const unsigned long long cl =
              ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)conf_hi, l) << 32) |
              (unsigned)__builtin_amdgcn_readlane((int)conf_lo, l);
          if (((cands >> l) & 1ull) && !(cl & kept)) {
            kept |= 1ull << l;
            --room;
          }
        }
        if ((kept >> lane) & 1ull) {
          const int k = nkept + __popcll(kept & ((1ull << lane) - 1ull));
          pz[k] = (short)z;
          py[k] = (short)y;
          px[k] = (short)x;
          const unsigned long long key = g.keys[base + srank[i]];
          g.peaks[3 * k + 0] = z;
          g.peaks[3 * k + 1] = y;
          g.peaks[3 * k + 2] = x;
          g.vals[k] = __uint_as_float(~(unsigned)(key >> 32));
        }
        wave_lds_sync();
        if (lane == 0) {
          // hash insertion in rank order
          const int nk = __popcll(kept);
          for (int t = 0; t < nk; ++t) {
            const int k = nkept + t;
            const int cell =
                ((int)(pz[k] / g.cell) * g.gy + (int)(py[k] / g.cell)) * g.gx + (int)(px[k] / g.cell);
            next[k] = head[cell];
            head[cell] = (short)k;
          }
          nkept += nk;
          if (nkept >= g.top_p) stop = 1;
        }
        wave_lds_sync();
      }
    }
    __syncthreads();
    if (stop) break;
  }
  // the hash and the count for the filter and the next walk
  const int nk = nkept;
  for (int i = tid; i < ncell; i += kGreedyThreads) g.hash[i] = head[i];
  for (int k = tid; k < nk; k += kGreedyThreads) {
    gnext[k] = next[k];
    gpz[k] = pz[k];
    gpy[k] = py[k];
    gpx[k] = px[k];
  }
  if (tid == 0) *g.n_found = nk;
}

// ---------------------------------------------------------------- filter
// Between two walks the rest of the sorted list is filtered on the whole
// GPU: a key dies when a peak kept so far lies within D (it could never be
// kept later, and only kept peaks decide anything), and the survivors are
// written in their order.  k_filter<false> counts the survivors of each
// block of kSortTile keys, k_scan turns the counts into offsets (the extra
// last entry becomes the total), k_filter<true> writes the survivors and the
// new list length.
struct FilterArgs {
  const unsigned long long* keys;
  int from;               // first key to filter (the walk took the keys before)
  int m;                  // list length, or
  const int* m_dev;       // read here when set
  int ny, nx;
  float d2, cell;
  int gz, gy, gx;
  int top_p;
  const int* n_found;
  const short* hash;      // as the greedy leaves it
  unsigned* counts;       // nb + 1 entries
  int nb;
  unsigned long long* out;
  int* m_next;
};

template <bool SCATTER>
__global__ __launch_bounds__(kSortBlock) void k_filter(FilterArgs f) {
  constexpr int NW = kSortBlock / 64;
  __shared__ short head[kMaxCells];
  __shared__ short next[kMaxPeaks], pz[kMaxPeaks], py[kMaxPeaks], px[kMaxPeaks];
  __shared__ unsigned wcnt[kSortIPT][NW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int np = *f.n_found;
  const int m = f.m_dev ? *f.m_dev : f.m;
  const bool done = np >= f.top_p;
  const int base = f.from + (int)blockIdx.x * kSortTile;
  if (blockIdx.x == 0 && tid == 0) {
    if (SCATTER) {
      *f.m_next = done ? 0 : (int)f.counts[f.nb];
    } else {
      f.counts[f.nb] = 0u;
    }
  }
  if (done || base >= m) {  // uniform per workgroup
    if (!SCATTER && tid == 0) f.counts[blockIdx.x] = 0u;
    return;
  }
  const int ncell = f.gz * f.gy * f.gx;
  for (int i = tid; i < ncell; i += kSortBlock) head[i] = f.hash[i];
  for (int k = tid; k < np; k += kSortBlock) {
    next[k] = f.hash[kMaxCells + k];
    pz[k] = f.hash[kMaxCells + kMaxPeaks + k];
    py[k] = f.hash[kMaxCells + 2 * kMaxPeaks + k];
    px[k] = f.hash[kMaxCells + 3 * kMaxPeaks + k];
  }
  __syncthreads();
  const unsigned yx = (unsigned)f.ny * (unsigned)f.nx, nxu = (unsigned)f.nx;
  unsigned long long key[kSortIPT];
  bool alive[kSortIPT];
#pragma unroll
  for (int j = 0; j < kSortIPT; ++j) {
    const int i = base + j * kSortBlock + tid;
    alive[j] = i < m;
    key[j] = alive[j] ? f.keys[i] : 0ull;
  }
  for (int j = 0; j < kSortIPT; ++j) {
    if (!alive[j]) continue;
    const unsigned lin = (unsigned)(key[j] & 0xffffffffull);
    const unsigned qz = lin / yx, rz = lin - qz * yx, qy = rz / nxu;
    const int cz = (int)qz, cy = (int)qy, cxx = (int)(rz - qy * nxu);
    const int hz = (int)(cz / f.cell), hy = (int)(cy / f.cell), hx = (int)(cxx / f.cell);
    bool al = true;
    for (int c = 0; c < 27 && al; ++c) {
      const int z2 = hz + c / 9 - 1, y2 = hy + (c / 3) % 3 - 1, x2 = hx + c % 3 - 1;
      if (z2 < 0 || z2 >= f.gz || y2 < 0 || y2 >= f.gy || x2 < 0 || x2 >= f.gx) continue;
      for (int q = head[(z2 * f.gy + y2) * f.gx + x2]; q >= 0; q = next[q]) {
        const float ddz = (float)(cz - pz[q]), ddy = (float)(cy - py[q]), ddx = (float)(cxx - px[q]);
        if (ddz * ddz + ddy * ddy + ddx * ddx < f.d2) {
          al = false;
          break;
        }
      }
    }
    alive[j] = al;
  }
  // survivors of each slice j, per wavefront; ranks follow (j, thread)
  unsigned long long bal[kSortIPT];
#pragma unroll
  for (int j = 0; j < kSortIPT; ++j) {
    bal[j] = __ballot(alive[j]);
    if (lane == 0) wcnt[j][wv] = __popcll(bal[j]);
  }
  __syncthreads();
  if (!SCATTER) {
    if (tid == 0) {
      unsigned t = 0;
      for (int j = 0; j < kSortIPT; ++j)
        for (int w = 0; w < NW; ++w) t += wcnt[j][w];
      f.counts[blockIdx.x] = t;
    }
    return;
  }
  unsigned run = f.counts[blockIdx.x];
  const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < kSortIPT; ++j) {
    unsigned before = 0, tot = 0;
    for (int w = 0; w < NW; ++w) {
      const unsigned v = wcnt[j][w];
      before += w < wv ? v : 0u;
      tot += v;
    }
    if (alive[j]) f.out[run + before + __popcll(bal[j] & lt)] = key[j];
    run += tot;
  }
}

// Index bytes of the keys (their low 32 bits) that are zero for every linear
// index of the map need no radix pass: the pass would keep the order.  The
// padding keys (all ones) still sort after every real key, because the real
// keys' index bytes that are sorted already stay below theirs or, at equality,
// stable passes keep the real keys (placed first) ahead.
bool index_byte_constant(int shift, const Region& r) {
  const unsigned long long total = (unsigned long long)r.nz * r.ny * r.nx;
  return shift < 32 && total <= (1ull << shift);
}

constexpr int kWalkRounds = 3;                // short walks, each followed by a filter
constexpr int kWalkKeys = 8 * kGreedyChunk;    // keys per short walk

// Bytes of the workspace before its tail (keys, histograms, counters,
// sort counts), and the tail: the kept peaks' hash and the list lengths.
size_t peaks_head_bytes(int64_t n_voxels) {
  const size_t cand = (size_t)n_voxels + kSortTile;
  const size_t nblk = (cand + kSortTile - 1) / kSortTile;
  const size_t b = 2 * cand * 8 + kHistBins * 4 + 256 * nblk * 4 + 256 + 1024;
  return (b + 255) / 256 * 256;
}
constexpr size_t kPeaksTailBytes = (kHashShorts * 2 + 256 + 255) / 256 * 256;

// The settling's arrays behind the tail: positions and states of at most
// kSettleMax candidates, the kept keys, the cells' best keys, leaders, starts and fills.
size_t settle_bytes(int64_t n_voxels) {
  const size_t m = ((size_t)std::min<int64_t>(n_voxels, kSettleMax) + 1) / 2 * 2;
  return m * 12 + (size_t)kMaxCells * 16 + (2 * kMaxCells + 64) * 4 + (size_t)kKeptMax * 8 + 1024;
}

// The greedy walk over m sorted keys in `srt` (`spare` holds as many):
// `rounds` times a walk over the first kWalkKeys keys of the list and the
// filter of the rest into the other buffer, then a walk over what is left.
// The result equals one walk over all m keys: a filtered key was within D of
// a peak kept before it, and the survivors keep their order.  The rounds pay
// when most keys die (every voxel a candidate, few peaks); over the top
// candidates alone one walk is as fast.
void greedy_walks(unsigned long long* srt, unsigned long long* spare, size_t m, const Region& r,
                  float min_dist, float cell, int gz, int gy, int gx, int top_p, int32_t* peaks,
                  float* vals, int32_t* n_found, unsigned* counts, char* tail, int rounds,
                  hipStream_t s) {
  short* hash = reinterpret_cast<short*>(tail);
  int* mdev = reinterpret_cast<int*>(tail + kHashShorts * 2);
  const int nb = m > (size_t)kWalkKeys ? (int)((m - kWalkKeys + kSortTile - 1) / kSortTile) : 0;
  unsigned long long* cur = srt;
  unsigned long long* other = spare;
  const int* mcur = nullptr;
  const float d2 = min_dist * min_dist;
  for (int round = 0;; ++round) {
    const bool last = round == rounds || nb == 0;
    GreedyArgs ga{cur, (int)m, mcur, last ? INT_MAX : kWalkKeys, round > 0 ? 1 : 0, r.nz, r.ny,
                  r.nx, d2, cell, gz, gy, gx, top_p, peaks, vals, n_found, hash};
    hipLaunchKernelGGL(k_greedy, dim3(1), dim3(kGreedyThreads), 0, s, ga);
    if (last) break;
    FilterArgs fa{cur, kWalkKeys, (int)m, mcur, r.ny, r.nx, d2, cell, gz, gy, gx, top_p, n_found,
                  hash, counts, nb, other, mdev + round};
    hipLaunchKernelGGL(k_filter<false>, dim3(nb), dim3(kSortBlock), 0, s, fa);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, counts, nb + 1);
    hipLaunchKernelGGL(k_filter<true>, dim3(nb), dim3(kSortBlock), 0, s, fa);
    mcur = mdev + round;
    std::swap(cur, other);
  }
}

}  // namespace

// Exact Find Peaks with every valid voxel as a candidate and no host
// synchronisation (the count stays on the device), for graph capture.
int find_peaks_async(const float* score, int nz, int ny, int nx, const int32_t lo[3],
                     const int32_t hi[3], int top_p, float min_dist, int32_t* peaks_out,
                     float* vals_out, int32_t* n_found_dev, void* ws, size_t ws_bytes,
                     hipStream_t s) {
  Region r{nz, ny, nx, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]};
  const int64_t nvalid = (int64_t)(hi[0] - lo[0] + 1) * (hi[1] - lo[1] + 1) * (hi[2] - lo[2] + 1);
  const size_t need = peaks_workspace(nvalid);
  if (ws_bytes < need) {
    set_error("ttm_find_peaks_async: workspace %zu < %zu bytes", ws_bytes, need);
    return -5;
  }
  const float cell = fmaxf(min_dist, 1.0f);
  const int gz = (int)(nz / cell) + 1, gy = (int)(ny / cell) + 1, gx = (int)(nx / cell) + 1;
  if ((int64_t)gz * gy * gx > kMaxCells || top_p > kMaxPeaks || nz > 32767 || ny > 32767 ||
      nx > 32767) {
    set_error("ttm_find_peaks_async: exclusion grid %dx%dx%d or top_p %d too large", gz, gy, gx,
              top_p);
    return -4;
  }
  char* w = static_cast<char*>(ws);
  const size_t cand_cap = (size_t)nvalid + kSortTile;
  unsigned long long* keys_a = reinterpret_cast<unsigned long long*>(w);
  unsigned long long* keys_b = keys_a + cand_cap;
  unsigned* hist = reinterpret_cast<unsigned*>(keys_b + cand_cap);
  unsigned* counter = hist + kHistBins;
  unsigned* shist = reinterpret_cast<unsigned*>(counter + 128);
  const dim3 cgrid(1, (hi[1] - lo[1] + kCompactRows) / kCompactRows,
                   hi[0] - lo[0] + 1);
  const size_t m = (size_t)nvalid;
  const size_t mpad = (m + kSortTile - 1) / kSortTile * kSortTile;
  const int nblk = (int)(mpad / kSortTile);
  fill_zero(counter, 4, s);
  hipLaunchKernelGGL(k_compact, cgrid, dim3(256), 0, s, score, r, nullptr, keys_a, counter);
  if (mpad > m) {
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((mpad - m + 255) / 256)), dim3(256), 0, s, keys_a, m,
                       mpad);
  }
  unsigned long long* src = keys_a;
  unsigned long long* dst = keys_b;
  for (int shift = 0; shift < 64; shift += 8) {
    if (index_byte_constant(shift, r)) continue;
    hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(kSortBlock), 0, s, src, shift, shist, nblk);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, shist, 256 * nblk);
    hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(kSortBlock), 0, s, src, dst, shift, shist,
                       nblk);
    std::swap(src, dst);
  }
  greedy_walks(src, dst, m, r, min_dist, cell, gz, gy, gx, top_p, peaks_out, vals_out,
               n_found_dev, shist, w + peaks_head_bytes(nvalid), kWalkRounds, s);
  TTM_HIP(hipGetLastError());
  return 0;
}

size_t peaks_workspace(int64_t n_voxels) {
  return peaks_head_bytes(n_voxels) + kPeaksTailBytes + settle_bytes(n_voxels);
}

int find_peaks(const float* score, int nz, int ny, int nx, const int32_t lo[3],
               const int32_t hi[3], int top_p, float min_dist, int32_t* peaks_out,
               float* vals_out, int32_t* n_found_host, void* ws, size_t ws_bytes,
               hipStream_t s) {
  Region r{nz, ny, nx, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]};
  const int64_t nvalid = (int64_t)(hi[0] - lo[0] + 1) * (hi[1] - lo[1] + 1) * (hi[2] - lo[2] + 1);
  const size_t need = peaks_workspace(nvalid);
  if (ws_bytes < need) {
    set_error("ttm_find_peaks: workspace %zu < %zu bytes", ws_bytes, need);
    return -5;
  }
  const float cell = fmaxf(min_dist, 1.0f);
  const int gz = (int)(nz / cell) + 1, gy = (int)(ny / cell) + 1, gx = (int)(nx / cell) + 1;
  if ((int64_t)gz * gy * gx > kMaxCells || top_p > kMaxPeaks || nz > 32767 || ny > 32767 ||
      nx > 32767) {
    set_error("ttm_find_peaks: exclusion grid %dx%dx%d or top_p %d too large", gz, gy, gx, top_p);
    return -4;
  }
  char* w = static_cast<char*>(ws);
  const size_t cand_cap = (size_t)nvalid + kSortTile;
  unsigned long long* keys_a = reinterpret_cast<unsigned long long*>(w);
  unsigned long long* keys_b = keys_a + cand_cap;
  unsigned* hist = reinterpret_cast<unsigned*>(keys_b + cand_cap);
  unsigned* counter = hist + kHistBins;
  int* nfound_dev = reinterpret_cast<int*>(counter + 64);
  unsigned* shist = reinterpret_cast<unsigned*>(nfound_dev + 64);

  const dim3 cgrid(1, (hi[1] - lo[1] + kCompactRows) / kCompactRows,
                   hi[0] - lo[0] + 1);
  const dim3 hgrid(1, (hi[1] - lo[1] + kHistRows) / kHistRows, hi[0] - lo[0] + 1);
  char* tail = w + peaks_head_bytes(nvalid) + kPeaksTailBytes;
  const size_t sm = ((size_t)std::min<int64_t>(nvalid, kSettleMax) + 1) / 2 * 2;
  Settle st;
  st.in = keys_a;
  st.key = keys_b;
  st.pos = reinterpret_cast<ushort4*>(tail);
  st.state = reinterpret_cast<int*>(tail + sm * 8);
  st.kept = reinterpret_cast<unsigned long long*>(tail + sm * 12);
  st.lead = reinterpret_cast<ushort4*>(st.kept + kKeptMax);
  const int ncell = gz * gy * gx;
  st.best = reinterpret_cast<unsigned long long*>(st.lead + kMaxCells);
  st.start = reinterpret_cast<unsigned*>(st.best + ncell);   // best, start and fill are cleared as one
  st.fill = st.start + ncell + 1;
  Pick* pick = reinterpret_cast<Pick*>(st.best + 2 * kMaxCells + 32);
  st.pick = pick;
  st.ny = ny;
  st.nx = nx;
  st.cell = cell;
  st.d2 = min_dist * min_dist;
  st.gz = gz;
  st.gy = gy;
  st.gx = gx;

  // The first threshold comes from a sample of at least 4 million voxels (every 16th
  // (slice, row block) pair of a large map): it only sets how many candidates
  // there are, not the answer.  A quarter more are asked of a sample, whose count
  // is off by a few percent: too few candidates cost the whole search once more.
  // 64 candidates a peak hold maps of noise or of small maxima; broad maxima, ramps and
  // plateaus need a second search, of 65 536 at least, then of four times the last.
  // The sorted walk takes lists of that length that do not settle; without a try those
  // of more than twice what was asked for (equal scores: chains of candidates that
  // wait for each other) and those after a list whose leaders left many open.
  const bool few = top_p <= kShortPeaks;
  const int64_t first = few ? kShortWant : std::max<int64_t>(64 * (int64_t)top_p, 4096);
  const int64_t second = std::max<int64_t>(64 * (int64_t)top_p, 1 << 16);
  Pick got;
  int counted = 0;      // the sample in `hist`
  bool slopes = true;   // the leaders are expected to drop most candidates
  for (int64_t want = first;; want = want < second ? second : want * 4) {
    const int sample = want == first ? (int)std::min<int64_t>(16, std::max<int64_t>(1, nvalid >> 22)) : 1;
    fill_zero(pick, sizeof(Pick), s);
    if (want < nvalid) {
      const unsigned want_s = (unsigned)std::max<int64_t>(1, sample > 1 ? want * 5 / 4 / sample : want);
      for (int level = 0; level < 2; ++level) {
        // the second level's bins lie where the kept keys go later: the first
        // level's, once they count every voxel, serve all searches
        unsigned* bins = level ? reinterpret_cast<unsigned*>(st.kept) : hist;
        if (level || counted != 1) {
          fill_zero(bins, kHistBins * 4, s);
          hipLaunchKernelGGL(k_hist, hgrid, dim3(256), 0, s, score, r, level, pick, sample, bins);
        }
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(1024), 0, s, bins, level, want_s, pick);
      }
      counted = sample;
    }
    hipLaunchKernelGGL(k_compact, cgrid, dim3(256), 0, s, score, r, &pick->key_lo, keys_a, &pick->count);
    if (few && want == first)
      hipLaunchKernelGGL(k_short, dim3(1), dim3(kShortThreads), 0, s, keys_a, &pick->count, &pick->n_found, ny, nx,
                         st.d2, top_p, peaks_out, vals_out);
    TTM_HIP(hipGetLastError());   // a launch that failed leaves counts that mean nothing
    TTM_HIP(hipMemcpyAsync(&got, pick, sizeof(Pick), hipMemcpyDeviceToHost, s));
    TTM_HIP(hipStreamSynchronize(s));
    int64_t m = got.count;
    const bool all = m >= nvalid || got.key_lo == 0;
    if (few && want == first && got.n_found >= 0) {
      if (got.n_found >= top_p || all) {
        *n_found_host = got.n_found;
        return 0;
      }
      slopes = false;
      continue;
    }
    if (slopes && m <= (int64_t)kSettleMax && m <= 2 * want) {
      st.m = (unsigned)m;
      const dim3 mg((unsigned)((m + 255) / 256));
      fill_zero(st.best, (size_t)ncell * 8 + (2 * (size_t)ncell + 1) * 4, s);
      hipLaunchKernelGGL(k_cells<false>, mg, dim3(256), 0, s, st);
      hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, st.start, ncell + 1);
      hipLaunchKernelGGL(k_cells<true>, mg, dim3(256), 0, s, st);
      hipLaunchKernelGGL(k_lead, dim3((ncell + 3) / 4), dim3(256), 0, s, st);
      hipLaunchKernelGGL(k_drop, mg, dim3(256), 0, s, st);
      unsigned before = 0;
      for (int look = 0; look < kSettleLooks; ++look) {
        fill_zero(&pick->undecided, 8, s);
        for (int k = 0; k < kSettleRounds; ++k)
          hipLaunchKernelGGL(k_settle, dim3((unsigned)((m + 4 * kSettlePer - 1) / (4 * kSettlePer))), dim3(256), 0, s, st);
        hipLaunchKernelGGL(k_gather, mg, dim3(256), 0, s, st);
        hipLaunchKernelGGL(k_rank, dim3(kKeptMax / 64), dim3(256), 0, s, st.kept, pick, ny, nx, top_p,
                           peaks_out, vals_out);
        TTM_HIP(hipGetLastError());
        TTM_HIP(hipMemcpyAsync(&got, pick, sizeof(Pick), hipMemcpyDeviceToHost, s));
        TTM_HIP(hipStreamSynchronize(s));
        if (look == 0) before = got.open;
        slopes = 4ull * got.open <= st.m;
        // a look that leaves more than half of the last one's: chains, one peak a round
        if (!got.undecided || 2ull * got.undecided > before || !rounds_pay(got, st.m)) break;
        before = got.undecided;
      }
      if (!got.undecided && got.kept <= kKeptMax) {
        if (got.n_found >= top_p || all) {
          *n_found_host = got.n_found;
          return 0;
        }
        continue;
      }
      if (want < second) continue;   // a short list is not worth a sort
      if (2 * ((int64_t)got.undecided + got.kept) < m) {
        fill_zero(counter, 4, s);
        hipLaunchKernelGGL(k_left, mg, dim3(256), 0, s, st, keys_a, counter);
        m = (int64_t)got.undecided + got.kept;
      }
    }
    const size_t mpad = ((size_t)m + kSortTile - 1) / kSortTile * kSortTile;
    const int nblk = (int)(mpad / kSortTile);
    if (mpad > (size_t)m) {
      hipLaunchKernelGGL(k_fill, dim3((unsigned)((mpad - m + 255) / 256)), dim3(256), 0, s, keys_a,
                         (size_t)m, mpad);
    }
    unsigned long long* src = keys_a;
    unsigned long long* dst = keys_b;
    // the scores' highest byte, where every candidate has the same
    const bool one_top = sample == 1 && want < nvalid && got.most >> 4 == got.key_lo >> 24;
    for (int shift = 0; shift < (one_top ? 56 : 64); shift += 8) {
      if (index_byte_constant(shift, r)) continue;
      hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(kSortBlock), 0, s, src, shift, shist, nblk);
      hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, shist, 256 * nblk);
      hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(kSortBlock), 0, s, src, dst, shift, shist,
                         nblk);
      std::swap(src, dst);
    }
    greedy_walks(src, dst, (size_t)m, r, min_dist, cell, gz, gy, gx, top_p, peaks_out, vals_out,
                 nfound_dev, shist, w + peaks_head_bytes(nvalid), 0, s);
    TTM_HIP(hipGetLastError());
    int nf = 0;
    TTM_HIP(hipMemcpyAsync(&nf, nfound_dev, 4, hipMemcpyDeviceToHost, s));
    TTM_HIP(hipStreamSynchronize(s));
    if (nf >= top_p || all) {
      *n_found_host = nf;
      return 0;
    }
  }
}

}  // namespace ttm

// near2d.h -- what the FP32 and FP64 near fields of the 2D log kernel share: the
// workgroup order, the leaf tile with its halo, and the walk over the leaves
// around a wave's targets.
#pragma once

#include <algorithm>

#include "device_common.h"

namespace sffmm {

// Workgroup order of the near-field kernels: chunks of kXcdChunk consecutive
// workgroups (consecutive sorted targets or tiles) go to one XCD, the chunks dealt over
// the 8 XCDs in the order the hardware deals workgroups, so that the waves that
// share a neighbourhood mostly read its sources through one XCD's L2.  The
// grid is a multiple of 8 kXcdChunk workgroups (chunked_grid) and the map is a
// permutation of it.
constexpr int kXcdChunk = 8;
__device__ __forceinline__ int64_t xcd_chunk_remap(int64_t bid) {
  const int64_t x = bid & 7, i = bid >> 3;
  return ((i / kXcdChunk) * 8 + x) * kXcdChunk + (i % kXcdChunk);
}
inline dim3 chunked_grid(int64_t blocks) {
  const int64_t per = 8 * kXcdChunk;
  return dim3((unsigned)((blocks + per - 1) / per * per));
}

constexpr int kP2pHalo = 6;  // 4 x 4-leaf tile + one leaf on each side
constexpr int kP2pHaloLeaves = kP2pHalo * kP2pHalo;

// LDS records staged per tile: 1.5 x the mean halo occupancy, in [512, most].
inline int p2p2d_tile_cap(const LevelTable& lt, int64_t n, int most) {
  const double leaves = (double)((int64_t)lt.nsys << (2 * lt.L));
  const double want = 1.5 * kP2pHaloLeaves * (double)n / leaves;
  const int cap = ((int)std::min(want, (double)most) + 127) / 128 * 128;
  return std::max(512, std::min(most, cap));
}

// Halo of tile `tile` (every thread of the workgroup calls it): first sorted
// position of each of its kP2pHaloLeaves leaves in hstart (rows of the halo
// one after the other; leaves outside the grid are empty) and the exclusive
// scan of their sizes in hoff[0..kP2pHaloLeaves].
__device__ __forceinline__ void tile_halo(const LevelTable& lt, const int32_t* leaf_start,
                                          uint32_t tile, int32_t* hstart, int32_t* hoff) {
  const int L = lt.L, nl = 1 << L, tid = threadIdx.x;
  const uint32_t k0 = tile << 4;  // first leaf key of the tile (system bits included)
  const uint32_t sysbits = k0 & ~local2(0xFFFFFFFFu, L);
  const uint32_t tm = local2(k0, L);
  const int bx0 = (int)compact2(tm), by0 = (int)compact2(tm >> 1);
  int cnt = 0;
  if (tid < kP2pHaloLeaves) {
    const int x = bx0 - 1 + tid % kP2pHalo, y = by0 - 1 + tid / kP2pHalo;
    int32_t s0 = 0;
    if (x >= 0 && x < nl && y >= 0 && y < nl) {
      const uint32_t k = sysbits | spread2((uint32_t)x) | (spread2((uint32_t)y) << 1);
      s0 = leaf_start[k];
      cnt = leaf_start[k + 1] - s0;
    }
    hstart[tid] = s0;
  }
  if (tid < 64) {  // offsets of the halo leaves: an inclusive scan across wave 0
    int v = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int u = __shfl_up(v, d, 64);
      if (tid >= d) v += u;
    }
    if (tid < kP2pHaloLeaves) hoff[tid + 1] = v;
    if (tid == 0) hoff[0] = 0;
  }
  __syncthreads();
}

// Calls f(e, i, column) for every source of the halo: its place in the stage, its
// sorted position and its leaf's halo column.  16 lanes take a leaf (a search
// for each source's leaf took three times the instructions).
template <class F>
__device__ __forceinline__ void stage_halo(const int32_t* hstart, const int32_t* hoff, int threads,
                                           F&& f) {
  const int u = threadIdx.x & 15;
  for (int h = threadIdx.x >> 4; h < kP2pHaloLeaves; h += threads >> 4) {
    const int e0 = hoff[h], m = hoff[h + 1] - e0, i0 = hstart[h], col = h % kP2pHalo;
    for (int c = u; c < m; c += 16) f(e0 + c, i0 + c, col);
  }
}

// Calls f(i0, i1, dx, dy) for every in-domain leaf next to this lane's leaf
// `key` (its sorted range, and the lane's leaf minus that leaf in columns and
// rows), rows in ascending order and columns within them.  lsh: leaf keys and
// offsets are those of a level lsh / 2 above the sorted keys' (adaptive depth).
//
// The wave's distinct leaves (its targets are consecutive in sorted order, so
// dense leaves give one or two): when there are at most four, of one system,
// whose neighbourhoods fit in a 4 x 4-leaf box, and the sources of that box
// are at most 1.2 x those of the largest single neighbourhood (a wave in one
// leaf always), the wave walks the box with uniform leaf ranges and sources
// (scalar loads), each lane taking the leaves next to its own; its leaves
// come in the order of its own 3 x 3 walk, so the sums are the same as with
// the per-lane walk, which reads sources with vector loads.
template <class F>
__device__ __forceinline__ void walk_near2d(const LevelTable& lt, uint32_t key,
                                            const int32_t* __restrict__ leaf_start, int lsh,
                                            F&& f) {
  const int nl = 1 << lt.L;
  const uint32_t lmask = local2(0xFFFFFFFFu, lt.L);
  const int lx = (int)compact2(key & lmask), ly = (int)compact2((key & lmask) >> 1);
  uint64_t todo = __ballot(true);
  int nd = 0, bx0 = 0, bx1 = -1, by0 = 0, by1 = -1;
  int dx0 = 0, dy0 = 0, dx1 = 0, dy1 = 0, dx2 = 0, dy2 = 0, dx3 = 0, dy3 = 0;
  uint32_t sys0 = 0;
  bool shared = true;
  while (todo != 0 && shared) {
    const uint32_t kk = __builtin_amdgcn_readlane(key, __ffsll((unsigned long long)todo) - 1);
    todo &= ~__ballot(key == kk);
    const int kx = (int)compact2(kk & lmask), ky = (int)compact2((kk & lmask) >> 1);
    const uint32_t ks = kk & ~lmask;
    if (nd == 0) {
      sys0 = ks;
      bx0 = kx - 1;
      bx1 = kx + 1;
      by0 = ky - 1;
      by1 = ky + 1;
    } else {
      bx0 = min(bx0, kx - 1);
      bx1 = max(bx1, kx + 1);
      by0 = min(by0, ky - 1);
      by1 = max(by1, ky + 1);
    }
    if (nd == 0) {
      dx0 = kx;
      dy0 = ky;
    } else if (nd == 1) {
      dx1 = kx;
      dy1 = ky;
    } else if (nd == 2) {
      dx2 = kx;
      dy2 = ky;
    } else {
      dx3 = kx;
      dy3 = ky;
    }
    ++nd;
    shared = nd <= 4 && ks == sys0 && (bx1 - bx0 + 1) * (by1 - by0 + 1) <= 16;
  }
  if (shared && nd > 1) {
    int usum = 0, o0 = 0, o1 = 0, o2 = 0, o3 = 0;
    for (int ny = max(by0, 0); ny <= min(by1, nl - 1); ++ny)
      for (int nx = max(bx0, 0); nx <= min(bx1, nl - 1); ++nx) {
        const uint32_t nk = sys0 | spread2(nx) | (spread2(ny) << 1);
        const int c = leaf_start[(int64_t)(nk + 1) << lsh] - leaf_start[(int64_t)nk << lsh];
        usum += c;
        if (abs(nx - dx0) <= 1 && abs(ny - dy0) <= 1) o0 += c;
        if (abs(nx - dx1) <= 1 && abs(ny - dy1) <= 1) o1 += c;
        if (nd > 2 && abs(nx - dx2) <= 1 && abs(ny - dy2) <= 1) o2 += c;
        if (nd > 3 && abs(nx - dx3) <= 1 && abs(ny - dy3) <= 1) o3 += c;
      }
    shared = 5 * usum <= 6 * max(max(o0, o1), max(o2, o3));
  }
  if (shared) {
    for (int ny = max(by0, 0); ny <= min(by1, nl - 1); ++ny) {
      for (int nx = max(bx0, 0); nx <= min(bx1, nl - 1); ++nx) {
        const uint32_t nk = sys0 | spread2(nx) | (spread2(ny) << 1);
        const int32_t i0 = leaf_start[(int64_t)nk << lsh], i1 = leaf_start[(int64_t)(nk + 1) << lsh];
        if (abs(nx - lx) <= 1 && abs(ny - ly) <= 1) f(i0, i1, lx - nx, ly - ny);
      }
    }
  } else {
    const uint32_t sysbits = key & ~lmask;
    for (int ny = ly - 1; ny <= ly + 1; ++ny) {
      if (ny < 0 || ny >= nl) continue;
      for (int nx = lx - 1; nx <= lx + 1; ++nx) {
        if (nx < 0 || nx >= nl) continue;
        const uint32_t nk = sysbits | spread2(nx) | (spread2(ny) << 1);
        f(leaf_start[(int64_t)nk << lsh], leaf_start[(int64_t)(nk + 1) << lsh], lx - nx, ly - ny);
      }
    }
  }
}

// FP64 near field (p2p2d_f64.hip): as launch_p2p2d with FP64 coordinates.
void launch_p2p2d_f64(const FmmArgs& a, hipStream_t st);

}  // namespace sffmm

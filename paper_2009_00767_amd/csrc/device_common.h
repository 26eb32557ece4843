// device_common.h -- Morton-code helpers, leaf-centre offsets, the P2M work
// plan and the point-charge (Lagrange) weights shared by the 2D and 3D kernels.
#pragma once

#include "fmm_internal.h"

namespace sffmm {

__device__ __forceinline__ uint32_t compact2(uint32_t v) {
  v &= 0x55555555u;
  v = (v | (v >> 1)) & 0x33333333u;
  v = (v | (v >> 2)) & 0x0F0F0F0Fu;
  v = (v | (v >> 4)) & 0x00FF00FFu;
  v = (v | (v >> 8)) & 0x0000FFFFu;
  return v;
}

__device__ __forceinline__ uint32_t spread2(uint32_t v) {
  v &= 0xFFFFu;
  v = (v | (v << 8)) & 0x00FF00FFu;
  v = (v | (v << 4)) & 0x0F0F0F0Fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

__device__ __forceinline__ uint32_t compact3(uint32_t v) {
  v &= 0x09249249u;
  v = (v | (v >> 2)) & 0x030C30C3u;
  v = (v | (v >> 4)) & 0x0300F00Fu;
  v = (v | (v >> 8)) & 0x030000FFu;
  v = (v | (v >> 16)) & 0x000003FFu;
  return v;
}

__device__ __forceinline__ uint32_t spread3(uint32_t v) {
  v &= 0x3FFu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// Offset of a leaf centre from the centre of its level-k ancestor, along one
// axis, in units of s_L: (r + 1/2) - 2^(L-k) / 2 with r the leaf index inside
// the ancestor.  Exact in FP32 and FP64.
template <typename T>
__device__ __forceinline__ T leaf_to_box(uint32_t leaf, int sh) {
  const uint32_t r = leaf & ((1u << sh) - 1u);
  return (T)r + (T)0.5 - (T)(1u << sh) * (T)0.5;
}

// P2M work plan: per level, G = 2^lgG lanes per box (at most 64) and S = 2^lgS
// waves (slices) per box when it holds far more than a wave's share.  Level
// thread ranges start on wave boundaries.  (Powers of two kept as shifts: the
// 64-bit divisions by G and S took more instructions than a lane's particles.)
struct P2mPlan {
  int klo, khi;
  int32_t lgG[kMaxLevels2D + 1];
  int32_t lgS[kMaxLevels2D + 1];
  int64_t thr_off[kMaxLevels2D + 2];
  int64_t part_off[kMaxLevels2D + 1];
};

// Each lane takes about `per` particles (16; where a lane's sum may be split,
// fewer: p2m_lane_particles), a box of at most 1.5 per a single lane.
inline P2mPlan make_p2m_plan(int dim, int klo, int khi, int64_t n, int nsys = 1, int per = 16) {
  P2mPlan pl{};
  pl.klo = klo;
  pl.khi = khi;
  int64_t t = 0, po = 0;
  for (int k = klo; k <= khi; ++k) {
    const int64_t nb = (int64_t)nsys << (dim * k);
    const int64_t avg = n / nb;
    int lg = 0, ls = 0;
    if (2 * avg > 3 * per) {
      while (lg < 6 && ((int64_t)per << lg) < avg) ++lg;
      if (avg > 2048)
        while (ls < 10 && ((int64_t)1024 << ls) < avg) ++ls;
    }
    pl.lgG[k] = lg;
    pl.lgS[k] = ls;
    pl.thr_off[k] = t;
    pl.part_off[k] = po;
    t += ((nb << (lg + ls)) + 63) / 64 * 64;
    if (ls > 0) po += nb << ls;
  }
  pl.thr_off[khi + 1] = t;
  return pl;
}

// Particles per lane.  FP32 sums keep 16, which their rounding follows.  FP64 sums
// take 4 up to 2^16 particles, where the waves of a level would not fill the chip
// and a launch lasts as long as one lane's chain (whole evaluations with 16, 8 and
// 4: 4096 particles 50.8, 48.5, 47.1 us, 65,536 103, 100, 98; 20,000 in 3D 251,
// 240, 238; 8192 with 8 x 8 Chebyshev points 116, 108, 107).  Beyond, shorter chains
// are what dense boxes need, most of all in 3D, whose boxes hold few particles on
// average (clustered: 100,000 at level 4 13.4, 4.0, 2.2 ms, 300,000 at level 5 13.2,
// 13.4, 10.8; uniform: 600,000 2.31, 2.33, 2.34); in 2D the further waves also take
// their places from the near field beside them (clustered: 150,000 at level 6 2022,
// 2043, 2312 us, 262,144 at level 7 1944, 1884, 1872, 100,000 with 8 x 8 points 1457,
// 1305, 1655; uniform: 400,000 254, 261, 273, 300,000 with 8 x 8 points 392, 452, 459).
inline int p2m_lane_particles(bool f64, int64_t n, int beyond) {
  return !f64 ? 16 : n > ((int64_t)1 << 16) ? beyond : 4;
}

// A particle's sorted place where lanes step through a range: unsigned, since a
// plan may hold up to 2^31 - 2 particles, and a lane's first place, or the one past
// its last, lies up to a step (at most 64 + 63) beyond the range's end.
typedef uint32_t place_t;

// The work item of thread t of level k: box b, slice j, lane r of its group, and
// (inside the box range) its particles lo + r, lo + r + G, ... below hi.
struct P2mItem {
  int64_t b;
  int j, r;
};
__device__ __forceinline__ P2mItem p2m_item_of(const P2mPlan& pl, int k, int64_t t) {
  const int64_t local = t - pl.thr_off[k];
  const int lg = pl.lgG[k], ls = pl.lgS[k];
  return P2mItem{local >> (lg + ls), (int)(local >> lg) & ((1 << ls) - 1),
                 (int)local & ((1 << lg) - 1)};
}
__host__ __device__ inline void p2m_slice(const P2mPlan& pl, int k, int j, int32_t s0, int32_t s1,
                                          place_t& lo, place_t& hi) {
  const int64_t len = s1 - s0;
  lo = (place_t)(s0 + (len * j >> pl.lgS[k]));
  hi = (place_t)(s0 + (len * (j + 1) >> pl.lgS[k]));
}

// Distance between the 64 probes of a search over n >= 1 places.
__host__ __device__ constexpr int32_t probe_step(int32_t n) {
  return (int32_t)(((place_t)n + 63) >> 6);
}

// Sums v[0..N) over the 2^lg lanes of each group (neighbouring lanes, lg uniform
// over the wave) and hands every value to one lane: store(i, sum) on the lane
// that ends up with value i.  Step d (lanes d apart) keeps half of the values a
// lane holds and sends the other half, so that N values cost N exchanges and
// not N per step, and a row is written by all lanes of its group.  The sums are
// those of a butterfly over d = 1, 2, 4, ..., bit for bit.
template <int N, int STEP = 0, int NV, typename T, class F>
__device__ __forceinline__ void group_sum(T (&v)[NV], int lg, F&& store, int base = 0,
                                          int lim = N) {
  if constexpr (STEP < 6) {
    if (lg > STEP) {
      constexpr int H = (N + 1) / 2;
      const bool up = (threadIdx.x >> STEP) & 1;
#pragma unroll
      for (int i = 0; i < H; ++i) {
        const T lo = v[i], hi = H + i < N ? v[H + i] : (T)0;
        v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, 1 << STEP, 64);
      }
      group_sum<H, STEP + 1>(v, lg, store, up ? base + H : base, up ? lim : min(lim, base + H));
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (base + i < lim) store(base + i, v[i]);
}

inline size_t p2m_partial_rows(int dim, int klo, int khi, int64_t maxn, int nsys = 1) {
  if (khi < klo) return 0;
  const P2mPlan pl = make_p2m_plan(dim, klo, khi, maxn, nsys);
  int64_t rows = 0;
  for (int k = klo; k <= khi; ++k)
    if (pl.lgS[k] > 0) rows += ((int64_t)nsys << (dim * k)) << pl.lgS[k];
  return (size_t)rows;
}

// Low 2k bits of a stacked 2D key / box index: the Morton code inside its system.
__device__ __forceinline__ uint32_t local2(uint32_t v, int k) {
  return v & ((k >= 16) ? 0xFFFFFFFFu : ((1u << (2 * k)) - 1u));
}

// Deals blocks round-robin over the 8 XCDs the way the hardware dispatches them
// and maps them back so that each XCD owns one contiguous range of work items.
// Adaptive depth: particles in the 3 x 3 level-k boxes around box (bx, by) of
// a one-system 2D tree of depth L (leaf_start: the level-L leaf offsets; a
// level-k box spans the leaf keys [b << 2 (L - k), (b + 1) << 2 (L - k))).
__device__ __forceinline__ int64_t around_count2(const int32_t* leaf_start, int L, int k, int bx,
                                                 int by) {
  const int nb = 1 << k, sh = 2 * (L - k);
  int64_t c = 0;
  for (int y = by - 1; y <= by + 1; ++y) {
    if (y < 0 || y >= nb) continue;
    for (int x = bx - 1; x <= bx + 1; ++x) {
      if (x < 0 || x >= nb) continue;
      const int64_t b = (int64_t)(spread2((uint32_t)x) | (spread2((uint32_t)y) << 1));
      c += leaf_start[(b + 1) << sh] - leaf_start[b << sh];
    }
  }
  return c;
}

__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nblocks) {
  const int64_t q8 = nblocks / 8, r8 = nblocks % 8;
  const int64_t xcd = bid % 8, idx = bid / 8;
  return xcd * q8 + (xcd < r8 ? xcd : r8) + idx;
}

// Fixed point-charge basis (Appendix STEP1-STEP2): 4 points per axis at
// a_n s / 5 from the box centre (node set NS: the paper's a = (-2, -1, 1, 2),
// or Chebyshev points), point i + 4 j + 16 l.  A charge at w = (r - r_b) / s
// becomes the 64 charges q f_i(5 w_x) f_j(5 w_y) f_l(5 w_z), f the cubic
// Lagrange basis of those nodes; with d_n = u - a_n and c_n the inverse
// denominators:
//   f = (d_1 d_2 d_3 c_0, d_0 d_2 d_3 c_1, d_0 d_1 d_3 c_2, d_0 d_1 d_2 c_3).
template <int NS, typename T>
__device__ __forceinline__ void lag4(T w, T (&f)[4]) {
  constexpr T a0 = (T)point_node(NS, 0), a1 = (T)point_node(NS, 1), a2 = (T)point_node(NS, 2),
              a3 = (T)point_node(NS, 3);
  constexpr T c0 = (T)point_node_inv_den(NS, 0), c1 = (T)point_node_inv_den(NS, 1),
              c2 = (T)point_node_inv_den(NS, 2), c3 = (T)point_node_inv_den(NS, 3);
  const T u = (T)5 * w;
  const T d0 = u - a0, d1 = u - a1, d2 = u - a2, d3 = u - a3;
  const T d23 = d2 * d3, d01 = d0 * d1;
  f[0] = d1 * d23 * c0;
  f[1] = d0 * d23 * c1;
  f[2] = d01 * d3 * c2;
  f[3] = d01 * d2 * c3;
}

// the weights and their derivatives in u
template <int NS, typename T>
__device__ __forceinline__ void lag4d(T w, T (&f)[4], T (&df)[4]) {
  constexpr T a0 = (T)point_node(NS, 0), a1 = (T)point_node(NS, 1), a2 = (T)point_node(NS, 2),
              a3 = (T)point_node(NS, 3);
  constexpr T c0 = (T)point_node_inv_den(NS, 0), c1 = (T)point_node_inv_den(NS, 1),
              c2 = (T)point_node_inv_den(NS, 2), c3 = (T)point_node_inv_den(NS, 3);
  const T u = (T)5 * w;
  const T d0 = u - a0, d1 = u - a1, d2 = u - a2, d3 = u - a3;
  const T d23 = d2 * d3, d01 = d0 * d1, d13 = d1 * d3, d12 = d1 * d2, d03 = d0 * d3,
          d02 = d0 * d2;
  f[0] = d1 * d23 * c0;
  f[1] = d0 * d23 * c1;
  f[2] = d01 * d3 * c2;
  f[3] = d01 * d2 * c3;
  df[0] = (d23 + d13 + d12) * c0;
  df[1] = (d23 + d03 + d02) * c1;
  df[2] = (d13 + d03 + d01) * c2;
  df[3] = (d12 + d02 + d01) * c3;
}

// acc[i + 4 j + 16 l] += q f_i(x) f_j(y) f_l(z)
template <int NS, typename T>
__device__ __forceinline__ void points_accumulate(T (&acc)[64], T q, T wx, T wy, T wz) {
  T fx[4], fy[4], fz[4];
  lag4<NS>(wx, fx);
  lag4<NS>(wy, fy);
  lag4<NS>(wz, fz);
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    const T ql = q * fz[l];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const T qjl = ql * fy[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i + 4 * j + 16 * l] += fx[i] * qjl;
    }
  }
}

}  // namespace sffmm

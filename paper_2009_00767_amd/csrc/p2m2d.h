// p2m2d.h -- the moments of the 2D log kernel: one work item's accumulation, for
// the moment kernels and for the launch that joins them with the near field.
#pragma once

#include <type_traits>

#include "device_common.h"

namespace sffmm {

#define SFFMM_PB_DISPATCH(fn, p, ...) \
  do {                                \
    switch (order_bucket(p)) {        \
      case 8: fn<8>(__VA_ARGS__); break;   \
      case 12: fn<12>(__VA_ARGS__); break; \
      case 16: fn<16>(__VA_ARGS__); break; \
      case 20: fn<20>(__VA_ARGS__); break; \
      case 24: fn<24>(__VA_ARGS__); break; \
      default: fn<30>(__VA_ARGS__); break; \
    }                                 \
  } while (0)

// Runs f(integral_constant<PK>) with PK the order bucket of p (at most PB), so
// that a level's work follows its own order and not the layout's: the loops
// over coefficients are unrolled to PK with no per-coefficient test.
// FULL: every level runs at the layout order PB.
template <int PB, bool FULL, class F>
__device__ __forceinline__ void with_order_bucket(int p, F&& f) {
  if (FULL) {
    f(std::integral_constant<int, PB>());
    return;
  }
  const int pk = order_bucket(p);
  if constexpr (PB > 8)
    if (pk == 8) {
      f(std::integral_constant<int, 8>());
      return;
    }
  if constexpr (PB > 12)
    if (pk == 12) {
      f(std::integral_constant<int, 12>());
      return;
    }
  if constexpr (PB > 16)
    if (pk == 16) {
      f(std::integral_constant<int, 16>());
      return;
    }
  if constexpr (PB > 20)
    if (pk == 20) {
      f(std::integral_constant<int, 20>());
      return;
    }
  if constexpr (PB > 24)
    if (pk == 24) {
      f(std::integral_constant<int, 24>());
      return;
    }
  f(std::integral_constant<int, PB>());
}

struct NegInverse {  // -1 / m
  double v[kMaxOrder2D + 1];
  constexpr NegInverse() : v() {
    for (int m = 1; m <= kMaxOrder2D; ++m) v[m] = -1.0 / m;
  }
};
static __constant__ const NegInverse kNegInverse;

// Moments of one (box, slice, lane) work item up to order PK (>= p): powers
// of w above p are formed too and dropped at the store, where every moment
// above p is written as zero.
template <typename T, int PB, int PK, bool LL>
__device__ __forceinline__ void p2m_item(const FmmArgs& a, const P2mPlan& pl, int k, int p,
                                         bool valid, const P2mItem& it) {
  const LevelTable& lt = a.lt;
  const int sh = lt.L - k, G = 1 << pl.lgG[k];
  const int64_t b = it.b;
  T v[2 * PK + 1];  // re / im of orders 1..PK, then order 0
#pragma unroll
  for (int i = 0; i <= 2 * PK; ++i) v[i] = (T)0;
  // adaptive depth: only the moments some interaction list reads, those of
  // boxes whose parent has an open box in its 3 x 3 (every box at kmin)
  if (valid && a.adapt_open && k > lt.kmin)
    valid = (a.adapt_open[adapt_open_off(k - 1) + (b >> 2)] & 2) != 0;
  if (valid) {
    place_t lo, hi;
    p2m_slice(pl, k, it.j, a.leaf_start[b << (2 * sh)], a.leaf_start[(b + 1) << (2 * sh)], lo, hi);
    const T is = (T)lt.inv_s[k];
    T cx = 0, cy = 0, sL = (T)lt.s[lt.L];
    if (!LL) {
      const uint32_t lb = local2((uint32_t)b, k);
      cx = (T)(lt.origin[0] + lt.s[k] * ((double)compact2(lb) + 0.5));
      cy = (T)(lt.origin[1] + lt.s[k] * ((double)compact2(lb >> 1) + 0.5));
    }
    // the next particle's inputs are loaded while this one is accumulated
    float4 npt = make_float4(0.f, 0.f, 0.f, 0.f);
    double nx = 0, ny = 0, nq = 0;
    if (lo + it.r < hi) {
      if (LL) {
        npt = a.pts[lo + it.r];
      } else {
        nx = a.xs[lo + it.r];
        ny = a.ys[lo + it.r];
        nq = a.qs[lo + it.r];
      }
    }
    for (place_t i = lo + it.r; i < hi; i += G) {
      T q, wr, wi;
      const float4 pt = npt;
      const double px = nx, py = ny, pq = nq;
      if (i + G < hi) {
        if (LL) {
          npt = a.pts[i + G];
        } else {
          nx = a.xs[i + G];
          ny = a.ys[i + G];
          nq = a.qs[i + G];
        }
      }
      if (LL) {
        const uint32_t lb = __float_as_uint(pt.w);  // the leaf's column | row << 16
        const T ox = leaf_to_box<T>(lb & 0xFFFFu, sh) * sL;
        const T oy = leaf_to_box<T>(lb >> 16, sh) * sL;
        q = (T)pt.z;
        wr = ((T)pt.x + ox) * is;
        wi = ((T)pt.y + oy) * is;
      } else {
        q = (T)pq;
        wr = ((T)px - cx) * is;
        wi = ((T)py - cy) * is;
      }
      v[2 * PK] += q;
      T pr = q * wr, pi = q * wi;  // q w^m
#pragma unroll
      for (int m = 1; m <= PK; ++m) {
        v[2 * (m - 1)] += pr;
        v[2 * (m - 1) + 1] += pi;
        const T nr = pr * wr - pi * wi;
        pi = pr * wi + pi * wr;
        pr = nr;
      }
    }
  }
  const int S = 1 << pl.lgS[k], cs = a.cs;
  T* out;
  if (S == 1)
    out = (sizeof(T) == 8 ? (T*)a.mom64 : (T*)a.mom32) + (lt.off[k] + b) * cs;
  else
    out = (sizeof(T) == 8 ? (T*)a.part64 : (T*)a.part32) + (pl.part_off[k] + b * S + it.j) * cs;
  group_sum<2 * PK + 1>(v, pl.lgG[k], [&](int i, T x) {
    if (!valid) return;
    if (i < 2 * PK) {
      const int m = i / 2 + 1;
      out[i] = m <= p ? x * (T)kNegInverse.v[m] : (T)0;
    } else {
      out[2 * PB] = x;
    }
  });
  if (!valid || it.r != 0) return;
#pragma unroll
  for (int i = 2 * PK; i < 2 * PB; ++i) out[i] = (T)0;
  out[2 * PB + 1] = (T)0;
}

// Work item of thread t of a launch over the plan's levels.
template <typename T, int PB, bool LL, bool FULL>
__device__ __forceinline__ void p2m_thread(const FmmArgs& a, const P2mPlan& pl, int64_t t) {
  if ((t & ~(int64_t)63) >= pl.thr_off[pl.khi + 1]) return;  // whole wave beyond the end
  const LevelTable& lt = a.lt;
  int k = pl.klo;
  while (k < pl.khi && t >= pl.thr_off[k + 1]) ++k;
  k = __builtin_amdgcn_readfirstlane(k);  // (waves never straddle levels)
  const P2mItem it = p2m_item_of(pl, k, t);
  const bool valid = it.b < (int64_t)lt.nsys << (2 * k);
  const int p = FULL ? PB : a.ord[k];  // this level's order
  with_order_bucket<PB, FULL>(p, [&](auto pk) {
    p2m_item<T, PB, decltype(pk)::value, LL>(a, pl, k, p, valid, it);
  });
}

// Adds up the slice partials of a launch over the plan's levels (order bucket
// pb), if it has any.
void launch_p2m2d_slices(const FmmArgs& a, const P2mPlan& pl, int pb, bool f64, hipStream_t st);

}  // namespace sffmm

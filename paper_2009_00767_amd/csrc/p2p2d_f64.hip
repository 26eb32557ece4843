// p2p2d_f64.hip -- the FP64 near field of the 2D log kernel (E-2 of Section
// 2.1), in sorted order (the local evaluation adds the far field and scatters
// back to input order).  Sources of a target: its leaf and the adjacent ones;
// pairs with r = 0 (the target itself, coincident points) contribute nothing.
//
// A pair needs log r^2 and 1 / r^2 in FP64; with the library's log and a correctly
// rounded division it took about 117 vector instructions.  Here the loop over four
// sources holds 111: the reciprocal is the hardware estimate with one third-order
// step, and the logarithm comes from a table in LDS.  Whole evaluations, before and
// now: 500,009 clustered particles at level 8 (8.5e8 to 9.8e8 pairs) 4.53 -> 1.62
// ms, 2^20 uniform at level 8 (1.5e8) 0.95 -> 0.52, 4096 at level 4 (sixteen lanes a
// target instead of one: 64 waves had left the chip idle) 112 -> 44 us.
//
// What bounds it, by counters of each kernel alone (vector instructions take 4
// cycles of a SIMD and more for the reciprocal, exponent and conversion):
//   direct form, the clustered case: 1.27 ms, 6.9e11 pairs/s, 29.4 instructions a
//     pair, the vector unit at work for 0.62 of the cycles.  Waves are 0.42 of their
//     time ready without a turn and 0.22 waiting for data, and 2.2 of them are on a
//     SIMD on average: those of the densest leaves outlast the others.  The LDS is
//     busy for 0.22 of the cycles, two thirds of that bank conflicts of the table.
//   tile form, the uniform case: 0.24 ms, 6.2e11 pairs/s, 39.8 instructions a pair
//     (lanes whose spans have ended, remainders taken one by one, staging), the vector
//     unit at work for 0.77 of the cycles, the LDS for 0.41, a third of that
//     conflicts; 2.8 waves on a SIMD.
#include "near2d.h"
#include "p2m2d.h"

namespace sffmm {

namespace {

// Targets up to which sixteen, and four, lanes share one (launch_p2p2d_f64).
constexpr int64_t kLanes16 = 1 << 14, kLanes4 = 1 << 16;

// log2 of a normal r2 > 0 from the hardware's mantissa m in [1/2, 1) and exponent:
// log2(m) is T_i + log2(1 + u) with u = m c_i - 1, c_i the reciprocal of the middle
// of m's interval of width 2^-8 and T_i = -log2 c_i.  |u| <= 2^-8, so the series of
// log2(1 + u) ends after u^6 (the next term is below 3e-18).
//
// UNIT (pairs can be about one unit apart, near_unit): exponent and mantissa
// parts must vanish together at r2 = 1, or a logarithm near zero loses its
// digits to their cancellation.  The mantissa then runs over [1/s, s), s = 1 +
// kLogLow / 128 (about the square root of 2): intervals below kLogLow stand for 2 m, T_i
// = -log2(c_i / 2), and the exponent is one less.  The intervals at m = 1/2 and
// below 1 take c = 2 and 1, for which u is exact and T = 0; |u| <= 2^-7 there,
// so the series goes up to u^7, its u^8 term folded into the lower ones over |u|
// <= 2^-7 by Chebyshev's T_7 (economisation; what is left is below 4e-18 of the
// logarithm).  Two instructions a pair more, so only where it matters: 500,009
// clustered particles (level 8 of a box of side 5) 1502 us a call, with it 1554.
constexpr int kLogBits = 7;
constexpr int kLogTable = 1 << kLogBits;
constexpr int kLogLow = 53;
constexpr uint32_t kLogBase = (1022u << 20) + ((uint32_t)kLogLow << (20 - kLogBits));
template <bool UNIT>
__device__ __forceinline__ void fill_log_table(double2* tab) {
  for (int i = threadIdx.x; i < kLogTable; i += blockDim.x) {
    double c = 1.0 / (0.5 + ((double)i + 0.5) * (0.5 / kLogTable));
    if (UNIT) c = i == 0 ? 2.0 : i == kLogTable - 1 ? 1.0 : c;
    tab[i] = make_double2(c, 0.0 - log2(UNIT && i < kLogLow ? 0.5 * c : c));
  }
}

// Whether sources of the leaves around a target (at most two leaf sides away in
// each direction) can reach r2 = 1: below, r2 lies in intervals where exponent and
// mantissa parts do not cancel.
bool near_unit(const LevelTable& lt) { return !(8.0 * lt.s[lt.L] * lt.s[lt.L] < 0.98); }

constexpr double kHalfLn2 = 0.34657359027997264;  // log r = log2(r^2) (ln 2) / 2

// Running sums of a target: log2(r^2) in two parts (the exponents' share is
// kept apart, so that neither part rounds at the other's magnitude), and the field.
struct NearSum {
  double fr = 0.0, ex2 = 0.0, ex = 0.0, ey = 0.0;
};

// Below thr (0 < r2 < 2^-900, or any r2 of a box too large for the reciprocal)
// a pair takes the library's functions.
__device__ __forceinline__ double near_threshold(double side) {
  return side < 0x1p400 ? 0x1p-900 : __builtin_inf();
}

// The sums of U pairs at dx, dy, r2 (a normal number of FP64's range).
template <int U, bool UNIT>
__device__ __forceinline__ void add_pairs2(const double (&dx)[U], const double (&dy)[U],
                                           const double (&r2)[U], const double (&q)[U],
                                           const double2* tab, NearSum& a) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t hi = (uint32_t)__double2hiint(r2[u]);
    const double2 t = tab[(hi >> (20 - kLogBits)) & (kLogTable - 1)];
    const double m = __builtin_amdgcn_frexp_mant(r2[u]);
    const double ef = UNIT ? (double)((int32_t)(hi - kLogBase) >> 20)
                           : (double)__builtin_amdgcn_frexp_exp(r2[u]);
    double y0 = __builtin_amdgcn_rcp(r2[u]);  // relative error e at most 2^-24.3 (measured)
    const double e = fma(-r2[u], y0, 1.0);
    y0 = fma(y0, fma(e, e, e), y0);  // 1 / r2 = y0 / (1 - e) = y0 (1 + e + e^2 + ...)
    const double w = q[u] * y0;
    const double v = fma(m, t.x, -1.0);
    double p;
    if constexpr (UNIT) {
      p = fma(v, 0.2060992915555662, -0.24046843553839053);  // (-1)^k / ((k + 1) ln 2), folded
      p = fma(p, v, 0.28853900817779266);
      p = fma(p, v, -0.3606737596344095);
      p = fma(p, v, 0.4808983469629878);
      p = fma(p, v, -0.7213475204444861);
    } else {
      p = fma(v, -0.24044917348149390, 0.28853900817779268);  // (-1)^k / ((k + 1) ln 2)
      p = fma(p, v, -0.36067376022224085);
      p = fma(p, v, 0.48089834696298780);
      p = fma(p, v, -0.72134752044448170);
    }
    p = fma(p, v, 1.4426950408889634);
    a.fr = fma(q[u], fma(p, v, t.y), a.fr);
    a.ex2 = fma(q[u], ef, a.ex2);
    a.ex = fma(-w, dx[u], a.ex);
    a.ey = fma(-w, dy[u], a.ey);
  }
}

// U sources at once.  Whether some lane has a pair at r = 0 or below thr is one
// compare a pair (its mask is joined in scalar registers); the batch then takes
// a path of its own, so that the others carry nothing of it.
template <int U, bool UNIT>
__device__ __forceinline__ void pairs2_f64(double x, double y, const double (&sx)[U],
                                           const double (&sy)[U], const double (&q)[U],
                                           double thr, const double2* tab, NearSum& a) {
  double dx[U], dy[U], r2[U];
  uint64_t odd = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    dx[u] = x - sx[u];
    dy[u] = y - sy[u];
    r2[u] = fma(dx[u], dx[u], dy[u] * dy[u]);
    odd |= __ballot(!(r2[u] >= thr));
  }
  if (odd != 0) {
    double r[U], c[U];
    uint64_t tiny = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool zero = r2[u] == 0.0;
      r[u] = zero ? 1.0 : r2[u];
      c[u] = zero ? 0.0 : q[u];
      tiny |= __ballot(!(r2[u] >= thr) && !zero);
    }
    if (tiny != 0) {
#pragma unroll 1
      for (int u = 0; u < U; ++u) {
        double ru = r[0], cu = c[0], du = dx[0], eu = dy[0];
#pragma unroll
        for (int v = 1; v < U; ++v)
          if (u == v) {
            ru = r[v];
            cu = c[v];
            du = dx[v];
            eu = dy[v];
          }
        a.fr += cu * log2(ru);
        const double w = cu / ru;
        a.ex -= w * du;
        a.ey -= w * eu;
      }
      return;
    }
    add_pairs2<U, UNIT>(dx, dy, r, c, tab, a);
    return;
  }
  add_pairs2<U, UNIT>(dx, dy, r2, q, tab, a);
}

// The potential of target j again, by the library's logarithm and one term at a
// time.  The two parts of a logarithm may differ in sign, and either may be zero:
// with infinite charges, or charges near the end of the range, their sums can be
// inf - inf, inf * 0 or beyond the range where the terms' own sum is not, so a
// target whose sum is not finite comes here (a sum of whole terms in the loops cost
// the clustered case 3 % more).  Everything is read again, so that the loops hold
// no register for it.  lsh: see walk_near2d.
__device__ __forceinline__ void near_by_terms(const FmmArgs& a, int64_t j,
                                              const double* __restrict__ xs,
                                              const double* __restrict__ ys,
                                              const double* __restrict__ qs,
                                              const int32_t* __restrict__ leaf_start, int lsh) {
  const LevelTable& lt = a.lt;
  const uint32_t key = a.keys[j] >> lsh;
  const uint32_t lmask = local2(0xFFFFFFFFu, lt.L), sysbits = key & ~lmask;
  const int lx = (int)compact2(key & lmask), ly = (int)compact2((key & lmask) >> 1);
  const int nl = 1 << lt.L;
  const double x = xs[j], y = ys[j];
  double sum = 0.0;
#pragma unroll 1
  for (int b = 0; b < 9; ++b) {
    const int nx = lx - 1 + b % 3, ny = ly - 1 + b / 3;
    if (nx < 0 || nx >= nl || ny < 0 || ny >= nl) continue;
    const int64_t nk = (int64_t)(sysbits | spread2(nx) | (spread2(ny) << 1));
    const int32_t i1 = leaf_start[(nk + 1) << lsh];
#pragma unroll 1
    for (int32_t i = leaf_start[nk << lsh]; i < i1; ++i) {
      const double dx = x - xs[i], dy = y - ys[i], r2 = fma(dx, dx, dy * dy);
      if (r2 != 0.0) sum += qs[i] * log2(r2);
    }
  }
  a.near_pot[j] = sum * kHalfLn2;
}

// Whether the potential is finite (else near_by_terms has to follow).
__device__ __forceinline__ bool store_near(const FmmArgs& a, int64_t j, const NearSum& s) {
  const double lg = s.fr + s.ex2;
  a.near_pot[j] = lg * kHalfLn2;
  a.near_ex[j] = s.ex;
  a.near_ey[j] = s.ey;
  return fabs(lg) < __builtin_inf();
}

// Sources i0 + P k (k = 0, 1, ...) below i1 in batches of four; the last batch
// repeats its first source with no charge.  (Places are compared by their distance:
// a plan may hold up to 2^31 - 2 particles, though few with P > 1.  Unsigned ones,
// which may wrap, keep a batch's loads from being joined: 500,009 clustered
// particles 1650 -> 1774 us.)
template <int P, bool UNIT>
__device__ __forceinline__ void range2_f64(const double* __restrict__ xs,
                                           const double* __restrict__ ys,
                                           const double* __restrict__ qs, int32_t i0, int32_t i1,
                                           double x, double y, double thr, const double2* tab,
                                           NearSum& s) {
  int32_t i = i0;
  for (; i1 - i > 3 * P; i += 4 * P) {
    double sx[4], sy[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sx[u] = xs[i + u * P];
      sy[u] = ys[i + u * P];
      q[u] = qs[i + u * P];
    }
    pairs2_f64<4, UNIT>(x, y, sx, sy, q, thr, tab, s);
  }
  if (i < i1) {
    double sx[4], sy[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = u * P < i1 - i;
      const int32_t iu = in ? i + u * P : i;
      sx[u] = xs[iu];
      sy[u] = ys[iu];
      q[u] = in ? qs[iu] : 0.0;
    }
    pairs2_f64<4, UNIT>(x, y, sx, sy, q, thr, tab, s);
  }
}

// Direct form.  P = 1: one thread per sorted target (walk_near2d; dense leaves
// share their sources as scalar loads).  P > 1 (few targets for the chip): P
// neighbouring lanes share a target, lane r taking every P-th source of the
// leaves' sources in a row, and their sums meet in a butterfly.
// lsh = 2 (L - d) when the launch works at level d = lt.L of an adaptive tree
// of depth L: leaf keys and leaf offsets are those of level d, and only the
// targets whose leaf lies at level d are taken.
// over: only the targets of tiles the tile kernel left.
template <int P, bool UNIT>
__device__ __forceinline__ void near_direct(const FmmArgs& a, int over,
                                            const double* __restrict__ xs,
                                            const double* __restrict__ ys,
                                            const double* __restrict__ qs,
                                            const int32_t* __restrict__ leaf_start, int lsh,
                                            int64_t block, double2* tab) {
  const int64_t t = xcd_chunk_remap(block) * 256 + threadIdx.x;
  const int64_t j = t / P;
  const LevelTable& lt = a.lt;
  bool mine = j < a.n && (!a.depth || a.depth[j] == lt.L);
  const uint32_t key = mine ? a.keys[j] >> lsh : 0u;
  if (over) mine = mine && a.p2p_over[key >> 4];
  if (!__syncthreads_or(mine)) return;
  fill_log_table<UNIT>(tab);
  __syncthreads();
  if (!mine) return;
  const double thr = near_threshold(lt.side);
  const double x = xs[j], y = ys[j];
  NearSum s;
  if constexpr (P == 1) {
    walk_near2d(lt, key, leaf_start, lsh, [&](int32_t i0, int32_t i1, int, int) {
      range2_f64<1, UNIT>(xs, ys, qs, i0, i1, x, y, thr, tab, s);
    });
  } else {
    const uint32_t lmask = local2(0xFFFFFFFFu, lt.L), sysbits = key & ~lmask;
    const int lx = (int)compact2(key & lmask), ly = (int)compact2((key & lmask) >> 1);
    const int nl = 1 << lt.L;
    int32_t i0[9], i1[9];
#pragma unroll
    for (int b = 0; b < 9; ++b) {  // every range up front: the loads overlap
      const int nx = lx - 1 + b % 3, ny = ly - 1 + b / 3;
      const bool in = nx >= 0 && nx < nl && ny >= 0 && ny < nl;
      const int64_t nk = in ? (int64_t)(sysbits | spread2(nx) | (spread2(ny) << 1)) : 0;
      i0[b] = in ? leaf_start[nk << lsh] : 0;
      i1[b] = in ? leaf_start[(nk + 1) << lsh] : 0;
    }
    int32_t off = (int32_t)(t % P);  // this lane's first source of the next leaf
#pragma unroll
    for (int b = 0; b < 9; ++b) {
      const int32_t len = i1[b] - i0[b];
      range2_f64<P, UNIT>(xs, ys, qs, i0[b] + off, i1[b], x, y, thr, tab, s);
      const int32_t left = len - off;  // sources from this lane's first one on
      off = left > 0 ? (P - left % P) % P : -left;
    }
#pragma unroll
    for (int d = 1; d < P; d <<= 1) {
      s.fr += __shfl_xor(s.fr, d, 64);
      s.ex2 += __shfl_xor(s.ex2, d, 64);
      s.ex += __shfl_xor(s.ex, d, 64);
      s.ey += __shfl_xor(s.ey, d, 64);
    }
    if (t % P != 0) return;
  }
  if (!store_near(a, j, s)) near_by_terms(a, j, xs, ys, qs, leaf_start, lsh);
}

template <int P, bool UNIT>
__global__ __launch_bounds__(256) void k_p2p2d_f64(FmmArgs a, int over,
                                                   const double* __restrict__ xs,
                                                   const double* __restrict__ ys,
                                                   const double* __restrict__ qs,
                                                   const int32_t* __restrict__ leaf_start,
                                                   int lsh) {
  __shared__ double2 tab[kLogTable];
  near_direct<P, UNIT>(a, over, xs, ys, qs, leaf_start, lsh, blockIdx.x, tab);
}

// Few particles: the near field and the moments of every level, which both
// need only the sort, as two kinds of workgroups of one launch: the moments'
// few workgroups first, rounded up to whole rounds of the 8 XCDs.  Both are
// bound by latency and leave most of the chip idle alone (20,011 particles,
// order 16, 5 levels: 23 and 12 us one after the other; a call on one stream 85
// -> 73 us).
template <int P, int PB, bool FULL, bool UNIT>
__global__ __launch_bounds__(256) void k_near_moments2d(FmmArgs a, P2mPlan pl, int moments,
                                                        const double* __restrict__ xs,
                                                        const double* __restrict__ ys,
                                                        const double* __restrict__ qs,
                                                        const int32_t* __restrict__ leaf_start) {
  __shared__ double2 tab[kLogTable];
  if ((int)blockIdx.x < moments)
    p2m_thread<double, PB, false, FULL>(a, pl, (int64_t)blockIdx.x * 256 + threadIdx.x);
  else
    near_direct<P, UNIT>(a, 0, xs, ys, qs, leaf_start, 0, blockIdx.x - moments, tab);
}

// Tile form: a workgroup stages the sources of a 4 x 4-leaf tile's 6 x 6-leaf
// halo in LDS, halo rows contiguous, so that a target's nine leaves are three
// spans.  Two lanes share a target (its spans' sources dealt round): a wave then
// holds 32 targets of two or three leaves, whose spans differ little in length
// (2^20 uniform particles at level 8, alone: one lane 282 us, two 239, four 249,
// eight 287).  Tiles whose halo exceeds the stage are flagged and left to the
// direct kernel.
constexpr int kTile64P = 2;
constexpr int kTile64Cap = 1536;  // records of 24 bytes

template <bool UNIT>
__global__ __launch_bounds__(256) void k_p2p2d_f64_tile(FmmArgs a, int cap) {
  constexpr int P = kTile64P;
  extern __shared__ double2 sxy[];  // cap positions, then as many charges
  __shared__ double2 tab[kLogTable];
  __shared__ int32_t hstart[kP2pHaloLeaves];
  __shared__ int32_t hoff[kP2pHaloLeaves + 1];
  double* sq = reinterpret_cast<double*>(sxy + cap);
  const LevelTable& lt = a.lt;
  const int L = lt.L, tid = threadIdx.x;
  const int64_t tl = xcd_chunk_remap(blockIdx.x);
  if (tl >= ((int64_t)lt.nsys << (2 * (L - 2)))) return;  // grid padding (workgroup-uniform)
  const uint32_t tile = (uint32_t)tl, k0 = tile << 4;
  const uint32_t tm = local2(k0, L);
  const int bx0 = (int)compact2(tm), by0 = (int)compact2(tm >> 1);
  fill_log_table<UNIT>(tab);
  tile_halo(lt, a.leaf_start, tile, hstart, hoff);
  const int total = hoff[kP2pHaloLeaves];
  if (tid == 0) a.p2p_over[tile] = total > cap ? 1 : 0;
  if (total > cap) return;  // workgroup-uniform
  stage_halo(hstart, hoff, 256, [&](int e, int32_t i, int) {
    sxy[e] = make_double2(a.xs[i], a.ys[i]);
    sq[e] = a.qs[i];
  });
  __syncthreads();
  const int32_t t0 = a.leaf_start[k0], t1 = a.leaf_start[k0 + 16];
  const double thr = near_threshold(lt.side);
  const int part = tid % P;
  bool again = false;
  for (int32_t j = t0 + tid / P; j < t1; j += 256 / P) {
    const uint32_t key = local2(a.keys[j], L);
    const int tx = (int)compact2(key) - bx0, ty = (int)compact2(key >> 1) - by0;
    const double x = a.xs[j], y = a.ys[j];
    NearSum s;
#pragma unroll 1
    for (int dy = 0; dy < 3; ++dy) {
      const int h = (ty + dy) * kP2pHalo + tx;  // halo leaves h, h + 1, h + 2
      const int c1 = hoff[h + 3];
      int c = hoff[h] + part;
      for (; c + 3 * P < c1; c += 4 * P) {
        double sx[4], sy[4], q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double2 p = sxy[c + u * P];
          sx[u] = p.x;
          sy[u] = p.y;
          q[u] = sq[c + u * P];
        }
        pairs2_f64<4, UNIT>(x, y, sx, sy, q, thr, tab, s);
      }
      for (; c < c1; c += P) {
        double sx[1] = {sxy[c].x}, sy[1] = {sxy[c].y}, q[1] = {sq[c]};
        pairs2_f64<1, UNIT>(x, y, sx, sy, q, thr, tab, s);
      }
    }
#pragma unroll
    for (int d = 1; d < P; d <<= 1) {
      s.fr += __shfl_xor(s.fr, d, 64);
      s.ex2 += __shfl_xor(s.ex2, d, 64);
      s.ex += __shfl_xor(s.ex, d, 64);
      s.ey += __shfl_xor(s.ey, d, 64);
    }
    if (part == 0 && !store_near(a, j, s)) again = true;
  }
  if (!again) return;
#pragma unroll 1
  for (int j = t0 + tid / P; j < t1; j += 256 / P)
    if (!(fabs(a.near_pot[j]) < __builtin_inf()))
      near_by_terms(a, j, a.xs, a.ys, a.qs, a.leaf_start, 0);
}

template <int P>
void direct_f64(const FmmArgs& a, int over, int lsh, hipStream_t st) {
  const dim3 grid = chunked_grid((a.n * P + 255) / 256);
  if (near_unit(a.lt))
    hipLaunchKernelGGL((k_p2p2d_f64<P, true>), grid, dim3(256), 0, st, a, over, a.xs, a.ys, a.qs,
                       a.leaf_start, lsh);
  else
    hipLaunchKernelGGL((k_p2p2d_f64<P, false>), grid, dim3(256), 0, st, a, over, a.xs, a.ys, a.qs,
                       a.leaf_start, lsh);
}

// Tiles from 1024 of them on (four workgroups a CU) and for 6 to 40 particles a
// leaf.  Below, a tile's staging costs more than its sources' second reads (uniform
// particles at levels 7, 8 and 9, whole calls with tiles and without: 5 a leaf
// 121, 241 and 824 us against 112, 235 and 832; 7: 128, 275, 969 against 127,
// 284, 1012; 0.1 a leaf 193, 281, 589 against 176, 266, 549).  Above, many a halo
// (36 leaves) outgrows the stage and the direct kernel does it again (39 a leaf at
// levels 7 and 8: 458 and 1580 against 453 and 1661; 45: 737 and 2260 against 534
// and 2022).
// Without tiles the chip wants more threads than targets.  Whole calls, order 12,
// with sixteen, four and one lane a target, uniform | clustered particles:
//      4096, level 4   44.8  48.7  64.2 |  60.7 103.9 259.4 us
//    16,384, level 5   62.3  58.2  75.3 | 118.7 167.1 377.8
//    24,000, level 5   69.5  64.0  84.1 | 172.2 236.7 523.9
//    32,768, level 6   85.9  68.4  75.6 | 178.8 188.3 376.6
//    65,536, level 6  121.4  94.0  93.3 | 398.5 474.1 671.6
//   100,000, level 6  157.3 120.9 122.7 (131,072: 187.3 151.2 135.9)
// Uniform particles turn from sixteen lanes to four near 12,000, clustered ones
// beyond 65,536; sixteen up to 2^14 lies between.  From four to one uniform ones
// turn at 65,536 to 100,000.
int64_t near_tiles(const FmmArgs& a) {  // 0: the direct form
  const int64_t tiles = a.lt.L >= 2 && a.p2p_over ? (int64_t)a.lt.nsys << (2 * (a.lt.L - 2)) : 0;
  const bool dense = a.n >= 6 * 16 * tiles && a.n <= 40 * 16 * tiles;
  return tiles >= 1024 && dense ? tiles : 0;
}

template <int P, int PB, bool FULL>
void near_moments(const FmmArgs& a, hipStream_t st) {
  const P2mPlan pl = make_p2m_plan(2, a.klo, a.khi, a.n, a.lt.nsys, p2m_lane_particles(true, a.n, 8));
  const int moments = (int)((pl.thr_off[a.khi + 1] + 256 * 8 - 1) / (256 * 8) * 8);
  const dim3 grid(chunked_grid((a.n * P + 255) / 256).x + moments);
  if (near_unit(a.lt))
    hipLaunchKernelGGL((k_near_moments2d<P, PB, FULL, true>), grid, dim3(256), 0, st, a, pl,
                       moments, a.xs, a.ys, a.qs, a.leaf_start);
  else
    hipLaunchKernelGGL((k_near_moments2d<P, PB, FULL, false>), grid, dim3(256), 0, st, a, pl,
                       moments, a.xs, a.ys, a.qs, a.leaf_start);
  launch_p2m2d_slices(a, pl, PB, true, st);
}

template <int PB>
void near_moments_pb(const FmmArgs& a, hipStream_t st) {
  if (a.n <= kLanes16)
    a.ord_full ? near_moments<16, PB, true>(a, st) : near_moments<16, PB, false>(a, st);
  else
    a.ord_full ? near_moments<4, PB, true>(a, st) : near_moments<4, PB, false>(a, st);
}

}  // namespace

bool near_moments2d_ok(const FmmArgs& a) {
  return !a.depth && a.n > 0 && a.n <= kLanes4 && a.lt.L >= a.lt.kmin && !near_tiles(a);
}

void launch_near_moments2d(const FmmArgs& a, hipStream_t st) {
  SFFMM_PB_DISPATCH(near_moments_pb, a.p, a, st);
}

void launch_p2p2d_f64(const FmmArgs& a, hipStream_t st) {
  if (a.n <= 0) return;
  if (a.depth) {
    // the uniform near field of depth d for the targets whose depth is d (the
    // others leave at once), one launch per level
    for (int d = a.lt.kmin; d <= a.lt.L; ++d) {
      FmmArgs b = a;
      b.lt.L = d;
      direct_f64<1>(b, 0, 2 * (a.lt.L - d), st);
    }
    return;
  }
  if (const int64_t tiles = near_tiles(a)) {
    const int cap = p2p2d_tile_cap(a.lt, a.n, kTile64Cap);
    const size_t lds = (size_t)cap * 3 * sizeof(double);
    if (near_unit(a.lt))
      hipLaunchKernelGGL(k_p2p2d_f64_tile<true>, chunked_grid(tiles), dim3(256), lds, st, a, cap);
    else
      hipLaunchKernelGGL(k_p2p2d_f64_tile<false>, chunked_grid(tiles), dim3(256), lds, st, a, cap);
    direct_f64<1>(a, 1, 0, st);
  } else if (a.n <= kLanes16) {
    direct_f64<16>(a, 0, 0, st);
  } else if (a.n <= kLanes4) {
    direct_f64<4>(a, 0, 0, st);
  } else {
    direct_f64<1>(a, 0, 0, st);
  }
}

}  // namespace sffmm

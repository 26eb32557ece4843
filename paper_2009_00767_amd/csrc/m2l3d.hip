// m2l3d.hip -- the interaction-list contraction (D-bar-1 of Section 2.2.1) for
// the 3D 1/r kernel on the matrix cores.
//
// L(t) = sum_{o in IL(t)} T_o M(t + o) with T_o the real (p+1)^2 x (p+1)^2
// operator of offset o (operators.cpp), or the 64 x 64 point-charge block of
// the fixed point-charge basis (Appendix STEP3; its degree-0 slot stays zero).  The 189 offsets of an interior box
// depend only on the parities of its indices, so one workgroup takes one parity
// class and a block of 4 x 4 x (NW MB) same-parity targets (an 8 x 8 x 2 NW MB
// box region) with NW waves: wave w owns the 16 targets of each of the
// z-layers w, w + NW, ... and, per offset, runs the dense products
// C[16 x N] += A_o[16 x K] . W_o[K x N] as v_mfma 16x16x4 instructions, each
// operator value read from LDS serving MB of them.  The operators stream from
// beyond the L2 (the 3D pack outgrows an XCD's L2), so the more targets a
// workgroup holds, the less operator traffic per target.
// The operator of the next offset is copied straight from global memory into
// the other of two LDS buffers while the current one is in use (the FP64
// operators of 125 point charges, which leave room for one buffer, pass through
// registers), in the lane-major order in which the MFMA steps consume it
// (conflict-free LDS reads).  Source moments are read straight from global
// memory (each is used by one target per offset): the next offset's row takes
// the registers of the current one part by part, as the steps finish with them.
// The degree-0 input enters as one more MFMA step (K = 1, lane group 0); the
// degree-0 output uses VALU fused multiply-adds.
// Bound by the matrix cores and, near their peak, by the clock they run at.
// Measured (FP32, order 8, 2^22 particles at level 7): 63.9 -> 52 ms; with operator
// values read from LDS right before their use, and rows waited for at the head
// of an offset, the cores were busy 0.64 of the time, now 0.81 of the time a CU
// holds work.
#include <type_traits>

#include "device_common.h"
#include "points3d.h"

namespace sffmm {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));

template <typename T>
struct Mfma16x;
template <>
struct Mfma16x<float> {
  using acc_t = floatx4;
  using vec_t = floatx4;
  static __device__ __forceinline__ acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma16x<double> {
  using acc_t = doublex4;
  using vec_t = doublex2;
  static __device__ __forceinline__ acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Copies 16 bytes a lane from global memory to LDS without passing through
// registers: lane l's go to dst + 16 l (dst uniform over the wave).
__device__ __forceinline__ void lds_copy16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)(uintptr_t)src,
      (__attribute__((address_space(3))) void*)(uintptr_t)(uint32_t)(uintptr_t)dst, 16, 0, 0);
}
// Waits until at most `newer` (0, 2 or 4) of this wave's vector memory accesses are
// outstanding; they return in order, so all but the `newer` issued last have
// arrived.  Nothing is moved across it.
__device__ __forceinline__ void lds_copy_wait(int newer) {
  __builtin_amdgcn_sched_barrier(0);
  if (newer == 4)
    __builtin_amdgcn_s_waitcnt(0x0f74);
  else if (newer == 2)
    __builtin_amdgcn_s_waitcnt(0x0f72);
  else
    __builtin_amdgcn_s_waitcnt(0x0f70);
  __builtin_amdgcn_sched_barrier(0);
}

// LDS of a workgroup: the operator slot double-buffered where two fit the
// 160 KB of a CU, else one buffer (the 128 x 128 point-charge operators of
// n = 5 in FP64), refilled between two barriers.
template <typename T, int KS, int NB>
__host__ __device__ constexpr int m2l3_lds_slots() {
  return 2 * (64 * (NB * (KS + 1) + KS) + 4) * (int)sizeof(T) <= 160 * 1024 ? 2 : 1;
}

// The row of a source outside the grid (a select on the values would wait for
// their loads where they are issued): read like a box row, up to value 4 KS (the
// degree-0 value's index is at most that) and 16 bytes at a time.
constexpr int kZeroRow = 132;
alignas(16) static __device__ const double g_zero_row[kZeroRow] = {0};

struct M2l3Tiles {
  int klo, khi;
  int64_t off[kMaxLevels3D + 2];  // first block of level k (split launches: finest level first)
  int64_t nblocks;
  int nsplit[kMaxLevels3D + 2];     // offset chunks per tile at level k (1: no split)
  int64_t pbase[kMaxLevels3D + 2];  // level k's first row in the partial buffer
};

// Accumulator register r of lane group g holds output row 4g + r (FP32) or
// g + 4r (FP64); row i is the target (2 (i & 3) + px, 2 (i >> 2) + py, 2w + pz).
template <typename T>
__device__ __forceinline__ int crow3(int r, int g) {
  return sizeof(T) == 8 ? g + 4 * r : 4 * g + r;
}

template <typename T, int KS, int NB, int MB, int NW, bool SPLIT>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 && KS < 32 ? 2 : 1) void k_m2l3d_mfma(FmmArgs a, M2l3Tiles tt, M2lLayout ly) {
  using acc_t = typename Mfma16x<T>::acc_t;
  using vec_t = typename Mfma16x<T>::vec_t;
  constexpr int VW = sizeof(vec_t) / sizeof(T);  // values per vector load
  constexpr int WGLB = 64 * (NB * (KS + 1) + KS) + 4;  // lane-major slot (operators.cpp)
  constexpr int WLDS = WGLB;
  constexpr int NV = WGLB / VW;                    // vectors per slot
  constexpr int NT = 64 * NW;
  constexpr int ZL = NW * MB;  // same-parity z-layers per block
  constexpr int PRE = (NV + NT - 1) / NT;
  constexpr bool kDB = m2l3_lds_slots<T, KS, NB>() == 2;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* wb0 = reinterpret_cast<T*>(smem_raw);
  T* wb1 = kDB ? wb0 + WLDS : wb0;

  // split levels, finest first: ns workgroups per tile, each over its own chunk
  // of the 189 offsets, writing FP64 partial sums (added in chunk order by
  // k_m2l3d_reduce)
  const int64_t blk = SPLIT ? (int64_t)blockIdx.x : xcd_remap(blockIdx.x, tt.nblocks);
  int k = SPLIT ? tt.khi : tt.klo;
  if (SPLIT)
    while (k > tt.klo && blk >= tt.off[k - 1]) --k;
  else
    while (k < tt.khi && blk >= tt.off[k + 1]) ++k;
  const int ns = SPLIT ? tt.nsplit[k] : 1;
  const int chunk = SPLIT ? (int)((blk - tt.off[k]) % ns) : 0;
  const int64_t local = SPLIT ? (blk - tt.off[k]) / ns : blk - tt.off[k];
  const int n = 1 << k;
  // blocks per parity: nxy x nxy x nz.  With nz = nxy or nxy / 2 (or nxy <= 2)
  // a 3D Morton index below nxy^2 nz decodes to x, y < nxy and z < nz, and the
  // blocks run in Morton order; with fewer z blocks (nz = nxy / 4, sixteen
  // layers per workgroup) the top Morton bits would also bound y, so there the
  // z block is the slab index and x, y run in 2D Morton order within it.
  const int nxy = n >= 8 ? n / 8 : 1;
  const int nz = n >= 2 * ZL ? n / (2 * ZL) : 1;
  const int64_t per = (int64_t)nxy * nxy * nz;
  const int par = (int)(local / per);
  const uint32_t bm = (uint32_t)(local - (int64_t)par * per);
  const int px = par & 1, py = (par >> 1) & 1, pz = par >> 2;
  int tx0, ty0, tz0;
  if (2 * nz >= nxy) {
    tx0 = 8 * (int)compact3(bm);
    ty0 = 8 * (int)compact3(bm >> 1);
    tz0 = 2 * ZL * (int)compact3(bm >> 2);
  } else {
    const uint32_t slab = bm / (uint32_t)(nxy * nxy), r = bm - slab * (uint32_t)(nxy * nxy);
    tx0 = 8 * (int)compact2(r);
    ty0 = 8 * (int)compact2(r >> 1);
    tz0 = 2 * ZL * (int)slab;
  }
  const int cs = ly.cs;
  constexpr bool kF64 = sizeof(T) == 8;
  const T* mom = (kF64 ? (const T*)a.mom64 : (const T*)a.mom32) + a.lt.off[k] * cs;
  T* loc = (kF64 ? (T*)a.loc64 : (T*)a.loc32) + a.lt.off[k] * cs;
  const T* ops = kF64 ? (const T*)a.opl64 : (const T*)a.opl32;
  const int i00 = ly.nr - 1;  // index of the degree-0 value
  static_assert(4 * KS + 1 <= kZeroRow, "the zero row is as long as a box row");
  static_assert(sizeof(vec_t) <= 16, "the zero row's alignment");
  // (global address space: a generic pointer chosen between the two would make
  // the loads flat ones)
  typedef const __attribute__((address_space(1))) T* row_t;
  typedef const __attribute__((address_space(1))) vec_t* row_vec_t;
  const row_t mom_rows = (row_t)mom, zero_row = (row_t)(const T*)g_zero_row;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int tx = tx0 + 2 * (i & 3) + px, ty = ty0 + 2 * (i >> 2) + py;
  int tzm[MB];  // the z of this lane's target in each of the wave's layers
#pragma unroll
  for (int m = 0; m < MB; ++m) tzm[m] = tz0 + 2 * (w + NW * m) + pz;
  const int xlo = px ? -3 : -2, ylo = py ? -3 : -2, zlo = pz ? -3 : -2;

  // offset q (0..215 over the 6 x 6 x 6 range; 27 of them are adjacent).  Along
  // x the window runs in steps of two, 0 2 4 1 3 5: consecutive offsets then
  // read sources of the same x parity, three quarters of them the same boxes,
  // which the L2 still holds.
  auto xstep = [](int r) { return r < 3 ? 2 * r : 2 * r - 5; };
  auto slot_of = [&](int q) -> int {
    return (xlo + xstep(q % 6) + 3) + 7 * (ylo + (q / 6) % 6 + 3) + 49 * (zlo + q / 36 + 3);
  };
  auto adjacent = [&](int q, int xl, int yl, int zl) {
    const int dx = xl + xstep(q % 6), dy = yl + (q / 6) % 6, dz = zl + q / 36;
    return dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
  };
  auto next_q = [&](int q) {
    do ++q;
    while (q < 216 && adjacent(q, xlo, ylo, zlo));
    return q;
  };
  auto nth_q = [&](int m) {  // the m-th (from 0) offset of the list, 216 past its end
    int q = -1;
    for (int e = 0; e <= m; ++e) q = next_q(q);
    return q;
  };
  const int q_stop = SPLIT ? nth_q((chunk + 1) * 189 / ns) : 216;
  // FP32: each offset's contribution is formed in the MFMA accumulators and
  // added into FP64 sums (the 189-offset sum is not left to FP32 rounding).
  acc_t acc[MB][NB];
  double sum[MB][NB][4];
  double b0p[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    b0p[m] = 0.0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      acc[m][nb] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[m][nb][r] = 0.0;
    }
  }

  // Operator of offset qq into LDS, lane-major as in memory (kDB: straight to
  // LDS, no registers; else through registers, fetched early and stored late).
  vec_t pre[kDB ? 1 : PRE];
  auto fetch = [&](int qq, T* buf) {
    const vec_t* W = reinterpret_cast<const vec_t*>(ops + (size_t)slot_of(qq) * WGLB);
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int e0 = NT * u + 64 * w, e = e0 + lane;
      if constexpr (kDB) {
        if ((u + 1) * NT <= NV || e < NV) lds_copy16(W + e, buf + (size_t)e0 * VW);
      } else {
        pre[u] = W[e < NV ? e : NV - 1];
      }
    }
  };
  // `newer`: loads issued after the copies that need not have arrived.  Right only
  // while at least that many loads stay behind the copies in issue order: fetch,
  // which issues the copies, stands before contract, whose scheduling barriers
  // keep each reload in its step, and every layer's last part and degree-0
  // value are reloaded there; neither may be moved across a barrier.
  auto settle = [&](T* buf, int newer) {
    if constexpr (kDB) {
      lds_copy_wait(newer);
    } else {
#pragma unroll
      for (int u = 0; u < PRE; ++u) {
        const int e = (tid + NT * u) * VW;
        if (e < WGLB) *reinterpret_cast<vec_t*>(buf + e) = pre[u];
      }
    }
  };
  // Source rows of offset qq for this lane's targets (the zero row outside the
  // grid).  The y and z parts of the box index change every sixth offset only.
  uint32_t yz[MB];
  bool yzok[MB];
  int qyz = -1;
  auto find_rows = [&](int qq, row_t (&row)[MB]) {
    if (qq / 6 != qyz) {  // (uniform)
      qyz = qq / 6;
      const int sy = ty + ylo + qyz % 6, dz = zlo + qyz / 6;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int sz = tzm[m] + dz;
        yzok[m] = sy >= 0 && sy < n && sz >= 0 && sz < n && tx < n && ty < n && tzm[m] < n;
        yz[m] = (spread3((uint32_t)sy) << 1) | (spread3((uint32_t)sz) << 2);
      }
    }
    const int sx = tx + xlo + xstep(qq % 6);
    const bool xok = sx >= 0 && sx < n;
    const uint32_t xs = spread3((uint32_t)sx);
#pragma unroll
    for (int m = 0; m < MB; ++m)
      row[m] = xok && yzok[m] ? mom_rows + (int64_t)(xs | yz[m]) * cs : zero_row;
  };
  // Values s0 .. s0 + RW - 1 of this lane's part of a row (one load).
  constexpr int RW = (KS * sizeof(T)) % 16 == 0 ? VW : 1;
  auto load_part = [&](const row_t (&row)[MB], int s0, T (&av)[MB][KS]) {
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      if constexpr (RW == 1) {
        av[m][s0] = row[m][g * KS + s0];
      } else {
        const vec_t v = *(row_vec_t)(row[m] + g * KS + s0);
#pragma unroll
        for (int c = 0; c < RW; ++c) av[m][s0 + c] = v[c];
      }
    }
  };
  // The products of the rows av, a0 with the operator in Wl, step by step: the
  // NB output blocks of a step follow each other, on independent accumulators,
  // while the next step's operator values are on their way from LDS (left to
  // itself the compiler read them just before their use and waited: 0.64 of
  // the matrix cores' time).  RELOAD: a part of the rows is dead after its last
  // step, and the next offset's takes its registers.
  auto contract = [&](auto reload, const T* Wl, T (&av)[MB][KS], T (&a0)[MB],
                      const row_t (&row)[MB]) {
    constexpr bool kReload = decltype(reload)::value;
    constexpr acc_t zero = {0, 0, 0, 0};
    const T* R = Wl + (size_t)NB * (KS + 1) * 64;
    T wv[2][NB + 1];  // a step's operator values and its degree-0 output weight
    auto read = [&](int s, T (&d)[NB + 1]) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) d[nb] = Wl[(nb * (KS + 1) + s) * 64 + lane];
      d[NB] = s < KS ? R[s * 64 + lane] : R[KS * 64];
    };
    T b0o[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) b0o[m] = (T)0;
    read(0, wv[0]);
#pragma unroll
    for (int s = 0; s <= KS; ++s) {  // (step KS: the degree-0 input, K = 1, lane group 0)
      if (s < KS) read(s + 1, wv[(s + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          acc[m][nb] = Mfma16x<T>::op(s < KS ? av[m][s < KS ? s : 0] : g == 0 ? a0[m] : (T)0,
                                      wv[s & 1][nb], s == 0 && !kF64 ? zero : acc[m][nb]);
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        if (s < KS)
          b0o[m] = fma(wv[s & 1][NB], av[m][s < KS ? s : 0], b0o[m]);
        else if (g == 0)
          b0o[m] = fma(wv[s & 1][NB], a0[m], b0o[m]);  // degree 0 -> degree 0
      }
      if constexpr (kReload) {
        if (s < KS && s % RW == RW - 1) load_part(row, s - RW + 1, av);
        if (s == KS)
#pragma unroll
          for (int m = 0; m < MB; ++m) a0[m] = row[m][i00];
      }
    }
#pragma unroll
    for (int m = 0; m < MB; ++m) b0p[m] += (double)b0o[m];
    if constexpr (!kF64) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[m][nb][r] += (double)acc[m][nb][r];
    }
  };

  int q = SPLIT ? nth_q(chunk * 189 / ns) : next_q(-1);
  row_t row[MB];
  T av[MB][KS], a0[MB];
  fetch(q, wb0);
  find_rows(q, row);
#pragma unroll
  for (int s = 0; s < KS; s += RW) load_part(row, s, av);
#pragma unroll
  for (int m = 0; m < MB; ++m) a0[m] = row[m][i00];
  settle(wb0, 0);
  __syncthreads();
  if constexpr (kDB) {
    T* cur = wb0;
    T* nxt = wb1;
    for (;;) {
      // past the last offset a repeat of it, never used: the same loads and
      // copies are in flight on every path
      const int qn = next_q(q);
      const bool more = qn < q_stop;
      fetch(more ? qn : q, nxt);
      find_rows(more ? qn : q, row);
      contract(std::true_type{}, cur, av, a0, row);
      static_assert(KS / RW + 1 >= 2, "two reloads a layer behind the copies");
      settle(nxt, 2 * MB);
      __syncthreads();
      if (!more) break;
      T* t = cur;
      cur = nxt;
      nxt = t;
      q = qn;
    }
  } else {
    for (;;) {
      const int qn = next_q(q);
      const bool more = qn < q_stop;
      fetch(more ? qn : q, wb0);
      find_rows(more ? qn : q, row);
      contract(std::true_type{}, wb0, av, a0, row);
      if (!more) break;
      __syncthreads();  // every wave done with the one buffer
      settle(wb0, 0);
      __syncthreads();
      q = qn;
    }
  }
  const int nout = ly.nr - 1;
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    double b0 = b0p[m];
    b0 += __shfl_xor(b0, 16, 64);
    b0 += __shfl_xor(b0, 32, 64);
    const int tz = tzm[m];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ci = crow3<T>(r, g);
      const int gx = tx0 + 2 * (ci & 3) + px, gy = ty0 + 2 * (ci >> 2) + py;
      // the C rows of this lane belong to the wave's layer (all lanes share tz)
      if (gx < n && gy < n && tz < n) {
        const int64_t bx = (int64_t)(spread3(gx) | (spread3(gy) << 1) | (spread3(tz) << 2));
        if constexpr (SPLIT) {
          double* pdst = a.m2l_part + (tt.pbase[k] + ((int64_t)chunk << (3 * k)) + bx) * cs;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const int j = 16 * nb + i;
            if (j < nout) pdst[j] = kF64 ? (double)acc[m][nb][r] : sum[m][nb][r];
          }
        } else {
          T* dst = loc + bx * cs;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const int j = 16 * nb + i;
            if (j < nout) dst[j] = kF64 ? (T)acc[m][nb][r] : (T)sum[m][nb][r];
          }
        }
      }
    }
    if (g == 0 && tx < n && ty < n && tz < n) {
      const int64_t bx = (int64_t)(spread3(tx) | (spread3(ty) << 1) | (spread3(tz) << 2));
      if constexpr (SPLIT)
        a.m2l_part[(tt.pbase[k] + ((int64_t)chunk << (3 * k)) + bx) * cs + i00] = b0;
      else
        loc[bx * cs + i00] = (T)b0;
    }
  }
}

// loc[b][j] = sum over chunks c (in order) of the partial rows of level k
template <typename T>
__global__ void k_m2l3d_reduce(const double* part, T* loc, int64_t nbox, int cs, int nr, int ns,
                               int64_t pbase) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nbox * nr) return;
  const int64_t b = g / nr;
  const int j = (int)(g - b * nr);
  double s = 0.0;
  for (int c = 0; c < ns; ++c) s += part[(pbase + c * nbox + b) * cs + j];
  loc[b * cs + j] = (T)s;
}

template <typename T, int KS, int NB, int MB, int NW, bool SPLIT>
static void m2l3_launch(const FmmArgs& a, const M2l3Tiles& tt, const M2lLayout& ly,
                        hipStream_t st) {
  const size_t lds = (size_t)m2l3_lds_slots<T, KS, NB>() * (64 * (NB * (KS + 1) + KS) + 4) *
                     sizeof(T);
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_m2l3d_mfma<T, KS, NB, MB, NW, SPLIT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_m2l3d_mfma<T, KS, NB, MB, NW, SPLIT>), dim3(tt.nblocks), dim3(64 * NW), lds,
                     st, a, tt, ly);
  if (SPLIT)
    for (int k = tt.klo; k <= tt.khi; ++k) {
      const int64_t nbox = (int64_t)1 << (3 * k), cnt = nbox * ly.nr;
      T* loc = (sizeof(T) == 8 ? (T*)a.loc64 : (T*)a.loc32) + a.lt.off[k] * ly.cs;
      hipLaunchKernelGGL(k_m2l3d_reduce<T>, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st,
                         a.m2l_part, loc, nbox, ly.cs, ly.nr, tt.nsplit[k], tt.pbase[k]);
    }
}

// Tile variant mb: 4 mb layers of 16 targets per workgroup (mb = 4, FP32 only:
// eight waves of two layers).  FP64, mb = 1: eight waves of one layer where the
// levels run unsplit: an operator pair of order 8 fills the LDS of a CU, and one
// workgroup of four waves left each SIMD a single wave, which nothing overlaps
// (300,007 particles, level 5, order 8: 2.17 -> 2.00 ms a step).
template <typename T, int KS, int NB, bool SPLIT>
static void m2l3_mb(const FmmArgs& a, const M2l3Tiles& tt, const M2lLayout& ly, hipStream_t st) {
  if constexpr (KS == 32) {  // K = N = 128: one layer per wave, one workgroup per CU
    m2l3_launch<T, KS, NB, 1, 4, SPLIT>(a, tt, ly, st);
  } else if constexpr (sizeof(T) == 8) {
    if (a.m2l_mb == 2)
      m2l3_launch<T, KS, NB, 2, 4, SPLIT>(a, tt, ly, st);
    else
      m2l3_launch<T, KS, NB, 1, SPLIT ? 4 : 8, SPLIT>(a, tt, ly, st);
  } else {
    if (a.m2l_mb == 4)
      m2l3_launch<T, KS, NB, 2, 8, SPLIT>(a, tt, ly, st);
    else if (a.m2l_mb == 2)
      m2l3_launch<T, KS, NB, 2, 4, SPLIT>(a, tt, ly, st);
    else
      m2l3_launch<T, KS, NB, 1, 4, SPLIT>(a, tt, ly, st);
  }
}

template <typename T, int KS, int NB>
static void m2l3_split(const FmmArgs& a, const M2l3Tiles& tt, const M2lLayout& ly, bool split,
                       hipStream_t st) {
  if (split)
    m2l3_mb<T, KS, NB, true>(a, tt, ly, st);
  else
    m2l3_mb<T, KS, NB, false>(a, tt, ly, st);
}

bool m2l3d_variant_ok(int mb, bool fp64) { return mb == 1 || mb == 2 || (mb == 4 && !fp64); }

void launch_m2l3d(const FmmArgs& a, bool fp64, hipStream_t st) {
  if (a.khi < a.klo) return;
  const M2lLayout ly = a.basis ? points3d_layout_n(a.p) : m2l3d_layout(order_bucket3(a.p));
  const int mb = ly.kpad == 128 ? 1 : m2l3d_variant_ok(a.m2l_mb, fp64) ? a.m2l_mb : 1;
  FmmArgs am = a;
  am.m2l_mb = mb;
  // Levels 2..4 have 8, 8 and (of four layers) 64 tiles: their own launch splits
  // each tile's offsets over several workgroups; the finer levels, whose tiles
  // are multiples of the 256 CUs, run unsplit (level 5 in FP64: two even rounds
  // where its 512 and level 4's 64 tiles made three).
  const int ksplit = a.m2l_part ? std::min(a.khi, kM2l3SplitLevel) : a.klo - 1;
  for (int part = 0; part < 2; ++part) {
    const bool split = part == 0;
    // same-parity z-layers per block (m2l3_mb)
    const int zl = fp64 && mb == 1 && !split && ly.kpad < 128 ? 8 : 4 * mb;
    const int klo = split ? a.klo : std::max(a.klo, ksplit + 1);
    const int khi = split ? ksplit : a.khi;
    if (khi < klo) continue;
    M2l3Tiles tt{};
    tt.klo = klo;
    tt.khi = khi;
    int64_t t = 0;
    for (int i = 0; i <= khi - klo; ++i) {
      const int k = split ? khi - i : klo + i;
      tt.off[k] = t;
      const int n = 1 << k;
      const int64_t nxy = n >= 8 ? n / 8 : 1, nz = n >= 2 * zl ? n / (2 * zl) : 1;
      tt.nsplit[k] = split ? m2l3_split_of(k) : 1;
      tt.pbase[k] = split ? m2l3_split_row(k) : 0;
      t += 8 * nxy * nxy * nz * tt.nsplit[k];
    }
    if (!split) tt.off[khi + 1] = t;
    tt.nblocks = t;
    if (a.basis && ly.kpad == 128) {  // 125 point charges: K = N = 128
      if (fp64)
        m2l3_split<double, 32, 8>(am, tt, ly, split, st);
      else
        m2l3_split<float, 32, 8>(am, tt, ly, split, st);
    } else if (a.basis) {  // up to 64 point charges: K = N = 64
      if (fp64)
        m2l3_split<double, 16, 4>(am, tt, ly, split, st);
      else
        m2l3_split<float, 16, 4>(am, tt, ly, split, st);
    } else if (ly.p == 4) {
      if (fp64)
        m2l3_split<double, 6, 2>(am, tt, ly, split, st);
      else
        m2l3_split<float, 6, 2>(am, tt, ly, split, st);
    } else {
      if (fp64)
        m2l3_split<double, 20, 5>(am, tt, ly, split, st);
      else
        m2l3_split<float, 20, 5>(am, tt, ly, split, st);
    }
  }
}

}  // namespace sffmm

// HIP kernels of the extraction path (gfx950), generic over the order N.
//
// Per element (Deville, Fischer & Mund 2002, ch. 4; Hunt, Wray & Moin 1988):
//   reference derivatives  f_r = D f (along i), f_s (along j), f_t (along k)
//   Jacobian               J = d(x,y,z)/d(r,s,t), J^-1 = adj(J) / det J
//   chain rule             A_ij = sum_a (d u_i / d r_a) (J^-1)_{a j}
//   Q = -tr(A^2)/2 (equal to Hunt's (|Omega|^2 - |S|^2)/2), |omega|.
// Marching cubes over the N^3 sub-hexahedra (Lorensen & Cline 1987) with a
// count / exclusive-scan / emit compaction.
//
// Every 1-D contraction subtracts the line's first value before applying D:
// sum_m D_im (f_m - f_0) equals (D f)_i exactly in exact arithmetic because
// D annihilates constants, but it removes the large common offset of
// coordinates and velocities before rounding.  In FP32 this is what keeps
// the Jacobian of a small element at a large absolute position accurate.
#include <cmath>
#include <cstdint>
#include <mutex>
#include <unordered_map>
#include <type_traits>

#include <hip/hip_ext.h>

#include "sem_internal.h"

namespace sem {
namespace {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ T neg_inf() { return -__builtin_huge_val(); }
template <>
__device__ __forceinline__ float neg_inf<float>() { return -__builtin_huge_valf(); }
template <typename T>
__device__ __forceinline__ T pos_inf() { return -neg_inf<T>(); }

// One DPP move of a 32- or 64-bit value (a 64-bit value as its two halves
// under the same control).  With every row enabled each lane reads a lane of
// its own row; lanes of rows that ROWS leaves out keep `fill`.
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_move(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit values");
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(
        T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
  } else {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  }
}
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_move(T v, T fill) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit values");
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, fill),
                                                             __builtin_bit_cast(int, v), CTRL,
                                                             ROWS, 0xf, false));
  } else {
    const uint64_t u = __builtin_bit_cast(uint64_t, v), f = __builtin_bit_cast(uint64_t, fill);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(
        (int)(uint32_t)f, (int)(uint32_t)u, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(
        (int)(uint32_t)(f >> 32), (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  }
}

// Minimum and maximum over the wave, left in lane 63 (other lanes hold
// partial results), by DPP moves only: within quads (quad_perm [1,0,3,2],
// [2,3,0,1]), half rows (row_half_mirror), rows (row_mirror), then lane 15
// of rows 0 and 2 into rows 1 and 3 (row_bcast:15) and lane 31 into rows 2
// and 3 (row_bcast:31).  No NaN may reach it: callers map NaN to -inf.
template <typename T>
__device__ __forceinline__ void wave_minmax(T& mn, T& mx) {
  const T pinf = pos_inf<T>(), ninf = neg_inf<T>();
  mn = fmin(mn, dpp_move<0xb1>(mn));
  mx = fmax(mx, dpp_move<0xb1>(mx));
  mn = fmin(mn, dpp_move<0x4e>(mn));
  mx = fmax(mx, dpp_move<0x4e>(mx));
  mn = fmin(mn, dpp_move<0x141>(mn));
  mx = fmax(mx, dpp_move<0x141>(mx));
  mn = fmin(mn, dpp_move<0x140>(mn));
  mx = fmax(mx, dpp_move<0x140>(mx));
  mn = fmin(mn, dpp_move<0x142, 0xa>(mn, pinf));
  mx = fmax(mx, dpp_move<0x142, 0xa>(mx, ninf));
  mn = fmin(mn, dpp_move<0x143, 0xc>(mn, pinf));
  mx = fmax(mx, dpp_move<0x143, 0xc>(mx, ninf));
}
// Inclusive sum of a 64-bit value over the lanes up to this one (lane 63:
// the wave's sum), by DPP moves of both halves: row shifts right by 1, 2,
// 4, 8 (lanes without a source add 0), then lane 15 of rows 0 and 2 into
// rows 1 and 3 (row_bcast:15) and lane 31 into rows 2 and 3
// (row_bcast:31).  Every lane of the wave must be active.
__device__ __forceinline__ int64_t wave_inclusive_sum(int64_t v) {
  const int64_t z = 0;
  v += dpp_move<0x111, 0xf>(v, z);
  v += dpp_move<0x112, 0xf>(v, z);
  v += dpp_move<0x114, 0xf>(v, z);
  v += dpp_move<0x118, 0xf>(v, z);
  v += dpp_move<0x142, 0xa>(v, z);
  v += dpp_move<0x143, 0xc>(v, z);
  return v;
}

// Block-wide (min, max) of per-thread values; result valid in every thread.
template <typename T, int THREADS>
__device__ __forceinline__ void block_minmax(T& mn, T& mx, T* scratch /*2*THREADS/64*/) {
  constexpr int W = THREADS / 64;
  wave_minmax(mn, mx);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) {
    scratch[w] = mn;
    scratch[W + w] = mx;
  }
  __syncthreads();
  mn = scratch[0];
  mx = scratch[W];
#pragma unroll
  for (int i = 1; i < W; ++i) {
    mn = scratch[i] < mn ? scratch[i] : mn;
    mx = scratch[W + i] > mx ? scratch[W + i] : mx;
  }
  __syncthreads();
}

// Block-wide sum of a 64-bit value; result valid in every thread.
template <int THREADS>
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t* scratch /*THREADS/64*/) {
  constexpr int W = THREADS / 64;
  v = wave_inclusive_sum(v);
  if ((threadIdx.x & 63) == 63) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < W; ++i) s += scratch[i];
  __syncthreads();
  return s;
}

// Exclusive block scan of a 64-bit value (THREADS multiple of 64).
template <int THREADS>
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* scratch,
                                                        int64_t* total) {
  constexpr int W = THREADS / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t inc = wave_inclusive_sum(v);
  if (lane == 63) scratch[w] = inc;
  __syncthreads();
  int64_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    before += (i < w) ? scratch[i] : 0;
    all += scratch[i];
  }
  __syncthreads();
  *total = all;
  return before + inc - v;
}

// Coefficient type of the line sums: FP64 with the FP64 D for FP64 fields;
// for FP32 fields FP32 with the FP32-rounded D up to order kF32SumOrder
// (within the FP32 bound there; FP32 FMAs need no conversions and half the
// registers), FP64 above it.
template <int N, typename T>
using coef_t = typename std::conditional<std::is_same<T, float>::value && f32_line_sums(N),
                                         float, double>::type;

// 1-D contractions at node (i, j, k) of a tile in LDS, line-shifted, summed
// in the coefficient type C.
template <int N, typename T, typename C>
__device__ __forceinline__ void ref_derivs(const T* __restrict__ f,
                                           const C* __restrict__ d, int i, int j, int k,
                                           T& fr, T& fs, T& ft) {
  constexpr int P = N + 1;
  const T* lr = f + (k * P + j) * P;   // line along i
  const T* ls = f + k * P * P + i;     // along j, stride P
  const T* lt = f + j * P + i;         // along k, stride P^2
  const C r0 = lr[0], s0 = ls[0], t0 = lt[0];
  C ar = C(0), as = C(0), at = C(0);
#pragma unroll
  for (int m = 1; m < P; ++m) {
    ar = fma(d[i * P + m], (C)lr[m] - r0, ar);
    as = fma(d[j * P + m], (C)ls[m * P] - s0, as);
    at = fma(d[k * P + m], (C)lt[m * P * P] - t0, at);
  }
  fr = (T)ar;
  fs = (T)as;
  ft = (T)at;
}

template <typename T>
struct InvJac {
  T rx, ry, rz, sx, sy, sz, tx, ty, tz;
};

// J^-1 = adj(J) / det J; returns det J > 0.
template <typename T>
__device__ __forceinline__ bool invert_jacobian(T xr, T xs, T xt, T yr, T ys, T yt, T zr,
                                                T zs, T zt, InvJac<T>& k) {
  const T c0 = ys * zt - yt * zs;
  const T c1 = yt * zr - yr * zt;
  const T c2 = yr * zs - ys * zr;
  const T det = xr * c0 + xs * c1 + xt * c2;
  // FP32: the hardware reciprocal (1 ulp) instead of the correctly rounded
  // division sequence, far inside the FP32 bound of the derived fields
  T inv;
  if constexpr (std::is_same<T, float>::value) inv = __builtin_amdgcn_rcpf(det);
  else inv = T(1) / det;
  k.rx = c0 * inv;
  k.ry = (xt * zs - xs * zt) * inv;
  k.rz = (xs * yt - xt * ys) * inv;
  k.sx = c1 * inv;
  k.sy = (xr * zt - xt * zr) * inv;
  k.sz = (xt * yr - xr * yt) * inv;
  k.tx = c2 * inv;
  k.ty = (xs * zr - xr * zs) * inv;
  k.tz = (xr * ys - xs * yr) * inv;
  return det > T(0);
}

// 1 / x from the hardware estimate and two Newton steps (an ulp at most; none
// of 8,388,608 random determinants differed from the correctly rounded
// division, which adds range scaling and a final correction and takes about
// 1 % longer in Q of orders 6 to 9); x outside [2^-1000, 2^1000] in magnitude,
// 0 and NaN take the division (a branch that a wave skips unless one of its
// lanes needs it).
__device__ __forceinline__ double recip_refined(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  const double a = fabs(x);
  const bool out = !(a >= 0x1p-1000 && a <= 0x1p+1000);
  if (__builtin_amdgcn_ballot_w64(out) != 0) {   // wave-uniform: skipped as a whole
    double xx = x;
    asm volatile("" : "+v"(xx));   // keeps the division from being hoisted out
    if (out) r = 1.0 / xx;
  }
  return r;
}

// sqrt(x) from the hardware estimate of 1 / sqrt(x), one Goldschmidt step and
// a Newton correction of the root (within an ulp or two); x outside
// [2^-1000, 2^1000], 0 and NaN take the library root.
__device__ __forceinline__ double sqrt_refined(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  double sq = x * r, hr = 0.5 * r;
  const double e = fma(-hr, sq, 0.5);
  sq = fma(sq, e, sq);
  hr = fma(hr, e, hr);
  sq = fma(fma(-sq, sq, x), hr, sq);
  const bool out = !(x >= 0x1p-1000 && x <= 0x1p+1000);
  if (__builtin_amdgcn_ballot_w64(out) != 0) {   // wave-uniform: skipped as a whole
    double xx = x;
    asm volatile("" : "+v"(xx));   // keeps the root from being hoisted out
    if (out) sq = sqrt(xx);
  }
  return sq;
}

// Root of |omega|^2: FP32 takes the hardware square root (v_sqrt_f32, within
// 1 ulp; the correctly rounded form adds range scaling and a correction of
// the last bit, a dozen instructions per node), FP64 the refined estimate
// above.
__device__ __forceinline__ float vort_root(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double vort_root(double x) { return sqrt_refined(x); }

// Coefficient tables (D, its even-odd halves) are read through the
// constant address space: the index is wave-uniform, so every read is a
// scalar load whatever stores precede it in the kernel.
using const_f64 = const __attribute__((address_space(4))) double*;
using const_f32 = const __attribute__((address_space(4))) float*;
__device__ __forceinline__ double coef(const double* p, int idx) {
  return ((const_f64)p)[idx];
}
__device__ __forceinline__ float coef(const float* p, int idx) {
  return ((const_f32)p)[idx];
}

// All P outputs of one line (line-shifted, summed in the coefficient type C,
// as ref_derivs) through the even-odd halves of D stored after D itself: an output pair (i, P-1-i)
// costs P multiply-adds instead of 2 (P - 1).
template <int P, typename T, typename C>
__device__ __forceinline__ void line_deriv_all(const C* __restrict__ d, const T (&g)[P],
                                               T (&out)[P]) {
  constexpr int H = P / 2, NE = (P + 1) / 2;
  const C* a = d + P * P;
  const C* b = a + NE * NE;
  const C g0 = g[0];
  C hv[P], e[NE], o[H > 0 ? H : 1];
#pragma unroll
  for (int m = 1; m < P; ++m) hv[m] = (C)g[m] - g0;
  // hv[0] = 0: e[0] = hv[P-1], o[0] = -hv[P-1] (written out, since 0 + x
  // does not fold for a possibly negative zero x)
  if constexpr (H > 0) {
    e[0] = hv[P - 1];
    o[0] = -hv[P - 1];
  }
#pragma unroll
  for (int m = 1; m < H; ++m) {
    e[m] = hv[m] + hv[P - 1 - m];
    o[m] = hv[m] - hv[P - 1 - m];
  }
  if constexpr (P % 2 == 1) e[H] = hv[H];   // P odd: H >= 1
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    C pe = coef(a, NE * i) * e[0];
#pragma unroll
    for (int m = 1; m < NE; ++m) pe = fma(coef(a, NE * i + m), e[m], pe);
    C ro = C(0);
    if constexpr (H > 0) ro = coef(b, H * i) * o[0];
#pragma unroll
    for (int m = 1; m < H; ++m) ro = fma(coef(b, H * i + m), o[m], ro);
    out[i] = (T)(ro + pe);
    if (P - 1 - i != i) out[P - 1 - i] = (T)(ro - pe);
  }
}

// Sum over the 16 lanes of each row of the wave, by DPP row shifts (lanes
// shifted in from outside the row read 0): lane 15 of the row ends with the
// row's sum (the others with partial sums).  Four VALU operations, no LDS.
__device__ __forceinline__ uint32_t row_sum16(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
  return v;
}

// Sum over each quad of lanes, in all of them (quad_perm [1,0,3,2], [2,3,0,1]).
__device__ __forceinline__ uint32_t quad_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, false);
  return v;
}

// Sum over the wave, left in lane 63 (other lanes hold partial sums): the
// row sums above, then lane 15 of rows 0 and 2 added into rows 1 and 3
// (row_bcast:15) and lane 31 into rows 2 and 3 (row_bcast:31); lanes of the
// rows a row mask leaves out add 0.  Every lane of the wave must be active.
__device__ __forceinline__ uint32_t wave_sum_to63(uint32_t v) {
  v = row_sum16(v);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Where a Q kernel also counts each isovalue's triangles and active cells per
// element (the count pass of the isosurface, fused).
template <typename T>
struct CountSink {
  int n_iso;
  IsoList<T> iso;
  const uint8_t* ntri;     // [256] triangles per case
  int32_t* cnt;            // [n_iso][n_elem], packed (below)
  int64_t* active;         // [n_iso] active-cell totals (may be NULL): set to 0
                           // here, summed by the scan's first kernel
  int64_t n_elem;
};

// A count slot holds an element's triangles (at most 5 x 729) and, from bit
// 16 on, its active cells (at most 729).  The totals of the active cells
// come from the scan, which reads the slots anyway: one atomic per element
// and isovalue on the n_iso totals instead bound the count kernels (all of
// them hit one cache line; 155,344 order-2 elements at three isovalues took
// 650 us, the Q kernel among it 76 us).
__device__ __forceinline__ int slot_tris(int32_t v) { return v & 0xffff; }
__device__ __forceinline__ int slot_active(int32_t v) { return v >> 16; }
__device__ __forceinline__ void clear_active(int64_t* active, int n_iso) {
  if (active && blockIdx.x == 0 && (int)threadIdx.x < n_iso) active[threadIdx.x] = 0;
}

#include "sem_lines.h"

// ---------------------------------------------------------------------------
// element tiles fetched by direct global->LDS loads (emission and counts)
// ---------------------------------------------------------------------------
//
// A tile is fetched with global_load_lds (16 bytes per lane, 1 KiB per wave
// instruction, fully coalesced, no registers held while the data is in
// flight).  A lane may fetch any 16-byte chunk (two neighbouring i of an
// order-7 FP64 element) and it lands at LDS slot base + lane, so the chunk
// placement is chosen freely:
//   slot(k, j, ip) = 4 (8k + (j ^ (k & 1))) + (ip ^ ((j >> 1) & 3)),
// i.e. rows j <-> j^1 swapped in odd slabs and the four chunks of a row
// rotated by j >> 1, which spreads reads along any direction over the banks.

namespace dma7 {
__device__ __forceinline__ constexpr int slot(int k, int j, int ip) {
  return 4 * (8 * k + (j ^ (k & 1))) + (ip ^ ((j >> 1) & 3));
}
__device__ __forceinline__ constexpr int at(int i, int j, int k) {
  return 2 * slot(k, j, i >> 1) + (i & 1);
}
}  // namespace dma7

struct DmaNode {
  __device__ __forceinline__ int operator()(int i, int j, int k) const {
    return dma7::at(i, j, k);
  }
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// One 16-byte direct load per lane into LDS at lds + 16 * lane, issued as
// inline assembly: the compiler then keeps no record of the LDS write and
// inserts no waits of its own for it (after LDS lowering it cannot tell the
// tiles apart and would wait for every load in flight before any tile
// read).  Every consumer waits explicitly (s_waitcnt on vmcnt, then a
// barrier) before reading the tile.
__device__ __forceinline__ void lds_load16(const double* src, double* lds) {
  const uint32_t m0 =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)lds);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(src), "s"(m0)
               : "memory", "m0");
}

// Fetch one 4 KiB tile: wave h issues the chunk groups h and h + 2.
__device__ __forceinline__ void dma_tile(const double* __restrict__ src, double* raw, int h,
                                         int lane) {
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    const int part = 2 * pp + h;
    const int s = 64 * part + lane;
    const int row = s >> 2, k = row >> 3, j = (row & 7) ^ (k & 1);
    const int ip = (s & 3) ^ ((j >> 1) & 3);
    lds_load16(src + 2 * (ip + 4 * j + 32 * k), raw + 128 * part);
  }
}

// s_waitcnt immediate (vmcnt in bits 3:0 and 15:14, expcnt at its maximum,
// lgkmcnt 0): wait until at most n vector-memory operations and no LDS
// operation of this wave are outstanding.
constexpr int waitcnt_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70; }

// Barrier after an explicit wait: a plain s_barrier (the compiler-level
// memory clobbers keep LDS accesses on their side of it).  __syncthreads()
// would add a workgroup fence, which must also wait for every direct load
// still in flight.
__device__ __forceinline__ void barrier_after_wait() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------------------
// marching cubes
// ---------------------------------------------------------------------------

// low corner and axis of each cube edge (edge id = 4*axis + rank)
// Low corner of edge e, packed as 4-bit fields (edge 0 lowest): edges
// 0..3 run along r from corners 0, 2, 4, 6; edges 4..7 along s from 0, 1,
// 4, 5; edges 8..11 along t from 0, 1, 2, 3.  The axis is e >> 2.  Decoded
// with a shift instead of a table, so the vertex loop reads no memory for it.
constexpr uint64_t kEdgeLoPacked = 0x321054106420ull;
__device__ __forceinline__ int edge_lo(int e) { return (int)((kEdgeLoPacked >> (4 * e)) & 15); }

// Exclusive prefix over the cells of a block of the per-cell triangle counts
// nt (0..7): one ballot per bit gives the wave prefix; wave totals go through
// LDS.  Returns the thread's offset; *block_total receives the block total.
template <int TH>
__device__ __forceinline__ int block_count_prefix(int nt, int32_t* s_wave, int* block_total) {
  constexpr int W = TH / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t m0 = __ballot(nt & 1), m1 = __ballot(nt & 2), m2 = __ballot(nt & 4);
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  int pre = __popcll(m0 & lt) + 2 * __popcll(m1 & lt) + 4 * __popcll(m2 & lt);
  if (lane == 0) s_wave[wv] = __popcll(m0) + 2 * __popcll(m1) + 4 * __popcll(m2);
  __syncthreads();
  int tot = 0;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    pre += q < wv ? s_wave[q] : 0;
    tot += s_wave[q];
  }
  __syncthreads();
  *block_total = tot;
  return pre;
}

// Balanced emission of one element's triangles for one isovalue.  First
// every cell (in rounds of TH threads, cell order) records its case and
// writes one descriptor (cell << 3 | slot) per triangle into `desc` at its
// running prefix; then thread v computes vertex v of that list.  Every lane
// does the same amount of work however unevenly the triangles fall on the
// cells, and consecutive lanes write consecutive vertices.  `node(i, j, k)`
// maps a node to its index in the field tile ft, `cnode(i, j, k)` to its
// index in the coordinate arrays sx, sy, sz (a tile in LDS, or the
// element's values in global memory).  Returns the element's triangle count.
template <int N, int TH, typename T, class NodeFn, class CoordFn>
__device__ __forceinline__ int emit_element(T c, NodeFn node, CoordFn cnode,
                                            const T* __restrict__ ft,
                                            const T* __restrict__ sx, const T* __restrict__ sy,
                                            const T* __restrict__ sz,
                                            const uint8_t* __restrict__ s_ntri,
                                            const int8_t* __restrict__ s_tri,
                                            uint8_t* __restrict__ cases,
                                            uint16_t* __restrict__ desc, int32_t* s_wave,
                                            T* __restrict__ out, int64_t g0, int64_t cap,
                                            uint64_t* __restrict__ keys, int64_t key_base) {
  constexpr int P = N + 1, NC = N * N * N, ROUNDS = (NC + TH - 1) / TH;
  const int t = threadIdx.x;
  int run = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int cell = r * TH + t;
    int cs = 0, nt = 0;
    if (cell < NC) {
      const int ci = cell % N, cj = (cell / N) % N, ck = cell / (N * N);
#pragma unroll
      for (int vtx = 0; vtx < 8; ++vtx)
        cs |= (ft[node(ci + (vtx & 1), cj + ((vtx >> 1) & 1), ck + (vtx >> 2))] > c) << vtx;
      nt = s_ntri[cs];
      cases[cell] = (uint8_t)cs;
    }
    int tot;
    const int pre = block_count_prefix<TH>(nt, s_wave, &tot);
    for (int sl = 0; sl < nt; ++sl) desc[run + pre + sl] = (uint16_t)((cell << 3) | sl);
    run += tot;
  }
  __syncthreads();
  for (int vv = t; vv < 3 * run; vv += TH) {
    const int tri = vv / 3, vtx = vv - 3 * tri;
    const int64_t g = g0 + tri;
    if (g >= cap) continue;
    const int dsc = desc[tri];
    const int cell = dsc >> 3, slot = dsc & 7;
    const int cs = cases[cell];
    const int ci = cell % N, cj = (cell / N) % N, ck = cell / (N * N);
    const int edge = s_tri[(cs * kMcMaxTri + slot) * 3 + vtx];
    const int v0 = edge_lo(edge);
    const int ax = edge >> 2;
    const int a0 = ci + (v0 & 1), b0 = cj + ((v0 >> 1) & 1), c0 = ck + (v0 >> 2);
    const int a1 = a0 + (ax == 0), b1 = b0 + (ax == 1), c1 = c0 + (ax == 2);
    const int lo = node(a0, b0, c0), hi = node(a1, b1, c1);
    const int clo = cnode(a0, b0, c0), chi = cnode(a1, b1, c1);
    T* o = out + g * 9 + 3 * vtx;
    {
#pragma clang fp contract(off)
      const T f0 = ft[lo], f1 = ft[hi];
      const T tt = (c - f0) / (f1 - f0);
      o[0] = sx[clo] + tt * (sx[chi] - sx[clo]);
      o[1] = sy[clo] + tt * (sy[chi] - sy[clo]);
      o[2] = sz[clo] + tt * (sz[chi] - sz[clo]);
    }
    if (keys)
      keys[g * 3 + vtx] = (uint64_t)(key_base + a0 + P * (b0 + P * c0)) * 3u + (uint64_t)ax;
  }
  __syncthreads();
  return run;
}

// Tile index functions for emit_element.
template <int RS, int SS>
struct StridedNode {
  __device__ __forceinline__ int operator()(int i, int j, int k) const {
    return i + RS * j + SS * k;
  }
};

// ---------------------------------------------------------------------------
// device-wide exclusive scan of int32 counts into int64 offsets
// ---------------------------------------------------------------------------

constexpr int kScanThreads = 256;

// Tile sums; a tile is kScanThreads x ITEMS counts (scan_tile).  PACKED: the
// counts are slots of triangles and active cells; the active cells of the
// isovalues that the tile holds (n_elem slots each) are added to `active`.
// CT: int32_t or int64_t counts, or uint8_t flags (nonzero counts as 1).  A tile of few
// isovalues sums each over the workgroup; from kScanActive on they are added up
// in LDS (8 elements at 64 isovalues: 24 us by workgroup sums, 5 so).
constexpr int kScanActive = 4;
template <typename CT>
using scan_t = typename std::conditional<sizeof(CT) == 8, int64_t, int32_t>::type;
template <typename CT>
__device__ __forceinline__ scan_t<CT> scan_value(CT v) {
  if constexpr (sizeof(CT) == 1) return v != 0;
  else return v;
}
template <int ITEMS, bool PACKED, typename CT>
__global__ void __launch_bounds__(kScanThreads)
scan_reduce(const CT* __restrict__ cnt, int64_t count, int64_t* __restrict__ partial,
            int64_t* __restrict__ active, int64_t n_elem) {
  __shared__ int64_t sred[kScanThreads / 64];
  const int64_t start = (int64_t)blockIdx.x * (kScanThreads * ITEMS);
  scan_t<CT> v[ITEMS];
  int64_t s = 0;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t idx = start + r * kScanThreads + threadIdx.x;
    v[r] = idx < count ? scan_value(cnt[idx]) : 0;
    // packed: both sums at once (a tile's stay below 2^24)
    if constexpr (PACKED) s += (int64_t)slot_tris(v[r]) | ((int64_t)slot_active(v[r]) << 32);
    else s += v[r];
  }
  s = block_sum<kScanThreads>(s, sred);
  if (threadIdx.x == 0) partial[blockIdx.x] = PACKED ? (int64_t)(uint32_t)s : s;
  if constexpr (PACKED) {
    if (!active) return;
    const int64_t end = start + kScanThreads * ITEMS < count ? start + kScanThreads * ITEMS : count;
    const int64_t i0 = start / n_elem, i1 = (end - 1) / n_elem;
    if (i1 - i0 >= kScanActive) {   // a few elements at many isovalues
      __shared__ uint32_t s_act[SEM_MAX_ISO];
      if (threadIdx.x < SEM_MAX_ISO) s_act[threadIdx.x] = 0;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const uint32_t at = (uint32_t)(start - i0 * n_elem) + r * kScanThreads + threadIdx.x;
        if (slot_active(v[r]) != 0)
          atomicAdd(&s_act[at / (uint32_t)n_elem], (uint32_t)slot_active(v[r]));
      }
      __syncthreads();
      if ((int64_t)threadIdx.x <= i1 - i0 && s_act[threadIdx.x] != 0)
        atomicAdd((unsigned long long*)&active[i0 + threadIdx.x],
                  (unsigned long long)s_act[threadIdx.x]);
      return;
    }
    for (int64_t i = i0; i <= i1; ++i) {
      int64_t a = s >> 32;
      if (i0 != i1) {
        a = 0;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
          const int64_t idx = start + r * kScanThreads + threadIdx.x;
          if (idx >= i * n_elem && idx < (i + 1) * n_elem) a += slot_active(v[r]);
        }
        a = block_sum<kScanThreads>(a, sred);
      }
      if (threadIdx.x == 0 && a)
        atomicAdd((unsigned long long*)&active[i], (unsigned long long)a);
    }
  }
}

__global__ void __launch_bounds__(1024)
scan_partials(int64_t* __restrict__ partial, int64_t nb) {
  __shared__ int64_t sred[1024 / 64];
  int64_t running = 0;
  for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
    const int64_t idx = c0 + threadIdx.x;
    const int64_t v = idx < nb ? partial[idx] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<1024>(v, sred, &total);
    if (idx < nb) partial[idx] = running + ex;
    running += total;
  }
  if (threadIdx.x == 0) partial[nb] = running;
}

// Tiles' exclusive offsets.  FOLD: partial holds the tiles' sums, not yet
// scanned (nb <= kScanFold), and each workgroup adds up the sums of the
// tiles before it, which saves the one-workgroup scan of the partials.
constexpr int64_t kScanFold = 1024;
template <bool FOLD, int ITEMS, bool PACKED, typename CT>
__global__ void __launch_bounds__(kScanThreads)
scan_apply(const CT* __restrict__ cnt, int64_t count, const int64_t* __restrict__ partial,
           int64_t nb, int64_t* __restrict__ offs) {
  __shared__ int64_t sred[kScanThreads / 64];
  const int64_t start =
      (int64_t)blockIdx.x * (kScanThreads * ITEMS) + (int64_t)threadIdx.x * ITEMS;
  scan_t<CT> v[ITEMS];
  int64_t s = 0;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    v[r] = (start + r < count) ? scan_value(cnt[start + r]) : 0;
    if constexpr (PACKED) v[r] = slot_tris(v[r]);
    s += v[r];
  }
  int64_t base;
  if constexpr (FOLD) {
    int64_t b = 0;
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) b += partial[i];
    base = block_sum<kScanThreads>(b, sred);
  } else {
    base = partial[blockIdx.x];
  }
  int64_t total;
  int64_t run = base + block_exclusive_scan<kScanThreads>(s, sred, &total);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    if (start + r < count) offs[start + r] = run;
    run += v[r];
  }
  if (blockIdx.x == nb - 1 && threadIdx.x == 0) offs[count] = FOLD ? base + total : partial[nb];
}

// Per-isovalue totals and the overflow flag, from the exclusive offsets
// (thread s < n_iso takes isovalue s).
template <typename T>
__device__ __forceinline__ void write_totals(int s, const int64_t* __restrict__ offs,
                                             int64_t n_elem, int n_iso,
                                             int64_t* __restrict__ tri_count,
                                             const IsoOut<T>& out, int32_t* __restrict__ status) {
  if (s < n_iso) {
    const int64_t c = offs[(int64_t)(s + 1) * n_elem] - offs[(int64_t)s * n_elem];
    tri_count[s] = c;
    if (status && out.per_iso && c > out.cap[s]) atomicOr(status, SEM_FLAG_TRI_OVERFLOW);
  }
  if (s == 0 && status && !out.per_iso && offs[(int64_t)n_iso * n_elem] > out.cap[0])
    atomicOr(status, SEM_FLAG_TRI_OVERFLOW);
}

template <typename T>
__global__ void iso_totals(const int64_t* __restrict__ offs, int64_t n_elem, int n_iso,
                           int64_t* __restrict__ tri_count, IsoOut<T> out,
                           int32_t* __restrict__ status) {
  write_totals<T>(threadIdx.x, offs, n_elem, n_iso, tri_count, out, status);
}

__global__ void fill_i64(int64_t* __restrict__ p, int n, int64_t value) {
  const int s = threadIdx.x;
  if (s < n) p[s] = value;
}

// ---------------------------------------------------------------------------
// emission from element tiles fetched by direct global->LDS loads
// ---------------------------------------------------------------------------

// Emission for N = 7, FP64: elements with triangles stage their field and
// coordinate tiles with direct loads and emit through emit_element.

// Odd N (an even number of nodes per edge: every tile is a whole number of
// 16-byte chunks and starts 16-byte aligned): a tile arrives in natural
// node order, wave h of W issuing the 1 KiB instructions h, h + W, ... (lanes
// past the tile's end load nothing).
template <int N, int W, typename T>
__device__ __forceinline__ void dma_tile_natural(const T* __restrict__ src, T* raw, int h,
                                                 int lane) {
  constexpr int CH = (N + 1) * (N + 1) * (N + 1) * (int)sizeof(T) / 16;   // 16-byte chunks
  static_assert((N + 1) * (N + 1) * (N + 1) * sizeof(T) % 16 == 0, "whole chunks");
#pragma unroll
  for (int q = h; q * 64 < CH; q += W) {
    if (q * 64 + lane < CH)
      lds_load16(reinterpret_cast<const double*>(src) + 2 * (q * 64 + lane),
                 reinterpret_cast<double*>(raw) + 128 * q);
  }
}

// Element tile of any order into LDS by W waves: direct loads where the
// tile is a whole number of 16-byte chunks at a 16-byte aligned address
// (odd N), plain loads otherwise.  Consumers wait with
// s_waitcnt(vm, lgkm = 0) and a barrier.
template <int N, int W, typename T>
__device__ __forceinline__ void tile_lds(const T* __restrict__ src, T* dst, int h, int lane) {
  constexpr int NP = (N + 1) * (N + 1) * (N + 1);
  if constexpr (N % 2 == 1) {
    dma_tile_natural<N, W>(src, dst, h, lane);
  } else {
    for (int q = 64 * h + lane; q < NP; q += 64 * W) dst[q] = src[q];
  }
}

// Threads of an emission workgroup: one wave where it has a lane for every cell
// (155,344 order-2 elements at four isovalues, FP32: the extraction 293 us with
// two waves, 216 with one; 524,288 order-1 elements 781 and 560).
constexpr int emit_threads(int n) { return n <= 4 ? 64 : 128; }

// Emission of element e, which has triangles: the isovalues s0, s0 + ds, ...
// with a nonzero count write their triangles at offs[s * n_elem + e] of out (or
// of out.ptr[s], relative to the isovalue's first offset, when out.per_iso).
template <int N, typename T, class IL = IsoList<T>, class OUT = IsoOut<T>>
__device__ __forceinline__ void emit_elem(int64_t e, int t, int64_t n_elem,
                                          const T* __restrict__ x, const T* __restrict__ y,
                                          const T* __restrict__ z, const T* __restrict__ field,
                                          int s0, int ds, int n_iso, const IL& iso,
                                          const OUT& out,
                                          const uint8_t* __restrict__ ntri_tab,
                                          const int32_t* __restrict__ cnt,
                                          const int64_t* __restrict__ offs,
                                          uint64_t* __restrict__ keys) {
  constexpr int P = N + 1, NP = P * P * P, NC = N * N * N, TH = emit_threads(N), W = TH / 64;
  constexpr bool SWZ = N == 7 && std::is_same<T, double>::value;
  // The coordinate tiles are staged in LDS too, except for FP32 at N = 8 and
  // 9, which read the coordinates where the vertices need them (edge
  // endpoints only, through the caches) and so need 13 and 16 instead of 22
  // and 28 KB of LDS. Staged against read: FP64 N = 7 0.319 and 0.379 ms, the
  // FP32 step at N = 7 0.679 and 0.712 ms; FP32 N = 8, 5,753 elements, four
  // isovalues, 71 and 58 us (the isosurface call), N = 9, 4,194 elements, 63.6
  // and 60.5 us, the FP32 batched step (orders 5, 7, 9) 12.20 and 11.90 ms.
  constexpr bool XYZ = std::is_same<T, double>::value || N <= 7;
  __shared__ __attribute__((aligned(16))) T s_f[NP];
  __shared__ __attribute__((aligned(16))) T s_x[XYZ ? NP : 1];
  __shared__ __attribute__((aligned(16))) T s_y[XYZ ? NP : 1];
  __shared__ __attribute__((aligned(16))) T s_z[XYZ ? NP : 1];
  static_assert(256 + 256 * kMcMaxTri * 3 == 4096, "tables fill one 4 KiB block");
  __shared__ uint4 s_tab[16];      // triangle counts (256 B)
  __shared__ uint8_t s_case[NC];
  __shared__ uint16_t s_desc[NC * kMcMaxTri];
  __shared__ int32_t s_wave[W];
  const uint8_t* s_ntri = reinterpret_cast<const uint8_t*>(s_tab);
  const int8_t* s_tri = reinterpret_cast<const int8_t*>(ntri_tab) + 256;   // through the caches
  __builtin_assume(t >= 0 && t < TH);
  const int h = __builtin_amdgcn_readfirstlane(t >> 6);
  const int p = t & 63;
  const int64_t base = e * NP;
  // the triangle counts (256 B) and the tiles arrive by direct loads before
  // the one wait below; the case table (3.75 KiB) is read through the caches
  // in the vertex loop, which takes the FP64 workgroup from 24.3 to 20.4 KB
  // of LDS, six to eight per CU (emission 0.319 -> 0.307 ms on the channel
  // snapshot)
  if (h == 0 && p < 16)
    lds_load16(reinterpret_cast<const double*>(ntri_tab) + 2 * p,
               reinterpret_cast<double*>(s_tab));
  if constexpr (SWZ) {
    dma_tile(field + base, s_f, h, p);
    dma_tile(x + base, s_x, h, p);
    dma_tile(y + base, s_y, h, p);
    dma_tile(z + base, s_z, h, p);
  } else {
    tile_lds<N, W>(field + base, s_f, h, p);
    if constexpr (XYZ) {
      tile_lds<N, W>(x + base, s_x, h, p);
      tile_lds<N, W>(y + base, s_y, h, p);
      tile_lds<N, W>(z + base, s_z, h, p);
    }
  }
  const T* gx = XYZ ? s_x : x + base;
  const T* gy = XYZ ? s_y : y + base;
  const T* gz = XYZ ? s_z : z + base;
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds(0));
  barrier_after_wait();
  for (int s = s0; s < n_iso; s += ds) {
    const int64_t flat = (int64_t)s * n_elem + e;
    if (slot_tris(cnt[flat]) == 0) continue;
    int64_t g = offs[flat];
    T* dst = out.ptr[0];
    int64_t cap = out.cap[0];
    if (out.per_iso) {
      g -= offs[(int64_t)s * n_elem];
      dst = out.ptr[s];
      cap = out.cap[s];
    }
    if constexpr (SWZ)
      emit_element<7, TH>(iso.v[s], DmaNode{}, DmaNode{}, s_f, gx, gy, gz, s_ntri, s_tri,
                          s_case, s_desc, s_wave, dst, g, cap, out.per_iso ? nullptr : keys,
                          base);
    else
      emit_element<N, TH>(iso.v[s], StridedNode<P, P * P>{}, StridedNode<P, P * P>{}, s_f, gx,
                          gy, gz, s_ntri, s_tri, s_case, s_desc, s_wave, dst, g, cap,
                          out.per_iso ? nullptr : keys, base);
  }
}

// A workgroup per element, at every order.  Most leave at once (of 65,536
// elements of order 7, 26 % have triangles; 31 of 124 us if none has), but
// workgroups that take several elements and look them up together are
// slower, 133 against 120 us: the triangles of one element must be written
// before the tiles of the next are known to be there.  Few
// elements leave the chip idle: if SLICED, gridDim.y workgroups share each
// one's isovalues (a kernel of its own: strides that are read cost the others
// 2 %, 12,228 elements of order 6 45.3 us against 44.1).
template <int N, typename T, bool SLICED>
__global__ void __launch_bounds__(emit_threads(N))
emit_direct(int64_t e_begin, int64_t n_elem, const T* __restrict__ x, const T* __restrict__ y,
            const T* __restrict__ z, const T* __restrict__ field, int n_iso,
            IsoList<T> iso, IsoOut<T> out, const uint8_t* __restrict__ ntri_tab,
            const int32_t* __restrict__ cnt, const int64_t* __restrict__ offs,
            uint64_t* __restrict__ keys, int64_t* __restrict__ tri_count,
            int32_t* __restrict__ status) {
  const int64_t e = e_begin + blockIdx.x;
  // the last workgroup also writes the totals (in place of a kernel of its own)
  if (e == n_elem - 1 && (!SLICED || blockIdx.y == 0))
    write_totals<T>(threadIdx.x, offs, n_elem, n_iso, tri_count, out, status);
  const int s0 = SLICED ? blockIdx.y : 0, ds = SLICED ? gridDim.y : 1;
  bool any = false;
  for (int s = s0; s < n_iso; s += ds) any |= slot_tris(cnt[(int64_t)s * n_elem + e]) > 0;
  if (any)
    emit_elem<N, T>(e, threadIdx.x, n_elem, x, y, z, field, s0, ds, n_iso, iso, out, ntri_tab,
                    cnt, offs, keys);
}

// Counts of the elements `mine` of a wave's lanes (in == false: none) at the
// isovalues s0, s0 + ds, ..., and their cells' cases if case_idx.  The lanes look their
// elements' ranges up at once; elements that no isovalue crosses get zero
// counts without being read, the others are counted one after the other from
// bit rows (count_rows).  mm == NULL: every element is read (a value that is
// not above an isovalue, NaN included, is below it).  bits: the wave's own
// LDS.
template <int N, typename T, class IL>
__device__ __forceinline__ void count_lanes(int64_t mine, bool in, int lane, int64_t n_elem,
                                            const T* __restrict__ field,
                                            const T* __restrict__ mm, int s0, int ds, int n_iso,
                                            const IL& iso, const uint8_t* tab, uint64_t* bits,
                                            int32_t* __restrict__ cnt,
                                            uint8_t* __restrict__ case_idx) {
  constexpr int P = N + 1, NP = P * P * P, NC = N * N * N, R = (NP + 63) / 64;
  T lo = neg_inf<T>(), hi = pos_inf<T>();
  if (mm && in) {
    lo = mm[2 * mine];
    hi = mm[2 * mine + 1];
  }
  bool need = false;
  for (int s = s0; s < n_iso; s += ds) {
    const T c = iso.v[s];
    const bool crossed = in && (!mm || (hi > c && !(lo > c)));
    need |= crossed;
    if (in && !crossed) cnt[(int64_t)s * n_elem + mine] = 0;
    if (case_idx) {   // uniform cases
      const uint64_t above = __ballot(hi > c);
      for (uint64_t out = __ballot(in && !crossed); out != 0; out &= out - 1) {
        const int from = __builtin_ctzll(out);
        uint8_t* cd = case_idx + ((int64_t)s * n_elem + __shfl(mine, from)) * NC;
        for (int q = lane; q < NC; q += 64) cd[q] = (above >> from) & 1 ? 255 : 0;
      }
    }
  }
  for (uint64_t live = __ballot(need); live != 0; live &= live - 1) {
    const int from = __builtin_ctzll(live);
    const int64_t e = __shfl(mine, from);
    const T* src = field + e * NP;
    T v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int q = 64 * r + lane;
      v[r] = src[q < NP ? q : NP - 1];
    }
    for (int s = s0; s < n_iso; s += ds) {
      const T c = iso.v[s];
      if (__ballot(lane == from && (!mm || (hi > c && !(lo > c)))) == 0) continue;
      uint64_t b[R];
#pragma unroll
      for (int r = 0; r < R; ++r) b[r] = __ballot(64 * r + lane < NP && v[r] > c);
      if (lane == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) bits[r] = b[r];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const int64_t flat = (int64_t)s * n_elem + e;
      const uint32_t sum = count_rows<N>(reinterpret_cast<const uint32_t*>(bits), 0, lane, tab,
                                         case_idx ? case_idx + flat * NC : nullptr);
      if (lane == 63) cnt[flat] = (int)sum;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

// count_waves<N, T>: the count pass of the two-pass isosurface, four
// independent waves a workgroup; wave w takes elements w, w + waves, ...; of
// few elements gridDim.y workgroups share the isovalues.
// Bound by the field's elements that an isovalue crosses, read once.  A
// workgroup per element spent its time on starting: 33 us for 24,389
// elements of order 6 (FP32, four isovalues) with or without any to read.
constexpr int kCountWaves = 4;
template <int N>
constexpr int kCountBits = ((N + 1) * (N + 1) * (N + 1) + 63) / 64 + 1;   // a word past the last row's

template <int N, typename T>
__global__ void __launch_bounds__(64 * kCountWaves)
count_waves(int64_t n_elem, const T* __restrict__ field, const T* __restrict__ mm,
            int n_iso, IsoList<T> iso, const uint8_t* __restrict__ ntri_tab,
            int32_t* __restrict__ cnt, int64_t* __restrict__ active_total,
            uint8_t* __restrict__ case_idx) {
  __shared__ uint32_t s_tab[64];
  __shared__ uint64_t s_bits[kCountWaves][kCountBits<N>];
  clear_active(active_total, n_iso);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  if (t < 64) s_tab[t] = reinterpret_cast<const uint32_t*>(ntri_tab)[t];
  __syncthreads();
  const int64_t step = (int64_t)gridDim.x * kCountWaves;
  for (int64_t e0 = (int64_t)blockIdx.x * kCountWaves + wave; e0 < n_elem; e0 += 64 * step) {
    const int64_t mine = e0 + lane * step;
    count_lanes<N, T>(mine, mine < n_elem, lane, n_elem, field, mm, blockIdx.y, gridDim.y, n_iso,
                      iso, reinterpret_cast<const uint8_t*>(s_tab), s_bits[wave], cnt, case_idx);
  }
}

// ---------------------------------------------------------------------------
// mixed precision, N = 7, FP32 storage: derivative contractions on MFMA
// ---------------------------------------------------------------------------
//
// The 1-D contractions run as v_mfma_f32_16x16x32_{bf16,f16}: low-precision
// operands, FP32 accumulation.  One workgroup of two waves per element; for
// each field and direction wave w differentiates the 32 lines 32w..32w+31,
// two sets of 16 at once through a block-diagonal D:
//   rows     i = output node along the line, 0..7 of the first set's lines,
//            8..15 of the second's,
//   columns  the 16 lines of a set,
//   depth    the 8 line values spread over the four lane groups (group g
//            holds values m0 = 2g and m1 = 2g + 1 of both sets' lines), each
//            with the products the mode needs:
//   plain            D_hi (f - f_0)_hi
//   split (x3)       D_hi f_hi, then D_lo f_hi + D_hi f_lo in a product of
//                    its own (Henry, Tang & Heinecke 2019: the lo*lo term is
//                    dropped)
// where x_hi = round(x) to the operand format and x_lo = round(x - x_hi).
// In the FP16 split the lo parts are scaled by 2^11 (out of FP16's subnormal
// range; Ootomo & Yokota 2022) and accumulate separately, then scaled back.
// Values enter line-shifted (f_m - f_0), which keeps the coordinates'
// absolute offset out of the rounding.  The Jacobian is inverted in FP64;
// the chain rule, Q and |omega| are FP32.
//
// A lane gets four neighbouring outputs of one line.  It owns those four
// nodes of its t line, whose t derivatives therefore stay in registers; the
// r and s derivatives reach their owners through LDS, in node order with a
// pitch of 72 words a slab, which spreads the accesses of all three
// directions over the banks.  Bound by the vector units and the wait for the
// element's fields with six workgroups per CU (162 registers; with 128 and
// eight workgroups the Jacobians spill: 475 us).  65,536 elements, FP16 split:
// 450 us with four waves, one set of 16 lines a product (half its rows zero,
// half the lanes without outputs) and all derivatives through LDS, 4,596
// vector instructions an element; 340 so, with 2,460.  The fields once in and
// Q and |omega| once out take 212 us at copy rate.

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

enum MixMode { kMixBF16 = 0, kMixFP16 = 1, kMixBF16x3 = 2, kMixFP16x3 = 3 };

template <int M>
struct MixT {
  typedef __bf16 E;
  typedef bf16x8 V;
};
template <>
struct MixT<kMixFP16> {
  typedef _Float16 E;
  typedef f16x8 V;
};
template <>
struct MixT<kMixFP16x3> {
  typedef _Float16 E;
  typedef f16x8 V;
};

constexpr float kF16LoScale = 2048.0f;   // 2^11

template <int M>
__device__ __forceinline__ f32x4 mfma_line(typename MixT<M>::V a, typename MixT<M>::V b,
                                           f32x4 c) {
  if constexpr (M == kMixBF16 || M == kMixBF16x3)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

template <int M>
constexpr bool kMixSplit = M == kMixBF16x3 || M == kMixFP16x3;
// scale of the lo parts
template <int M>
constexpr float kMixLo = M == kMixFP16x3 ? kF16LoScale : 1.0f;

// A operands of one lane (row i = lane % 16, lane group g = lane / 16).
template <int M>
struct MixOps {
  typename MixT<M>::V a;    // main product
  typename MixT<M>::V ac;   // correction (splits only)
};

template <int M>
__device__ __forceinline__ MixOps<M> mix_ops(const double* __restrict__ d, int lane) {
  using E = typename MixT<M>::E;
  MixOps<M> o;
  const int i = lane & 15, g = lane >> 4;
  // an unconditional load (row i & 7): no branch holds the caller's later
  // loads behind its wait
  const double r0 = d[(i & 7) * 8 + 2 * g], r1 = d[(i & 7) * 8 + 2 * g + 1];
  const E zero = E(0.f), h0 = E((float)r0), h1 = E((float)r1);
  const E l0 = E((float)((r0 - (double)(float)h0) * kMixLo<M>));
  const E l1 = E((float)((r1 - (double)(float)h1) * kMixLo<M>));
#pragma unroll
  for (int q = 0; q < 2; ++q) {   // the set whose rows these are
    const bool on = (i >> 3) == q;
    o.a[2 * q] = on ? h0 : zero;
    o.a[2 * q + 1] = on ? h1 : zero;
    o.a[4 + 2 * q] = o.a[5 + 2 * q] = zero;
    o.ac[4 * q] = on ? l0 : zero;
    o.ac[4 * q + 1] = on ? l1 : zero;
    o.ac[4 * q + 2] = on ? h0 : zero;
    o.ac[4 * q + 3] = on ? h1 : zero;
  }
  return o;
}

// Derivatives along two line sets: v[q] are this lane's shifted values
// f[2g] - f[0], f[2g + 1] - f[0] of line lane % 16 of set q; lane group g
// receives the outputs 4 (g & 1) .. + 3 of that line of set g >> 1.
template <int M>
__device__ __forceinline__ f32x4 mix_contract(const MixOps<M>& o, const f32x2 (&v)[2]) {
  using E = typename MixT<M>::E;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  typename MixT<M>::V b, bc;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    // a pair at a time: one packed conversion, and its result is both
    // products' operand
    typedef E E2 __attribute__((ext_vector_type(2)));
    const E2 h = __builtin_convertvector(v[q], E2);
    b[2 * q] = bc[4 * q] = h[0];
    b[2 * q + 1] = bc[4 * q + 1] = h[1];
    b[4 + 2 * q] = b[5 + 2 * q] = E(0.f);
    if constexpr (kMixSplit<M>) {
#pragma unroll
      for (int m = 0; m < 2; ++m)   // (v - h) scaled, exact in one operation
        bc[4 * q + 2 + m] = E(fmaf((float)h[m], -kMixLo<M>, v[q][m] * kMixLo<M>));
    }
  }
  f32x4 acc = mfma_line<M>(o.a, b, zero);
  if constexpr (M == kMixBF16x3) acc = mfma_line<M>(o.ac, bc, acc);
  if constexpr (M == kMixFP16x3) {
    const f32x4 c = mfma_line<M>(o.ac, bc, zero);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = fmaf(c[r], 1.0f / kF16LoScale, acc[r]);
  }
  return acc;
}

constexpr int kMixSlab = 72;             // words of a slab of 64 nodes in LDS
constexpr int kMixTile = 8 * kMixSlab;

// Where a lane finds things in a tile (words): node 0 and node 2g of its line
// of the first set in each direction (the second set's lie kMixSet further),
// its four outputs along r and along s, and its first own node.
struct MixLane {
  int line0[3], line2g[3], out_r, out_s, own;
};
constexpr int kMixSet[3] = {2 * kMixSlab, 2 * kMixSlab, 16};
constexpr int kMixStride[3] = {1, 8, kMixSlab};
__device__ __forceinline__ MixLane mix_lane(int wv, int lane) {
  const int n = lane & 15, g = lane >> 4, lo = n & 7, hi = 4 * wv + (n >> 3);
  MixLane m;
  m.line0[0] = 8 * lo + kMixSlab * hi;
  m.line0[1] = lo + kMixSlab * hi;
  m.line0[2] = lo + 8 * hi;
#pragma unroll
  for (int d = 0; d < 3; ++d) m.line2g[d] = m.line0[d] + 2 * g * kMixStride[d];
  m.out_r = m.line0[0] + (g >> 1) * kMixSet[0] + 4 * (g & 1);
  m.out_s = m.line0[1] + (g >> 1) * kMixSet[1] + 32 * (g & 1);
  m.own = m.line0[2] + (g >> 1) * kMixSet[2] + 4 * kMixSlab * (g & 1);
  return m;
}

// One field (tile f) -> its r and s derivatives (tiles dr, ds), and the t
// derivatives of the lane's own nodes.
template <int M>
__device__ __forceinline__ f32x4 mix_field(const float* __restrict__ f, float* __restrict__ dr,
                                           float* __restrict__ ds, const MixOps<M>& o,
                                           const MixLane& at) {
  f32x4 acc[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    f32x2 v[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float f0 = f[at.line0[d] + q * kMixSet[d]];
      const float* p = f + at.line2g[d] + q * kMixSet[d];
      v[q][0] = p[0] - f0;
      v[q][1] = p[kMixStride[d]] - f0;
    }
    acc[d] = mix_contract<M>(o, v);
  }
  *reinterpret_cast<f32x4*>(dr + at.out_r) = acc[0];
#pragma unroll
  for (int r = 0; r < 4; ++r) ds[at.out_s + 8 * r] = acc[1][r];
  return acc[2];
}

// QC: Q, |omega| and the element range of Q from (x, y, z, u, v, w);
// otherwise the physical gradient of f = u into (o0, o1, o2).
// COUNT (with QC): also the per-(isovalue, element) triangle and active-cell
// counts from the element's Q, by bit rows.
template <int M, bool QC, bool COUNT = false>
__global__ void __launch_bounds__(128, 3)
mixed7(const double* __restrict__ dmat, const float* __restrict__ x,
       const float* __restrict__ y, const float* __restrict__ z, const float* __restrict__ u,
       const float* __restrict__ v, const float* __restrict__ w, float* __restrict__ o0,
       float* __restrict__ o1, float* __restrict__ o2, float* __restrict__ qmm,
       int32_t* __restrict__ status, CountSink<float> sink) {
  static_assert(QC || !COUNT, "counting needs Q");
  constexpr int NF = QC ? 6 : 4;
  __shared__ __align__(16) float s_in[NF][kMixTile];
  __shared__ __align__(16) float s_d[2][2][kMixTile];
  __shared__ float s_red[4];
  __shared__ uint32_t s_tab[COUNT ? 64 : 1];
  if constexpr (COUNT) clear_active(sink.active, sink.n_iso);
  const int t = threadIdx.x, lane = t & 63;
  __builtin_assume(t >= 0 && t < 128);
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t base = (int64_t)blockIdx.x * 512;
  const MixOps<M> ops = mix_ops<M>(dmat, lane);   // its loads first: in flight with the tiles'
  const int64_t off = base + 4 * t;
  f32x4 in[NF];
  in[0] = *reinterpret_cast<const f32x4*>(x + off);
  in[1] = *reinterpret_cast<const f32x4*>(y + off);
  in[2] = *reinterpret_cast<const f32x4*>(z + off);
  in[3] = *reinterpret_cast<const f32x4*>(u + off);
  if constexpr (NF == 6) {
    in[4] = *reinterpret_cast<const f32x4*>(v + off);
    in[5] = *reinterpret_cast<const f32x4*>(w + off);
  }
  if (COUNT && t < 64) s_tab[t] = reinterpret_cast<const uint32_t*>(sink.ntri)[t];
#pragma unroll
  for (int c = 0; c < NF; ++c)
    *reinterpret_cast<f32x4*>(s_in[c] + kMixSlab * (t >> 4) + 4 * (t & 15)) = in[c];
  __syncthreads();

  const MixLane at = mix_lane(wv, lane);
  float gd[3][4][3];   // geometry: [coordinate][node][r, s, t]
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const f32x4 ft = mix_field<M>(s_in[c], s_d[c & 1][0], s_d[c & 1][1], ops, at);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      gd[c][r][0] = s_d[c & 1][0][at.own + kMixSlab * r];
      gd[c][r][1] = s_d[c & 1][1][at.own + kMixSlab * r];
      gd[c][r][2] = ft[r];
    }
  }
  int bad = 0;
  InvJac<float> kk[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    InvJac<double> k64;
    bad |= !invert_jacobian<double>(gd[0][r][0], gd[0][r][1], gd[0][r][2], gd[1][r][0],
                                    gd[1][r][1], gd[1][r][2], gd[2][r][0], gd[2][r][1],
                                    gd[2][r][2], k64);
    kk[r] = InvJac<float>{(float)k64.rx, (float)k64.ry, (float)k64.rz,
                          (float)k64.sx, (float)k64.sy, (float)k64.sz,
                          (float)k64.tx, (float)k64.ty, (float)k64.tz};
    __builtin_amdgcn_sched_barrier(0);   // one node's FP64 values at a time
  }
  // an inverted element (rare) is flagged by its own lanes: no block vote
  if (bad && status) atomicOr(status, SEM_FLAG_BAD_JACOBIAN);
  float a[4][NF - 3][3];
#pragma unroll
  for (int c = 0; c < NF - 3; ++c) {
    const int buf = (3 + c) & 1;
    const f32x4 tt = mix_field<M>(s_in[3 + c], s_d[buf][0], s_d[buf][1], ops, at);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float fr = s_d[buf][0][at.own + kMixSlab * r];
      const float fs = s_d[buf][1][at.own + kMixSlab * r];
      const float ft = tt[r];
      const InvJac<float>& K = kk[r];
      a[r][c][0] = fr * K.rx + fs * K.sx + ft * K.tx;
      a[r][c][1] = fr * K.ry + fs * K.sy + ft * K.ty;
      a[r][c][2] = fr * K.rz + fs * K.sz + ft * K.tz;
    }
  }
  // the lane's nodes: 4 (g & 1) + r along its t line
  const int g = lane >> 4, k0 = 4 * (g & 1);
  const int64_t own = base + 64 * k0 + 32 * wv + 16 * (g >> 1) + (lane & 15);
  if constexpr (!QC) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      o0[own + 64 * r] = a[r][0][0];
      o1[own + 64 * r] = a[r][0][1];
      o2[own + 64 * r] = a[r][0][2];
    }
  } else {
    float mn = pos_inf<float>(), mx = neg_inf<float>();
    float qn[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float(&A)[3][3] = a[r];
      const float tr2 = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2] +
                        2.f * (A[0][1] * A[1][0] + A[0][2] * A[2][0] + A[1][2] * A[2][1]);
      const float w1 = A[2][1] - A[1][2], w2 = A[0][2] - A[2][0], w3 = A[1][0] - A[0][1];
      const float qv = -0.5f * tr2;
      if (o0) o0[own + 64 * r] = qv;
      if (o1) o1[own + 64 * r] = vort_root(w1 * w1 + w2 * w2 + w3 * w3);
      qn[r] = qv;
      const float c = qv != qv ? neg_inf<float>() : qv;
      mn = c < mn ? c : mn;
      mx = c > mx ? c : mx;
    }
    if (qmm) {
      block_minmax<float, 128>(mn, mx, s_red);
      if (t == 0) {
        qmm[2 * (int64_t)blockIdx.x] = mn;
        qmm[2 * (int64_t)blockIdx.x + 1] = mx;
      }
    }
    if constexpr (COUNT) {
      // 16 lanes of a ballot are 16 consecutive nodes
      __shared__ uint32_t s_bits[kBitGroup][18];
      for (int i = 0; i < sink.n_iso; i += kBitGroup) {
        const int m = sink.n_iso - i < kBitGroup ? sink.n_iso - i : kBitGroup;
        if (i > 0) __syncthreads();   // both waves are done with the previous bits
#pragma unroll
        for (int q = 0; q < kBitGroup; ++q) {
          if (q >= m) break;
          const float c = sink.iso.v[i + q];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint64_t b = __ballot(qn[r] > c);
            if ((lane & 15) == 0)
              reinterpret_cast<uint16_t*>(s_bits[q])[4 * (k0 + r) + 2 * wv + (g >> 1)] =
                  (uint16_t)(b >> (16 * g));
          }
        }
        __syncthreads();
        for (int q = wv; q < m; q += 2) {
          const uint32_t sum =
              count_rows<7>(s_bits[q], 0, lane, reinterpret_cast<const uint8_t*>(s_tab));
          if (lane == 63) sink.cnt[(int64_t)(i + q) * sink.n_elem + blockIdx.x] = (int)sum;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// batched snapshots: one persistent launch over every snapshot's elements
// ---------------------------------------------------------------------------
//
// Work item = `chunk` consecutive elements of one snapshot; snapshots may
// differ in order N and element count.  Each workgroup takes items
// blockIdx.x, blockIdx.x + gridDim.x, ... ; for an item it finds the
// snapshot (binary search over the items' prefix) and computes Q, |omega| and
// the element ranges with the order's instantiation: by default the line
// exchange of sem_qcrit, or the LDS-tile form (six tiles and D staged) if the
// caller or the tuner chose it, where small elements leave threads idle unless
// several share a workgroup.

constexpr int kBatchThreads = 256;
constexpr int kBatchTile = 6144;   // LDS values for 6 fields x chunk x (N+1)^3

template <int N, typename T>
__device__ __forceinline__ int batch_chunk(const coef_t<N, T>* dmat, const T* const (&fp)[6], T* oq,
                                           T* oom, T* oqmm, int64_t e0, int ne, T* tiles,
                                           coef_t<N, T>* sd) {
  constexpr int P = N + 1, P3 = P * P * P;
  constexpr int MAXQ = kBatchTile / 6 / kBatchThreads;   // node values per thread
  const int t = threadIdx.x;
  const int nn = ne * P3;
  for (int q = t; q < P * P; q += kBatchThreads) sd[q] = dmat[q];
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    const T* src = fp[f] + e0 * P3;
    for (int q = t; q < nn; q += kBatchThreads) tiles[f * nn + q] = src[q];
  }
  __syncthreads();
  int bad = 0;
  T qkeep[MAXQ];
#pragma unroll
  for (int r = 0; r < MAXQ; ++r) {
    const int q = t + r * kBatchThreads;
    qkeep[r] = neg_inf<T>();
    if (q >= nn) continue;
    const int c = q / P3, node = q - c * P3;
    const int i = node % P, j = (node / P) % P, k = node / (P * P);
    const T* tl[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) tl[f] = tiles + f * nn + c * P3;
    T xr, xs, xt, yr, ys, yt, zr, zs, zt;
    ref_derivs<N>(tl[0], sd, i, j, k, xr, xs, xt);
    ref_derivs<N>(tl[1], sd, i, j, k, yr, ys, yt);
    ref_derivs<N>(tl[2], sd, i, j, k, zr, zs, zt);
    InvJac<T> kk;
    bad |= !invert_jacobian(xr, xs, xt, yr, ys, yt, zr, zs, zt, kk);
    T a[3][3];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      T fr, fs, ft;
      ref_derivs<N>(tl[3 + cc], sd, i, j, k, fr, fs, ft);
      a[cc][0] = fr * kk.rx + fs * kk.sx + ft * kk.tx;
      a[cc][1] = fr * kk.ry + fs * kk.sy + ft * kk.ty;
      a[cc][2] = fr * kk.rz + fs * kk.sz + ft * kk.tz;
    }
    const T tr2 = a[0][0] * a[0][0] + a[1][1] * a[1][1] + a[2][2] * a[2][2] +
                  T(2) * (a[0][1] * a[1][0] + a[0][2] * a[2][0] + a[1][2] * a[2][1]);
    const T w1 = a[2][1] - a[1][2], w2 = a[0][2] - a[2][0], w3 = a[1][0] - a[0][1];
    const T qv = T(-0.5) * tr2;
    const int64_t o = e0 * P3 + q;
    if (oq) oq[o] = qv;
    if (oom) oom[o] = vort_root(w1 * w1 + w2 * w2 + w3 * w3);
    qkeep[r] = qv != qv ? neg_inf<T>() : qv;
    // one node at a time: no overlap of the unrolled iterations (which
    // would multiply the live registers)
    asm volatile("" ::: "memory");
  }
  if (oqmm) {
    __syncthreads();                     // every tile read is done
#pragma unroll
    for (int r = 0; r < MAXQ; ++r) {
      const int q = t + r * kBatchThreads;
      if (q < nn) tiles[q] = qkeep[r];
    }
    __syncthreads();
    const int wv = t >> 6, lane = t & 63;
    if (wv < ne) {                       // wave c reduces element c
      T mn = pos_inf<T>(), mx = neg_inf<T>();
      for (int q = lane; q < P3; q += 64) {
        const T v = tiles[wv * P3 + q];
        mn = v < mn ? v : mn;
        mx = v > mx ? v : mx;
      }
      wave_minmax(mn, mx);
      if (lane == 63) {
        oqmm[2 * (e0 + wv)] = mn;
        oqmm[2 * (e0 + wv) + 1] = mx;
      }
    }
  }
  return bad;
}

// A descriptor field read inside the persistent loop comes through vector
// loads (the loop's stores precede it); moving it to a scalar register keeps
// every pointer and address computation off the VGPRs.
template <typename P>
__device__ __forceinline__ P* uniform_ptr(P* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<P*>(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t uniform_i64(int64_t x) {
  const uint64_t v = (uint64_t)x;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One instantiation per (order, precision, form), so that no form's register
// demand limits another's occupancy.  kBatchLines runs the body of
// qcrit_lines on its workgroup's elements.
template <int N, typename T, int FORM>
constexpr int batch_threads() {
  return FORM == kBatchLines ? LineOf<N, T>::TH : kBatchThreads;
}

// Waves per SIMD to hold: the LDS tile leaves room for three workgroups a CU in
// FP64 and six in FP32; a few registers more than three (four) waves allow cost
// the tile form a quarter (12,228 order-6 elements, FP64: 168 us, 226 with two).
// Order 9 in FP64 would spill too much for three (188 us with two, 195).  The
// line form at FP64 N = 8 and 9 spills two registers in the loop over items
// (12 bytes a lane; a launch of sem_qcrit holds them): within 10 % of sem_qcrit,
// and a wave less would cost more.
template <int N, typename T, int FORM>
constexpr int batch_waves() {
  return FORM == kBatchLines ? line_waves<N, T, LineOf<N, T>>()
         : sizeof(T) == 4    ? 4
                             : N < 9 ? 3 : 2;
}

template <int N, typename T, int FORM>
__global__ void __launch_bounds__((batch_threads<N, T, FORM>()), (batch_waves<N, T, FORM>()))
qcrit_batch(const BatchHeader* __restrict__ hdr, const BatchSnap* __restrict__ snaps,
            int32_t* __restrict__ status) {
  const int s0 = hdr->snap_begin[N], s1 = hdr->snap_begin[N + 1];
  const int64_t total = hdr->items[N];
  int bad = 0;
  // The descriptor of the current snapshot stays in scalar registers; a
  // workgroup's items increase, so it is looked up again only when an item
  // passes the next snapshot's first item.
  int cur = s0 - 1;
  int64_t begin = 0, next_begin = 0, n_elem = 0;
  int chunk = 1;
  const coef_t<N, T>* dmat = nullptr;
  const T *f0 = nullptr, *f1 = nullptr, *f2 = nullptr, *f3 = nullptr, *f4 = nullptr,
          *f5 = nullptr;
  T *oq = nullptr, *oom = nullptr, *oqmm = nullptr;
  for (int64_t item = blockIdx.x; item < total; item += gridDim.x) {
    if (cur < s0 || item >= next_begin) {
      int lo = cur < s0 ? s0 : cur, hi = s1 - 1;   // last snapshot with item_begin <= item
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (snaps[mid].item_begin <= item) lo = mid;
        else hi = mid - 1;
      }
      cur = __builtin_amdgcn_readfirstlane(lo);
      const BatchSnap& sn = snaps[cur];
      begin = uniform_i64(sn.item_begin);
      next_begin = uniform_i64(cur + 1 < s1 ? snaps[cur + 1].item_begin : total);
      n_elem = uniform_i64(sn.n_elem);
      chunk = __builtin_amdgcn_readfirstlane(sn.chunk);
      dmat = uniform_ptr(static_cast<const coef_t<N, T>*>(sn.dmat));
      f0 = uniform_ptr(static_cast<const T*>(sn.f[0]));
      f1 = uniform_ptr(static_cast<const T*>(sn.f[1]));
      f2 = uniform_ptr(static_cast<const T*>(sn.f[2]));
      f3 = uniform_ptr(static_cast<const T*>(sn.f[3]));
      f4 = uniform_ptr(static_cast<const T*>(sn.f[4]));
      f5 = uniform_ptr(static_cast<const T*>(sn.f[5]));
      oq = uniform_ptr(static_cast<T*>(sn.q));
      oom = uniform_ptr(static_cast<T*>(sn.om));
      oqmm = uniform_ptr(static_cast<T*>(sn.qmm));
    }
    const int64_t e0 = (item - begin) * chunk;
    // the thread index is made opaque per item, so that no index arithmetic
    // of the body is hoisted out of the loop and held in registers across it
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    if constexpr (FORM == kBatchChunk) {
      __shared__ T tiles[kBatchTile];
      __shared__ coef_t<N, T> sd[(N + 1) * (N + 1)];
      const int64_t left = n_elem - e0;
      const int ne = (int)(left < chunk ? left : chunk);
      const T* fp[6] = {f0, f1, f2, f3, f4, f5};
      bad |= batch_chunk<N, T>(dmat, fp, oq, oom, oqmm, e0, ne, tiles, sd);
    } else {
      constexpr int E = LineOf<N, T>::E;   // the item's chunk
      const int64_t left = n_elem - e0;
      const int ne = (int)(left < E ? left : E);
      qcrit_lines_elem<N, T, false, LineOf<N, T>>(e0, t, ne, dmat, f0, f1, f2, f3, f4, f5, oq, oom, oqmm,
                                    status);
    }
    __syncthreads();                   // the next item reuses the LDS
  }
  if constexpr (FORM == kBatchChunk) {
    bad = __syncthreads_or(bad);
    if (bad && threadIdx.x == 0 && status) atomicOr(status, SEM_FLAG_BAD_JACOBIAN);
  }
}

// ---------------------------------------------------------------------------
// batched isosurfaces: persistent count and emission over (job, element)
// ---------------------------------------------------------------------------
//
// A job is one field of one snapshot at up to four isovalues.  The plan
// lists the jobs grouped by order; within an order, work item k is element
// k - item_begin of the job whose item range holds k.  Count slots of a job
// are [slot_begin, slot_begin + n_iso * n_elem), isovalue-major, so one
// exclusive scan over every slot of every job gives each (job, isovalue,
// element) its first triangle in one soup ordered by job, isovalue,
// element, cell and slot.

// Isovalues read through a pointer (the job descriptor's copy).
template <typename T>
struct IsoPtr {
  const T* v;
};

// One soup with global offsets (the per-isovalue form of IsoOut is never
// taken, so nothing is indexed by isovalue).
template <typename T>
struct SoupOut {
  T* ptr[1];
  int64_t cap[1];
  static constexpr int per_iso = 0;
};

template <typename T>
__device__ __forceinline__ const T* job_iso(const IsoBatchJob& jb);
template <>
__device__ __forceinline__ const double* job_iso<double>(const IsoBatchJob& jb) {
  return jb.isod;
}
template <>
__device__ __forceinline__ const float* job_iso<float>(const IsoBatchJob& jb) {
  return jb.isof;
}

// The job descriptor a workgroup is in, kept in scalar registers and looked
// up again (binary search over the jobs' first items) only when the work
// item passes the next job's first item.
template <typename T>
struct JobCursor {
  int cur = -1;
  int64_t begin = 0, next_begin = 0, n_elem = 0, slot = 0;
  int n_iso = 0, job = 0;
  const T *x = nullptr, *y = nullptr, *z = nullptr, *field = nullptr, *mm = nullptr;
  const T* iso = nullptr;

  __device__ __forceinline__ void seek(const IsoBatchJob* __restrict__ jobs, int j0, int j1,
                                       int64_t total, int64_t item) {
    if (cur >= j0 && item < next_begin) return;
    int lo = cur < j0 ? j0 : cur, hi = j1 - 1;   // last job with item_begin <= item
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (jobs[mid].item_begin <= item) lo = mid;
      else hi = mid - 1;
    }
    cur = __builtin_amdgcn_readfirstlane(lo);
    const IsoBatchJob& jb = jobs[cur];
    begin = uniform_i64(jb.item_begin);
    next_begin = uniform_i64(cur + 1 < j1 ? jobs[cur + 1].item_begin : total);
    n_elem = uniform_i64(jb.n_elem);
    slot = uniform_i64(jb.slot_begin);
    n_iso = __builtin_amdgcn_readfirstlane(jb.n_iso);
    job = __builtin_amdgcn_readfirstlane(jb.job);
    x = uniform_ptr(static_cast<const T*>(jb.x));
    y = uniform_ptr(static_cast<const T*>(jb.y));
    z = uniform_ptr(static_cast<const T*>(jb.z));
    field = uniform_ptr(static_cast<const T*>(jb.field));
    mm = uniform_ptr(static_cast<const T*>(jb.mm));
    iso = uniform_ptr(job_iso<T>(jb));
  }
};

// Waves take runs of consecutive items, a lane each (a run is cut where a job
// ends), as long as one round of waves covers them all: on the batched
// snapshots 109 us in all for the three orders, 127 with a run of one.
template <int N, typename T>
__global__ void __launch_bounds__(64 * kCountWaves)
iso_batch_count(const IsoBatchHeader* __restrict__ hdr, const IsoBatchJob* __restrict__ jobs,
                const uint8_t* __restrict__ ntri_tab, int32_t* __restrict__ cnt) {
  __shared__ uint32_t s_tab[64];
  __shared__ uint64_t s_bits[kCountWaves][kCountBits<N>];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  if (t < 64) s_tab[t] = reinterpret_cast<const uint32_t*>(ntri_tab)[t];
  __syncthreads();
  const int j0 = hdr->job_begin[N], j1 = hdr->job_begin[N + 1];
  const int64_t total = hdr->items[N];
  const int64_t waves = (int64_t)gridDim.x * kCountWaves;
  const int64_t each = (total + waves - 1) / waves;
  const int run = each > 64 ? 64 : (int)each;
  JobCursor<T> c;
  for (int64_t i0 = ((int64_t)blockIdx.x * kCountWaves + wave) * run; i0 < total;
       i0 += waves * run) {
    const int64_t end = i0 + run < total ? i0 + run : total;
    for (int64_t i = i0; i < end;) {
      c.seek(jobs, j0, j1, total, i);
      const int64_t stop = end < c.next_begin ? end : c.next_begin;
      const int64_t mine = i - c.begin + lane;
      count_lanes<N, T>(mine, i + lane < stop, lane, c.n_elem, c.field, c.mm, 0, 1, c.n_iso,
                        IsoPtr<T>{c.iso}, reinterpret_cast<const uint8_t*>(s_tab),
                        s_bits[wave], cnt + c.slot, nullptr);
      i = stop;
    }
  }
}

template <int N, typename T>
__global__ void __launch_bounds__(emit_threads(N))
iso_batch_emit(const IsoBatchHeader* __restrict__ hdr, const IsoBatchJob* __restrict__ jobs,
               const uint8_t* __restrict__ ntri_tab, const int32_t* __restrict__ cnt,
               const int64_t* __restrict__ offs, T* __restrict__ tri, int64_t cap) {
  const int j0 = hdr->job_begin[N], j1 = hdr->job_begin[N + 1];
  const int64_t total = hdr->items[N];
  SoupOut<T> out;
  out.ptr[0] = tri;
  out.cap[0] = cap;
  JobCursor<T> c;
  for (int64_t item = blockIdx.x; item < total; item += gridDim.x) {
    c.seek(jobs, j0, j1, total, item);
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int64_t e = item - c.begin;
    bool any = false;
    for (int s = 0; s < c.n_iso; ++s) any |= slot_tris(cnt[c.slot + s * c.n_elem + e]) > 0;
    if (any)
      emit_elem<N, T>(e, t, c.n_elem, c.x, c.y, c.z, c.field, 0, 1, c.n_iso, IsoPtr<T>{c.iso},
                      out, ntri_tab, cnt + c.slot, offs + c.slot, nullptr);
  }
}

// Per (job, isovalue): first triangle and count (isovalues past a job's
// n_iso get count 0 at the job's end), by the first `totals` workgroups; the
// overflow flag if the soup does not fit.  Each later workgroup adds up the
// active cells of one (job, isovalue) from its slots (0 past the job's isovalues).
__global__ void __launch_bounds__(256)
iso_batch_totals(const IsoBatchHeader* __restrict__ hdr, const IsoBatchJob* __restrict__ jobs,
                 const int32_t* __restrict__ cnt, const int64_t* __restrict__ offs,
                 int64_t* __restrict__ tri_offset, int64_t* __restrict__ tri_count,
                 int64_t* __restrict__ active, int totals, int64_t cap,
                 int32_t* __restrict__ status) {
  __shared__ int64_t sred[256 / 64];
  if ((int)blockIdx.x >= totals) {
    const int at = blockIdx.x - totals, s = at & 3;
    const IsoBatchJob& jb = jobs[at >> 2];
    int64_t a = 0;
    if (s < jb.n_iso)
      for (int64_t e = threadIdx.x; e < jb.n_elem; e += 256)
        a += slot_active(cnt[jb.slot_begin + s * jb.n_elem + e]);
    a = block_sum<256>(a, sred);
    if (threadIdx.x == 0) active[4 * jb.job + s] = a;
    return;
  }
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx < 4 * hdr->n_job) {
    const IsoBatchJob& jb = jobs[idx >> 2];
    const int s = idx & 3;
    const int64_t lo = jb.slot_begin + (int64_t)(s < jb.n_iso ? s : jb.n_iso) * jb.n_elem;
    const int64_t hi = s < jb.n_iso ? lo + jb.n_elem : lo;
    if (tri_offset) tri_offset[4 * jb.job + s] = offs[lo];
    tri_count[4 * jb.job + s] = offs[hi] - offs[lo];
  }
  if (idx == 0 && status && offs[hdr->n_slots] > cap) atomicOr(status, SEM_FLAG_TRI_OVERFLOW);
}

// Synthetic unit-cube elements on a 16 x 16 x ... lattice with node
// spacing 1/N and a smooth velocity: timing input for the autotuner.
template <typename T>
__global__ void tune_fill(int order, int64_t n_elem, T* x, T* y, T* z, T* u, T* v, T* w) {
  const int p = order + 1;
  const int64_t p3 = (int64_t)p * p * p;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n_elem * p3) return;
  const int64_t e = idx / p3;
  const int node = (int)(idx - e * p3);
  const int i = node % p, j = (node / p) % p, k = node / (p * p);
  const T xv = T(e % 16) + T(i) / T(order), yv = T((e / 16) % 16) + T(j) / T(order);
  const T zv = T(e / 256) + T(k) / T(order);
  x[idx] = xv;
  y[idx] = yv;
  z[idx] = zv;
  u[idx] = sin(xv + T(2) * yv);
  v[idx] = cos(yv - zv);
  w[idx] = sin(zv + T(0.5) * xv);
}

// ---------------------------------------------------------------------------
// dispatch over the order
// ---------------------------------------------------------------------------

#define SEM_ORDER_SWITCH(order, ...) \
  switch (order) {                    \
    case 1: { constexpr int N = 1; __VA_ARGS__; } break; \
    case 2: { constexpr int N = 2; __VA_ARGS__; } break; \
    case 3: { constexpr int N = 3; __VA_ARGS__; } break; \
    case 4: { constexpr int N = 4; __VA_ARGS__; } break; \
    case 5: { constexpr int N = 5; __VA_ARGS__; } break; \
    case 6: { constexpr int N = 6; __VA_ARGS__; } break; \
    case 7: { constexpr int N = 7; __VA_ARGS__; } break; \
    case 8: { constexpr int N = 8; __VA_ARGS__; } break; \
    case 9: { constexpr int N = 9; __VA_ARGS__; } break; \
    default: return hipErrorInvalidValue;          \
  }

// D and its even-odd halves in the line sums' type of (order, T).
template <int N, typename T>
const coef_t<N, T>* dmat_of(const DeviceTables& tab) {
  if constexpr (std::is_same<coef_t<N, T>, float>::value) return tab.d32[N];
  else return tab.d64[N];
}

// A launch holds fewer than 2^32 work-items: more elements than that (at
// `threads` for every `per` of them) take several.  go(first element, element
// past the last one, workgroups, start event, stop event).
template <class Go>
void launch_parts(int64_t n_elem, int per, int threads, hipEvent_t start, hipEvent_t stop,
                  const Go& go) {
  const int64_t most = 0xffffffffll / threads * per;
  for (int64_t b = 0; b < n_elem; b += most) {
    const int64_t end = n_elem - b < most ? n_elem : b + most;
    go(b, end, dim3((unsigned)((end - b + per - 1) / per)), b == 0 ? start : nullptr,
       end == n_elem ? stop : nullptr);
  }
}

template <typename T>
hipError_t derivs_t(int order, const DeviceTables& tab, int64_t n_elem, const void* x,
                    const void* y, const void* z, const void* f, void* gx, void* gy, void* gz,
                    int32_t* status, hipStream_t s) {
  SEM_ORDER_SWITCH(order, {
    using C = LineOf<N, T>;
    launch_parts(n_elem, C::E, C::TH, nullptr, nullptr,
                 [&](int64_t b, int64_t end, dim3 grid, hipEvent_t, hipEvent_t) {
                   hipLaunchKernelGGL((derivs_lines<N, T, C>), grid, dim3(C::TH), 0, s,
                                      dmat_of<N, T>(tab), (const T*)x, (const T*)y, (const T*)z,
                                      (const T*)f, (T*)gx, (T*)gy, (T*)gz, status, b, end);
                 });
  });
  return hipGetLastError();
}

template <typename T>
hipError_t qcrit_t(int order, const DeviceTables& tab, int64_t n_elem, const void* x,
                   const void* y, const void* z, const void* u, const void* v, const void* w,
                   void* q, void* om, void* qmm, int32_t* status, hipStream_t s) {
  const PhaseTimer pt = phase_timer(SEM_PHASE_QCRIT);
  SEM_ORDER_SWITCH(order, {
    auto go = [&](auto shape) {
      using C = decltype(shape);
      launch_parts(n_elem, C::E, C::TH, pt.start, pt.stop,
                   [&](int64_t b, int64_t end, dim3 grid, hipEvent_t e0, hipEvent_t e1) {
                     hipExtLaunchKernelGGL((qcrit_lines<N, T, C>), grid, dim3(C::TH), 0, s, e0,
                                           e1, 0, dmat_of<N, T>(tab), (const T*)x, (const T*)y,
                                           (const T*)z, (const T*)u, (const T*)v, (const T*)w,
                                           (T*)q, (T*)om, (T*)qmm, status, b, end);
                   });
    };
    if (n_elem * (int64_t)(8 * sizeof(T) * LineOf<N, T>::NP) > kLineNear)
      go(typename LineQ<N, T, true>::Shape{});
    else
      go(typename LineQ<N, T, false>::Shape{});
  });
  phase_done(pt);
  return hipGetLastError();
}

bool is_mixed(sem_dtype dt) {
  return dt == SEM_MIXED_BF16 || dt == SEM_MIXED_FP16 || dt == SEM_MIXED_BF16X3 ||
         dt == SEM_MIXED_FP16X3;
}

// Mixed-precision kernels (N = 7, FP32 storage).  QC: Q / |omega| / range
// into (o0, o1, qmm); otherwise the gradient of u into (o0, o1, o2).
template <bool QC>
hipError_t mixed_t(sem_dtype dt, const DeviceTables& tab, int64_t n_elem, const void* x,
                   const void* y, const void* z, const void* u, const void* v, const void* w,
                   void* o0, void* o1, void* o2, void* qmm, int32_t* status, hipStream_t s,
                   const PhaseTimer& pt, const CountSink<float>* sink = nullptr) {
  const CountSink<float> none{};
  const CountSink<float>& sk = sink ? *sink : none;
  auto go = [&](auto kern) {
    hipExtLaunchKernelGGL(kern, dim3((unsigned)n_elem), dim3(128), 0, s, pt.start, pt.stop, 0,
                          tab.d64[7], (const float*)x, (const float*)y, (const float*)z,
                          (const float*)u, (const float*)v, (const float*)w, (float*)o0,
                          (float*)o1, (float*)o2, (float*)qmm, status, sk);
  };
  constexpr bool kC = QC;   // counting variants exist with Q only
  switch (dt) {
    case SEM_MIXED_BF16:
      sink ? go(mixed7<kMixBF16, QC, kC>) : go(mixed7<kMixBF16, QC>);
      break;
    case SEM_MIXED_FP16:
      sink ? go(mixed7<kMixFP16, QC, kC>) : go(mixed7<kMixFP16, QC>);
      break;
    case SEM_MIXED_BF16X3:
      sink ? go(mixed7<kMixBF16x3, QC, kC>) : go(mixed7<kMixBF16x3, QC>);
      break;
    case SEM_MIXED_FP16X3:
      sink ? go(mixed7<kMixFP16x3, QC, kC>) : go(mixed7<kMixFP16x3, QC>);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
IsoList<T> make_isolist(int n_iso, const double* iso_host) {
  IsoList<T> iso;
  for (int q = 0; q < SEM_MAX_ISO; ++q) iso.v[q] = q < n_iso ? (T)iso_host[q] : T(0);
  return iso;
}

// Scan of the per-(isovalue, element) counts, totals, then emission.
// Exclusive scan of count int32 values into offs[0..count]: tile sums,
// then the tiles' offsets (folded into the apply kernel when there are at
// most kScanFold tiles, else through a one-workgroup scan of the sums).
// Tiles of 1,024 counts up to kScanSmall counts (always folded), else of
// 4,096 (scan_tile).  `start` and `stop` (may be null) stamp the first and
// the last kernel.
template <int ITEMS, bool PACKED, typename CT>
void scan_kernels_t(const CT* cnt, int64_t count, int64_t* partial, int64_t* offs,
                    int64_t* active, int64_t n_elem, hipStream_t s, hipEvent_t start,
                    hipEvent_t stop) {
  static_assert(kScanThreads * ITEMS == 1024 || kScanThreads * ITEMS == 4096, "scan_tile");
  const int64_t nb = scan_blocks(count);
  hipExtLaunchKernelGGL((scan_reduce<ITEMS, PACKED, CT>), dim3((unsigned)nb), dim3(kScanThreads), 0, s,
                        start, nullptr, 0, cnt, count, partial, active, n_elem);
  if (nb <= kScanFold) {
    hipExtLaunchKernelGGL((scan_apply<true, ITEMS, PACKED, CT>), dim3((unsigned)nb),
                          dim3(kScanThreads), 0, s, nullptr, stop, 0, cnt, count,
                          (const int64_t*)partial, nb, offs);
  } else {
    hipLaunchKernelGGL(scan_partials, dim3(1), dim3(1024), 0, s, partial, nb);
    hipExtLaunchKernelGGL((scan_apply<false, ITEMS, PACKED, CT>), dim3((unsigned)nb),
                          dim3(kScanThreads), 0, s, nullptr, stop, 0, cnt, count,
                          (const int64_t*)partial, nb, offs);
  }
}
// PACKED: count slots (active, if not NULL, receives the n_iso totals of the
// active cells, n_elem slots each); otherwise plain counts.
template <bool PACKED, typename CT>
void scan_kernels(const CT* cnt, int64_t count, int64_t* partial, int64_t* offs,
                  int64_t* active, int64_t n_elem, hipStream_t s, hipEvent_t start,
                  hipEvent_t stop) {
  if (scan_tile(count) == 1024)
    scan_kernels_t<1024 / kScanThreads, PACKED>(cnt, count, partial, offs, active, n_elem, s,
                                                start, stop);
  else
    scan_kernels_t<4096 / kScanThreads, PACKED>(cnt, count, partial, offs, active, n_elem, s,
                                                start, stop);
}

// Workgroups that share the isovalues of each element in the emission and in the
// count kernel: some 2,048 in all (order 9, FP64: the extraction of 8 elements at
// 64 isovalues 319 us with one each, 90 so, of 64 at 16 88 and 43; order 8: the
// isosurfaces of the same 285 and 24, 81 and 24).
unsigned iso_slices(int64_t n_elem, int n_iso) {
  const int64_t k = 2048 / n_elem;
  return (unsigned)(k < 1 ? 1 : k < n_iso ? k : n_iso);
}

// Workgroups of the count kernel: an element per wave while the chip has room
// for more waves, then as many waves as it holds.
unsigned count_grid(int64_t n_elem) {
  const int64_t waves = n_elem < 8192 ? n_elem : 8192;
  return (unsigned)((waves + kCountWaves - 1) / kCountWaves);
}

template <typename T>
hipError_t iso_scan_emit(int order, const DeviceTables& tab, int64_t n_elem, const void* x,
                         const void* y, const void* z, const void* field, int n_iso,
                         const IsoList<T>& iso, const IsoOut<T>& out, uint64_t* keys,
                         int64_t* tri_count, int64_t* active, const IsoWorkspace& ws,
                         int32_t* status, hipStream_t s) {
  const int64_t count = (int64_t)n_iso * n_elem;
  const PhaseTimer ps = phase_timer(SEM_PHASE_SCAN);
  scan_kernels<true>(ws.cnt, count, ws.partial, ws.offs, active, n_elem, s, ps.start, ps.stop);
  phase_done(ps);
  bool any_cap = false;
  for (int q = 0; q < (out.per_iso ? n_iso : 1); ++q) any_cap = any_cap || out.cap[q] > 0;
  if (!any_cap)   // otherwise the emission kernel writes the totals
    hipLaunchKernelGGL((iso_totals<T>), dim3(1), dim3(SEM_MAX_ISO), 0, s, (const int64_t*)ws.offs,
                       n_elem, n_iso, tri_count, out, status);
  if (!any_cap) return hipGetLastError();
  const PhaseTimer pe = phase_timer(SEM_PHASE_EMIT);
  SEM_ORDER_SWITCH(order, {
    launch_parts(n_elem, 1, emit_threads(N), pe.start, pe.stop,
                 [&](int64_t b, int64_t, dim3 grid, hipEvent_t e0, hipEvent_t e1) {
                   grid.y = iso_slices(n_elem, n_iso);
                   auto go = [&](auto kern) {
                     hipExtLaunchKernelGGL(kern, grid, dim3(emit_threads(N)), 0, s, e0, e1, 0, b,
                                           n_elem, (const T*)x, (const T*)y, (const T*)z,
                                           (const T*)field, n_iso, iso, out, tab.ntri,
                                           (const int32_t*)ws.cnt, (const int64_t*)ws.offs, keys,
                                           tri_count, status);
                   };
                   if (grid.y > 1) go(emit_direct<N, T, true>);
                   else go(emit_direct<N, T, false>);
                 });
  });
  phase_done(pe);
  return hipGetLastError();
}

// Two-pass isosurface of a given field: count, exclusive scan, emit.
template <typename T>
hipError_t iso_pipeline(int order, const DeviceTables& tab, int64_t n_elem, const void* x,
                        const void* y, const void* z, const void* field, const void* mm,
                        int n_iso, const double* iso_host, const IsoOut<T>& out,
                        uint64_t* keys, int64_t* tri_count, int64_t* active,
                        uint8_t* case_idx, const IsoWorkspace& ws, int32_t* status,
                        hipStream_t s) {
  const IsoList<T> iso = make_isolist<T>(n_iso, iso_host);
  const PhaseTimer pt = phase_timer(SEM_PHASE_COUNT);
  SEM_ORDER_SWITCH(order, {
    hipExtLaunchKernelGGL((count_waves<N, T>), dim3(count_grid(n_elem), iso_slices(n_elem, n_iso)),
                          dim3(64 * kCountWaves), 0, s, pt.start, pt.stop, 0, n_elem,
                          (const T*)field, (const T*)mm, n_iso, iso, tab.ntri, ws.cnt, active,
                          case_idx);
  });
  phase_done(pt);
  return iso_scan_emit<T>(order, tab, n_elem, x, y, z, field, n_iso, iso, out, keys, tri_count,
                          active, ws, status, s);
}

template <typename T>
hipError_t iso_t(int order, const DeviceTables& tab, int64_t n_elem, const void* x,
                 const void* y, const void* z, const void* field, const void* mm, int n_iso,
                 const double* iso_host, void* tri_xyz, int64_t cap, uint64_t* keys,
                 int64_t* tri_count, int64_t* active, uint8_t* case_idx,
                 const IsoWorkspace& ws, int32_t* status, hipStream_t s) {
  IsoOut<T> out{};
  out.ptr[0] = static_cast<T*>(tri_xyz);
  out.cap[0] = cap;
  out.per_iso = 0;
  return iso_pipeline<T>(order, tab, n_elem, x, y, z, field, mm, n_iso, iso_host, out, keys,
                         tri_count, active, case_idx, ws, status, s);
}

// sem_extract: q and qmm always point at storage (the caller's or the
// workspace's); `ws` is the isosurface part of the workspace.
template <typename T>
hipError_t extract_t(int order, sem_dtype dt, const DeviceTables& tab, int64_t n_elem,
                     const void* x,
                     const void* y, const void* z, const void* u, const void* v,
                     const void* w, void* q, void* om, void* qmm, int n_iso,
                     const double* iso_host, void* const* tri_xyz, const int64_t* cap,
                     int64_t* tri_count, int64_t* active, const IsoWorkspace& ws,
                     int32_t* status, hipStream_t s) {
  IsoOut<T> out{};
  for (int k = 0; k < n_iso; ++k) {
    out.ptr[k] = static_cast<T*>(tri_xyz[k]);
    out.cap[k] = cap[k];
  }
  out.per_iso = 1;
  CountSink<T> sink;
  sink.n_iso = n_iso;
  sink.iso = make_isolist<T>(n_iso, iso_host);
  sink.ntri = tab.ntri;
  sink.cnt = ws.cnt;
  sink.active = active;
  sink.n_elem = n_elem;
  const PhaseTimer pt = phase_timer(SEM_PHASE_QCRIT);
  hipError_t err = hipSuccess;
  bool done = false;
  if constexpr (std::is_same<T, float>::value) {
    if (is_mixed(dt)) {
      err = mixed_t<true>(dt, tab, n_elem, x, y, z, u, v, w, q, om, nullptr, qmm, status, s, pt,
                          &sink);
      done = true;
    }
  }
  if (!done) {
    SEM_ORDER_SWITCH(order, {
      using C = LineOf<N, T>;
      launch_parts(n_elem, C::E, C::TH, pt.start, pt.stop,
                   [&](int64_t b, int64_t, dim3 grid, hipEvent_t e0, hipEvent_t e1) {
                     hipExtLaunchKernelGGL((qcount_lines<N, T, C>), grid, dim3(C::TH), 0, s, e0, e1,
                                           0, dmat_of<N, T>(tab), (const T*)x, (const T*)y,
                                           (const T*)z, (const T*)u, (const T*)v, (const T*)w,
                                           (T*)q, (T*)om, (T*)qmm, status, b, sink);
                   });
    });
  }
  phase_done(pt);
  if (err == hipSuccess) err = hipGetLastError();
  if (err != hipSuccess) return err;
  return iso_scan_emit<T>(order, tab, n_elem, x, y, z, q, n_iso, sink.iso, out, nullptr, tri_count,
                          active, ws, status, s);
}

}  // namespace

int64_t scan_blocks(int64_t count) { return scan_tiles(count); }

size_t batch_plan_bytes(int n_snap) {
  return 256 + (((size_t)n_snap * sizeof(BatchSnap) + 255) & ~size_t(255));
}

int batch_variant_chunk(int order, sem_dtype dt, int variant) {
  if (variant < 3) return 1 << variant;
  return batch_variant_form(variant) == kBatchLines ? line_cfg(order, dt == SEM_F64, 0) : 1;
}

int batch_variant_form(int variant) {
  static const int form[kBatchVariants] = {kBatchChunk, kBatchChunk, kBatchChunk, kBatchLines,
                                           kBatchLines, kBatchLines};
  return form[variant];
}

bool batch_variant_ok(int order, sem_dtype dt, int variant) {
  if (variant < 0 || variant >= kBatchVariants) return false;
  if (order < 1 || order > kMaxOrder) return false;
  if (variant == 4 && (order != 7 || dt != SEM_F64)) return false;
  const int p3 = (order + 1) * (order + 1) * (order + 1);
  return batch_variant_form(variant) != kBatchChunk ||
         batch_variant_chunk(order, dt, variant) * p3 <= kBatchTile / 6;
}

// untuned: the form sem_qcrit itself uses for this order and precision
int batch_default_variant(int order, sem_dtype dt) {
  if (order == 7 && dt == SEM_F64) return 4;
  return (order <= 7 || dt == SEM_F32) ? 3 : 5;
}

template <int N, typename T>
const void* batch_kernel_nt(int form) {
  if (form == kBatchLines)
    return reinterpret_cast<const void*>(&qcrit_batch<N, T, kBatchLines>);
  return form == kBatchChunk ? reinterpret_cast<const void*>(&qcrit_batch<N, T, kBatchChunk>)
                             : nullptr;
}

int batch_threads_of(int n, bool f64, int form) {
  return form == kBatchLines ? line_cfg(n, f64, 1) : kBatchThreads;
}

template <int N>
const void* batch_kernel_n(bool f64, int form) {
  return f64 ? batch_kernel_nt<N, double>(form) : batch_kernel_nt<N, float>(form);
}

const void* batch_kernel(int n, bool f64, int form) {
  switch (n) {
    case 1: return batch_kernel_n<1>(f64, form);
    case 2: return batch_kernel_n<2>(f64, form);
    case 3: return batch_kernel_n<3>(f64, form);
    case 4: return batch_kernel_n<4>(f64, form);
    case 5: return batch_kernel_n<5>(f64, form);
    case 6: return batch_kernel_n<6>(f64, form);
    case 7: return batch_kernel_n<7>(f64, form);
    case 8: return batch_kernel_n<8>(f64, form);
    case 9: return batch_kernel_n<9>(f64, form);
    default: return nullptr;
  }
}

// Workgroups of a persistent launch: every CU filled to the kernel's
// occupancy (queried once per kernel).
int batch_grid(const void* fn, int threads, int cu_count) {
  static std::mutex mu;
  static std::unordered_map<const void*, int> occ;
  std::lock_guard<std::mutex> lock(mu);
  auto it = occ.find(fn);
  if (it == occ.end()) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, threads, 0) != hipSuccess ||
        blocks < 1)
      blocks = 2;
    it = occ.emplace(fn, blocks).first;
  }
  return it->second * cu_count;
}

hipError_t launch_qcrit_batch(sem_dtype dt, const void* plan, unsigned launch_code, int cu_count,
                              int32_t* status, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const BatchHeader* hdr = static_cast<const BatchHeader*>(plan);
  const BatchSnap* snaps =
      reinterpret_cast<const BatchSnap*>(static_cast<const char*>(plan) + 256);
  int first = -1, last = -1;
  for (int n = 1; n <= kMaxOrder; ++n)
    if (launch_code_form(launch_code, n) >= 0) {
      if (first < 0) first = n;
      last = n;
    }
  if (first < 0) return hipSuccess;
  for (int n = first; n <= last; ++n) {
    const int form = launch_code_form(launch_code, n);
    if (form < 0) continue;
    const void* fn = batch_kernel(n, dt == SEM_F64, form);
    if (!fn) return hipErrorInvalidValue;
    hipEvent_t a = n == first ? e0 : nullptr, b = n == last ? e1 : nullptr;
    void* args[] = {const_cast<BatchHeader**>(&hdr), const_cast<BatchSnap**>(&snaps), &status};
    const int threads = batch_threads_of(n, dt == SEM_F64, form);
    const hipError_t err = hipExtLaunchKernel(fn, dim3(batch_grid(fn, threads, cu_count)),
                                              dim3(threads), args, 0, s, a, b, 0);
    if (err != hipSuccess) return err;
  }
  return hipGetLastError();
}

size_t iso_batch_plan_bytes(int n_job) {
  return 256 + (((size_t)n_job * sizeof(IsoBatchJob) + 255) & ~size_t(255));
}

namespace {
template <int N>
hipError_t iso_batch_phase(bool f64, bool emit, const IsoBatchHeader* hdr,
                           const IsoBatchJob* jobs, const DeviceTables& tab,
                           const IsoWorkspace& ws, void* tri, int64_t cap,
                           hipStream_t s, hipEvent_t a, hipEvent_t b) {
  const void* fn;
  if (emit)
    fn = f64 ? reinterpret_cast<const void*>(&iso_batch_emit<N, double>)
             : reinterpret_cast<const void*>(&iso_batch_emit<N, float>);
  else
    fn = f64 ? reinterpret_cast<const void*>(&iso_batch_count<N, double>)
             : reinterpret_cast<const void*>(&iso_batch_count<N, float>);
  const uint8_t* ntri = tab.ntri;
  int32_t* cnt = ws.cnt;
  int64_t* offs = ws.offs;
  void* count_args[] = {&hdr, &jobs, &ntri, &cnt};
  void* emit_args[] = {&hdr, &jobs, &ntri, &cnt, &offs, &tri, &cap};
  // Emission with four times the workgroups the CUs hold at once: the cost of an element
  // varies with its triangles, and with a grid of exactly the resident
  // workgroups the unluckiest one sets the end (measured on the batched
  // benchmark snapshots: 4.54 ms at 1x, 3.58 at 4x, 3.60 at 16x, 3.84 at 64x;
  // 48 separate sem_isosurface calls: 4.4 ms).  Workgroups that start later
  // take the slots the early finishers free.
  const int threads = emit ? emit_threads(N) : 64 * kCountWaves;
  return hipExtLaunchKernel(fn, dim3((emit ? 4 : 1) * batch_grid(fn, threads, tab.cu_count)),
                            dim3(threads), emit ? emit_args : count_args, 0, s, a, b, 0);
}
}  // namespace

hipError_t launch_iso_batch(sem_dtype dt, const DeviceTables& tab, const void* plan,
                            unsigned launch_code, int n_job, int64_t n_slots, void* tri,
                            int64_t cap, int64_t* tri_offset, int64_t* tri_count,
                            int64_t* active, const IsoWorkspace& ws, int32_t* status,
                            hipStream_t s) {
  const IsoBatchHeader* hdr = static_cast<const IsoBatchHeader*>(plan);
  const IsoBatchJob* jobs =
      reinterpret_cast<const IsoBatchJob*>(static_cast<const char*>(plan) + 256);
  const bool f64 = dt == SEM_F64;
  int first = -1, last = -1;
  for (int n = 1; n <= kMaxOrder; ++n)
    if (launch_code >> n & 1u) {
      if (first < 0) first = n;
      last = n;
    }
  for (int pass = 0; pass < 2; ++pass) {
    const PhaseTimer pt = phase_timer(pass == 0 ? SEM_PHASE_COUNT : SEM_PHASE_EMIT);
    for (int n = first; n >= 1 && n <= last; ++n) {
      if (!(launch_code >> n & 1u)) continue;
      hipEvent_t a = n == first ? pt.start : nullptr, b = n == last ? pt.stop : nullptr;
      hipError_t err = hipSuccess;
      switch (n) {
        case 1: err = iso_batch_phase<1>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 2: err = iso_batch_phase<2>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 3: err = iso_batch_phase<3>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 4: err = iso_batch_phase<4>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 5: err = iso_batch_phase<5>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 6: err = iso_batch_phase<6>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 7: err = iso_batch_phase<7>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 8: err = iso_batch_phase<8>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        case 9: err = iso_batch_phase<9>(f64, pass, hdr, jobs, tab, ws, tri, cap, s, a, b); break;
        default: err = hipErrorInvalidValue;
      }
      if (err != hipSuccess) return err;
    }
    phase_done(pt);
    if (pass == 0) {
      // one exclusive scan over every count slot, then the per-(job,
      // isovalue) totals
      const PhaseTimer ps = phase_timer(SEM_PHASE_SCAN);
      scan_kernels<true>(ws.cnt, n_slots, ws.partial, ws.offs, nullptr, 1, s, ps.start, nullptr);
      const unsigned tb = n_job > 0 ? (unsigned)((4 * (int64_t)n_job + 255) / 256) : 1;
      hipExtLaunchKernelGGL(iso_batch_totals, dim3(tb + (active ? 4 * (unsigned)n_job : 0)),
                            dim3(256), 0, s, nullptr, ps.stop, 0, hdr, jobs,
                            (const int32_t*)ws.cnt, (const int64_t*)ws.offs, tri_offset,
                            tri_count, active, (int)tb, cap, status);
      phase_done(ps);
      if (cap <= 0) break;
    }
  }
  return hipGetLastError();
}

hipError_t launch_tune_fill(sem_dtype dt, int order, int64_t n_elem, void* const* f,
                            hipStream_t s) {
  const int64_t p = order + 1, n = n_elem * p * p * p;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (dt == SEM_F64)
    hipLaunchKernelGGL(tune_fill<double>, dim3(blocks), dim3(256), 0, s, order, n_elem,
                       (double*)f[0], (double*)f[1], (double*)f[2], (double*)f[3],
                       (double*)f[4], (double*)f[5]);
  else
    hipLaunchKernelGGL(tune_fill<float>, dim3(blocks), dim3(256), 0, s, order, n_elem,
                       (float*)f[0], (float*)f[1], (float*)f[2], (float*)f[3], (float*)f[4],
                       (float*)f[5]);
  return hipGetLastError();
}

hipError_t launch_flag_scan(const uint8_t* flag, int64_t count, int64_t* partial, int64_t* offs,
                            hipStream_t s) {
  scan_kernels<false>(flag, count, partial, offs, nullptr, 1, s, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_exclusive_scan(const int64_t* cnt, int64_t count, int64_t* partial,
                                 int64_t* offs, hipStream_t s) {
  scan_kernels<false>(cnt, count, partial, offs, nullptr, 1, s, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_exclusive_scan(const int32_t* cnt, int64_t count, int64_t* partial,
                                 int64_t* offs, hipStream_t s) {
  scan_kernels<false>(cnt, count, partial, offs, nullptr, 1, s, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_derivs(int order, sem_dtype dt, const DeviceTables& tab, int64_t n_elem,
                         const void* x, const void* y, const void* z, const void* f, void* gx,
                         void* gy, void* gz, int32_t* status, hipStream_t s) {
  if (is_mixed(dt))
    return mixed_t<false>(dt, tab, n_elem, x, y, z, f, nullptr, nullptr, gx, gy, gz, nullptr,
                          status, s, PhaseTimer{});
  return dt == SEM_F64 ? derivs_t<double>(order, tab, n_elem, x, y, z, f, gx, gy, gz, status, s)
                       : derivs_t<float>(order, tab, n_elem, x, y, z, f, gx, gy, gz, status, s);
}

hipError_t launch_qcrit(int order, sem_dtype dt, const DeviceTables& tab, int64_t n_elem,
                        const void* x, const void* y, const void* z, const void* u,
                        const void* v, const void* w, void* q, void* om, void* qmm,
                        int32_t* status, hipStream_t s) {
  if (is_mixed(dt)) {
    const PhaseTimer pt = phase_timer(SEM_PHASE_QCRIT);
    const hipError_t e =
        mixed_t<true>(dt, tab, n_elem, x, y, z, u, v, w, q, om, nullptr, qmm, status, s, pt);
    phase_done(pt);
    return e;
  }
  return dt == SEM_F64
             ? qcrit_t<double>(order, tab, n_elem, x, y, z, u, v, w, q, om, qmm, status, s)
             : qcrit_t<float>(order, tab, n_elem, x, y, z, u, v, w, q, om, qmm, status, s);
}

hipError_t launch_extract(int order, sem_dtype dt, const DeviceTables& tab, int64_t n_elem,
                          const void* x, const void* y, const void* z, const void* u,
                          const void* v, const void* w, void* q, void* om, void* qmm,
                          int n_iso, const double* iso_host, void* const* tri_xyz,
                          const int64_t* tri_capacity, int64_t* tri_count,
                          int64_t* active_cells, const IsoWorkspace& ws, int32_t* status,
                          hipStream_t s) {
  return dt == SEM_F64
             ? extract_t<double>(order, dt, tab, n_elem, x, y, z, u, v, w, q, om, qmm, n_iso,
                                 iso_host, tri_xyz, tri_capacity, tri_count, active_cells, ws,
                                 status, s)
             : extract_t<float>(order, dt, tab, n_elem, x, y, z, u, v, w, q, om, qmm, n_iso,
                                iso_host, tri_xyz, tri_capacity, tri_count, active_cells, ws,
                                status, s);
}

hipError_t launch_isosurface(int order, sem_dtype dt, const DeviceTables& tab, int64_t n_elem,
                             const void* x, const void* y, const void* z, const void* field,
                             const void* mm, int n_iso, const double* iso_host, void* tri_xyz,
                             int64_t cap, uint64_t* keys, int64_t* tri_count,
                             int64_t* active, uint8_t* case_idx, const IsoWorkspace& ws,
                             int32_t* status, hipStream_t s) {
  if (n_elem == 0) {
    hipLaunchKernelGGL(fill_i64, dim3(1), dim3(64), 0, s, tri_count, n_iso, (int64_t)0);
    if (active) hipLaunchKernelGGL(fill_i64, dim3(1), dim3(64), 0, s, active, n_iso, (int64_t)0);
    return hipGetLastError();
  }
  return dt == SEM_F64
             ? iso_t<double>(order, tab, n_elem, x, y, z, field, mm, n_iso, iso_host, tri_xyz,
                             cap, keys, tri_count, active, case_idx, ws, status, s)
             : iso_t<float>(order, tab, n_elem, x, y, z, field, mm, n_iso, iso_host, tri_xyz,
                            cap, keys, tri_count, active, case_idx, ws, status, s);
}

}  // namespace sem

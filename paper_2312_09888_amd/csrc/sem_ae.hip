// Per-element autoencoder compression of order-7 snapshots (u, v, w, theta)
// for the in-transit hand-off (section 4.2 ships every snapshot to separate
// visualisation nodes; here its bytes shrink first).
//
// Blocks are kept in Morton order: value (i, j, k) of channel c of element e
// at X[e][m][c] with m the bit interleave (i0 j0 k0 i1 j1 k1 i2 j2 k2, from
// the least significant bit).  Then node 8 p + d of a grid is position d =
// dx + 2 dy + 4 dz of the 2^3 patch p of the grid one level coarser, so a
// kernel-2 stride-2 convolution reads each output position's 8 x Cin inputs
// as one contiguous row, and a transposed one writes 8 x Cout contiguous
// outputs: every layer is a plain row-major GEMM
//   conv:  Y[rows][Cout]   = X[rows][8 Cin] W[8 Cin][Cout] + b
//   convT: Y[rows][8 Cout] = X[rows][Cin]   W[Cin][8 Cout] + b (b per Cout)
// with rows = element x output position, and the parameter layouts
// W[(d Cin + i) Cout + o] (conv) and W[(i 8 + d) Cout + o] (convT).
//
// Training: forward, loss and gradient in sem_ae_train.hip, Adam here.
// Initialisation: layer-wise principal components
// from FP64 Gram matrices and a cyclic Jacobi eigensolver.  Compression:
// encode, decode, per-element error check, raw blocks compacted by an
// exclusive scan; decompression reverses it.

#include <cmath>
#include <cstdint>

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "sem_internal.h"

namespace sem {
namespace {

constexpr int kT = 256;

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ __forceinline__ int morton8(int i, int j, int k) {
  int m = 0;
#pragma unroll
  for (int l = 0; l < 3; ++l)
    m |= (((i >> l) & 1) << (3 * l)) | (((j >> l) & 1) << (3 * l + 1)) |
         (((k >> l) & 1) << (3 * l + 2));
  return m;
}

// Several floats of a caller's buffer at once; its alignment is a float's.
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// One DPP move of a 32-bit value; lanes of rows that ROWS leaves out read 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_zero(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}

// Maximum of non-negative, non-NaN values over the wave, in every lane: DPP
// moves within quads (quad_perm [1,0,3,2], [2,3,0,1]), half rows
// (row_half_mirror) and rows (row_mirror), then lane 15 of rows 0 and 2 into
// rows 1 and 3 (row_bcast:15) and lane 31 into rows 2 and 3 (row_bcast:31)
// leave it in lane 63 (0 is neutral for the rows a mask leaves out), which
// is read back as a scalar.  Every lane of the wave must be active.
__device__ __forceinline__ float wave_max_pos(float v) {
  v = fmaxf(v, dpp_or_zero<0xb1, 0xf>(v));
  v = fmaxf(v, dpp_or_zero<0x4e, 0xf>(v));
  v = fmaxf(v, dpp_or_zero<0x141, 0xf>(v));
  v = fmaxf(v, dpp_or_zero<0x140, 0xf>(v));
  v = fmaxf(v, dpp_or_zero<0x142, 0xa>(v));
  v = fmaxf(v, dpp_or_zero<0x143, 0xc>(v));
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

template <typename T>
__device__ __forceinline__ T block_max_pos(T v, T* red) {
  // max of non-negative values over a 256-thread block
  if constexpr (std::is_same<T, float>::value) {
    v = wave_max_pos(v);
  } else {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const T o = __shfl_xor(v, off);
      v = o > v ? o : v;
    }
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  T r = red[0];
#pragma unroll
  for (int i = 1; i < kT / 64; ++i) r = red[i] > r ? red[i] : r;
  __syncthreads();
  return r;
}

__global__ void fill_f32(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// blocks: per-channel element maxima, normalised Morton blocks
// ---------------------------------------------------------------------------

// s[e][c] = max |f_c| over element e
__global__ void __launch_bounds__(kT)
ae_scales(int64_t e_begin, const float* __restrict__ u, const float* __restrict__ v,
          const float* __restrict__ w, const float* __restrict__ th, float* __restrict__ scale) {
  __shared__ float red[kT / 64];
  const int64_t e = e_begin + blockIdx.x;
  const float* f[4] = {u, v, w, th};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float* src = f[c] + e * 512;
    const float a = fabsf(src[threadIdx.x]), b = fabsf(src[threadIdx.x + 256]);
    const float m = block_max_pos(a > b ? a : b, red);
    if (threadIdx.x == 0) scale[e * 4 + c] = m;
  }
}

// gmax_bits[c] = bits of max_e s[e][c] (non-negative floats order like their
// bit patterns): one atomic per block and channel
__global__ void __launch_bounds__(kT)
gmax_k(const float* __restrict__ scale, int64_t n, uint32_t* __restrict__ gmax_bits) {
  // the four channels of an entry by one 16-byte load, reduced together
  __shared__ float red[kT / 64][4];
  float m[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const float4 x = reinterpret_cast<const float4*>(scale)[e];
    m[0] = x.x > m[0] ? x.x : m[0];
    m[1] = x.y > m[1] ? x.y : m[1];
    m[2] = x.z > m[2] ? x.z : m[2];
    m[3] = x.w > m[3] ? x.w : m[3];
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) m[c] = wave_max_pos(m[c]);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int c = 0; c < 4; ++c) red[w][c] = m[c];
  __syncthreads();
  if (threadIdx.x < 4) {
    float r = red[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < kT / 64; ++i) r = red[i][threadIdx.x] > r ? red[i][threadIdx.x] : r;
    atomicMax(gmax_bits + threadIdx.x, __float_as_uint(r));
  }
}

// X[r][m][c] = f_c(node of m) / s[e][c] (0 for a vanishing channel), element
// e = e_begin + r.
__global__ void __launch_bounds__(kT)
ae_pack(int64_t e_begin, const float* __restrict__ u, const float* __restrict__ v,
        const float* __restrict__ w, const float* __restrict__ th,
        const float* __restrict__ scale, float* __restrict__ x) {
  const int64_t e = e_begin + blockIdx.x;
  const float* f[4] = {u, v, w, th};
  float s[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) s[c] = scale[e * 4 + c];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = threadIdx.x + 256 * h;
    const int m = morton8(n & 7, (n >> 3) & 7, n >> 6);
    float4 o;
    float* op = reinterpret_cast<float*>(&o);
#pragma unroll
    for (int c = 0; c < 4; ++c) op[c] = s[c] > 0.f ? f[c][e * 512 + n] / s[c] : 0.f;
    reinterpret_cast<float4*>(x + (int64_t)blockIdx.x * 2048)[m] = o;
  }
}

// ---------------------------------------------------------------------------
// One layer as a GEMM (FP32)
// ---------------------------------------------------------------------------
//
// C[m][n] = sum_k A[m][k] B[k][n] + bias[n % bias_mod], row-major operands;
// 16-deep k steps.

constexpr int kBK = 16;

struct GemmArgs {
  int64_t M;
  int N;
  int K;
  const float* A;        // [M][K]
  const float* B;        // [K][N]
  float* C;              // [M][N]
  const float* bias;
  int bias_mod;
};

// BM x BN tile on the matrix cores: four waves in a 2 x 2 arrangement, each
// with a (BM / 2) x (BN / 2) block of 16 x 16 tiles of
// v_mfma_f32_16x16x4f32 (FP32 products, FP32 sums).  Lane l of a wave
// holds A(row l % 16, k l / 16) and B(k l / 16, col l % 16) of a 4-deep
// step, and C rows 4 (l / 16) + r, r < 4, of column l % 16.  The k-major
// LDS tiles have rows of BM + 16 (BN + 16) floats, so the four k rows of a
// step fall on disjoint bank halves.  Narrow layers (N = 32) use 128 x 32
// tiles.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int BM, int BN>
__global__ void __launch_bounds__(kT) gemm_f32(GemmArgs g) {
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 16, FN = WN / 16;
  __shared__ float As[kBK][BM + 16];
  __shared__ float Bs[kBK][BN + 16];
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int wm = (wave & 1) * WM, wn = (wave >> 1) * WN;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * BM;   // rows on x: up to 2^31 - 1 tiles
  const int n0 = blockIdx.y * BN;
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < g.K; k0 += kBK) {
#pragma unroll
    for (int q = 0; q < (BM * kBK) / kT; ++q) {
      const int idx = t + q * kT, kk = idx % kBK, mm = idx / kBK;
      const int64_t m = m0 + mm;
      As[kk][mm] = (m < g.M && k0 + kk < g.K) ? g.A[m * g.K + k0 + kk] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < (BN * kBK) / kT; ++q) {
      const int idx = t + q * kT, nn = idx % BN, kk = idx / BN;
      const int n = n0 + nn;
      Bs[kk][nn] = (n < g.N && k0 + kk < g.K) ? g.B[(int64_t)(k0 + kk) * g.N + n] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 4) {
      float a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = As[kk + lk][wm + 16 * i + lr];
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = Bs[kk + lk][wn + 16 * j + lr];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = m0 + wm + 16 * i + 4 * lk + r;
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = n0 + wn + 16 * j + lr;
        if (n >= g.N) continue;
        float v = acc[i][j][r];
        v += g.bias[n % g.bias_mod];
        g.C[m * g.N + n] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Adam, binary16 conversion
// ---------------------------------------------------------------------------

__global__ void adam_step(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                          float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                          float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// W^T: out[c][r] = in[r][c]
__global__ void transpose_f32(const float* __restrict__ in, int rows, int cols,
                              float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= (int64_t)rows * cols) return;
  const int r = (int)(i / cols), c = (int)(i % cols);
  out[(int64_t)c * rows + r] = in[i];
}

__global__ void identity_f32(float* __restrict__ w, int n) {
  const int i = blockIdx.x * kT + threadIdx.x;
  if (i < n * n) w[i] = (i / n == i % n) ? 1.f : 0.f;
}

// ---------------------------------------------------------------------------
// principal components: FP64 Gram matrix and cyclic Jacobi
// ---------------------------------------------------------------------------

// part[z][i][j] = sum over rows of slice z of a[r][i] a[r][j]  (32 x 32 tiles)
__global__ void __launch_bounds__(kT)
gram_f64(const float* __restrict__ a, int64_t rows, int k, int64_t rows_per,
         double* __restrict__ part) {
  __shared__ double Ai[32][33];
  __shared__ double Aj[32][33];
  const int i0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
  const int t = threadIdx.x;
  const int ti = t & 31, tj4 = (t >> 5) * 4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t r0 = (int64_t)blockIdx.z * rows_per;
  const int64_t r1 = r0 + rows_per < rows ? r0 + rows_per : rows;
  for (int64_t rb = r0; rb < r1; rb += 32) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = t + q * kT;            // 32 rows x 32 columns
      const int rr = idx >> 5, cc = idx & 31;
      const int64_t r = rb + rr;
      Ai[rr][cc] = r < r1 ? (double)a[r * k + i0 + cc] : 0.0;
      Aj[rr][cc] = r < r1 ? (double)a[r * k + j0 + cc] : 0.0;
    }
    __syncthreads();
#pragma unroll 8
    for (int rr = 0; rr < 32; ++rr) {
      const double ai = Ai[rr][ti];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = fma(ai, Aj[rr][tj4 + q], acc[q]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    part[(int64_t)blockIdx.z * k * k + (int64_t)(i0 + ti) * k + j0 + tj4 + q] = acc[q];
}

__global__ void sum_splits_f64(const double* __restrict__ part, int64_t n, int splits,
                               double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int z = 0; z < splits; ++z) s += part[(int64_t)z * n + i];
  out[i] = s;
}

// Cyclic Jacobi on the symmetric n x n matrix a (n even, in place): each
// round rotates the n/2 disjoint pairs (p, q) of the round-robin tournament
// ordering at once, a <- J^T a J, v <- v J, with the rotation that zeroes
// a_pq (t = sign(th) / (|th| + sqrt(th^2 + 1)), th = (a_qq - a_pp) /
// (2 a_pq); Rutishauser's formulas, e.g. Golub & Van Loan, Matrix
// Computations, section 8.5).  Sweeps of n - 1 rounds repeat until the
// off-diagonal mass (sum of squares) is below 1e-28 of the total, or below
// 1e-20 and no longer falling fourfold per sweep (the rounding floor of a
// large matrix), or 40 sweeps.
//
// A round is two launches over the whole GPU: jacobi_rot computes the n/2
// rotations from a (one workgroup), jacobi_apply updates every 2 x 2 block
// (rows of pair i, columns of pair j) of a as R_i^T A_ij R_j and every
// row's pair columns of v, one thread each; the convergence test
// (jacobi_check) runs once per sweep.
constexpr int kJacobiThreads = 1024;
constexpr int kJacobiMaxN = 512;

struct JacobiState {
  double prev_off;
  int done;
  int sweep;
};

__global__ void jacobi_init(int n, double* __restrict__ v, JacobiState* __restrict__ st) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < (int64_t)n * n) v[i] = (i / n == i % n) ? 1.0 : 0.0;
  if (i == 0) {
    st->prev_off = 0.0;
    st->done = 0;
    st->sweep = 0;
  }
}

// pairs and rotations of round r: pq[2i], pq[2i + 1] = p < q; cs[2i] = c,
// cs[2i + 1] = s
__global__ void __launch_bounds__(kT)
jacobi_rot(int n, int r, const double* __restrict__ a, int* __restrict__ pq,
           double* __restrict__ cs, const JacobiState* __restrict__ st) {
  if (st->done) return;
  const int half = n / 2;
  for (int i = threadIdx.x; i < half; i += kT) {
    const int x = i == 0 ? 0 : 1 + (i - 1 + r) % (n - 1);
    const int y = 1 + (n - 2 - i + r) % (n - 1);
    const int p = x < y ? x : y, q = x < y ? y : x;
    const double apq = a[(int64_t)p * n + q];
    double c = 1.0, sn = 0.0;
    if (apq != 0.0) {
      const double th = (a[(int64_t)q * n + q] - a[(int64_t)p * n + p]) / (2.0 * apq);
      const double tt = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
      c = 1.0 / sqrt(tt * tt + 1.0);
      sn = tt * c;
    }
    pq[2 * i] = p;
    pq[2 * i + 1] = q;
    cs[2 * i] = c;
    cs[2 * i + 1] = sn;
  }
}

// Column rotation of pair j: col p <- c col p - s col q, col q <- s col p +
// c col q; row rotation likewise on rows.
__global__ void __launch_bounds__(kT)
jacobi_apply(int n, const int* __restrict__ pq, const double* __restrict__ cs,
             double* __restrict__ a, double* __restrict__ v, const JacobiState* __restrict__ st) {
  if (st->done) return;
  const int half = n / 2;
  const int64_t nblk = (int64_t)half * half;
  for (int64_t w = (int64_t)blockIdx.x * kT + threadIdx.x; w < nblk + (int64_t)n * half;
       w += (int64_t)gridDim.x * kT) {
    if (w < nblk) {
      const int bi = (int)(w / half), bj = (int)(w % half);
      const int pi = pq[2 * bi], qi = pq[2 * bi + 1], pj = pq[2 * bj], qj = pq[2 * bj + 1];
      const double ci = cs[2 * bi], si = cs[2 * bi + 1], cj = cs[2 * bj], sj = cs[2 * bj + 1];
      double* rp = a + (int64_t)pi * n;
      double* rq = a + (int64_t)qi * n;
      const double x00 = rp[pj], x01 = rp[qj], x10 = rq[pj], x11 = rq[qj];
      const double y00 = cj * x00 - sj * x01, y01 = sj * x00 + cj * x01;
      const double y10 = cj * x10 - sj * x11, y11 = sj * x10 + cj * x11;
      rp[pj] = ci * y00 - si * y10;
      rq[pj] = si * y00 + ci * y10;
      rp[qj] = ci * y01 - si * y11;
      rq[qj] = si * y01 + ci * y11;
    } else {
      const int64_t u = w - nblk;
      const int row = (int)(u / half), bj = (int)(u % half);
      const int pj = pq[2 * bj], qj = pq[2 * bj + 1];
      const double cj = cs[2 * bj], sj = cs[2 * bj + 1];
      double* vr = v + (int64_t)row * n;
      const double vp = vr[pj], vq = vr[qj];
      vr[pj] = cj * vp - sj * vq;
      vr[qj] = sj * vp + cj * vq;
    }
  }
}

// Convergence test before sweep st->sweep (one workgroup): sets st->done.
__global__ void __launch_bounds__(kJacobiThreads)
jacobi_check(int n, const double* __restrict__ a, JacobiState* __restrict__ st) {
  __shared__ double red[2][kJacobiThreads / 64];
  const int t = threadIdx.x;
  if (st->done) return;
  double off = 0.0, tot = 0.0;
  for (int64_t i = t; i < (int64_t)n * n; i += kJacobiThreads) {
    const double x = a[i] * a[i];
    tot += x;
    if (i / n != i % n) off += x;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    off += __shfl_xor(off, o);
    tot += __shfl_xor(tot, o);
  }
  if ((t & 63) == 0) {
    red[0][t >> 6] = off;
    red[1][t >> 6] = tot;
  }
  __syncthreads();
  if (t == 0) {
    double so = 0.0, stot = 0.0;
    for (int i = 0; i < kJacobiThreads / 64; ++i) {
      so += red[0][i];
      stot += red[1][i];
    }
    const int sweep = st->sweep;
    st->done = !(so > 1e-28 * stot) ||
               (sweep > 0 && so >= 0.25 * st->prev_off && so <= 1e-20 * stot) || sweep >= 40;
    st->prev_off = so;
    if (!st->done) st->sweep = sweep + 1;
  }
}

// The r largest eigenvalues (diagonal of a) in decreasing order into lam and
// their eigenvectors (columns of v) into w[k][rank] (FP32; sign chosen so
// that the entry of largest magnitude, first on ties, is positive).
__global__ void __launch_bounds__(kJacobiThreads)
select_leading(int n, int r, const double* __restrict__ a, const double* __restrict__ v,
               double* __restrict__ lam, float* __restrict__ w) {
  for (int i = threadIdx.x; i < n; i += kJacobiThreads) {
    const double li = a[(int64_t)i * n + i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = a[(int64_t)j * n + j];
      rank += (lj > li) || (lj == li && j < i);
    }
    if (rank >= r) continue;
    if (lam) lam[rank] = li;
    int arg = 0;
    double best = -1.0;
    for (int k = 0; k < n; ++k) {
      const double x = fabs(v[(int64_t)k * n + i]);
      if (x > best) {
        best = x;
        arg = k;
      }
    }
    const double sg = v[(int64_t)arg * n + i] < 0.0 ? -1.0 : 1.0;
    for (int k = 0; k < n; ++k) w[(int64_t)k * r + rank] = (float)(sg * v[(int64_t)k * n + i]);
  }
}

// ---------------------------------------------------------------------------
// compression: error check, raw packing, decompression, modal baseline
// ---------------------------------------------------------------------------

__device__ __forceinline__ float fallback_bound(float s, uint32_t gbits) {
  const float g = __uint_as_float(gbits);
  const float floor_ = 1e-3f * g;
  return 1e-3f * (s > floor_ ? s : floor_);
}

// flag[e] = 1 if any channel's max |f - s xhat| exceeds the bound; element
// e = e_begin + r, xhat[r] in Morton order.
__global__ void __launch_bounds__(kT)
ae_check(int64_t e_begin, const float* __restrict__ u, const float* __restrict__ v,
         const float* __restrict__ w, const float* __restrict__ th,
         const float* __restrict__ scale, const uint32_t* __restrict__ gmax_bits,
         const float* __restrict__ xhat, uint8_t* __restrict__ flag) {
  __shared__ float red[kT / 64];
  const int64_t e = e_begin + blockIdx.x;
  const float* f[4] = {u, v, w, th};
  int bad = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float s = scale[e * 4 + c];
    float err = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = threadIdx.x + 256 * h;
      const int m = morton8(n & 7, (n >> 3) & 7, n >> 6);
      const float r = s * xhat[(int64_t)blockIdx.x * 2048 + m * 4 + c];
      const float d = fabsf(f[c][e * 512 + n] - r);
      err = d > err ? d : err;
    }
    err = block_max_pos(err, red);
    bad |= err > fallback_bound(s, gmax_bits[c]);
  }
  if (threadIdx.x == 0) flag[e] = bad;
}

// raw[offs[e]] = the element's four channels (GLL layout) for flagged e.
// A workgroup takes `per` consecutive elements, wave w the flagged ones of
// w, w + 4, ... (8 KiB each, 16-byte loads and stores).  The number of
// flagged elements goes out as n_raw.
__global__ void __launch_bounds__(kT)
pack_raw(int64_t n_elem, int per, const float* __restrict__ u, const float* __restrict__ v,
         const float* __restrict__ w, const float* __restrict__ th,
         const uint8_t* __restrict__ flag, const int64_t* __restrict__ offs, int64_t cap,
         float* __restrict__ raw, int64_t* __restrict__ n_raw, int32_t* __restrict__ status) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t e0 = (int64_t)blockIdx.x * per;
  const int ne = n_elem - e0 < per ? (int)(n_elem - e0) : per;
  if (blockIdx.x == 0 && t == 0 && n_raw) *n_raw = offs[n_elem];
  const float* f[4] = {u, v, w, th};
  for (int q = wv; q < ne; q += kT / 64) {
    const int64_t e = e0 + q;
    if (!flag[e]) continue;
    const int64_t o = offs[e];
    if (o >= cap) {
      if (lane == 0 && status) atomicOr(status, SEM_FLAG_RAW_OVERFLOW);
      continue;
    }
    f32x4u val[4][2];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        val[c][h] = reinterpret_cast<const f32x4u*>(f[c] + e * 512)[lane + 64 * h];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        reinterpret_cast<f32x4u*>(raw + (o * 4 + c) * 512)[lane + 64 * h] = val[c][h];
  }
}

// fields of elements e_begin + r: raw copy if flagged, else s * xhat
__global__ void __launch_bounds__(kT)
ae_unpack(int64_t e_begin, const float* __restrict__ xhat, const float* __restrict__ scale,
          const uint8_t* __restrict__ flag, const int64_t* __restrict__ offs,
          const float* __restrict__ raw, int64_t raw_count, float* __restrict__ u,
          float* __restrict__ v, float* __restrict__ w, float* __restrict__ th,
          int32_t* __restrict__ status) {
  const int64_t e = e_begin + blockIdx.x;
  float* f[4] = {u, v, w, th};
  const bool flagged = flag && flag[e];
  const int64_t o = flagged ? offs[e] : 0;
  // a flagged element beyond the raw blocks given decodes from its latent
  const bool is_raw = flagged && raw && o < raw_count;
  if (flagged && !is_raw && threadIdx.x == 0 && status)
    atomicOr(status, SEM_FLAG_RAW_OVERFLOW);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float s = scale[e * 4 + c];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = threadIdx.x + 256 * h;
      const int m = morton8(n & 7, (n >> 3) & 7, n >> 6);
      f[c][e * 512 + n] = is_raw ? raw[(o * 4 + c) * 512 + n]
                                 : s * xhat[(int64_t)blockIdx.x * 2048 + m * 4 + c];
    }
  }
}

struct Gll7 {
  float xi[8];
  float l0[8];   // w_n / 2: row 0 of the inverse Legendre Vandermonde matrix
  float l1[8];   // 3 w_n xi_n / 2: row 1
};

// Legendre modal truncation to degrees {0, 1}^3 per channel, coefficients
// stored as binary16 of c / s; reconstruction, fallback flag.
__global__ void __launch_bounds__(kT)
modal_k(const float* __restrict__ u, const float* __restrict__ v, const float* __restrict__ w,
        const float* __restrict__ th, Gll7 g, const uint32_t* __restrict__ gmax_bits,
        const float* __restrict__ scale, uint16_t* __restrict__ coef,
        uint8_t* __restrict__ flag, float* __restrict__ ru, float* __restrict__ rv,
        float* __restrict__ rw, float* __restrict__ rth) {
  __shared__ float red[kT / 64];
  __shared__ float part[kT / 64][8];
  __shared__ float cq[8];
  const int64_t e = blockIdx.x;
  const float* f[4] = {u, v, w, th};
  float* r[4] = {ru, rv, rw, rth};
  int bad = 0;
  for (int c = 0; c < 4; ++c) {
    const float s = scale[e * 4 + c];
    float acc[8] = {};
    float val[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = threadIdx.x + 256 * h;
      const int i = n & 7, j = (n >> 3) & 7, k = n >> 6;
      val[h] = f[c][e * 512 + n];
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const float li = (d & 1) ? g.l1[i] : g.l0[i];
        const float lj = (d & 2) ? g.l1[j] : g.l0[j];
        const float lk = (d & 4) ? g.l1[k] : g.l0[k];
        acc[d] = fmaf(li * lj * lk, val[h], acc[d]);
      }
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      float x = acc[d];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
      if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][d] = x;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
      const int d = threadIdx.x;
      const float cd = part[0][d] + part[1][d] + part[2][d] + part[3][d];
      const __half hq = __float2half_rn(s > 0.f ? cd / s : 0.f);
      if (coef) coef[(e * 4 + c) * 8 + d] = __half_as_ushort(hq);
      cq[d] = s * __half2float(hq);
    }
    __syncthreads();
    float err = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = threadIdx.x + 256 * h;
      const int i = n & 7, j = (n >> 3) & 7, k = n >> 6;
      float rec = 0.f;
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const float pi = (d & 1) ? g.xi[i] : 1.f;
        const float pj = (d & 2) ? g.xi[j] : 1.f;
        const float pk = (d & 4) ? g.xi[k] : 1.f;
        rec = fmaf(cq[d], pi * pj * pk, rec);
      }
      if (r[c]) r[c][e * 512 + n] = rec;
      const float dd = fabsf(val[h] - rec);
      err = dd > err ? dd : err;
    }
    err = block_max_pos(err, red);
    bad |= err > fallback_bound(s, gmax_bits[c]);
  }
  if (threadIdx.x == 0) flag[e] = bad;
}

// ---------------------------------------------------------------------------
// fused compression for the linear network (no tanh)
// ---------------------------------------------------------------------------
//
// With every layer linear, layers 0 and 1 compose into one map per octant
// (256 Morton-ordered inputs of the octant -> 64 outputs), and layers 4 and
// 5 likewise (64 -> the octant's 256 outputs):
//   W01[(d1 32 + d0 4 + c) 64 + o] = sum_j W1[(d1 32 + j) 64 + o] W0[(d0 4 + c) 32 + j]
//   b01[o] = b1[o] + sum_{d1, j} W1[(d1 32 + j) 64 + o] b0[j]
//   W45[i 256 + d4 32 + d5 4 + c] = sum_j W4[(i 8 + d4) 32 + j] W5[(j 8 + d5) 4 + c]
//   b45[d4 32 + d5 4 + c] = b5[c] + sum_j b4[j] W5[(j 8 + d5) 4 + c]
// (the same function, rounded differently).
//
// ae_encode takes elements from the GLL fields to their binary16 latents,
// ae_decode from the latents to the error check (compression) or the fields
// (decompression); no activation goes to memory.  A wave owns whole elements
// from start to end (rows (element, octant) of the matrix-core tiles), so
// after the weights are in LDS no barrier follows.  The weights (64 KB of the
// folded map, 64 KB of the 512 x 32 one) stay in LDS while a persistent
// workgroup walks the elements, laid out so that every lane's operands of
// four column tiles are one conflict-free 16-byte read.
//
// Operands without staging: v_mfma_f32_16x16x4f32 computes D(m, n) with lane
// l holding A(m = l % 16, k = l / 16), B(k = l / 16, n = l % 16) and outputs
// m = 4 (l / 16) + r, n = l % 16.  Weights are the A side, so a lane's column
// n is its own row (element, octant).  Encoder: input k = 4 s + c (s the
// Morton node of the octant, c the channel) is in lane group c for step s, so
// lane (row, c) needs exactly the 4 x 4 x 4 nodes of its octant in channel c:
// 16 direct 16-byte loads, no transposition.  Decoder: output column
// 32 d4 + 4 d5 + c is m = 4 (l / 16) + r with r = c: a lane holds all four
// channels of its nodes.
//
// Bound: the FP32 matrix cores, 2 x 131,072 multiply-adds per element and
// direction (0.11 ms for 65,536 elements at 157 TFLOP/s), with the 8 KB of
// fields per element close behind (0.10 ms at 5.1 TB/s); the vector work
// (layers 2 and 3: 16,384 multiply-adds per element each) hardly overlaps the
// matrix instructions.  65,536 elements: encode 0.21, check 0.23, decode
// 0.28 ms (with raw blocks for 72 % of them: 0.18 ms of traffic).  Four
// elements per workgroup with the tiles transposed through LDS, every wave
// reading every row and the weights coming from L2 took 0.30, 0.32 and
// 0.35 ms.  Sixteen waves of two elements instead of eight of four were
// slower (check 0.28 ms): every weight read then feeds one product.  The sums
// keep their order, so latents, flags and fields are the same bits.

constexpr int kFoldW01 = 0;                        // [step][lane][4 column tiles]
constexpr int kFoldB01 = kFoldW01 + 256 * 64;
constexpr int kFoldW45 = kFoldB01 + 64;            // [4 tile groups][step][lane][4 tiles]
constexpr int kFoldB45 = kFoldW45 + 64 * 256;
constexpr int kFoldW2 = kFoldB45 + 256;            // [k % 64][octant][32]
constexpr int kFoldW3 = kFoldW2 + 512 * 32;        // [i][2][lane][4] (ae_decode)
constexpr int kFoldFloats = kFoldW3 + 32 * 512;
constexpr int kCodecT = 512;                       // threads of a full workgroup
constexpr int kH1Pitch = 36;                       // half a layer-1 output row, padded

__global__ void __launch_bounds__(kT)
ae_fold(const float* __restrict__ prm, int64_t ow0, int64_t ob0, int64_t ow1, int64_t ob1,
        int64_t ow2, int64_t ow3, int64_t ow4, int64_t ob4, int64_t ow5, int64_t ob5,
        float* __restrict__ fold) {
  const int idx = blockIdx.x * kT + threadIdx.x;
  if (idx < kFoldB01) {
    const int j = idx & 3, lane = (idx >> 2) & 63, s = idx >> 8;
    const int o = 16 * j + (lane & 15), r = 4 * s + (lane >> 4), d1 = r / 32, dc = r % 32;
    float acc = 0.f;
    for (int q = 0; q < 32; ++q)
      acc = fmaf(prm[ow1 + (d1 * 32 + q) * 64 + o], prm[ow0 + dc * 32 + q], acc);
    fold[idx] = acc;
  } else if (idx < kFoldW45) {
    const int o = idx - kFoldB01;
    float acc = prm[ob1 + o];
    for (int d1 = 0; d1 < 8; ++d1)
      for (int q = 0; q < 32; ++q)
        acc = fmaf(prm[ow1 + (d1 * 32 + q) * 64 + o], prm[ob0 + q], acc);
    fold[idx] = acc;
  } else if (idx < kFoldB45) {
    const int p = idx - kFoldW45, jj = p & 3, lane = (p >> 2) & 63, s = (p >> 8) & 15;
    const int i = 4 * s + (lane >> 4), col = 64 * (p >> 12) + 16 * jj + (lane & 15);
    const int d4 = col / 32, d5 = (col / 4) % 8, c = col % 4;
    float acc = 0.f;
    for (int q = 0; q < 32; ++q)
      acc = fmaf(prm[ow4 + (i * 8 + d4) * 32 + q], prm[ow5 + (q * 8 + d5) * 4 + c], acc);
    fold[idx] = acc;
  } else if (idx < kFoldW2) {
    const int col = idx - kFoldB45, d5 = (col / 4) % 8, c = col % 4;
    float acc = prm[ob5 + c];
    for (int q = 0; q < 32; ++q) acc = fmaf(prm[ob4 + q], prm[ow5 + (q * 8 + d5) * 4 + c], acc);
    fold[idx] = acc;
  } else if (idx < kFoldW3) {
    const int p = idx - kFoldW2, o = p & 31, oct = (p >> 5) & 7, k = p >> 8;
    fold[idx] = prm[ow2 + (64 * oct + k) * 32 + o];
  } else if (idx < kFoldFloats) {
    const int p = idx - kFoldW3, lane = (p >> 2) & 63, i = p >> 9;
    const int s = 8 * ((lane >> 3) & 1) + 4 * ((p >> 8) & 1) + (p & 3);
    fold[idx] = prm[ow3 + i * 512 + (lane & 7) * 64 + 4 * s + (lane >> 4)];
  }
}

// A workgroup's copy of `n` weights (a multiple of 4) into LDS.
__device__ __forceinline__ void weights_lds(const float* __restrict__ src, float* dst, int n) {
#pragma unroll 8
  for (int q = threadIdx.x; q < n / 4; q += kCodecT)
    reinterpret_cast<f32x4*>(dst)[q] = reinterpret_cast<const f32x4*>(src)[q];
}

// Orders a wave's own LDS accesses (its lanes exchange data without a
// barrier: LDS operations of one wave complete in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// m = max(m, |a|, |b|) in one instruction, for m that is no NaN: a quiet NaN
// counts as smaller.  A signalling one would replace m, so a and b are results
// of arithmetic (loaded values are quieted first).
__device__ __forceinline__ void max_abs(float& m, float a, float b) {
  asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
}

// Node 0 of the lane's octant: octant bits (i2, j2, k2).
__device__ __forceinline__ int octant_node(int oct) {
  return 4 * (oct & 1) + 32 * ((oct >> 1) & 1) + 256 * (oct >> 2);
}

// Fields -> element maxima (scale), per-workgroup channel maxima (gpart) and
// binary16 latents, two elements per wave and pass.
__global__ void __launch_bounds__(kCodecT)
ae_encode(int64_t n_elem, int nw, const float* __restrict__ u, const float* __restrict__ v,
          const float* __restrict__ w, const float* __restrict__ th,
          const float* __restrict__ fold, const float* __restrict__ b2,
          float* __restrict__ scale, float* __restrict__ gpart, uint16_t* __restrict__ latent) {
  __shared__ __align__(16) float s_w01[256 * 64];
  __shared__ __align__(16) float s_w2[512 * 32];
  __shared__ __align__(16) float s_h1[kCodecT / 64][16 * kH1Pitch];   // per wave
  __shared__ float s_max[kCodecT / 64][4];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int el = lr >> 3, oct = lr & 7;
  const float* f = lk == 0 ? u : lk == 1 ? v : lk == 2 ? w : th;   // the lane's channel
  const int64_t step = (int64_t)gridDim.x * nw * 2;
  const int64_t first = ((int64_t)blockIdx.x * nw + wv) * 2;
  // the octant's values in Morton order (bits i0 j0 k0 i1 j1 k1)
  auto load = [&](float(&x)[64], int64_t e0) {
    const int64_t e = e0 + el < n_elem ? e0 + el : n_elem - 1;
    const float* src = f + e * 512 + octant_node(oct);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4u r = *reinterpret_cast<const f32x4u*>(src + 8 * j + 64 * k);
        const int s = 2 * (j & 1) + 4 * (k & 1) + 16 * (j >> 1) + 32 * (k >> 1);
        x[s] = r.x;
        x[s + 1] = r.y;
        x[s + 8] = r.z;
        x[s + 9] = r.w;
      }
  };
  float xa[64], xb[64];
  load(xa, first);
  weights_lds(fold + kFoldW01, s_w01, 256 * 64);
  weights_lds(fold + kFoldW2, s_w2, 512 * 32);
  __syncthreads();
  float* h1 = s_h1[wv];
  const int p = lane >> 3, oq = lane & 7;   // layer 2: octant, output quad
  float top = 0.f;                          // largest value of the lane's channel
  // biases held in registers: a load inside the pass would wait for the
  // fields requested before it
  f32x4 bias[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bias[j] = *reinterpret_cast<const f32x4*>(fold + kFoldB01 + 16 * j + 4 * lk);
    asm volatile("" : "+v"(bias[j]));
  }
  float bias2 = b2[lane & 31];
  asm volatile("" : "+v"(bias2));
  auto pass = [&](float(&x)[64], int64_t e0) {
    // the weights' offsets anew in every pass: the reads stay in it
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));
    const int lane4 = lane_now * 4;
    float mx = 0.f;   // a NaN counts as smaller
#pragma unroll
    for (int s = 0; s < 64; s += 2)
      max_abs(mx, __builtin_canonicalizef(x[s]), __builtin_canonicalizef(x[s + 1]));
    // over the element's octants (lanes of eight): quads, then half rows
    mx = fmaxf(mx, dpp_or_zero<0xb1, 0xf>(mx));
    mx = fmaxf(mx, dpp_or_zero<0x4e, 0xf>(mx));
    mx = fmaxf(mx, dpp_or_zero<0x141, 0xf>(mx));
    top = mx > top ? mx : top;
    if (oct == 0 && e0 + el < n_elem) scale[(e0 + el) * 4 + lk] = mx;
    // normalised by one reciprocal per channel (the latent is checked
    // against the exact encoder to within its binary16 step, and the error
    // check compares the fields with s x_hat, not with x)
    const float inv = mx > 0.f ? 1.f / mx : 0.f;
#pragma unroll
    for (int s = 0; s < 64; ++s) x[s] *= inv;
    // layers 0-1: outputs o = 16 j + 4 lk + r of the lane's row
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 64; ++s) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(&s_w01[s * 256 + lane4]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], x[s], acc[j], 0, 0, 0);
    }
    // layer 2: z[o] = b2[o] + sum_k h1[k] W2[k 32 + o]; lane (p, oq) sums the
    // 64 inputs of octant p for four outputs of both elements, 32 inputs at a
    // time through LDS
    float z[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      wave_lds_fence();
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *reinterpret_cast<f32x4*>(&h1[lr * kH1Pitch + 16 * j + 4 * lk]) =
            acc[2 * h + j] + bias[2 * h + j];
      wave_lds_fence();
#pragma unroll
      for (int k4 = 0; k4 < 8; ++k4) {
        f32x4 hv[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
          hv[q] = *reinterpret_cast<const f32x4*>(&h1[(8 * q + p) * kH1Pitch + 4 * k4]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const f32x4 wk = *reinterpret_cast<const f32x4*>(
              &s_w2[(32 * h + 4 * k4 + k) * 256 + lane4]);
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int o = 0; o < 4; ++o) z[q][o] = fmaf(hv[q][k], wk[o], z[q][o]);
        }
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<f32x4*>(&h1[(8 * q + p) * 32 + 4 * oq]) =
          f32x4{z[q][0], z[q][1], z[q][2], z[q][3]};
    wave_lds_fence();
    const int q = lane >> 5, o = lane & 31;
    float sum = bias2;
#pragma unroll
    for (int s = 0; s < 8; ++s) sum += h1[(8 * q + s) * 32 + o];
    if (e0 + q < n_elem) latent[(e0 + q) * 32 + o] = __half_as_ushort(__float2half_rn(sum));
  };
  // two passes a round, each with the next one's fields in flight (requested
  // without a branch, past the end the last element's again: behind a branch
  // the compiler would wait for them with the current ones)
  // (a small snapshot gives elements to the first nw waves only)
  for (int64_t e0 = wv < nw ? first : n_elem; e0 < n_elem; e0 += 2 * step) {
    load(xb, e0 + step);
    pass(xa, e0);
    if (e0 + step >= n_elem) break;
    load(xa, e0 + 2 * step);
    pass(xb, e0 + step);
  }
  // channel maxima of the workgroup (both elements' lanes of a channel)
  top = fmaxf(top, dpp_or_zero<0x140, 0xf>(top));
  if (lr == 0) s_max[wv][lk] = top;
  __syncthreads();
  if (t < 4) {
    float g = 0.f;
    for (int q = 0; q < kCodecT / 64; ++q) g = s_max[q][t] > g ? s_max[q][t] : g;
    gpart[blockIdx.x * 4 + t] = g;
  }
}

// Exchange between lanes 16 apart (odd rows of a with even rows of b).
__device__ __forceinline__ void swap_rows16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// The 32 latents of element e as 16 words, two halves a word.  The address is
// the same in every lane, so these become scalar loads, and those drop the two
// low address bits: `words` is the caller's pointer rounded down to a multiple
// of four, and latents that begin `shift` bits into it are moved into place.
// (The rounding is done on the host: here it would hide from the compiler that
// nothing writes to the latents, and the loads would be vector loads.)
__device__ __forceinline__ void latent_words(const uint32_t* __restrict__ words, int shift,
                                             int64_t e, uint32_t (&z)[16]) {
  const uint32_t* w = words + e * 16;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = w[i];
  if (shift != 0) {
    const uint32_t last = w[16];   // the rest of the last latent
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint64_t pair = ((uint64_t)(i < 15 ? z[i + 1] : last) << 32) | z[i];
      z[i] = (uint32_t)(pair >> shift);
    }
  }
}

// Latents -> reconstruction, 2 RT elements per wave and pass.  CHECK: compared
// with the fields (flag_out[e] = some channel exceeds the fallback bound);
// else written to the fields, raw blocks copied for flagged elements.
template <bool CHECK, int RT>
__global__ void __launch_bounds__(kCodecT)
ae_decode(int64_t n_elem, int nw, const uint32_t* __restrict__ latent, int latent_shift,
          const float* __restrict__ scale, const float* __restrict__ gpart, int n_gpart,
          const float* __restrict__ fold,
          const float* __restrict__ b3, const float* __restrict__ iu,
          const float* __restrict__ iv, const float* __restrict__ iw,
          const float* __restrict__ ith, float* __restrict__ ou, float* __restrict__ ov,
          float* __restrict__ ow, float* __restrict__ oth, const uint8_t* __restrict__ flag,
          const int64_t* __restrict__ offs, const float* __restrict__ raw, int64_t raw_count,
          uint8_t* __restrict__ flag_out, int32_t* __restrict__ status) {
  __shared__ __align__(16) float s_w3[32 * 512];
  __shared__ __align__(16) float s_w45[64 * 256];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int el = lr >> 3, oct = lr & 7;
  __shared__ float s_gmax[CHECK ? kCodecT / 64 : 1][4];
  weights_lds(fold + kFoldW3, s_w3, 32 * 512);
  weights_lds(fold + kFoldW45, s_w45, 64 * 256);
  if constexpr (CHECK) {
    // the channels' global maxima from the encoder's workgroups (<= kCodecT)
    float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < n_gpart) g = reinterpret_cast<const float4*>(gpart)[t];
    g.x = wave_max_pos(g.x);
    g.y = wave_max_pos(g.y);
    g.z = wave_max_pos(g.z);
    g.w = wave_max_pos(g.w);
    if (lane == 0) *reinterpret_cast<float4*>(s_gmax[wv]) = g;
  }
  __syncthreads();
  // the lane's nodes: i pair from its octant and (after the exchange) the
  // parity of lk, j0 from lk; the tile index gives j1, k0 and k1
  const int node0 = octant_node(oct) + 2 * (lk & 1) + 8 * (lk >> 1);
  const int64_t step = (int64_t)gridDim.x * nw * (2 * RT);
  // (a small snapshot gives elements to the first nw waves only)
  for (int64_t e0 = wv < nw ? ((int64_t)blockIdx.x * nw + wv) * (2 * RT) : n_elem; e0 < n_elem;
       e0 += step) {
    int64_t e[RT];      // the lane's elements e0 + 2 q + el
    bool ok[RT];
    f32x4u sc[RT];
    uint32_t zw[2 * RT][16];   // every element's latents, two halves a word
#pragma unroll
    for (int q = 0; q < RT; ++q) {
      e[q] = e0 + 2 * q + el;
      ok[q] = e[q] < n_elem;
      if (!ok[q]) e[q] = n_elem - 1;
      // elements with a raw block are not written from their latents
      if constexpr (!CHECK) ok[q] = ok[q] & !((flag[e[q]] != 0) & (offs[e[q]] < raw_count));
      sc[q] = *reinterpret_cast<const f32x4u*>(scale + e[q] * 4);
    }
#pragma unroll
    for (int x = 0; x < 2 * RT; ++x)
      latent_words(latent, latent_shift, e0 + x < n_elem ? e0 + x : n_elem - 1, zw[x]);
    // the weights' offsets anew in every pass: the reads stay in it
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));
    const int lane4 = lane_now * 4;
    // layer 3: of the outputs 4 s + lk (s < 16) of octant oct, this lane sums
    // s = 8 el .. 8 el + 7 for every element (64 lanes, 64 different weights)
    float a[2 * RT][8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float b = b3[4 * (8 * el + s) + lk];
#pragma unroll
      for (int x = 0; x < 2 * RT; ++x) a[x][s] = b;
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      if (i % 4 == 0) asm volatile("" ::: "memory");   // at most eight reads in flight
      float z[2 * RT];
#pragma unroll
      for (int x = 0; x < 2 * RT; ++x) {
        const uint32_t word = zw[x][i >> 1];
        z[x] = __half2float(__ushort_as_half((uint16_t)(i & 1 ? word >> 16 : word & 0xffffu)));
      }
#pragma unroll
      for (int s4 = 0; s4 < 2; ++s4) {
        const f32x4 wi = *reinterpret_cast<const f32x4*>(&s_w3[(i * 2 + s4) * 256 + lane4]);
#pragma unroll
        for (int x = 0; x < 2 * RT; ++x)
#pragma unroll
          for (int s = 0; s < 4; ++s) a[x][4 * s4 + s] = fmaf(z[x], wi[s], a[x][4 * s4 + s]);
      }
    }
    // the lane eight on in the row (row_ror:8) has the other half of this
    // lane's element
    float h3[RT][16];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float other = dpp_or_zero<0x128, 0xf>(el ? a[2 * q][s] : a[2 * q + 1][s]);
        h3[q][s] = el ? other : a[2 * q][s];
        h3[q][8 + s] = el ? a[2 * q + 1][s] : other;
      }
    float worst[RT][4];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c) worst[q][c] = 0.f;
    // layers 4-5, four column tiles at a time: tiles 4 g + jj, whose nodes
    // differ in i1 (jj / 2) and k0 (jj % 2); g gives j1 and k1
#pragma unroll 1
    for (int g = 0; g < 4; ++g) {
      const int node = node0 + 16 * (g & 1) + 128 * (g >> 1);
      f32x2u ref[RT][2][4];
      if constexpr (CHECK) {
#pragma unroll
        for (int q = 0; q < RT; ++q)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const int64_t at = e[q] * 512 + node + 64 * b;
            ref[q][b][0] = *reinterpret_cast<const f32x2u*>(iu + at);
            ref[q][b][1] = *reinterpret_cast<const f32x2u*>(iv + at);
            ref[q][b][2] = *reinterpret_cast<const f32x2u*>(iw + at);
            ref[q][b][3] = *reinterpret_cast<const f32x2u*>(ith + at);
          }
      }
      f32x4 acc[RT][4];
#pragma unroll
      for (int q = 0; q < RT; ++q)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) acc[q][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const f32x4 wv4 = *reinterpret_cast<const f32x4*>(&s_w45[(g * 16 + s) * 256 + lane4]);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int q = 0; q < RT; ++q)
            acc[q][jj] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(wv4[jj], h3[q][s], acc[q][jj], 0, 0, 0);
      }
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const f32x4 b =
            *reinterpret_cast<const f32x4*>(fold + kFoldB45 + 64 * g + 16 * jj + 4 * lk);
#pragma unroll
        for (int q = 0; q < RT; ++q) {
          acc[q][jj][0] = sc[q].x * (acc[q][jj][0] + b[0]);
          acc[q][jj][1] = sc[q].y * (acc[q][jj][1] + b[1]);
          acc[q][jj][2] = sc[q].z * (acc[q][jj][2] + b[2]);
          acc[q][jj][3] = sc[q].w * (acc[q][jj][3] + b[3]);
        }
      }
#pragma unroll
      for (int q = 0; q < RT; ++q)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            // values at i1 = 0 and 1 of this lane's i0 -> neighbours i, i + 1
            float lo = acc[q][b][c], hi = acc[q][2 + b][c];
            swap_rows16(lo, hi);
            if constexpr (CHECK) {
              max_abs(worst[q][c], ref[q][b][c].x - lo, ref[q][b][c].y - hi);
            } else if (ok[q]) {
              float* out = c == 0 ? ou : c == 1 ? ov : c == 2 ? ow : oth;
              *reinterpret_cast<f32x2u*>(out + e[q] * 512 + node + 64 * b) = f32x2u{lo, hi};
            }
          }
    }
    if constexpr (CHECK) {
#pragma unroll
      for (int q = 0; q < RT; ++q) {
        int bad = 0;
        const float s4[4] = {sc[q].x, sc[q].y, sc[q].z, sc[q].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          // over the element's lanes: octants, then lk
          float m = worst[q][c];
          m = fmaxf(m, dpp_or_zero<0xb1, 0xf>(m));
          m = fmaxf(m, dpp_or_zero<0x4e, 0xf>(m));
          m = fmaxf(m, dpp_or_zero<0x141, 0xf>(m));
          m = fmaxf(m, __shfl_xor(m, 16));
          m = fmaxf(m, __shfl_xor(m, 32));
          float gm = 0.f;
          for (int w = 0; w < kCodecT / 64; ++w) gm = fmaxf(gm, s_gmax[w][c]);
          bad |= m > fallback_bound(s4[c], __float_as_uint(gm));
        }
        if (ok[q] && oct == 0 && lk == 0) flag_out[e[q]] = (uint8_t)bad;
      }
    } else {
      // flagged elements: their raw blocks, by the whole wave
      for (int x = 0; x < 2 * RT; ++x) {
        const int64_t ex = e0 + x;
        if (ex >= n_elem || !flag[ex]) continue;
        const int64_t o = offs[ex];
        if (o >= raw_count) {
          // beyond the raw blocks given: decoded from its latent
          if (lane == 0 && status) atomicOr(status, SEM_FLAG_RAW_OVERFLOW);
          continue;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float* out = (c == 0 ? ou : c == 1 ? ov : c == 2 ? ow : oth) + ex * 512;
          const float* src = raw + (o * 4 + c) * 512;
#pragma unroll
          for (int h = 0; h < 2; ++h)
            reinterpret_cast<f32x4u*>(out)[lane + 64 * h] =
                reinterpret_cast<const f32x4u*>(src)[lane + 64 * h];
        }
      }
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct Layer {
  bool conv;
  int cin, cout;
  int64_t w_off, b_off;
};

constexpr int kLayers = 6;
const Layer* layers() {
  static Layer L[kLayers];
  static bool init = false;
  if (!init) {
    const int spec[kLayers][3] = {{1, 4, 32}, {1, 32, 64}, {1, 64, 32},
                                  {0, 32, 64}, {0, 64, 32}, {0, 32, 4}};
    int64_t off = 0;
    for (int l = 0; l < kLayers; ++l) {
      L[l].conv = spec[l][0] != 0;
      L[l].cin = spec[l][1];
      L[l].cout = spec[l][2];
      L[l].w_off = off;
      off += (int64_t)8 * L[l].cin * L[l].cout;
      L[l].b_off = off;
      off += L[l].cout;
    }
    init = true;
  }
  return L;
}

// GEMM rows of layer l for n elements: output positions of a convolution,
// input positions of a transposed one
int64_t out_rows(int l, int64_t n) {
  static const int pos[kLayers] = {64, 8, 1, 1, 8, 64};
  return n * pos[l];
}
int out_width(int l) {
  const Layer& L = layers()[l];
  return L.conv ? L.cout : 8 * L.cout;
}
int in_width(int l) {
  const Layer& L = layers()[l];
  return L.conv ? 8 * L.cin : L.cin;
}

hipError_t gemm(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.N <= 32) {
    dim3 grid((unsigned)cdiv(g.M, 128), (unsigned)cdiv(g.N, 32));
    hipLaunchKernelGGL((gemm_f32<128, 32>), grid, dim3(kT), 0, s, g);
  } else {
    dim3 grid((unsigned)cdiv(g.M, 64), (unsigned)cdiv(g.N, 64));
    hipLaunchKernelGGL((gemm_f32<64, 64>), grid, dim3(kT), 0, s, g);
  }
  return hipGetLastError();
}

// Y = X W + b for layer l on n elements
hipError_t layer_forward(int l, int64_t n, const float* params, const float* x, float* y,
                         hipStream_t s) {
  const Layer& L = layers()[l];
  GemmArgs g{};
  g.M = out_rows(l, n);
  g.K = in_width(l);
  g.N = out_width(l);
  g.A = x;
  g.B = params + L.w_off;
  g.C = y;
  g.bias = params + L.b_off;
  g.bias_mod = L.cout;
  return gemm(g, s);
}

constexpr int64_t kSplitRows = 512;   // least rows per Gram-matrix slice

// Workspace of a training step
struct AeWs {
  float* act[kLayers];   // act[l + 1] = output of layer l < 5 (act[0] unused)
  float* g;              // output gradient
  float* slices;         // weight-gradient slice per workgroup
  double* lpart;         // loss partial per workgroup
  size_t bytes;
};

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

AeWs ae_layout(void* base, int64_t n) {
  AeWs w{};
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char* q = p ? p + off : nullptr;
    off += align256(b);
    return q;
  };
  for (int l = 0; l < kLayers - 1; ++l)
    w.act[l + 1] = reinterpret_cast<float*>(take((size_t)out_rows(l, n) * out_width(l) * 4));
  w.g = reinterpret_cast<float*>(take((size_t)n * 2048 * 4));
  w.slices = reinterpret_cast<float*>(take((size_t)ae_net_groups(n) * kAeNetParams * 4));
  w.lpart = reinterpret_cast<double*>(take((size_t)ae_net_groups(n) * 8));
  w.bytes = off;
  return w;
}

}  // namespace

int64_t ae_param_count() {
  const Layer& L = layers()[kLayers - 1];
  return L.b_off + L.cout;
}

size_t ae_workspace_bytes(int64_t n) { return ae_layout(nullptr, n).bytes; }

hipError_t launch_ae_scales(int64_t n_elem, const float* const* f, float* scale,
                            uint32_t* gmax_bits, hipStream_t s) {
  if (gmax_bits) hipLaunchKernelGGL(fill_u32, dim3(1), dim3(kT), 0, s, gmax_bits, 4, 0u);
  if (n_elem > 0) {
    hipLaunchKernelGGL(ae_scales, dim3((unsigned)n_elem), dim3(kT), 0, s, (int64_t)0, f[0], f[1],
                       f[2], f[3], scale);
    if (gmax_bits) {
      const int64_t nb = cdiv(n_elem, kT);
      hipLaunchKernelGGL(gmax_k, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(kT), 0, s, scale,
                         n_elem, gmax_bits);
    }
  }
  return hipGetLastError();
}

hipError_t launch_ae_pack(int64_t e_begin, int64_t n, const float* const* f, const float* scale,
                          float* x, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(ae_pack, dim3((unsigned)n), dim3(kT), 0, s, e_begin, f[0], f[1], f[2],
                       f[3], scale, x);
  return hipGetLastError();
}

hipError_t launch_ae_forward(int64_t n, const float* blocks, const float* params, int tanh_mask,
                             float* recon, uint16_t* latent, hipStream_t s) {
  return n <= 0 ? hipSuccess : launch_net_forward(n, blocks, params, tanh_mask, recon, latent, s);
}

hipError_t launch_ae_grad(int64_t n, const float* pool, int64_t n_pool, const int64_t* idx,
                          const float* params, int tanh_mask, int loss_kind, float* grad,
                          float* loss, void* ws, int32_t* status, hipStream_t s) {
  const AeWs w = ae_layout(ws, n);
  if (n <= 0) return hipSuccess;
  return launch_net_grad(n, pool, n_pool, idx, params, tanh_mask, loss_kind, w.act, w.g, w.slices,
                         w.lpart, grad, loss, status, s);
}

hipError_t launch_ae_adam(int64_t n, float* p, const float* g, float* m, float* v, int step,
                          float lr, float b1, float b2, float eps, hipStream_t s) {
  const double c1 = 1.0 / (1.0 - std::pow((double)b1, step));
  const double c2 = 1.0 / (1.0 - std::pow((double)b2, step));
  if (n > 0)
    hipLaunchKernelGGL(adam_step, dim3((unsigned)cdiv(n, kT)), dim3(kT), 0, s, n, p, g, m, v, lr,
                       b1, b2, eps, (float)c1, (float)c2);
  return hipGetLastError();
}

size_t eig_workspace_bytes(int n) {
  return align256((size_t)n * n * 8) * 2 + align256((size_t)n * 8) + align256((size_t)n * 4) +
         256;
}

__global__ void jacobi_sweeps_out(const JacobiState* __restrict__ st, int* __restrict__ out) {
  *out = st->sweep;
}

// Sweeps until jacobi_check sets the done flag: the host reads the flag
// once per sweep (a stream synchronisation), so the launches stop there.
hipError_t jacobi_run(int n, double* a, double* v, int* pq, double* cs, JacobiState* st,
                      int* sweeps, hipStream_t s) {
  hipLaunchKernelGGL(jacobi_init, dim3((unsigned)cdiv((int64_t)n * n, kT)), dim3(kT), 0, s, n,
                     v, st);
  const int64_t work = (int64_t)(n / 2) * (n / 2) + (int64_t)n * (n / 2);
  const unsigned grid = (unsigned)cdiv(work, kT);
  for (int sweep = 0; sweep <= 40; ++sweep) {
    hipLaunchKernelGGL(jacobi_check, dim3(1), dim3(kJacobiThreads), 0, s, n, a, st);
    int done = 0;
    hipError_t e = hipMemcpyAsync(&done, &st->done, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    if (done) break;
    for (int r = 0; r < n - 1; ++r) {
      hipLaunchKernelGGL(jacobi_rot, dim3(1), dim3(kT), 0, s, n, r, a, pq, cs, st);
      hipLaunchKernelGGL(jacobi_apply, dim3(grid), dim3(kT), 0, s, n, pq, cs, a, v, st);
    }
  }
  if (sweeps) hipLaunchKernelGGL(jacobi_sweeps_out, dim3(1), dim3(1), 0, s, st, sweeps);
  return hipGetLastError();
}

hipError_t launch_sym_eig(int n, const double* a_in, int r, double* lam, float* w, void* ws,
                          int* sweeps, hipStream_t s) {
  char* p = static_cast<char*>(ws);
  const size_t nn = align256((size_t)n * n * 8);
  double* a = reinterpret_cast<double*>(p);
  double* v = reinterpret_cast<double*>(p + nn);
  double* cs = reinterpret_cast<double*>(p + 2 * nn);
  int* pq = reinterpret_cast<int*>(p + 2 * nn + align256((size_t)n * 8));
  JacobiState* st = reinterpret_cast<JacobiState*>(p + 2 * nn + align256((size_t)n * 8) +
                                                   align256((size_t)n * 4));
  hipError_t e = hipMemcpyAsync(a, a_in, (size_t)n * n * 8, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = jacobi_run(n, a, v, pq, cs, st, sweeps, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(select_leading, dim3(1), dim3(kJacobiThreads), 0, s, n, r, a, v, lam, w);
  return hipGetLastError();
}

// Gram matrices: at most 64 row slices (each at least kSplitRows rows)
int64_t gram_splits(int64_t rows) {
  const int64_t s = cdiv(rows, kSplitRows);
  return s < 64 ? s : 64;
}

size_t pca_workspace_bytes(int64_t n_pool) {
  const int64_t splits = gram_splits(n_pool * 8);
  return align256((size_t)n_pool * 512 * 4) +                 // layer-1 outputs
         align256((size_t)splits * 512 * 512 * 8) +          // Gram partials
         align256((size_t)512 * 512 * 8) + eig_workspace_bytes(512);
}

hipError_t launch_ae_pca_init(int64_t n_pool, const float* pool, float* params, double* lams,
                              void* ws, hipStream_t s) {
  const Layer* L = layers();
  char* p = static_cast<char*>(ws);
  float* a2 = reinterpret_cast<float*>(p);
  size_t off = align256((size_t)n_pool * 512 * 4);
  double* part = reinterpret_cast<double*>(p + off);
  off += align256((size_t)gram_splits(n_pool * 8) * 512 * 512 * 8);
  double* gram = reinterpret_cast<double*>(p + off);
  off += align256((size_t)512 * 512 * 8);
  void* eig_ws = p + off;
  hipLaunchKernelGGL(fill_f32, dim3((unsigned)cdiv(ae_param_count(), kT)), dim3(kT), 0, s, params,
                     ae_param_count(), 0.f);
  // layer 0: identity on each patch (its input and output rows coincide)
  hipLaunchKernelGGL(identity_f32, dim3((unsigned)cdiv(32 * 32, kT)), dim3(kT), 0, s,
                     params + L[0].w_off, 32);
  // layers 1 and 2: leading eigenvectors of the second moments of their inputs
  const float* in = pool;                    // layer-1 inputs: [n_pool * 8][256]
  for (int l = 1; l <= 2; ++l) {
    const int k = in_width(l), r = L[l].cout;
    const int64_t rows = l == 1 ? n_pool * 8 : n_pool;
    const int splits = (int)gram_splits(rows);
    hipLaunchKernelGGL(gram_f64, dim3(k / 32, k / 32, splits), dim3(kT), 0, s, in, rows, k,
                       cdiv(rows, splits), part);
    hipLaunchKernelGGL(sum_splits_f64, dim3((unsigned)cdiv((int64_t)k * k, kT)), dim3(kT), 0, s,
                       part, (int64_t)k * k, splits, gram);
    hipError_t e = launch_sym_eig(k, gram, r, lams ? lams + (l == 1 ? 0 : 64) : nullptr,
                                  params + L[l].w_off, eig_ws, nullptr, s);
    if (e != hipSuccess) return e;
    if (l == 1) {
      e = layer_forward(1, n_pool, params, pool, a2, s);   // [n_pool * 8][64]
      if (e != hipSuccess) return e;
      in = a2;                               // layer-2 inputs: [n_pool][512]
    }
  }
  // decoder layers: transposes of the encoder layers
  hipLaunchKernelGGL(transpose_f32, dim3((unsigned)cdiv(512 * 32, kT)), dim3(kT), 0, s,
                     params + L[2].w_off, 512, 32, params + L[3].w_off);
  hipLaunchKernelGGL(transpose_f32, dim3((unsigned)cdiv(256 * 64, kT)), dim3(kT), 0, s,
                     params + L[1].w_off, 256, 64, params + L[4].w_off);
  hipLaunchKernelGGL(identity_f32, dim3((unsigned)cdiv(32 * 32, kT)), dim3(kT), 0, s,
                     params + L[5].w_off, 32);
  return hipGetLastError();
}

// Compression in chunks of kChunk elements.
constexpr int64_t kChunk = 16384;
// Workgroups of a codec kernel at most (one per CU).
constexpr int kCodecGroups = 256;

struct CompressWs {
  float* blocks;    // packed elements of a chunk and their reconstruction
  float* recon;     //   (tanh network; the linear one needs neither)
  int64_t* offs;
  int64_t* partial;
  uint32_t* gmax;
  float* fold;      // folded layers 0-1 and 4-5 (linear network)
  float* gpart;     // per-workgroup channel maxima of the fused encoder
  size_t bytes;
};

CompressWs compress_layout(void* base, int64_t n_elem) {
  CompressWs c{};
  const int64_t chunk = n_elem < kChunk ? n_elem : kChunk;
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char* q = p ? p + off : nullptr;
    off += align256(b);
    return q;
  };
  c.blocks = reinterpret_cast<float*>(take((size_t)chunk * 2048 * 4));
  c.recon = reinterpret_cast<float*>(take((size_t)chunk * 2048 * 4));
  c.offs = reinterpret_cast<int64_t*>(take((size_t)(n_elem + 1) * 8));
  c.partial = reinterpret_cast<int64_t*>(take((size_t)(scan_partials_capacity(n_elem) + 1) * 8));
  c.gmax = reinterpret_cast<uint32_t*>(take(16));
  c.fold = reinterpret_cast<float*>(take((size_t)kFoldFloats * 4));
  c.gpart = reinterpret_cast<float*>(take((size_t)kCodecGroups * 4 * 4));
  c.bytes = off;
  return c;
}

hipError_t launch_fold(const float* params, float* fold, hipStream_t s) {
  const Layer* L = layers();
  hipLaunchKernelGGL(ae_fold, dim3((unsigned)cdiv(kFoldFloats, kT)), dim3(kT), 0, s, params,
                     L[0].w_off, L[0].b_off, L[1].w_off, L[1].b_off, L[2].w_off, L[3].w_off,
                     L[4].w_off, L[4].b_off, L[5].w_off, L[5].b_off, fold);
  return hipGetLastError();
}

// Waves per workgroup that take elements, `per` a wave and pass (the weights
// fill the CU's LDS: one workgroup per CU): as few as take the elements in
// one pass, so that a small snapshot spreads over the chip, at most all.
int codec_waves(int64_t n_elem, int per) {
  int w = 1;
  while (w < kCodecT / 64 && n_elem > (int64_t)kCodecGroups * w * per) w *= 2;
  return w;
}
unsigned codec_groups(int64_t n_elem, int per) {
  const int64_t g = cdiv(n_elem, codec_waves(n_elem, per) * per);
  return (unsigned)(g < kCodecGroups ? g : kCodecGroups);
}

// Four elements a wave and pass (every weight read feeds two products) where
// that still fills the chip, else two.
template <bool CHECK>
hipError_t launch_decode(int64_t n_elem, const uint16_t* latent, const float* scale,
                         const CompressWs& c, const float* params, const float* const* in,
                         float* const* out, const uint8_t* flag, const float* raw,
                         int64_t raw_count, uint8_t* flag_out, int32_t* status, hipStream_t s) {
  const int per = n_elem >= (int64_t)kCodecGroups * (kCodecT / 64) * 4 ? 4 : 2;
  const uintptr_t at = reinterpret_cast<uintptr_t>(latent);
  const uint32_t* words = reinterpret_cast<const uint32_t*>(at & ~uintptr_t(3));
  const int shift = 8 * (int)(at & 3);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(codec_groups(n_elem, per)), dim3(kCodecT), 0, s, n_elem,
                       codec_waves(n_elem, per), words, shift, scale, (const float*)c.gpart,
                       (int)codec_groups(n_elem, 2), (const float*)c.fold,
                       params + layers()[3].b_off, in[0], in[1], in[2], in[3], out[0], out[1],
                       out[2], out[3], flag, (const int64_t*)c.offs, raw, raw ? raw_count : 0,
                       flag_out, status);
  };
  if (per == 4) go(ae_decode<CHECK, 2>);
  else go(ae_decode<CHECK, 1>);
  return hipGetLastError();
}

size_t compress_workspace_bytes(int64_t n_elem) { return compress_layout(nullptr, n_elem).bytes; }

hipError_t launch_ae_compress(int64_t n_elem, const float* const* f, const float* params,
                              int tanh_mask, uint16_t* latent, float* scale, uint8_t* flags,
                              float* raw, int64_t raw_cap, int64_t* n_raw, void* ws,
                              int32_t* status, hipStream_t s) {
  CompressWs c = compress_layout(ws, n_elem);
  hipError_t e;
  if (tanh_mask == 0 && n_elem > 0) {
    // linear network: fused encoder and decoder-check
    const unsigned grid = codec_groups(n_elem, 2);
    e = launch_fold(params, c.fold, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ae_encode, dim3(grid), dim3(kCodecT), 0, s, n_elem,
                       codec_waves(n_elem, 2), f[0], f[1], f[2], f[3], c.fold,
                       params + layers()[2].b_off, scale, c.gpart, latent);
    float* const none[4] = {nullptr, nullptr, nullptr, nullptr};
    e = launch_decode<true>(n_elem, latent, scale, c, params, f, none, nullptr, nullptr, 0, flags,
                            status, s);
    if (e != hipSuccess) return e;
  } else {
    e = launch_ae_scales(n_elem, f, scale, c.gmax, s);
    if (e != hipSuccess) return e;
  }
  for (int64_t b = 0; b < n_elem && tanh_mask != 0; b += kChunk) {
    const int64_t n = n_elem - b < kChunk ? n_elem - b : kChunk;
    e = launch_ae_pack(b, n, f, scale, c.blocks, s);
    if (e != hipSuccess) return e;
    e = launch_net_forward(n, c.blocks, params, tanh_mask, c.recon,
                           latent + b * 32, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ae_check, dim3((unsigned)n), dim3(kT), 0, s, b, f[0], f[1], f[2], f[3],
                       scale, c.gmax, c.recon, flags);
  }
  e = launch_flag_scan(flags, n_elem, c.partial, c.offs, s);
  if (e != hipSuccess) return e;
  // elements per workgroup: one a wave up to some 8,192 elements (the copies
  // of a wave follow one another), 16 a wave for large snapshots
  const int64_t four = cdiv(cdiv(n_elem, 2048), 4);
  const int per = 4 * (int)(four < 1 ? 1 : four > 16 ? 16 : four);
  hipLaunchKernelGGL(pack_raw, dim3((unsigned)(n_elem > 0 ? cdiv(n_elem, per) : 1)), dim3(kT), 0,
                     s, n_elem, per, f[0], f[1], f[2], f[3], (const uint8_t*)flags,
                     (const int64_t*)c.offs, raw_cap, raw, n_raw, status);
  return hipGetLastError();
}

hipError_t launch_ae_decompress(int64_t n_elem, const uint16_t* latent, const float* scale,
                                const uint8_t* flags, const float* raw, int64_t raw_count,
                                const float* params, int tanh_mask, float* const* f, void* ws,
                                int32_t* status, hipStream_t s) {
  CompressWs c = compress_layout(ws, n_elem);
  if (n_elem <= 0) return hipSuccess;
  hipError_t e = launch_flag_scan(flags, n_elem, c.partial, c.offs, s);
  if (e != hipSuccess) return e;
  if (tanh_mask == 0) {
    e = launch_fold(params, c.fold, s);
    if (e != hipSuccess) return e;
    const float* const none[4] = {nullptr, nullptr, nullptr, nullptr};
    return launch_decode<false>(n_elem, latent, scale, c, params, none, f, flags, raw, raw_count,
                                nullptr, status, s);
  }
  for (int64_t b = 0; b < n_elem; b += kChunk) {
    const int64_t n = n_elem - b < kChunk ? n_elem - b : kChunk;
    e = launch_net_decode(n, latent + b * 32, params, tanh_mask, c.recon, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ae_unpack, dim3((unsigned)n), dim3(kT), 0, s, b, c.recon, scale,
                       flags, c.offs, raw, raw_count, f[0], f[1], f[2], f[3], status);
  }
  return hipGetLastError();
}

hipError_t launch_modal(int64_t n_elem, const float* const* f, const double* xi,
                        const double* wq, float* scale, uint16_t* coef, uint8_t* flags,
                        float* const* recon, void* ws, hipStream_t s) {
  CompressWs c = compress_layout(ws, n_elem);
  hipError_t e = launch_ae_scales(n_elem, f, scale, c.gmax, s);
  if (e != hipSuccess || n_elem <= 0) return e;
  Gll7 g{};
  for (int i = 0; i < 8; ++i) {
    g.xi[i] = (float)xi[i];
    g.l0[i] = (float)(0.5 * wq[i]);
    g.l1[i] = (float)(1.5 * wq[i] * xi[i]);
  }
  float* r[4] = {nullptr, nullptr, nullptr, nullptr};
  if (recon)
    for (int k = 0; k < 4; ++k) r[k] = recon[k];
  hipLaunchKernelGGL(modal_k, dim3((unsigned)n_elem), dim3(kT), 0, s, f[0], f[1], f[2], f[3], g,
                     c.gmax, scale, coef, flags, r[0], r[1], r[2], r[3]);
  return hipGetLastError();
}

}  // namespace sem

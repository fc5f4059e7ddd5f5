// Training step of the compressor's network (order 7, FP32): forward pass,
// loss and gradient in three launches.
//
// Layer shapes per block (rows x depth -> width), every one a row-major GEMM
// on Morton-ordered blocks:
//   0: 64 x 32 -> 32    1: 8 x 256 -> 64    2: 1 x 512 -> 32   (encoder)
//   3: 1 x 32 -> 512    4: 8 x 64 -> 256    5: 64 x 32 -> 32   (decoder)
// The output of a layer, read row by row, is the input of the next one.
//
// net_forward keeps kNB = 8 blocks per workgroup (eight waves) in LDS from
// the first layer to the loss; net_backward takes the same blocks from the
// output gradient back to layer 0 and writes its weight gradients to a slice
// of its own; net_reduce adds the slices in a fixed order, in FP64.
//
// Bound: 2.56 MFLOP per block and step on the FP32 matrix cores (2,048
// blocks: 33 us at 157 TFLOP/s), and the chain of layers inside a workgroup
// (one workgroup of eight waves per CU; layer 2 is two chains of 128
// dependent steps).  Measured on 2,048 blocks: forward 58 us, backward
// 59 us, reduction 15 us; a step with Adam 151 us.  One launch per layer and
// product (17 GEMMs of 64-row tiles plus 23 small reductions) took 1,795 us:
// the narrow GEMMs left most of the chip idle, and the column sums and their
// one-workgroup folds (85 us a layer) ran one after the other.
//
// Eight blocks per workgroup: a wave owns a block in the layers with 64 rows,
// and the tiles of a pass (92 KB forward, 111 KB backward) fit in LDS; with 16
// they would not, with four the 16-row tiles of layers 2 and 3 would be three
// quarters padding.  A pass of the 256 workgroups then takes 2,048 blocks,
// and the time goes up in steps of a pass: tanh loss and gradient of 1 block 87
// us, 8 99, 256 110 (32 workgroups: the rest of the chip idles, but the chain
// of layers is as long), 1,000 140, 2,048 148, 2,049 239 (a second pass for
// one block), 4,096 280, 16,384 1,183.
//
// All products run as v_mfma_f32_16x16x4f32: lane l holds A(row l % 16,
// k l / 16) and B(k l / 16, column l % 16) of a four-deep step and the
// outputs of rows 4 (l / 16) + r, column l % 16.  The forward sums keep the
// step order k = 0..3, 4..7, ... of a plain loop, so that the binary16 latent
// does not depend on the tiling.  To feed four steps with one 16-byte LDS
// read, activations lie in LDS with each 16 values of a row transposed as
// 4 x 4 (kperm): lane group g then finds its k = g, 4 + g, 8 + g, 12 + g side
// by side.  The backward products have no such order to keep: there a lane
// group takes four neighbouring k instead, so natural rows serve both as A
// and as B operand.  Row pitches are 4 (or 20) modulo 64 words: the 16 rows
// of a 16-byte read fall on different banks.
#include <cmath>
#include <cstdint>

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "sem_internal.h"

namespace sem {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats at any float address (the caller's parameter vector)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kNB = 8;      // blocks per workgroup pass, one per wave
constexpr int kNT = 64 * kNB;

// parameter vector: weights then biases of each layer
constexpr int kW0 = 0, kB0 = kW0 + 32 * 32;
constexpr int kW1 = kB0 + 32, kB1 = kW1 + 256 * 64;
constexpr int kW2 = kB1 + 64, kB2 = kW2 + 512 * 32;
constexpr int kW3 = kB2 + 32, kB3 = kW3 + 32 * 512;
constexpr int kW4 = kB3 + 64, kB4 = kW4 + 64 * 256;
constexpr int kW5 = kB4 + 32, kB5 = kW5 + 32 * 32;
constexpr int kParams = kB5 + 4;

__device__ __forceinline__ constexpr int kperm(int k) {
  return (k & ~15) | ((k & 3) << 2) | ((k >> 2) & 3);
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Four steps of A (four k per lane) with B (four k per lane).
template <class VA, class VB>
__device__ __forceinline__ f32x4 mfma16(const VA& a, const VB& b, f32x4 c) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = mfma4(a[s], b[s], c);
  return c;
}

template <bool TANH>
__device__ __forceinline__ float epi(float v, int tanh_mask, int l) {
  if (TANH && ((tanh_mask >> l) & 1)) v = tanhf(v);
  return v;
}

// A lane's byte offset (from its offset in floats), made anew in every pass:
// what is loaded with it stays inside the pass (hoisted out of the loop, the
// weights of all layers would need some 250 registers and spill).  Accesses
// go to a wave-uniform base plus such an offset: one address register serves
// all of a pattern's loads.
__device__ __forceinline__ uint32_t pass_offset(uint32_t v) {
  v *= 4;
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ float ld(const float* base, uint32_t off) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off);
}
__device__ __forceinline__ f32x4 ld4(const float* base, uint32_t off) {
  return *reinterpret_cast<const f32x4u*>(reinterpret_cast<const char*>(base) + off);
}
__device__ __forceinline__ void st(float* base, uint32_t off, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(base) + off) = v;
}

struct NetArgs {
  int64_t n;
  const float* pool;       // [n_pool][512][4]
  const int64_t* idx;      // [n] or NULL (the first n)
  int64_t n_pool;
  const float* params;
  int tanh_mask;
  int max_loss;
  float inv2;              // 2 / (values or channels of the loss)
  float* act[6];           // outputs of layers 0..4 at [1..5] (NULL: not kept)
  float* g;                // output gradient [n][2048] (NULL: no loss)
  const uint16_t* given;   // binary16 latent [n][32] to decode
  float* recon;            // output [n][2048] or NULL
  uint16_t* latent;        // binary16 latent [n][32] or NULL
  double* lpart;           // loss partial per workgroup
  float* slices;           // weight-gradient slice per workgroup
  int32_t* status;
};

// First value of block b of the batch in the pool; NULL for a bad index.
__device__ __forceinline__ const float* net_input(const NetArgs& a, int64_t b) {
  if (b >= a.n) return nullptr;
  const int64_t src = a.idx ? a.idx[b] : b;
  return src < 0 || src >= a.n_pool ? nullptr : a.pool + src * 2048;
}

constexpr int kP1 = 260;    // pitch of a layer-1 input row (256 values)
constexpr int kP2 = 516;    // layer-2 input row (512)
constexpr int kP3 = 36;     // latent row, layer-5 input row (32)
constexpr int kP4 = 68;     // layer-4 input row (64)

// DECODE starts from given latents: the reconstruction that a compressor
// checked is what its receiver gets, bit for bit, because both come from
// this body.  Decoding 65,536 elements took 1,090 us with a GEMM launch for
// each of the layers 3 to 5, and takes 764; 64 elements 39 and 25.
template <bool TANH, bool DECODE>
__global__ void __launch_bounds__(kNT) net_forward(NetArgs a) {
  // layer-1 input, later the layer-5 input (512 rows x kP3)
  __shared__ __align__(16) float s_big[512 * kP3];
  __shared__ __align__(16) float s_mid[64 * kP4];   // layer-2 input, later layer-4 input
  __shared__ __align__(16) float s_lat[kNB * kP3];
  __shared__ double s_loss[kNB];
  static_assert(512 * kP3 >= 64 * kP1 && 64 * kP4 >= kNB * kP2, "overlaid tiles fit");
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const float* __restrict__ prm = a.params;
  double sq = 0.0;
  for (int64_t c0 = (int64_t)blockIdx.x * kNB; c0 < a.n; c0 += (int64_t)gridDim.x * kNB) {
    const int64_t blk = c0 + w;
    const bool own = blk < a.n;
    const float* __restrict__ x = DECODE ? nullptr : net_input(a, blk);
    if (!DECODE && own && !x && lane == 0 && a.status) atomicOr(a.status, SEM_FLAG_BAD_ID);
    const int ct1 = w & 3, rp1 = 2 * (w >> 2);
    const uint32_t xo = pass_offset(32 * lr + lk), o32 = pass_offset(32 * lk + lr),
                   o1 = pass_offset(64 * lk + 16 * ct1 + lr),
                   o3 = pass_offset(512 * lk + 64 * w + lr),
                   o4 = pass_offset(256 * lk + 32 * w + lr), ob = pass_offset(lr),
                   oc32 = pass_offset(128 * lk + lr), oc64 = pass_offset(256 * lk + lr),
                   oc256 = pass_offset(1024 * lk + lr), oc512 = pass_offset(2048 * lk + lr);
    float wb[2][8];
    if constexpr (!DECODE) {
      // ---- layer 0: the wave's own block, 64 rows x 32 -> 32
      float xa[4][8];
  #pragma unroll
      for (int i = 0; i < 4; ++i)
  #pragma unroll
        for (int s = 0; s < 8; ++s) xa[i][s] = x ? ld(x + 512 * i + 4 * s, xo) : 0.f;
  #pragma unroll
      for (int j = 0; j < 2; ++j)
  #pragma unroll
        for (int s = 0; s < 8; ++s) wb[j][s] = ld(prm + kW0 + 128 * s + 16 * j, o32);
      // layer 1's weights of this wave's column tile, requested early
      float w1[64];
  #pragma unroll
      for (int s = 0; s < 64; ++s) w1[s] = ld(prm + kW1 + 256 * s, o1);
  #pragma unroll
      for (int i = 0; i < 4; ++i) {
  #pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  #pragma unroll
          for (int s = 0; s < 8; ++s) acc = mfma4(xa[i][s], wb[j][s], acc);
          const int col = 16 * j + lr;
          const float bias = ld(prm + kB0 + 16 * j, ob);
  #pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * i + 4 * lk + r;
            const float v = epi<TANH>(acc[r] + bias, a.tanh_mask, 0);
            s_big[(8 * w + (row >> 3)) * kP1 + kperm((row & 7) * 32 + col)] = v;
            if (a.act[1] && own) 
              st(a.act[1] + blk * 2048 + 512 * i + 32 * r + 16 * j, oc32, v);
          }
        }
      }
      __syncthreads();
      // ---- layer 1: 64 rows x 256 -> 64, a column tile and two row tiles a wave
      {
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  #pragma unroll
        for (int c = 0; c < 16; ++c) {
          const f32x4 b = {w1[4 * c], w1[4 * c + 1], w1[4 * c + 2], w1[4 * c + 3]};
  #pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i] = mfma16(*reinterpret_cast<const f32x4*>(
                                &s_big[(16 * (rp1 + i) + lr) * kP1 + 16 * c + 4 * lk]),
                            b, acc[i]);
        }
        const int col = 16 * ct1 + lr;
        const float bias = ld(prm + kB1 + 16 * ct1, ob);
  #pragma unroll
        for (int i = 0; i < 2; ++i)
  #pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int R = 16 * (rp1 + i) + 4 * lk + r;
            const float v = epi<TANH>(acc[i][r] + bias, a.tanh_mask, 1);
            s_mid[(R >> 3) * kP2 + kperm((R & 7) * 64 + col)] = v;
            if (a.act[2] && c0 + (R >> 3) < a.n)
              st(a.act[2] + c0 * 512 + 1024 * (rp1 + i) + 64 * r + 16 * ct1, oc64, v);
          }
      }
    }
    // layer 3's weights of this wave's 64 columns, requested before the wait
    float w3[4][8];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        w3[j][s] = ld(prm + kW3 + 2048 * s + 16 * j, o3);
    if constexpr (DECODE) {
      if (t < kNB * 32) {
        const int b = t >> 5, col = t & 31;
        s_lat[b * kP3 + kperm(col)] =
            c0 + b < a.n ? __half2float(__ushort_as_half(a.given[(c0 + b) * 32 + col])) : 0.f;
      }
    } else {
      __syncthreads();
      // ---- layer 2: 8 rows x 512 -> 32 on two waves (rows 8..15 of the tile
      // repeat rows 0..7; one chain of 128 steps per column tile)
      if (w < 2) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float b0[32], b1[32];
        const float* wp = prm + kW2 + 16 * w;
  #pragma unroll
        for (int s = 0; s < 32; ++s) b0[s] = ld(wp + s * 128, o32);
  #pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q < 3) {
  #pragma unroll
            for (int s = 0; s < 32; ++s) b1[s] = ld(wp + (32 * (q + 1) + s) * 128, o32);
          }
  #pragma unroll
          for (int c = 0; c < 8; ++c) {
            const f32x4 b = {b0[4 * c], b0[4 * c + 1], b0[4 * c + 2], b0[4 * c + 3]};
            acc = mfma16(*reinterpret_cast<const f32x4*>(
                             &s_mid[(lr & 7) * kP2 + 16 * (8 * q + c) + 4 * lk]),
                         b, acc);
          }
          if (q < 3) {
  #pragma unroll
            for (int s = 0; s < 32; ++s) b0[s] = b1[s];
          }
        }
        const int col = 16 * w + lr;
        const float bias = ld(prm + kB2 + 16 * w, ob);
        if (lk < 2) {
  #pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int b = 4 * lk + r;
            const __half h = __float2half_rn(epi<TANH>(acc[r] + bias, a.tanh_mask, 2));
            const float v = __half2float(h);
            s_lat[b * kP3 + kperm(col)] = v;
            if (c0 + b < a.n) {
              if (a.act[3]) a.act[3][(c0 + b) * 32 + col] = v;
              if (a.latent) a.latent[(c0 + b) * 32 + col] = __half_as_ushort(h);
            }
          }
        }
      }
    }
    __syncthreads();
    // ---- layer 3: 8 rows x 32 -> 512, four column tiles a wave
    {
      f32x4 acc[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&s_lat[(lr & 7) * kP3 + 16 * c + 4 * lk]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 b = {w3[j][4 * c], w3[j][4 * c + 1], w3[j][4 * c + 2], w3[j][4 * c + 3]};
          acc[j] = mfma16(v, b, acc[j]);
        }
      }
      if (lk < 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int o = 16 * j + lr;
          const float bias = ld(prm + kB3 + 16 * j, ob);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int b = 4 * lk + r;
            const float v = epi<TANH>(acc[j][r] + bias, a.tanh_mask, 3);
            s_mid[(8 * b + w) * kP4 + kperm(o)] = v;
            if (a.act[4] && c0 + b < a.n)
              st(a.act[4] + (c0 + r) * 512 + 64 * w + 16 * j, oc512, v);
          }
        }
      }
    }
    float w4[2][16];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int s = 0; s < 16; ++s)
        w4[j][s] = ld(prm + kW4 + 1024 * s + 16 * j, o4);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int s = 0; s < 8; ++s) wb[j][s] = ld(prm + kW5 + 128 * s + 16 * j, o32);
    __syncthreads();
    // ---- layer 4: 64 rows x 64 -> 256, two column tiles (position w) a wave
    {
      f32x4 acc[4][2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 v =
              *reinterpret_cast<const f32x4*>(&s_mid[(16 * i + lr) * kP4 + 16 * c + 4 * lk]);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const f32x4 b = {w4[j][4 * c], w4[j][4 * c + 1], w4[j][4 * c + 2], w4[j][4 * c + 3]};
            acc[i][j] = mfma16(v, b, acc[i][j]);
          }
        }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int o = 16 * j + lr;
        const float bias = ld(prm + kB4 + 16 * j, ob);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int R = 16 * i + 4 * lk + r;
            const float v = epi<TANH>(acc[i][j][r] + bias, a.tanh_mask, 4);
            s_big[(8 * R + w) * kP3 + kperm(o)] = v;
            if (a.act[5] && c0 + (R >> 3) < a.n)
              st(a.act[5] + c0 * 2048 + 4096 * i + 256 * r + 32 * w + 16 * j, oc256, v);
          }
      }
    }
    __syncthreads();
    // ---- layer 5 and the loss: the wave's own block, 64 rows x 32 -> 32
    f32x4 y[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) y[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(
            &s_big[(64 * w + 16 * i + lr) * kP3 + 16 * c + 4 * lk]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4 b = {wb[j][4 * c], wb[j][4 * c + 1], wb[j][4 * c + 2], wb[j][4 * c + 3]};
          y[i][j] = mfma16(v, b, y[i][j]);
        }
      }
    const float bias5 = ld(prm + kB5, ob & 15);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = 512 * i + 32 * r + 16 * j;
          const float v = epi<TANH>(y[i][j][r] + bias5, a.tanh_mask, 5);
          if (a.recon && own) st(a.recon + blk * 2048 + at, oc32, v);
          y[i][j][r] = a.g ? v - (x ? ld(x + at, oc32) : 0.f) : 0.f;   // the error from here on
        }
    if (a.g && own) {
      float* __restrict__ g = a.g + blk * 2048;
      if (!a.max_loss) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float d = y[i][j][r];
              st(g + 512 * i + 32 * r + 16 * j, oc32, a.inv2 * d);
              sq += (double)d * d;
            }
      } else {
        // the lane's 32 values belong to channel lr % 4: the channel's largest
        // error and how many nodes reach it, over the lanes of that channel
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float d = fabsf(y[i][j][r]);
              m = d > m ? d : m;
            }
#pragma unroll
        for (int off = 4; off < 64; off <<= 1) {
          const float o = __shfl_xor(m, off);
          m = o > m ? o : m;
        }
        int k = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) k += fabsf(y[i][j][r]) == m;
#pragma unroll
        for (int off = 4; off < 64; off <<= 1) k += __shfl_xor(k, off);
        const float share = m > 0.f ? a.inv2 * m / (float)k : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float d = y[i][j][r];
              st(g + 512 * i + 32 * r + 16 * j, oc32,
                 (m > 0.f && fabsf(d) == m) ? copysignf(share, d) : 0.f);
            }
        if (lane < 4) sq += (double)m * m;
      }
    }
    __syncthreads();   // s_big is written again by the next pass
  }
  if (a.lpart) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (lane == 0) s_loss[w] = sq;
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int i = 0; i < kNB; ++i) s += s_loss[i];
      a.lpart[blockIdx.x] = s;
    }
  }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------

constexpr int kG1 = 276;    // pitch of a layer-4 output / layer-0 output row pair (256 values)
constexpr int kG2 = 84;     // layer-1 output row (64)
constexpr int kG3 = 532;    // layer-3 output row (512)
constexpr int kG4 = 52;     // layer-2 output row (32)

// A 16 x 16 weight-gradient tile at row m0, column n0 of dW [.][ldw] in the
// workgroup's slice: the passes after the first one add to it.
// `off` is the lane's byte offset 4 (4 lk ldw + lr).
__device__ __forceinline__ f32x4 tile_begin(const float* tile, int ldw, uint32_t off,
                                            bool first) {
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
  if (!first) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = ld(tile + r * ldw, off);
  }
  return c;
}
__device__ __forceinline__ void tile_end(float* tile, int ldw, uint32_t off, f32x4 c) {
#pragma unroll
  for (int r = 0; r < 4; ++r) st(tile + r * ldw, off, c[r]);
}
// An input gradient times tanh' = 1 - d^2 of the layer it belongs to.
__device__ __forceinline__ float tanh_grad(float v, float d) { return v * (1.f - d * d); }

template <bool TANH>
__global__ void __launch_bounds__(kNT) net_backward(NetArgs a) {
  __shared__ __align__(16) float s_g1[64 * kG1];    // dL/d(layer 4 output), later layer 0's
  __shared__ __align__(16) float s_g2[64 * kG2];    // layer 1 output
  __shared__ __align__(16) float s_g3[kNB * kG3];   // layer 3 output
  __shared__ __align__(16) float s_g4[kNB * kG4];   // layer 2 output
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const float* __restrict__ prm = a.params;
  float* __restrict__ slice = a.slices + (int64_t)blockIdx.x * kParams;
  const float* __restrict__ act1 = a.act[1];
  const float* __restrict__ act2 = a.act[2];
  const float* __restrict__ act3 = a.act[3];
  const float* __restrict__ act4 = a.act[4];
  const float* __restrict__ act5 = a.act[5];
  f32x4 dw0[2][2], dw5[2][2];
  float db0[2] = {0.f, 0.f}, db1[4] = {0.f, 0.f, 0.f, 0.f}, db2[2] = {0.f, 0.f};
  float db3[4] = {0.f, 0.f, 0.f, 0.f}, db4[2] = {0.f, 0.f}, db5[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) dw0[i][j] = dw5[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bool first = true;
  for (int64_t c0 = (int64_t)blockIdx.x * kNB; c0 < a.n; c0 += (int64_t)gridDim.x * kNB) {
    const int64_t blk = c0 + w;
    const bool own = blk < a.n;
    // rows past the last block: gradients are 0 there, activations are read
    // from the last block (finite where the batch's are)
    const int last = (int)(a.n - 1 - c0 < kNB - 1 ? a.n - 1 - c0 : kNB - 1);
    auto bc = [&](int b) { return c0 + (b < last ? b : last); };
    const uint32_t o32 = pass_offset(32 * lk + lr), oc32 = pass_offset(128 * lk + lr),
                   q32 = pass_offset(32 * lr + 4 * lk), q64 = pass_offset(64 * lr + 4 * lk),
                   q256 = pass_offset(256 * lr + 4 * lk), q512 = pass_offset(512 * lr + 4 * lk),
                   oc64 = pass_offset(256 * lk + lr), oc256 = pass_offset(1024 * lk + lr),
                   oc512 = pass_offset(2048 * lk + lr), o64 = pass_offset(64 * lk + lr),
                   o256 = pass_offset(256 * lk + lr);
    // ---- layer 5 (own block): dW5 = act5^T g, dX5 = g W5^T
    {
      const float* __restrict__ g = a.g + bc(w) * 2048;
      const float* __restrict__ in = act5 + bc(w) * 2048;
#pragma unroll 8
      for (int s = 0; s < 16; ++s) {
        float av[2], bv[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          av[i] = ld(in + 128 * s + 16 * i, o32);
          bv[i] = own ? ld(g + 128 * s + 16 * i, o32) : 0.f;
          db5[i] += bv[i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) dw5[i][j] = mfma4(av[i], bv[j], dw5[i][j]);
      }
      f32x4 b[2][2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          b[j][c] = ld4(prm + kW5 + 512 * j + 16 * c, q32);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 av[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
          av[c] = own ? ld4(g + 512 * i + 16 * c, q32) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < 2; ++c) acc = mfma16(av[c], b[j][c], acc);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * i + 4 * lk + r, col = 16 * j + lr;
            float v = acc[r];
            if (TANH && (a.tanh_mask & 16)) v = tanh_grad(v, ld(in + 512 * i + 32 * r + 16 * j, oc32));
            s_g1[(8 * w + (row >> 3)) * kG1 + (row & 7) * 32 + col] = v;
          }
        }
      }
    }
    __syncthreads();
    // ---- layer 4: dW4 [64][256] (columns 32 w ..), dX4 = g W4^T [64 rows][64]
    {
      f32x4 acc[4][2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = tile_begin(slice + kW4 + 4096 * i + 32 * w + 16 * j, 256, oc256, first);
#pragma unroll 8
      for (int s = 0; s < 16; ++s) {
        const float* in = act4 + bc(s >> 1) * 512 + 256 * (s & 1);
        float av[4], bv[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) av[i] = ld(in + 16 * i, o64);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          bv[j] = s_g1[(4 * s + lk) * kG1 + 32 * w + 16 * j + lr];
          db4[j] += bv[j];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma4(av[i], bv[j], acc[i][j]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          tile_end(slice + kW4 + 4096 * i + 32 * w + 16 * j, 256, oc256, acc[i][j]);
      const int ct = w & 3, rp = 2 * (w >> 2);
      f32x4 dx[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const f32x4 b = ld4(prm + kW4 + 4096 * ct + 16 * c, q256);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          dx[i] = mfma16(*reinterpret_cast<const f32x4*>(
                             &s_g1[(16 * (rp + i) + lr) * kG1 + 16 * c + 4 * lk]),
                         b, dx[i]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int R = 16 * (rp + i) + 4 * lk + r, col = 16 * ct + lr;
          float v = dx[i][r];
          if (TANH && (a.tanh_mask & 8)) v = tanh_grad(v, act4[bc(R >> 3) * 512 + (R & 7) * 64 + col]);
          s_g3[(R >> 3) * kG3 + (R & 7) * 64 + col] = v;
        }
    }
    __syncthreads();
    // ---- layer 3: dW3 [32][512] (columns 64 w ..); dX3 = g W3^T [8 rows][32],
    // the 512-deep sum in four parts over the waves
    {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float bv[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          bv[s] = s_g3[(4 * s + lk) * kG3 + 64 * w + 16 * j + lr];
          db3[j] += bv[s];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          f32x4 acc = tile_begin(slice + kW3 + 8192 * i + 64 * w + 16 * j, 512, oc512, first);
#pragma unroll
          for (int s = 0; s < 2; ++s)
            acc = mfma4(act3[bc(4 * s + lk) * 32 + 16 * i + lr], bv[s], acc);
          tile_end(slice + kW3 + 8192 * i + 64 * w + 16 * j, 512, oc512, acc);
        }
      }
      const int ct = w & 1, q = w >> 1;
      f32x4 dx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 8; ++c)
        dx = mfma16(*reinterpret_cast<const f32x4*>(
                        &s_g3[(lr & 7) * kG3 + 128 * q + 16 * c + 4 * lk]),
                    ld4(prm + kW3 + 8192 * ct + 128 * q + 16 * c, q512),
                    dx);
      // partial sums into the (free) layer-4 tile
      if (lk < 2) {
#pragma unroll
        for (int r = 0; r < 4; ++r) s_g1[(q * 8 + 4 * lk + r) * 32 + 16 * ct + lr] = dx[r];
      }
      __syncthreads();
      if (t < 256) {
        const int b = t >> 5, col = t & 31;
        float v = (s_g1[t] + s_g1[256 + t]) + (s_g1[512 + t] + s_g1[768 + t]);
        if (TANH && (a.tanh_mask & 4)) v = tanh_grad(v, act3[bc(b) * 32 + col]);
        s_g4[b * kG4 + col] = v;
      }
    }
    __syncthreads();
    // ---- layer 2: dW2 [512][32] (rows 64 w ..), dX2 = g W2^T [8 rows][512]
    {
      float bv[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          bv[s][j] = s_g4[(4 * s + lk) * kG4 + 16 * j + lr];
          db2[j] += bv[s][j];
        }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float av[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) av[s] = act2[bc(4 * s + lk) * 512 + 64 * w + 16 * i + lr];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 acc = tile_begin(slice + kW2 + 2048 * w + 512 * i + 16 * j, 32, oc32, first);
#pragma unroll
          for (int s = 0; s < 2; ++s) acc = mfma4(av[s], bv[s][j], acc);
          tile_end(slice + kW2 + 2048 * w + 512 * i + 16 * j, 32, oc32, acc);
        }
      }
      f32x4 av[2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
        av[c] = *reinterpret_cast<const f32x4*>(&s_g4[(lr & 7) * kG4 + 16 * c + 4 * lk]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = 64 * w + 16 * j + lr;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc = mfma16(av[c],
                       ld4(prm + kW2 + 2048 * w + 512 * j + 16 * c, q32),
                       acc);
        if (lk < 2) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int b = 4 * lk + r;
            float v = acc[r];
            if (TANH && (a.tanh_mask & 2)) v = tanh_grad(v, act2[bc(b) * 512 + col]);
            s_g2[(8 * b + w) * kG2 + 16 * j + lr] = v;
          }
        }
      }
    }
    __syncthreads();
    // ---- layer 1: dW1 [256][64] (rows 32 w ..), dX1 = g W1^T [64 rows][256]
    {
      f32x4 acc[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = tile_begin(slice + kW1 + 2048 * w + 1024 * i + 16 * j, 64, oc64, first);
#pragma unroll 8
      for (int s = 0; s < 16; ++s) {
        const float* in = act1 + bc(s >> 1) * 2048 + 1024 * (s & 1) + 32 * w;
        float av[2], bv[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) av[i] = ld(in + 16 * i, o256);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          bv[j] = s_g2[(4 * s + lk) * kG2 + 16 * j + lr];
          db1[j] += bv[j];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mfma4(av[i], bv[j], acc[i][j]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          tile_end(slice + kW1 + 2048 * w + 1024 * i + 16 * j, 64, oc64, acc[i][j]);
      f32x4 b[2][4];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          b[j][c] = ld4(prm + kW1 + 2048 * w + 1024 * j + 16 * c, q64);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 dx[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const f32x4 v =
              *reinterpret_cast<const f32x4*>(&s_g2[(16 * i + lr) * kG2 + 16 * c + 4 * lk]);
#pragma unroll
          for (int j = 0; j < 2; ++j) dx[j] = mfma16(v, b[j][c], dx[j]);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int R = 16 * i + 4 * lk + r, col = 32 * w + 16 * j + lr;
            float v = dx[j][r];
            if (TANH && (a.tanh_mask & 1)) v = tanh_grad(v, act1[bc(R >> 3) * 2048 + (R & 7) * 256 + col]);
            s_g1[R * kG1 + col] = v;
          }
      }
    }
    __syncthreads();
    // ---- layer 0 (own block): dW0 = x^T g
    {
      const float* __restrict__ x = net_input(a, blk);
#pragma unroll 8
      for (int s = 0; s < 16; ++s) {
        const int row = 4 * s + lk;
        float av[2], bv[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          av[i] = x ? ld(x + 128 * s + 16 * i, o32) : 0.f;
          bv[i] = s_g1[(8 * w + (row >> 3)) * kG1 + (row & 7) * 32 + 16 * i + lr];
          db0[i] += bv[i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) dw0[i][j] = mfma4(av[i], bv[j], dw0[i][j]);
      }
    }
    first = false;
    __syncthreads();   // the tiles are written again by the next pass
  }
  // Sums over the waves: the two 32 x 32 weight gradients through s_g1
  // ([wave][1024] each), the bias sums through s_g2 ([wave][sum][16]).
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float* p = s_g1 + 2048 * w + 512 * i + 16 * j + 128 * lk + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[32 * r] = dw0[i][j][r];
        p[1024 + 32 * r] = dw5[i][j][r];
      }
    }
  float sums[16];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    sums[j] = db0[j];
    sums[2 + j] = db2[j];
    sums[4 + j] = db4[j];
    sums[6 + j] = db5[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sums[8 + j] = db1[j];
    sums[12 + j] = db3[j];
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    sums[q] += __shfl_xor(sums[q], 16);
    sums[q] += __shfl_xor(sums[q], 32);
    if (lk == 0) s_g2[(16 * w + q) * 16 + lr] = sums[q];
  }
  __syncthreads();
  for (int q = t; q < 2048; q += kNT) {
    float v = 0.f;
    for (int i = 0; i < kNB; ++i) v += s_g1[2048 * i + q];
    slice[q < 1024 ? kW0 + q : kW5 + q - 1024] = v;
  }
  // sum number q0 + column / 16 of every wave, or of wave 0 where all hold
  // the same rows
  auto bsum = [&](int q0, int col, int waves) {
    float v = 0.f;
    for (int i = 0; i < waves; ++i) v += s_g2[(16 * i + q0 + (col >> 4)) * 16 + (col & 15)];
    return v;
  };
  if (t < 32) slice[kB0 + t] = bsum(0, t, kNB);
  else if (t < 64) slice[kB2 + t - 32] = bsum(2, t - 32, 1);
  else if (t < 96) slice[kB4 + t - 64] = bsum(4, t - 64, kNB);
  else if (t < 100) {
    float v = 0.f;
    for (int d = 0; d < 8; ++d) v += bsum(6, 4 * d + t - 96, kNB);
    slice[kB5 + t - 96] = v;
  } else if (t >= 128 && t < 192) slice[kB1 + t - 128] = bsum(8, t - 128, 1);
  else if (t >= 192 && t < 256) slice[kB3 + t - 192] = bsum(12, t - 192, kNB);
}

// grad[i] = sum of the slices' value i (FP64, fixed order); the loss from the
// workgroups' partials.  64 neighbouring values per workgroup, the slices in
// 16 groups: every wave reads 256 contiguous bytes of a slice.
constexpr int kRedT = 1024;
__global__ void __launch_bounds__(kRedT)
net_reduce(const float* __restrict__ slices, int n_slice, float* __restrict__ grad,
           const double* __restrict__ lpart, double inv_n, float* __restrict__ loss) {
  __shared__ double red[kRedT / 64][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (i < kParams) {
#pragma unroll 8
    for (int z = grp; z < n_slice; z += kRedT / 64) s += (double)slices[(int64_t)z * kParams + i];
  }
  red[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && i < kParams) {
#pragma unroll
    for (int q = 1; q < kRedT / 64; ++q) s += red[q][lane];
    grad[i] = (float)s;
  }
  if (loss && blockIdx.x == 0 && grp == 1) {
    double v = 0.0;
    for (int z = lane; z < n_slice; z += 64) v += lpart[z];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) *loss = (float)(v * inv_n);
  }
}

}  // namespace

static_assert(kAeNetParams == kParams, "the slices' size in the workspace layout");

hipError_t launch_net_forward(int64_t n, const float* blocks, const float* params, int tanh_mask,
                              float* recon, uint16_t* latent, hipStream_t s) {
  NetArgs a{};
  a.n = n;
  a.pool = blocks;
  a.n_pool = n;
  a.params = params;
  a.tanh_mask = tanh_mask;
  a.recon = recon;
  a.latent = latent;
  hipLaunchKernelGGL((tanh_mask ? net_forward<true, false> : net_forward<false, false>),
                     dim3((unsigned)ae_net_groups(n)), dim3(kNT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_net_decode(int64_t n, const uint16_t* latent, const float* params,
                             int tanh_mask, float* recon, hipStream_t s) {
  NetArgs a{};
  a.n = n;
  a.params = params;
  a.tanh_mask = tanh_mask;
  a.given = latent;
  a.recon = recon;
  hipLaunchKernelGGL((net_forward<true, true>), dim3((unsigned)ae_net_groups(n)), dim3(kNT), 0, s,
                     a);
  return hipGetLastError();
}

hipError_t launch_net_grad(int64_t n, const float* pool, int64_t n_pool, const int64_t* idx,
                           const float* params, int tanh_mask, int loss_kind, float* const* act,
                           float* g, float* slices, double* lpart, float* grad, float* loss,
                           int32_t* status, hipStream_t s) {
  NetArgs a{};
  const bool mx = loss_kind == SEM_AE_LOSS_MAX;
  const double values = (mx ? 4.0 : 2048.0) * (double)n;
  a.n = n;
  a.pool = pool;
  a.idx = idx;
  a.n_pool = n_pool;
  a.params = params;
  a.tanh_mask = tanh_mask;
  a.max_loss = mx;
  a.inv2 = (float)(2.0 / values);
  for (int l = 1; l <= 5; ++l) a.act[l] = act[l];
  a.g = g;
  a.lpart = lpart;
  a.slices = slices;
  a.status = status;
  const int groups = ae_net_groups(n);
  hipLaunchKernelGGL((tanh_mask ? net_forward<true, false> : net_forward<false, false>),
                     dim3((unsigned)groups), dim3(kNT), 0, s, a);
  hipLaunchKernelGGL((tanh_mask ? net_backward<true> : net_backward<false>),
                     dim3((unsigned)groups), dim3(kNT), 0, s, a);
  hipLaunchKernelGGL(net_reduce, dim3((kParams + 63) / 64), dim3(kRedT), 0, s, slices, groups,
                     grad, lpart, 1.0 / values, loss);
  return hipGetLastError();
}

}  // namespace sem

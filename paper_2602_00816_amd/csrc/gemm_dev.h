// Device helpers shared by the GEMM kernels.
#pragma once
#include "gemm.h"

namespace fdh {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

__device__ inline int64_t batch_off(int z, int inner_count, int64_t s_outer, int64_t s_inner, int div) {
  return (int64_t)(z / inner_count) * s_outer + (int64_t)((z % inner_count) / div) * s_inner;
}

// Workgroup ids are dealt to the 8 XCDs in turn; renumber them so that each
// XCD takes a contiguous run of tiles (neighbouring tiles share operand rows
// and columns in that XCD's L2).
__device__ inline int xcd_order(int lin, int nb) {
  const int per = nb / 8;
  return lin < per * 8 ? (lin % 8) * per + lin / 8 : lin;
}

template <int N>
__device__ inline void wait_vm() {
  // s_waitcnt with vmcnt = N (bits 3:0 and 15:14), expcnt and lgkmcnt left at their maxima
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Four consecutive outputs at C[idx..idx+3], 16-byte (fp32) or 8-byte (bf16)
// aligned: one vector store, with the residual and previous C read as vectors
template <typename T>
__device__ inline void store_quad(const GemmArgs& a, const float (&x)[4], int64_t idx) {
  if (a.out_type == OUT_F32) {
    float* C = reinterpret_cast<float*>(a.C);
    float4 v = make_float4(x[0], x[1], x[2], x[3]);
    if (a.resid) {
      const float4 r = *reinterpret_cast<const float4*>(a.resid + idx);
      v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
    }
    if (a.beta != 0.f) {
      const float4 c = *reinterpret_cast<const float4*>(C + idx);
      v.x += a.beta * c.x; v.y += a.beta * c.y; v.z += a.beta * c.z; v.w += a.beta * c.w;
    }
    *reinterpret_cast<float4*>(C + idx) = v;
  } else {
    T* C = reinterpret_cast<T*>(a.C);
    if constexpr (sizeof(T) == 2) {
      uint2 u;
      u.x = (uint32_t)f32_to_bf16(x[0]) | ((uint32_t)f32_to_bf16(x[1]) << 16);
      u.y = (uint32_t)f32_to_bf16(x[2]) | ((uint32_t)f32_to_bf16(x[3]) << 16);
      *reinterpret_cast<uint2*>(C + idx) = u;
    } else {
      *reinterpret_cast<float4*>(C + idx) = make_float4(x[0], x[1], x[2], x[3]);
    }
  }
}

// Shared epilogue: accumulator block (i, j) of a wavefront whose 32x32 block
// origin is (rb, cb).  Every MFMA takes the B fragment as its first operand, so
// the block holds C^T in the MFMA output layout: lane l owns row rb + (l & 31)
// of C and, for g = 0..3, the four consecutive columns cb + 8g + 4(l >> 5) + 0..3
// (accumulator elements 4g..4g+3).  Each such quad is stored, and the residual
// or previous C loaded, as one vector where the addresses are aligned.
template <typename T>
__device__ inline void store_block(const GemmArgs& a, const f32x16_t& acc, int64_t coff, int rb, int cb, int lane) {
  const int row = rb + (lane & 31);
  if (row >= a.M) return;
  const int64_t rbase = coff + (int64_t)row * a.ldc;
  // vector path: row starts and column quads aligned for 16-byte (fp32) or
  // 8-byte (bf16) accesses
  const size_t ob = a.out_type == OUT_F32 ? 4 : sizeof(T);
  const bool aligned = a.ldc % 4 == 0 && coff % 4 == 0 && (uintptr_t)a.C % (4 * ob) == 0 &&
                       (!a.resid || (uintptr_t)a.resid % 16 == 0);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int col0 = cb + 8 * g + 4 * (lane >> 5);
    if (col0 >= a.N) continue;
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = min(col0 + r, a.N - 1);
      float badd = 0.f;
      if (a.bias_theta) badd += a.bias_theta_scale * ldf(reinterpret_cast<const T*>(a.bias_theta), col);
      if (a.bias_v) badd += a.bias_v_scale * a.bias_v[col];
      x[r] = a.alpha * acc[4 * g + r] + badd;
    }
    if (aligned && col0 + 3 < a.N) {
      store_quad<T>(a, x, rbase + col0);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (col0 + r >= a.N) break;
        const int64_t idx = rbase + col0 + r;
        float y = x[r];
        if (a.out_type == OUT_F32) {
          float* C = reinterpret_cast<float*>(a.C);
          if (a.resid) y += a.resid[idx];
          if (a.beta != 0.f) y += a.beta * C[idx];
          C[idx] = y;
        } else {
          stf(reinterpret_cast<T*>(a.C), idx, y);
        }
      }
    }
  }
}

// LDS-staged epilogue of one 32x32 block: the wavefront writes its block
// (scaled by alpha) to its own staging area of 32 rows x 36 floats, then reads
// it back so that lane l holds row 8k + (l >> 3), columns 4(l & 7) + 0..3:
// every global access then covers eight rows of 128 contiguous bytes.  The
// caller guarantees the staging area is not in use by the main loop any more.
constexpr int STG_LD = 36;
constexpr int STG_FLOATS = 32 * STG_LD;
// four staging areas fit one ring stage of the DMA kernels (256 x 32 + 128 x 32 bf16 at the smallest)
static_assert(4 * STG_FLOATS * 4 <= (256 + 128) * 32 * 2, "staging areas exceed a ring stage");
static_assert(4 * STG_FLOATS * 4 <= (256 + 256) * 32 * 2, "four blocks of staging exceed a 256 x 256 ring stage");
// (the eight-wavefront kernel gives each pair of wavefronts one 256 x 256 stage, two blocks each)

__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ inline void store_block_lds(const GemmArgs& a, const f32x16_t& acc, int64_t coff, int rb, int cb, int lane,
                                       float* stg) {
  {
    const int wr = lane & 31, wh = lane >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(stg + wr * STG_LD + 8 * g + 4 * wh) =
          make_float4(a.alpha * acc[4 * g], a.alpha * acc[4 * g + 1], a.alpha * acc[4 * g + 2], a.alpha * acc[4 * g + 3]);
  }
  wave_lds_order();
  const int c4 = 4 * (lane & 7);
  const int col0 = cb + c4;
  float badd[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int col = min(col0 + r, a.N - 1);
    if (a.bias_theta) badd[r] += a.bias_theta_scale * ldf(reinterpret_cast<const T*>(a.bias_theta), col);
    if (a.bias_v) badd[r] += a.bias_v_scale * a.bias_v[col];
  }
  const size_t ob = a.out_type == OUT_F32 ? 4 : sizeof(T);
  const bool aligned = a.ldc % 4 == 0 && coff % 4 == 0 && (uintptr_t)a.C % (4 * ob) == 0 &&
                       (!a.resid || (uintptr_t)a.resid % 16 == 0);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int lr = 8 * k + (lane >> 3);
    const float4 v = *reinterpret_cast<const float4*>(stg + lr * STG_LD + c4);
    const int row = rb + lr;
    if (row >= a.M || col0 >= a.N) continue;
    const float x[4] = {v.x + badd[0], v.y + badd[1], v.z + badd[2], v.w + badd[3]};
    const int64_t base = coff + (int64_t)row * a.ldc + col0;
    if (aligned && col0 + 3 < a.N) {
      store_quad<T>(a, x, base);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (col0 + r >= a.N) break;
        float y = x[r];
        if (a.out_type == OUT_F32) {
          float* C = reinterpret_cast<float*>(a.C);
          if (a.resid) y += a.resid[base + r];
          if (a.beta != 0.f) y += a.beta * C[base + r];
          C[base + r] = y;
        } else {
          stf(reinterpret_cast<T*>(a.C), base + r, y);
        }
      }
    }
  }
  wave_lds_order();   // the next block's writes come after these reads
}

// LDS-staged epilogue of NB 32x32 blocks of one wavefront (blocks (rb, cb[j]),
// j < NB) in one round: all NB are written to the wavefront's staging area
// (NB x 32 rows x 36 floats), then every lane reads its 4 NB quads, issues
// every global read the epilogue needs (residual, previous C) before any
// store, and stores.  One round has the latency of one block where the
// one-block form pays it NB times (a wavefront that is alone on its SIMD has
// nothing else to hide it with).  Global accesses cover eight rows of
// 128 contiguous bytes, as in store_block_lds.
template <typename T, int NB>
__device__ inline void store_blocks_lds(const GemmArgs& a, const f32x16_t (&acc)[NB], int64_t coff, int rb,
                                        const int (&cb)[NB], int lane, float* stg) {
  {
    const int wr = lane & 31, wh = lane >> 5;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(stg + j * STG_FLOATS + wr * STG_LD + 8 * g + 4 * wh) =
            make_float4(a.alpha * acc[j][4 * g], a.alpha * acc[j][4 * g + 1], a.alpha * acc[j][4 * g + 2],
                        a.alpha * acc[j][4 * g + 3]);
  }
  wave_lds_order();
  const int c4 = 4 * (lane & 7);
  float4 v[NB][4];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int k = 0; k < 4; ++k) v[j][k] = *reinterpret_cast<const float4*>(stg + j * STG_FLOATS + (8 * k + (lane >> 3)) * STG_LD + c4);
  wave_lds_order();   // the next round's writes come after these reads
  const size_t ob = a.out_type == OUT_F32 ? 4 : sizeof(T);
  const bool aligned = a.ldc % 4 == 0 && coff % 4 == 0 && (uintptr_t)a.C % (4 * ob) == 0 &&
                       (!a.resid || (uintptr_t)a.resid % 16 == 0);
  const bool full = aligned && rb + 32 <= a.M && cb[NB - 1] + 32 <= a.N;
  if (full && a.out_type == OUT_F32 && !a.bias_theta && !a.bias_v) {
    // the common case of the residual stream and the weight gradients: all
    // reads first, then all stores
    float* C = reinterpret_cast<float*>(a.C);
    float4 r[NB][4];
    const bool rd = a.resid != nullptr, bt = a.beta != 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t idx = coff + (int64_t)(rb + 8 * k + (lane >> 3)) * a.ldc + cb[j] + c4;
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        if (rd) t = *reinterpret_cast<const float4*>(a.resid + idx);
        if (bt) {
          const float4 c = *reinterpret_cast<const float4*>(C + idx);
          t.x += a.beta * c.x; t.y += a.beta * c.y; t.z += a.beta * c.z; t.w += a.beta * c.w;
        }
        r[j][k] = t;
      }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t idx = coff + (int64_t)(rb + 8 * k + (lane >> 3)) * a.ldc + cb[j] + c4;
        *reinterpret_cast<float4*>(C + idx) =
            make_float4(v[j][k].x + r[j][k].x, v[j][k].y + r[j][k].y, v[j][k].z + r[j][k].z, v[j][k].w + r[j][k].w);
      }
    return;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int col0 = cb[j] + c4;
    float badd[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = min(col0 + q, a.N - 1);
      if (a.bias_theta) badd[q] += a.bias_theta_scale * ldf(reinterpret_cast<const T*>(a.bias_theta), col);
      if (a.bias_v) badd[q] += a.bias_v_scale * a.bias_v[col];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int row = rb + 8 * k + (lane >> 3);
      if (row >= a.M || col0 >= a.N) continue;
      const float x[4] = {v[j][k].x + badd[0], v[j][k].y + badd[1], v[j][k].z + badd[2], v[j][k].w + badd[3]};
      const int64_t base = coff + (int64_t)row * a.ldc + col0;
      if (aligned && col0 + 3 < a.N) {
        store_quad<T>(a, x, base);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (col0 + q >= a.N) break;
          float y = x[q];
          if (a.out_type == OUT_F32) {
            float* C = reinterpret_cast<float*>(a.C);
            if (a.resid) y += a.resid[base + q];
            if (a.beta != 0.f) y += a.beta * C[base + q];
            C[base + q] = y;
          } else {
            stf(reinterpret_cast<T*>(a.C), base + q, y);
          }
        }
      }
    }
  }
}

}  // namespace
}  // namespace fdh

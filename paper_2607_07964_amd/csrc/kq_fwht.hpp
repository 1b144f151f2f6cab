// Butterflies of the fast Walsh-Hadamard transform in LDS, shared by the rotation passes and the
// online transforms (Sylvester order: entry (i, j) of H is (-1)^popcount(i & j)).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace kq {

template <int R>
__device__ __forceinline__ void hadamard_reg(float* x) {
#pragma unroll
  for (int s = 1; s < R; s <<= 1)
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (!(k & s)) {
        const float a = x[k], b = x[k + s];
        x[k] = a + b;
        x[k + s] = a - b;
      }
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}

// Butterfly stages across the lanes of a wave (lane xor 1 ... 8, then 16 and 32 as far as stages,
// 4 to 6, goes) on N registers a lane (N even). Strides 1 ... 8 take the partner by DPP and x = y -+ x in one FMA (exact); strides 16 and
// 32 exchange rows between two registers, add and subtract them, and exchange back. No LDS
// traffic: as __shfl_xor these stages were half of a row's LDS time.
template <int N>
__device__ __forceinline__ void hadamard_lanes(float (&x)[N], int lane, int stages = 6) {
  const float s0 = (lane & 1) ? -1.f : 1.f, s1 = (lane & 2) ? -1.f : 1.f;
  const float s2 = (lane & 4) ? -1.f : 1.f, s3 = (lane & 8) ? -1.f : 1.f;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    x[e] = fmaf(x[e], s0, dpp_mov<0xB1>(x[e]));                  // quad_perm [1, 0, 3, 2]
    x[e] = fmaf(x[e], s1, dpp_mov<0x4E>(x[e]));                  // quad_perm [2, 3, 0, 1]
    x[e] = fmaf(x[e], s2, dpp_mov<0x1B>(dpp_mov<0x141>(x[e])));  // half mirror, quad mirror
    x[e] = fmaf(x[e], s3, dpp_mov<0x128>(x[e]));                 // row_ror 8
  }
  auto pair = [](float& a, float& b, auto swap) {
    swap(a, b);
    const float s = a + b, d = a - b;
    a = s, b = d;
    swap(a, b);
  };
  auto swap16 = [](float& a, float& b) {
    const auto r =
        __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
  };
  auto swap32 = [](float& a, float& b) {
    const auto r =
        __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
  };
  if (stages < 5) return;
#pragma unroll
  for (int e = 0; e < N; e += 2) pair(x[e], x[e + 1], swap16);
  if (stages < 6) return;
#pragma unroll
  for (int e = 0; e < N; e += 2) pair(x[e], x[e + 1], swap32);
}

// One group of up to 3 butterfly stages (strides h, 2h, 4h; h = 2^lgh) over a buffer of n
// floats in LDS (n <= 2^24, so 32-bit indices; shifts and masks instead of divisions).
template <int R>
__device__ __forceinline__ void fwht_stage_group(float* buf, int n, int lgh, int tid,
                                                 int nthreads) {
  const int groups = n / R, hm = (1 << lgh) - 1;
  for (int q = tid; q < groups; q += nthreads) {
    const int base = (q >> lgh) * (R << lgh) + (q & hm);
    float x[R];
#pragma unroll
    for (int k = 0; k < R; ++k) x[k] = buf[base + (k << lgh)];
    hadamard_reg<R>(x);
#pragma unroll
    for (int k = 0; k < R; ++k) buf[base + (k << lgh)] = x[k];
  }
}

// FWHT of every length-m segment (m a power of 2) of buf[0, n), from the stage of stride
// 2^lgh0 on
__device__ inline void fwht_lds(float* buf, int64_t n, int64_t m, int tid, int nthreads,
                                int lgh0 = 0) {
  int lgh = lgh0;  // stages of strides below 2^lgh0 already applied
  while ((int64_t(1) << lgh) < m) {
    const int64_t left = m >> lgh;
    if (left >= 8) {
      fwht_stage_group<8>(buf, int(n), lgh, tid, nthreads);
      lgh += 3;
    } else if (left == 4) {
      fwht_stage_group<4>(buf, int(n), lgh, tid, nthreads);
      lgh += 2;
    } else {
      fwht_stage_group<2>(buf, int(n), lgh, tid, nthreads);
      lgh += 1;
    }
    __syncthreads();
  }
}

}  // namespace kq

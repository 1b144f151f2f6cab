// Lazy-block column-wise OBS with group quantisation (eq. obs_update; Prop. 1 eq. kronq_update
// with or without the drift correction P; Alg. 2).
//
// Rows are independent given U. A sweep launch takes one lazy group of up to 4 blocks of 128
// columns. Four waves share 32 rows of a block, each holding one 32-column tile of it in the
// accumulator layout of the 32 x 32 matrix instructions (lane l and l + 32 share row l; of each
// four columns in turn one half holds them), so that most updates are matrix instructions on the
// registers the sweep works in:
//   * pending: what the block owes to the lazy group's earlier blocks, sum_k E[row, k] U[k, col]
//     over the K <= 384 columns swept before it (and X P with the drift correction), on the
//     bf16 matrix cores from operands split into bf16 high and low parts and kept in
//     MFMA-fragment order;
//   * group parameters: a group of 128 columns takes them from the row's current 128 values; a
//     wider group (256, ..., d_in: the paper's per-channel grid is group = d_in) in a reduction
//     kernel launched when the sweep reaches the group's first block;
//   * the columns: the wave that holds the tile sweeps it, four columns at a time (a quad). Both
//     halves of the wave hold the quad's four values, quantise them one after another
//     (e_j = (w_j - w_hat_j) / U_jj reaches the quad's later columns by FMAs) and apply the four
//     errors to the next quad, taken from the half that holds it by v_permlane32_swap; the rest
//     of the tile gets the rank-4 update from two v_mfma_f32_32x32x2f32. The errors go through
//     LDS, one barrier a quad, to the waves of the later tiles, which apply the same update to
//     theirs while the sweep goes on, and to the wave that writes the tile's results. With the
//     drift correction w_j P[j, :], w_j as it stood before quantisation, is added the same way.
// Between lazy groups, products on the bf16 matrix cores bring the errors to the columns beyond
// (gemm_frag_add; see obs_launch for their order). Every column receives all updates of earlier
// columns before its own sweep, so this equals the paper's one-block-at-a-time update up to
// summation order.
//
// What bounds it: the chain of 128 quantisations a block. A wave that also updated the three
// later tiles and wrote the results took 870 cycles a quad (fp32 matrix instructions hold up the
// wave that issues them: 128 cycles a tile and quad); eight lanes a row with 16 columns in each
// lane, one DPP broadcast and 16 FMAs a column, 26 us a block at 4096 rows and 103 us at 28672.
// As it stands a block takes 20k cycles of sweep (625 a quad) and 4k to 12k of loads and pending
// products before it: the sweeps of a 4096 x 4096 layer 0.56 ms (0.83 ms before), 28672 x 8192
// 2.47 ms (6.6 ms before), 4096 x 4096 with P 0.69 ms (0.77 ms, and 0.41 ms of separate updates
// within the lazy groups).
//
// The quantiser (reading of the paper's "quant"): xmin = min(0, min w), xmax = max(0, max w),
// (-1, 1) when both are 0; scale = float32((xmax - xmin) / (2^b - 1)) in float64;
// zero = rint(-xmin / scale); q = clamp(rint(w / scale) + zero, 0, 2^b - 1);
// w_hat = float32(scale * (q - zero)). The code must be the one of the exact quotient w / scale
// rounded half to even: the kernel forms t = w * (1 / scale) in fp32 (relative error below
// 2.4e-7) and takes rint(t); when some t of a quad lies within 1e-6 (2^b + 1) of a half-integer
// (beyond |t| = 2^b the code is clamped whatever t is) the quad is quantised again with the side
// of the half-integer h decided by the sign of fma(-h, scale, w), which is exact. w_hat in fp32
// equals the float64 form exactly (scale and q - zero are exact fp32 operands of one correctly
// rounded product).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "kq_common.hpp"

namespace kq {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
#define KQ_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int OB = 128;                  // block (and the smallest group)
constexpr int LZMAX = 4;                 // blocks per lazy group (at most)

// a and b rounded to bf16 in one dword
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const bf16x2_t v = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
  return __builtin_bit_cast(uint32_t, v);
}
// four values as bf16 high and low parts, two dwords each
__device__ __forceinline__ void split4(const float (&v)[4], uint32_t (&h)[2], uint32_t (&l)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    h[i] = pack_bf16(v[2 * i], v[2 * i + 1]);
    l[i] = pack_bf16(v[2 * i] - __uint_as_float(h[i] << 16),
                     v[2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u));
  }
}

// (scale, zero) of a group from its range, the same float64 steps as the oracle's reading
__device__ __forceinline__ void grid_params(float xmin, float xmax, int bits, float& scale,
                                            float& fzero) {
  if (xmax == xmin) {
    xmin = -1.f;
    xmax = 1.f;
  }
  const double maxq = double((1 << bits) - 1);
  scale = float((double(xmax) - double(xmin)) / maxq);
  fzero = float(__builtin_rint(-double(xmin) / double(scale)));
}

// Group parameters of groups wider than one block: one wave per row reduces the row's current
// values over the group's columns [c0, c0 + g) (taken when the sweep reaches the group).
__global__ __launch_bounds__(256) void obs_group_params(const float* __restrict__ W,
                                                        int64_t d_out, int64_t ldw, int64_t c0,
                                                        int64_t g, int bits,
                                                        float* __restrict__ scales,
                                                        float* __restrict__ zeros, int64_t ldsz,
                                                        int64_t gi) {
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= d_out) return;  // uniform per wave
  const float* wr = W + row * ldw + c0;
  float xmin = 0.f, xmax = 0.f;
  for (int64_t c = int64_t(lane) * 4; c < g; c += 256) {
    const float4 v = *reinterpret_cast<const float4*>(wr + c);
    xmin = fminf(xmin, fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
    xmax = fmaxf(xmax, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    xmin = fminf(xmin, __shfl_xor(xmin, o));
    xmax = fmaxf(xmax, __shfl_xor(xmax, o));
  }
  if (lane == 0) {
    float scale, fzero;
    grid_params(xmin, xmax, bits, scale, fzero);
    scales[row * ldsz + gi] = scale;
    zeros[row * ldsz + gi] = fzero;
  }
}

// LDS image of a 128 x 128 block of U (or P): its ten 32 x 32 tiles (I <= J), row by row (the two
// rows a matrix operand reads at once lie in different banks)
__device__ __forceinline__ int utile(int I, int J) { return (I * (9 - I) / 2 + J - I) * 1024; }
constexpr int UTILES = 10;

// a block of U into LDS in that image, one kilobyte (8 rows of a tile) per wave and load
template <int NW>
__device__ __forceinline__ void stage_block(const float* __restrict__ src, int64_t ld, float* dst,
                                            int wave, int lane) {
#pragma unroll
  for (int i = 0; i < UTILES * 4 / NW; ++i) {
    const int u = wave + NW * i, tile = u >> 2;  // tile, quarter u % 4
    const int I = tile < 4 ? 0 : tile < 7 ? 1 : tile < 9 ? 2 : 3;
    const int J = tile - I * (9 - I) / 2 + I;
    const int j = 32 * I + 8 * (u & 3) + (lane >> 3), c = 32 * J + 4 * (lane & 7);
    __builtin_amdgcn_global_load_lds(src + int64_t(j) * ld + c, KQ_LDS(dst + u * 256), 16, 0, 0);
  }
}

// acc += sum_k U[kp + k, col m] E[row, k], k < K (a multiple of 128), for one tile of 32 columns
// and 32 rows: a wave's fragment loads are contiguous kilobytes, requested one step of KS k ahead
// of the step's products; the three split products accumulate in three independent chains (with
// KS = 32, where more waves share the registers and the matrix cores, in one). (The
// scheduling barriers keep each step's loads ahead of the other step's products; left to itself
// the compiler interleaves them and each product waits for a load issued just before. The load
// after the last step re-reads it, in bounds: a skipped load would make the wait before the
// products a full one on every step.)
template <int KS>
__device__ __forceinline__ void pending_update(const uint16_t* __restrict__ eh,
                                               const uint16_t* __restrict__ el,
                                               const uint16_t* __restrict__ uh,
                                               const uint16_t* __restrict__ ul, int K,
                                               f32x16_t& acc) {
  constexpr int S = KS / 16;
  constexpr bool SPLIT = KS == 64;
  bf16x8_t f0[4][S], f1[4][S];  // [eh, el, uh, ul][k step of 16]
  f32x16_t lh = {}, hl = {};
  auto load = [&](bf16x8_t (&f)[4][S], int k0) {
#pragma unroll
    for (int ks = 0; ks < S; ++ks) {
      const int kk = (k0 + 16 * ks) * 32;  // next 16-k unit: 512 elements on
      f[0][ks] = *reinterpret_cast<const bf16x8_t*>(eh + kk);
      f[1][ks] = *reinterpret_cast<const bf16x8_t*>(el + kk);
      f[2][ks] = *reinterpret_cast<const bf16x8_t*>(uh + kk);
      f[3][ks] = *reinterpret_cast<const bf16x8_t*>(ul + kk);
    }
  };
  auto mfmas = [&](const bf16x8_t (&f)[4][S]) {
#pragma unroll
    for (int ks = 0; ks < S; ++ks) {
      f32x16_t& l = SPLIT ? lh : acc;
      f32x16_t& h = SPLIT ? hl : acc;
      l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[3][ks], f[0][ks], l, 0, 0, 0);
      h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[2][ks], f[1][ks], h, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[2][ks], f[0][ks], acc, 0, 0, 0);
    }
  };
  load(f0, 0);
  for (int k0 = 0; k0 < K; k0 += 2 * KS) {
    load(f1, k0 + KS);
    __builtin_amdgcn_sched_barrier(0);
    mfmas(f0);
    __builtin_amdgcn_sched_barrier(0);
    load(f0, k0 + 2 * KS < K ? k0 + 2 * KS : K - KS);
    __builtin_amdgcn_sched_barrier(0);
    mfmas(f1);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (SPLIT) acc[r] += lh[r] + hl[r];
}

// LDS writes of this wave done, then the workgroup barrier (global stores stay in flight)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Where a row's results of a block go (a lane's row; rows past the end repeat the last row, value
// for value)
struct SweepOut {
  float *w, *wh, *err;  // W, W_hat and the errors (the last two or NULL) at the block's column 0
  uint8_t* codes;
  uint16_t *eh, *el;    // -errors, split, in fragment order
  uint16_t *xh, *xl;    // pre-quantisation values, the same (drift)
};

struct SweepIn {
  const float* ub;    // U block in LDS (utile)
  const float* pb;    // P block in LDS (drift)
  const float4* rec;  // the quads' records in LDS (QuadU)
  float4* pub;        // this row group's published quads: [2 tiles][8][NP][32 rows]
  float scale, inv_s, lo, hi, fzero, near;  // near: 0.5 - the distance that asks for the exact side
  int l32, half;
};

// What a quad needs of U (and P) in every lane, one record of float4s in LDS per quad, read a
// quad ahead: slots 0, 1 hold U[j, k] of the quad's own columns (01 02 03 12 | 13 23), slot 2 the
// 1 / U_jj, slots 3 .. 6 the rows' entries in the next quad's columns; 7, 8 and 9 .. 12 the same
// of P.
constexpr int REC = 8, RECD = 16;  // float4 per record (without, with P)
template <bool DRIFT>
struct QuadU {
  float4 a, b, rc, nx[4];
  float4 pa, pb, pnx[DRIFT ? 4 : 1];
};
__device__ __forceinline__ float comp(const float4& v, int i) {
  return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}
__device__ __forceinline__ float in_quad(const float4& a, const float4& b, int k, int i) {
  return k == 0 ? comp(a, i - 1) : k == 1 ? (i == 2 ? a.w : b.x) : b.y;
}

template <bool DRIFT>
__device__ __forceinline__ void read_quad(QuadU<DRIFT>& u, const float4* r, bool next) {
  u.a = r[0], u.b = r[1], u.rc = r[2];
  if (next) {
#pragma unroll
    for (int k = 0; k < 4; ++k) u.nx[k] = r[3 + k];
  }
  if (DRIFT) {
    u.pa = r[7], u.pb = r[8];
    if (next) {
#pragma unroll
      for (int k = 0; k < 4; ++k) u.pnx[DRIFT ? k : 0] = r[9 + k];
    }
  }
}

// row j = 4 q + k of the block into quad q's record (k = 0 .. 3), from memory
__device__ __forceinline__ void write_rec(const float* __restrict__ row, int q, int k, float* rec,
                                          int slot, bool diag) {
  const float4 in = *reinterpret_cast<const float4*>(row + 4 * q);
  const float4 nx = q < 31 ? *reinterpret_cast<const float4*>(row + 4 * q + 4) : in;
  if (k == 0) rec[4 * slot] = in.y, rec[4 * slot + 1] = in.z, rec[4 * slot + 2] = in.w;
  if (k == 1) rec[4 * slot + 3] = in.z, rec[4 * slot + 4] = in.w;
  if (k == 2) rec[4 * slot + 5] = in.w;
  if (diag) rec[8 + k] = 1.f / comp(in, k);
  reinterpret_cast<float4*>(rec)[slot + (diag ? 3 : 2) + k] = nx;
}

// quantise the quad's four columns: t by the reciprocal, or (EXACT) the side of the nearest
// half-integer by an exact residual
template <bool DRIFT, bool EXACT>
__device__ __forceinline__ float quant4(const float (&x0)[4], const QuadU<DRIFT>& u,
                                        const SweepIn& a, float (&x)[4], float (&ne)[4],
                                        float (&qz)[4]) {
  float far = 0.f;  // largest distance from the nearest integer
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = x0[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float t = x[k] * a.inv_s;
    float r = __builtin_rintf(t);
    const float d = t - r;
    if (EXACT) {
      const float h = r + copysignf(0.5f, d);            // the half-integer next to t
      const float res = fmaf(-h, a.scale, x[k]);         // exact sign of x / scale - h
      const float up = h + 0.5f, dn = h - 0.5f;
      const float even = 2.f * __builtin_rintf(0.5f * h);  // h +- 0.5, whichever is even
      r = res > 0.f ? up : res < 0.f ? dn : res == 0.f ? even : r;
    } else {
      far = fmaxf(far, fabsf(d));
    }
    qz[k] = __builtin_amdgcn_fmed3f(r, a.lo, a.hi);      // q - zero
    ne[k] = (a.scale * qz[k] - x[k]) * comp(u.rc, k);
#pragma unroll
    for (int i = k + 1; i < 4; ++i) {
      x[i] = fmaf(ne[k], in_quad(u.a, u.b, k, i), x[i]);
      if (DRIFT) x[i] = fmaf(x[k], in_quad(u.pa, u.pb, k, i), x[i]);
    }
  }
  return far;
}

// the low half's value of four registers in every lane (hi: the upper half's)
__device__ __forceinline__ void half_bcast(const float (&v)[4], bool hi, float (&o)[4]) {
  float a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = v[i], b[i] = v[i];
  // (one wait state between the copies and the swaps, for all four)
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %4\n\tv_permlane32_swap_b32 %1, %5\n\t"
      "v_permlane32_swap_b32 %2, %6\n\tv_permlane32_swap_b32 %3, %7"
      : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]),
        "+v"(b[3]));
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = hi ? b[i] : a[i];
}

// published values of a quad: -errors, q - zero (and x with the drift correction)
template <bool DRIFT>
constexpr int NP = DRIFT ? 3 : 2;
template <bool DRIFT>
__device__ __forceinline__ float4* pub_at(const SweepIn& a, int t, int q) {
  return a.pub + ((t & 1) * 8 + q) * NP<DRIFT> * 32;
}

// the tile t sweep, by the wave that holds it
template <bool DRIFT>
__device__ __forceinline__ void sweep_tile(f32x16_t& acc, int t, const SweepIn& a) {
  const float* ut = a.ub + utile(t, t) + a.half * 32 + a.l32;
  const float* pt = DRIFT ? a.pb + utile(t, t) + a.half * 32 + a.l32 : nullptr;
  const float4* rec = a.rec + t * 8 * (DRIFT ? RECD : REC);
  QuadU<DRIFT> u;
  read_quad<DRIFT>(u, rec, true);
  float s[4];  // the quad's values, in both halves
  {
    const float held[4] = {acc[0], acc[1], acc[2], acc[3]};
    half_bcast(held, false, s);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    // this quad's update operands and the next quad's record; the reads go out before this
    // quad's work
    float ua[2], pa[2];
    QuadU<DRIFT> un;
    if (q < 6) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ua[h] = ut[(4 * q + 2 * h) * 32];
        if (DRIFT) pa[h] = pt[(4 * q + 2 * h) * 32];
      }
    }
    if (q < 7) read_quad<DRIFT>(un, rec + (q + 1) * (DRIFT ? RECD : REC), q < 6);
    __builtin_amdgcn_sched_barrier(0);
    float x[4], ne[4], qz[4];
    const float far = quant4<DRIFT, false>(s, u, a, x, ne, qz);
    if (__builtin_expect(__any(far >= a.near), 0)) quant4<DRIFT, true>(s, u, a, x, ne, qz);
    float4* pub = pub_at<DRIFT>(a, t, q);
    // the low half writes the errors, the upper half q - zero
    float4 v;
    v.x = a.half ? qz[0] : ne[0], v.y = a.half ? qz[1] : ne[1];
    v.z = a.half ? qz[2] : ne[2], v.w = a.half ? qz[3] : ne[3];
    pub[a.half * 32 + a.l32] = v;
    if (DRIFT && a.half) pub[64 + a.l32] = make_float4(x[0], x[1], x[2], x[3]);
    if (q < 7) {
      // the next quad from the half that holds it, with this quad's errors; then the rest of
      // the tile
      const int r = 4 * ((q + 1) >> 1);
      const float held[4] = {acc[r], acc[r + 1], acc[r + 2], acc[r + 3]};
      half_bcast(held, (q + 1) & 1, s);
      if (q < 6) {
        const float e0 = a.half ? ne[1] : ne[0], e1 = a.half ? ne[3] : ne[2];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ua[0], e0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ua[1], e1, acc, 0, 0, 0);
        if (DRIFT) {
          const float x0 = a.half ? x[1] : x[0], x1 = a.half ? x[3] : x[2];
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[0], x0, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[1], x1, acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[i] = fmaf(ne[k], comp(u.nx[k], i), s[i]);
          if (DRIFT) s[i] = fmaf(x[k], comp(u.pnx[DRIFT ? k : 0], i), s[i]);
        }
      u = un;
    }
    lds_barrier();
  }
}

// results of the pair of quads 2 p, 2 p + 1 of tile t: the low half writes the first, the upper
// half the second
template <bool DRIFT>
__device__ __forceinline__ void write_pair(int t, int p, const SweepIn& a, const SweepOut& o) {
  const float4* pub = pub_at<DRIFT>(a, t, 2 * p + a.half) + a.l32;
  const float4 e4 = pub[0], z4 = pub[32];
  const int c = 32 * t + 8 * p + 4 * a.half;  // the quad's first column
  const int f = (2 * t + (p >> 1)) * 512 + (p & 1) * 256 + 4 * a.half;  // in fragment order
  const float4 w4 =
      make_float4(a.scale * z4.x, a.scale * z4.y, a.scale * z4.z, a.scale * z4.w);
  *reinterpret_cast<float4*>(o.w + c) = w4;
  if (o.wh) *reinterpret_cast<float4*>(o.wh + c) = w4;
  if (o.err) *reinterpret_cast<float4*>(o.err + c) = make_float4(-e4.x, -e4.y, -e4.z, -e4.w);
  *reinterpret_cast<uint32_t*>(o.codes + c) =
      uint32_t(z4.x + a.fzero) | (uint32_t(z4.y + a.fzero) << 8) |
      (uint32_t(z4.z + a.fzero) << 16) | (uint32_t(z4.w + a.fzero) << 24);
  uint32_t hi[2], lo[2];
  const float e[4] = {e4.x, e4.y, e4.z, e4.w};
  split4(e, hi, lo);
  *reinterpret_cast<uint2*>(o.eh + f) = make_uint2(hi[0], hi[1]);
  *reinterpret_cast<uint2*>(o.el + f) = make_uint2(lo[0], lo[1]);
  if (DRIFT) {
    const float4 x4 = pub[64];
    const float x[4] = {x4.x, x4.y, x4.z, x4.w};
    split4(x, hi, lo);
    *reinterpret_cast<uint2*>(o.xh + f) = make_uint2(hi[0], hi[1]);
    *reinterpret_cast<uint2*>(o.xl + f) = make_uint2(lo[0], lo[1]);
  }
}

// the tile t sweep as seen by another wave: the update of its own tile (mine > t), and the
// results when it is the tile's writer
template <bool DRIFT>
__device__ __forceinline__ void follow_tile(f32x16_t& acc, int t, int mine, bool writer,
                                            const SweepIn& a, const SweepOut& o) {
  const bool upd = mine > t;  // uniform over the wave
  const int at = utile(t, upd ? mine : t) + a.half * 32 + a.l32;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    float ua[2], pa[2];
    if (upd) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ua[h] = a.ub[at + (4 * q + 2 * h) * 32];
        if (DRIFT) pa[h] = a.pb[at + (4 * q + 2 * h) * 32];
      }
    }
    lds_barrier();  // quad q is published
    if (upd) {
      const float4* pub = pub_at<DRIFT>(a, t, q) + a.l32;
      const float4 e = pub[0];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ua[0], a.half ? e.y : e.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ua[1], a.half ? e.w : e.z, acc, 0, 0, 0);
      if (DRIFT) {
        const float4 x = pub[64];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[0], a.half ? x.y : x.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[1], a.half ? x.w : x.z, acc, 0, 0, 0);
      }
    }
    if (writer && (q & 1)) write_pair<DRIFT>(t, q >> 1, a, o);
  }
}

struct SweepArgs {
  float* W;
  int64_t d_out, ldw;
  const float* U;
  int64_t ldu;
  const float* P;
  int64_t ldp, c_first;  // first column of the lazy group
  int nblocks, bits;
  uint8_t* codes;
  int64_t ldq;
  float *scales, *zeros;
  int64_t ldsz;
  int group;
  float *err, *W_hat;
  int64_t ldo;  // of err and W_hat
  int cus;
  uint16_t *Efh, *Efl, *Xfh, *Xfl;
  const uint16_t *Ufh, *Ufl, *Pfh, *Pfl;
  int64_t d_in;
};

// One lazy group for RG x 32 rows per workgroup, four waves per 32 rows. RG = 2 halves the LDS a
// row takes (the U block is shared), so that a CU holds 128 rows: taken when RG = 1 would need
// more than two workgroups a CU (see obs_launch). (RG = 2 without P has 128 registers: five values
// go to scratch once a launch and come back once a block, none in the quads.)
template <bool DRIFT, int RG>
__global__ __launch_bounds__(256 * RG, DRIFT ? RG : 2 * RG) void obs_sweep(SweepArgs g) {
  __shared__ __attribute__((aligned(16))) float ub[UTILES * 1024];
  __shared__ __attribute__((aligned(16))) float pb[DRIFT ? UTILES * 1024 : 4];
  __shared__ float4 rec[32 * (DRIFT ? RECD : REC)];
  __shared__ float4 pub[RG * 16 * NP<DRIFT> * 32];
  __shared__ float2 mm[RG][4][32];  // a tile's range of each row
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), rg = wave >> 2;
  // This wave's tile. The waves of a SIMD (wave % 4; of both row groups, and of the workgroup
  // that shares the CU, dispatched a round of CUs later) sweep at different times.
  const int mine = (wave + 2 * rg + int(blockIdx.x / g.cus)) & 3;
  const int64_t row0 = (int64_t(blockIdx.x) * RG + rg) * 32;
  const bool active = row0 < g.d_out;  // uniform over the wave
  const int64_t rf = active ? row0 : 0;  // (a row group past the end works on the first)
#pragma unroll 1
  for (int b = 0; b < g.nblocks; ++b) {
    // an opaque copy of the thread index per block: the lane-dependent addresses are formed
    // here, not hoisted out of the loop into (spilled) registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int64_t row = rf + l32 < g.d_out ? rf + l32 : g.d_out - 1;
    const int64_t eo =
        split_frag_index(rf + l32, g.c_first + 8 * half, g.d_in / 16);  // operand
    const int64_t c0 = g.c_first + int64_t(b) * OB;
    stage_block<4 * RG>(g.U + c0 * g.ldu + c0, g.ldu, ub, wave, lane);
    if (DRIFT) stage_block<4 * RG>(g.P + c0 * g.ldp + c0, g.ldp, pb, wave, lane);
    if (tid < (DRIFT ? 256 : 128)) {
      const int q = (tid & 127) >> 2, k = tid & 3;
      float* r = reinterpret_cast<float*>(rec + q * (DRIFT ? RECD : REC));
      if (tid < 128)
        write_rec(g.U + (c0 + 4 * q + k) * g.ldu + c0, q, k, r, 0, true);
      else if (DRIFT)
        write_rec(g.P + (c0 + 4 * q + k) * g.ldp + c0, q, k, r, 7, false);
    }
    f32x16_t acc = {};
    {
      float4 w[4];
      const float* wr = g.W + row * g.ldw + c0 + 32 * mine + 4 * half;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const float4*>(wr + 8 * i);
      if (b > 0) {
        const int64_t uo =
            split_frag_index(c0 + 32 * mine + l32, g.c_first + 8 * half, g.d_in / 16);
        constexpr int KS = RG == 1 ? 64 : 32;
        pending_update<KS>(g.Efh + eo, g.Efl + eo, g.Ufh + uo, g.Ufl + uo, b * OB, acc);
        if (DRIFT) pending_update<KS>(g.Xfh + eo, g.Xfl + eo, g.Pfh + uo, g.Pfl + uo, b * OB, acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[4 * i] += w[i].x, acc[4 * i + 1] += w[i].y;
        acc[4 * i + 2] += w[i].z, acc[4 * i + 3] += w[i].w;
      }
    }
    if (g.group == OB) {
      float xmin = 0.f, xmax = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xmin = fminf(xmin, acc[r]);
        xmax = fmaxf(xmax, acc[r]);
      }
      xmin = fminf(xmin, __shfl_xor(xmin, 32));
      xmax = fmaxf(xmax, __shfl_xor(xmax, 32));
      if (!half) mm[rg][mine][l32] = make_float2(xmin, xmax);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's part of the U block is in LDS
    __syncthreads();
    const int64_t gi = c0 / g.group;
    float scale, fzero;
    if (g.group > OB) {  // taken at the group's first block by obs_group_params
      scale = g.scales[row * g.ldsz + gi];
      fzero = g.zeros[row * g.ldsz + gi];
    } else {
      float xmin = 0.f, xmax = 0.f;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float2 m = mm[rg][t][l32];
        xmin = fminf(xmin, m.x);
        xmax = fmaxf(xmax, m.y);
      }
      grid_params(xmin, xmax, g.bits, scale, fzero);
      if (mine == 3 && active) {
        g.scales[row * g.ldsz + gi] = scale;
        g.zeros[row * g.ldsz + gi] = fzero;
      }
    }
    const float maxq = float((1 << g.bits) - 1);
    const SweepIn in{ub, pb, rec, pub + rg * 16 * NP<DRIFT> * 32, scale, 1.f / scale, -fzero,
                     maxq - fzero, fzero, 0.5f - 1e-6f * (maxq + 2.f), l32, half};
    const int64_t f = split_frag_index(rf + l32, c0, g.d_in / 16);  // its row as written
    const SweepOut out{g.W + row * g.ldw + c0,
                       g.W_hat ? g.W_hat + row * g.ldo + c0 : nullptr,
                       g.err ? g.err + row * g.ldo + c0 : nullptr,
                       g.codes + row * g.ldq + c0,
                       g.Efh + f,
                       g.Efl + f,
                       DRIFT ? g.Xfh + f : nullptr,
                       DRIFT ? g.Xfl + f : nullptr};
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
      if (mine == t)
        sweep_tile<DRIFT>(acc, t, in);
      else  // the writer: the wave that has just swept its own tile (for tile 0 the last one)
        follow_tile<DRIFT>(acc, t, mine, active && mine == ((t + 3) & 3), in, out);
    }
    __syncthreads();  // the errors are visible to the workgroup, the U block is free
  }
}

// Blocks per lazy group. Pending updates reach a block only when the sweep gets there, so a
// quantisation group's columns are all current at its first block only if that block starts a
// lazy group (then every earlier update has been applied to everything after it): the lazy group
// divides the quantisation group (up to LZMAX blocks); a group of one block, or the whole row
// (parameters from the initial row), allows LZMAX. 0 when the group is not supported.
int lazy_blocks(int64_t d_in, int group) {
  if (group < OB || group % OB != 0 || d_in % group != 0) return 0;
  const int m = group / OB;
  if (m == 1 || group == d_in) return LZMAX;
  for (int k = m < LZMAX ? m : LZMAX; k > 1; --k)
    if (m % k == 0) return k;
  return 1;
}

}  // namespace

int obs_group_ok(int64_t d_in, int group) { return lazy_blocks(d_in, group); }

// the split errors (and pre-quantisation values) and the split U^T (and P^T), in fragment order
size_t obs_ws_bytes(int64_t d_out, int64_t d_in, bool drift) {
  if (d_out <= 0 || d_in <= 0) return 0;
  const size_t rows = size_t(cdiv(d_out, 32) * 32);
  const size_t one = 2 * align256(rows * size_t(d_in) * sizeof(uint16_t)) +
                     2 * align256(size_t(d_in) * size_t(d_in) * sizeof(uint16_t));
  return (drift ? 2 : 1) * one + 256;
}

int obs_launch(float* W, int64_t d_out, int64_t d_in, int64_t ldw, const float* U, int64_t ldu,
               int bits, int group, const float* P, int64_t ldp, uint8_t* codes, float* scales,
               float* zeros, float* err, float* W_hat, void* ws, hipStream_t s) {
  const bool drift = P != nullptr;
  const int64_t nblk = d_in / OB, ldsz = d_in / group;
  const int lz = lazy_blocks(d_in, group);
  KQ_REQUIRE(lz > 0, KRONQ_ERR_UNSUPPORTED, "group %d not supported for d_in %lld", group,
             (long long)d_in);
  Carver cv(ws);
  const size_t fe = size_t(cdiv(d_out, 32) * 32) * size_t(d_in), fu = size_t(d_in) * size_t(d_in);
  SweepArgs a{};
  a.W = W, a.d_out = d_out, a.ldw = ldw, a.U = U, a.ldu = ldu, a.P = P, a.ldp = ldp;
  a.bits = bits, a.codes = codes, a.ldq = d_in, a.scales = scales, a.zeros = zeros;
  a.ldsz = ldsz, a.group = group, a.err = err, a.W_hat = W_hat, a.ldo = d_in, a.d_in = d_in;
  a.Efh = cv.take<uint16_t>(fe), a.Efl = cv.take<uint16_t>(fe);
  uint16_t* ufh = cv.take<uint16_t>(fu);
  uint16_t* ufl = cv.take<uint16_t>(fu);
  KQ_TRY(split_transpose_launch(U, ldu, d_in, ufh, ufl, s, "obs_split_u"));
  a.Ufh = ufh, a.Ufl = ufl;
  if (drift) {
    a.Xfh = cv.take<uint16_t>(fe), a.Xfl = cv.take<uint16_t>(fe);
    uint16_t* pfh = cv.take<uint16_t>(fu);
    uint16_t* pfl = cv.take<uint16_t>(fu);
    KQ_TRY(split_transpose_launch(P, ldp, d_in, pfh, pfl, s, "obs_split_p"));
    a.Pfh = pfh, a.Pfl = pfl;
  }
  // 32 rows a workgroup while the chip holds all of them (two workgroups per CU, one with the
  // drift correction's P block), else 64. Measured (whole solve, 32 rows and 64): 4096 x 4096 694
  // and 835 us; 4096 x 14336 4.23 and 4.65 ms; 14336 x 4096 1414 and 1421 us; 28672 x 8192 7.76 and
  // 7.22 ms; with P 4096 x 4096 1159 and 1372 us, 14336 x 4096 2720 and 2285 us. Beside H_G on the
  // rest of the chip, whole layers: 4096 x 4096 with 262144 tokens 9.10 and 9.19 ms, with 65536 4.48
  // and 4.64, 14336 x 4096 with 65536 16.74 and 16.84.
  a.cus = device_cus();
  const int64_t g32 = cdiv(d_out, 32);
  const int rg = g32 <= int64_t(a.cus) * (drift ? 1 : 2) ? 1 : 2;
  const dim3 grid(unsigned(cdiv(g32, rg))), block(unsigned(256 * rg));
  auto kern = drift ? (rg == 1 ? obs_sweep<true, 1> : obs_sweep<true, 2>)
                    : (rg == 1 ? obs_sweep<false, 1> : obs_sweep<false, 2>);
  // Trailing products by halving: every earlier lazy group s reaches group g through the product
  // at the t of s < t <= g with the most trailing zeros, so a column of W is read and written
  // about log2(groups) times instead of once per earlier lazy group, and most of the work has a
  // long K. A wide quantisation group takes its parameters from current columns at its first
  // block t: all of [t, t + 2^v) are current then, so it must be a power of two of lazy groups
  // (or the whole row, which takes them from the initial row).
  const int64_t gl = cdiv(group, int64_t(lz) * OB);
  const bool halving = group == d_in || (gl & (gl - 1)) == 0;
  for (int64_t g0 = 0; g0 < nblk; g0 += lz) {
    const int64_t gend = g0 + lz < nblk ? g0 + lz : nblk;
    a.c_first = g0 * OB;
    a.nblocks = int(gend - g0);
    if (group > OB && a.c_first % group == 0)
      KQ_TRY(launch("obs_group_params", obs_group_params, dim3(unsigned(cdiv(d_out, 4))),
                    dim3(256), 0, s, static_cast<const float*>(W), d_out, ldw, a.c_first,
                    int64_t(group), bits, scales, zeros, ldsz, a.c_first / group));
    KQ_TRY(launch("obs_sweep", kern, grid, block, 0, s, a));
    if (gend * OB >= d_in) break;
    // after lazy group t - 1: with halving, the p = 2^v lazy groups before t update the p after it
    // (v the number of trailing zeros of t), else the last one everything after it
    const int64_t t = gend / lz, p = halving ? (t & -t) : 1;
    const int64_t k0 = (t - p) * lz * OB, K = p * lz * OB, n0 = gend * OB;
    const int64_t N = halving && K < d_in - n0 ? K : d_in - n0;
    const int64_t ks = d_in / 16, ea = split_frag_index(0, k0, ks), ub = split_frag_index(n0, k0, ks);
    const FragPair pu{a.Efh + ea, a.Efl + ea, ks, a.Ufh + ub, a.Ufl + ub, ks, K};
    FragPair pp{};
    if (drift) pp = FragPair{a.Xfh + ea, a.Xfl + ea, ks, a.Pfh + ub, a.Pfl + ub, ks, K};
    KQ_TRY(gemm_frag_add(d_out, N, pu, pp, W + n0, ldw, s, "obs_trailing_update"));
  }
  return KRONQ_OK;
}

}  // namespace kq

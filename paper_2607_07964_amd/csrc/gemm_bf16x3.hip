// C += A B^T with both operands fp32 matrices split beforehand into bf16 high and low parts, on the
// bf16 matrix cores (v_mfma_f32_32x32x16_bf16), fp32-accurate through three products:
// x = x_hi + x_lo with x_hi = bf16(x), x_lo = bf16(x - x_hi), and A B ~ A_hi B_hi + A_hi B_lo +
// A_lo B_hi (the dropped A_lo B_lo term and the parts of x below x_lo are ~2^-16 of each
// product). The OBS trailing updates W[:, rest] -= E U[blk, rest] and, with the drift correction,
// a second product W_blk P[blk, rest] in the same pass. Both operands are kept in MFMA-fragment
// order (split_frag_index): the sweep writes its errors (negated) that way, split_transpose the
// rows of U^T.
//   * 64 x 64 output tile per workgroup, 4 waves in a 2 x 2 grid, each wave one 32 x 32 MFMA block
//     with fp32 accumulators: for outputs too small for the 128 x 128 tiles of gemm_frag.hip.
//   * K advances 32 at a time, first over the K of the first pair, then over the second's,
//     through two LDS stages (one barrier per stage): the next stage is fetched into registers
//     during the current stage's MFMAs and written to the other buffer. LDS rows are padded to 80
//     bytes so that the 16-byte operand reads of 8 consecutive lanes hit distinct banks.
#include <type_traits>

#include "kq_common.hpp"

namespace kq {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 32;      // K per stage
constexpr int RS = 40;      // LDS row stride in bf16 (32 + 8 pad = 80 bytes)

constexpr int TM = 64;

__global__ __launch_bounds__(256, 2) void gemm3_frag_add(int64_t M, int64_t N, FragPair p1,
                                                         FragPair p2, float* __restrict__ C,
                                                         int64_t ldc) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][2][TM * RS], sB[2][2][TM * RS];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1, l32 = lane & 31, lhi = lane >> 5;
  const int64_t m0 = int64_t(blockIdx.y) * TM, n0 = int64_t(blockIdx.x) * TM;
  // this thread's 16-byte chunk of each array per stage: row r of the tile, k offset kc within the
  // stage, 32 consecutive threads on the 32 rows of a fragment (512 contiguous bytes)
  const int r = (tid >> 7) * 32 + (tid & 31), kc = ((tid >> 5) & 3) * 8, so = r * RS + kc;
  const int64_t ra = m0 + r < M ? m0 + r : M - 1, rb = n0 + r < N ? n0 + r : N - 1;
  u32x4_t rah, ral, rbh, rbl;
  f32x16_t acc = {};
  // this lane's elements of the C tile (in the accumulator layout), requested first so that
  // their latency hides behind the whole K loop instead of ending the tile
  const int64_t gm0 = m0 + wm * 32 + 4 * lhi, gn = n0 + wn * 32 + l32;
  float cin[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t gm = gm0 + 8 * (e >> 2) + (e & 3);
    cin[e] = (gm < M && gn < N) ? C[gm * ldc + gn] : 0.f;
  }
  const int n1 = int(p1.K / BK), nst = n1 + int(p2.K / BK);  // even: K is a multiple of 64
  // stage st of the concatenated K: the first pair for st < n1, else the second
  auto fetch = [&](int st) {
    const FragPair& p = st < n1 ? p1 : p2;
    const int64_t k0 = int64_t(st < n1 ? st : st - n1) * BK;
    const int64_t a = split_frag_index(ra, k0 + kc, p.aks);
    const int64_t b = split_frag_index(rb, k0 + kc, p.bks);
    rah = *reinterpret_cast<const u32x4_t*>(p.Ah + a);
    ral = *reinterpret_cast<const u32x4_t*>(p.Al + a);
    rbh = *reinterpret_cast<const u32x4_t*>(p.Bh + b);
    rbl = *reinterpret_cast<const u32x4_t*>(p.Bl + b);
  };
  auto stash = [&](int b) {
    *reinterpret_cast<u32x4_t*>(&sA[b][0][so]) = rah;
    *reinterpret_cast<u32x4_t*>(&sA[b][1][so]) = ral;
    *reinterpret_cast<u32x4_t*>(&sB[b][0][so]) = rbh;
    *reinterpret_cast<u32x4_t*>(&sB[b][1][so]) = rbl;
  };
  // one stage from buffer B (compile-time), while the next stage (clamped to the last one at
  // the end: a harmless reload) is fetched into registers and then written to the other buffer
  auto stage = [&](auto bc, int st) {
    constexpr int B = decltype(bc)::value;
    __syncthreads();  // stage st is in LDS; the other buffer is free
    fetch(st + 1 < nst ? st + 1 : st);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      const int k = ks * 16 + 8 * lhi;  // this lane's 8 k of the 16
      const int m = wm * 32 + l32, n = wn * 32 + l32;
      const bf16x8_t ah = *reinterpret_cast<const bf16x8_t*>(&sA[B][0][m * RS + k]);
      const bf16x8_t al = *reinterpret_cast<const bf16x8_t*>(&sA[B][1][m * RS + k]);
      const bf16x8_t bh = *reinterpret_cast<const bf16x8_t*>(&sB[B][0][n * RS + k]);
      const bf16x8_t bl = *reinterpret_cast<const bf16x8_t*>(&sB[B][1][n * RS + k]);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
    }
    stash(1 - B);
  };
  fetch(0);
  stash(0);
  for (int st = 0; st < nst; st += 2) {
    stage(std::integral_constant<int, 0>{}, st);
    stage(std::integral_constant<int, 1>{}, st + 1);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t gm = gm0 + 8 * (e >> 2) + (e & 3);
    if (gm < M && gn < N) C[gm * ldc + gn] = cin[e] + acc[e];
  }
}

// Fh[n][k] + Fl[n][k] = U[k][n], the bf16 split of U^T in MFMA-fragment order, 64 x 64 tiles
// through LDS: 16-byte loads of U rows, 16-byte stores (eight k of one n; 32 lanes fill 512
// contiguous bytes). U is upper triangular (strictly, for P) and the products read Ut[n][k]
// only for k < n, so tiles wholly below that (k0 >= n0 + 64) are not written. d is a multiple of
// 64.
__global__ __launch_bounds__(256) void split_transpose(const float* __restrict__ U, int64_t ldu,
                                                       int64_t d, uint16_t* __restrict__ Fh,
                                                       uint16_t* __restrict__ Fl) {
  __shared__ float t[64][65];
  const int64_t k0 = int64_t(blockIdx.y) * 64, n0 = int64_t(blockIdx.x) * 64;
  if (k0 >= n0 + 64) return;
  const int tid = threadIdx.x, q = (tid & 15) * 4, r = tid >> 4;  // 16 x 16
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kk = r + 16 * i;
    const float4 v = *reinterpret_cast<const float4*>(U + (k0 + kk) * ldu + n0 + q);
    t[kk][q] = v.x, t[kk][q + 1] = v.y, t[kk][q + 2] = v.z, t[kk][q + 3] = v.w;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = tid + 256 * i, nn = (e & 31) + 32 * (e >> 8), kk = ((e >> 5) & 7) * 8;
    uint32_t h[4], l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float a = t[kk + 2 * c][nn], b = t[kk + 2 * c + 1][nn];
      const bf16x2_t hv = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
      h[c] = __builtin_bit_cast(uint32_t, hv);
      const bf16x2_t lv = __builtin_convertvector(
          f32x2_t{a - __uint_as_float(h[c] << 16), b - __uint_as_float(h[c] & 0xFFFF0000u)},
          bf16x2_t);
      l[c] = __builtin_bit_cast(uint32_t, lv);
    }
    const int64_t f = split_frag_index(n0 + nn, k0 + kk, d / 16);
    *reinterpret_cast<uint4*>(Fh + f) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint4*>(Fl + f) = make_uint4(l[0], l[1], l[2], l[3]);
  }
}

}  // namespace

int split_transpose_launch(const float* U, int64_t ldu, int64_t d, uint16_t* Fh, uint16_t* Fl,
                           hipStream_t s, const char* name) {
  KQ_REQUIRE(d % 64 == 0, KRONQ_ERR_INVALID_ARG, "split_transpose: d %% 64 must be 0");
  const dim3 grid(unsigned(d / 64), unsigned(d / 64));
  return launch(name, split_transpose, grid, dim3(256), 0, s, U, ldu, d, Fh, Fl);
}

int gemm_frag_add(int64_t M, int64_t N, const FragPair& p1, const FragPair& p2, float* C,
                  int64_t ldc, hipStream_t s, const char* name) {
  if (M <= 0 || N <= 0 || p1.K + p2.K <= 0) return KRONQ_OK;
  KQ_REQUIRE(p1.K % (2 * BK) == 0 && p2.K % (2 * BK) == 0, KRONQ_ERR_INVALID_ARG,
             "gemm_frag_add: K %% 64 must be 0");
  // the largest tile that fills three quarters of the chip: 256 x 256 (one workgroup a CU) reads
  // its operands half as often as 128 x 128 (two a CU)
  const int64_t cus = device_cus();
  const int tile = cdiv(M, 256) * cdiv(N, 256) * 4 >= cus * 3   ? 256
                   : cdiv(M, 128) * cdiv(N, 128) * 4 >= cus * 3 ? 128
                                                                : 64;
  if (tile > 64) {
    FragJob j{};
    j.Ph = p1.Ah, j.Pl = p1.Al, j.pks = p1.aks, j.Qh = p1.Bh, j.Ql = p1.Bl, j.qks = p1.bks;
    j.M = M, j.N = N, j.K = p1.K, j.K2 = p2.K;
    j.P2h = p2.Ah, j.P2l = p2.Al, j.Q2h = p2.Bh, j.Q2l = p2.Bl;
    j.alpha = 1.f, j.C = C, j.ldc = ldc, j.add = true;
    return gemm_frag_bf16(j, tile, s, name);
  }
  return launch(name, gemm3_frag_add, dim3(unsigned(cdiv(N, 64)), unsigned(cdiv(M, 64))),
                dim3(256), 0, s, M, N, p1, p2, C, ldc);
}

}  // namespace kq

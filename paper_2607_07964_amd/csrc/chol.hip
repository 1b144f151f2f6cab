// Damping and the inverse-Cholesky factor (Alg. 2 first two lines; Prop. 1 uses rows of it).
//
// inv(H~) = U^T U with U upper. With J the index reversal, J H~ J = L L^T (ordinary lower
// Cholesky) gives H~ = (J L J)(J L J)^T, so U = (J L J)^-1 = J L^-1 J. Steps:
//   1. damping: H~ = H + damp * mean(diag H) * I (in place); M = C J H~ J C (workspace copy), C
//      the powers of two that bring the diagonal into [1, 4);
//   2. L and X = L^-1 together, recursively on [[M11, .], [M21, M22]] split at a multiple of 128:
//        factor and invert M11 (X11 = L11^-1);
//        L21 = M21 X11^T                  (written to the X21 slot, which is still free);
//        M22 -= L21 L21^T                 (lower tiles only) and T = L21 X11 (scratch kept
//                                          until the last step), both in one launch;
//        factor and invert M22 (X22);
//        X21 = -X22 T                     (over L21).
//      Leaves of at most 128 columns are factored and inverted in LDS by one workgroup; every
//      other step is a product with a long K: on the fp32 matrix cores, and from order FRAG_MIN
//      on fp16 planes, three products a term (gemm_frag.hip): an operand keeps 23 significant bits
//      down to 2^-16 of its row's largest value and is good to 2^-39 of that below, and the sums in
//      fp32 decide the error, as in an fp32 product. Three dependent launches per split (nine with
//      planes): the chain of small ones, not the flops, sets the time at d = 4096;
//   3. U[i][j] = c_j X[d-1-i][d-1-j] for i <= j, 0 below the diagonal.
// A non-positive pivot sets *info to its 1-based column in the original order (first failure).
#include <algorithm>
#include <cmath>
#include <utility>

#include "kq_common.hpp"

namespace kq {
namespace {

constexpr int NB = 128;
constexpr int DLD = NB + 1;  // LDS leading dimension of the diagonal block

__global__ __launch_bounds__(1024) void diag_shift(const float* __restrict__ H, int64_t d,
                                                   int64_t ldh, float damp,
                                                   float* __restrict__ shift,
                                                   int* __restrict__ info) {
  __shared__ double red[1024];
  const int tid = threadIdx.x;
  double s = 0.0;
  // 8 entries a thread in flight at once (each is a cache line of its own)
  for (int64_t i0 = tid; i0 < d; i0 += 8 * 1024) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = i0 + 1024 * k;
      v[k] = H[(i < d ? i : d - 1) * ldh + (i < d ? i : d - 1)];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i0 + 1024 * k < d) s += v[k];
  }
  red[tid] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    *shift = float(double(damp) * (red[0] / double(d)));
    *info = 0;
  }
}

// the damped diagonal, and the power of two c_i = 2^-floor(e / 2), e its exponent, that brings it
// into [1, 4) (1 for an entry that is not positive and finite); the large nodes' maxima start at 0
__global__ void add_diag(float* __restrict__ H, int64_t d, int64_t ldh,
                         const float* __restrict__ shift, float* __restrict__ cn,
                         float* __restrict__ mx, int64_t n_mx) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= d) return;
  for (int64_t e = i; e < n_mx; e += d) mx[e] = 0.f;
  const float v = H[i * ldh + i] + *shift;
  H[i * ldh + i] = v;
  cn[i] = v > 0.f && v <= 3.0e38f ? ldexpf(1.f, -(ilogbf(v) >> 1)) : 1.f;
}

// M[i][j] = c_i' c_j' H[i'][j'], i' = d-1-i, j' = d-1-j: reversed, and normalised to a diagonal in
// [1, 4) (exact: powers of two), so that the columns of X11 and X22, whose rows the planes scale
// as wholes, do not differ with the channels' sizes.
__global__ void reverse_copy(const float* __restrict__ H, int64_t d, int64_t ldh,
                             const float* __restrict__ cn, float* __restrict__ M, int64_t ldm) {
  const int64_t i = blockIdx.y;
  const float ci = cn[d - 1 - i];
  for (int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < d;
       j += int64_t(gridDim.x) * blockDim.x)
    M[i * ldm + j] = H[(d - 1 - i) * ldh + (d - 1 - j)] * ci * cn[d - 1 - j];
}

// the same with four columns per thread (d divisible by 4; rows 16-byte aligned); only the lower
// triangle, up to the end of its diagonal blocks, is read afterwards
__global__ void reverse_copy4(const float* __restrict__ H, int64_t d, int64_t ldh,
                              const float* __restrict__ cn, float* __restrict__ M, int64_t ldm) {
  const int64_t i = blockIdx.y, jend = d < (i | 127) + 1 ? d : (i | 127) + 1;
  const float ci = cn[d - 1 - i];
  for (int64_t j = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * 4; j < jend;
       j += int64_t(gridDim.x) * blockDim.x * 4) {
    const float4 h = *reinterpret_cast<const float4*>(H + (d - 1 - i) * ldh + (d - 4 - j));
    const float4 c = *reinterpret_cast<const float4*>(cn + (d - 4 - j));
    *reinterpret_cast<float4*>(M + i * ldm + j) =
        make_float4(h.w * ci * c.w, h.z * ci * c.z, h.y * ci * c.y, h.x * ci * c.x);
  }
}

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// One 32 x 32 block C = alpha * A op(B) + beta * C on LDS arrays, by one wave on the fp32
// matrix cores (v_mfma_f32_32x32x2f32, two k per instruction). A is 32 x k (row stride lda);
// op(B) is k x 32: B[k][n] at B[k * ldb + n], or with bt, B^T with (k, n) at B[n * ldb + k].
// k is even. The caller orders the LDS traffic (a wave's LDS accesses complete in order).
__device__ __forceinline__ void mfma_block(float* C, int ldc, const float* A, int lda,
                                           const float* B, int ldb, bool bt, int k, float alpha,
                                           float beta, int lane) {
  const int l32 = lane & 31, lhi = lane >> 5;
  f32x16_t acc = {};
  for (int k0 = 0; k0 < k; k0 += 2) {
    const float av = A[l32 * lda + k0 + lhi];
    const float bv = bt ? B[l32 * ldb + k0 + lhi] : B[(k0 + lhi) * ldb + l32];
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float* c = C + (8 * (r >> 2) + 4 * lhi + (r & 3)) * ldc + l32;
    *c = beta == 0.f ? alpha * acc[r] : alpha * acc[r] + beta * *c;
  }
}

// v of lane K of each 16-lane row, in the whole row (folds into the FMA that uses it)
template <int K>
__device__ __forceinline__ float bcast16(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xF, 0xF, true));
}

// The panel's state in one wave: v and u are rows 0 .. 15 and 16 .. 31 of the diagonal block, row
// lane % 16 in every 16-lane row (so that a column's entries can be broadcast within each by DPP),
// x a row of the panel below or a column of the identity of this lane's own.
struct PanelRows {
  float v[16], u[32], x[32], own;  // own: the pivot of column `lane` (lanes 0 .. 31)
};

// w += ng raw(lane K of the 16-lane row), one instruction with the broadcast as its DPP operand
// (left to itself the compiler keeps the broadcasts as moves of their own, half as many
// instructions again). A DPP read of raw needs two wait states after its write: ng depends on raw
// through four instructions.
template <int K>
__device__ __forceinline__ void fmac_bcast(float& w, float raw, float ng) {
  asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
               : "+v"(w)
               : "v"(raw), "v"(ng), "i"(K));
}

// w[k] += ng raw_k for the columns k = J + 1 + K of the panel, raw column J of the block's rows
template <int J, int N, int... K>
__device__ __forceinline__ void eliminate(std::integer_sequence<int, K...>, float (&w)[N],
                                          float ng, const PanelRows& r) {
  (fmac_bcast<(J + 1 + K) & 15>(w[J + 1 + K], J + 1 + K < 16 ? r.v[J & 15] : r.u[J], ng), ...);
}

// Column J of the panel: entry k > J of every row loses (w_J / L_JJ) L_kJ = w_J rl rl raw_k, with
// raw the column before scaling and rl = 1 / L_JJ. On the rows that is the rank-1 update, on the
// identity's columns the forward substitution, so that x ends as a row of L or a column of the
// inverse.
template <int J>
__device__ __forceinline__ void panel_column(PanelRows& r, int lane) {
  constexpr bool LO = J < 16;
  float& at = LO ? r.v[J & 15] : r.u[J];
  asm volatile("s_nop 1" : "+v"(at));  // (its last write is an asm the compiler does not look into)
  const float piv = bcast16<J & 15>(at);
  if (lane == J) r.own = piv;
  const float rl = __builtin_amdgcn_rsqf(piv);  // pivots are normal or the factor fails
  const float lu = r.u[J] * rl, lx = r.x[J] * rl, nu = -lu * rl, nx = -lx * rl;
  if constexpr (LO) {
    const float lv = r.v[J & 15] * rl, nv = -lv * rl;
    eliminate<J>(std::make_integer_sequence<int, 15 - (J & 15)>{}, r.v, nv, r);
    eliminate<J>(std::make_integer_sequence<int, 31 - J>{}, r.x, nx, r);
    eliminate<J>(std::make_integer_sequence<int, 31 - J>{}, r.u, nu, r);
    r.v[J & 15] = lv;
  } else {
    // the next column's rows first: its pivot waits for them
    eliminate<J>(std::make_integer_sequence<int, 31 - J>{}, r.u, nu, r);
    eliminate<J>(std::make_integer_sequence<int, 31 - J>{}, r.x, nx, r);
  }
  r.u[J] = lu;
  r.x[J] = lx;
}
template <int... J>
__device__ __forceinline__ void panel_columns(std::integer_sequence<int, J...>, PanelRows& r,
                                              int lane) {
  (panel_column<J>(r, lane), ...);
}

// Panel p (32 columns) by one of two waves, both of which eliminate the diagonal block: part 0
// takes the inverse Y_pp and the rows of block p + 1, part 1 those of blocks p + 2 and p + 3.
__device__ __forceinline__ void factor_panel(float* a, float* y, int p, int part, int64_t kb,
                                             int64_t d, int* info, int lane) {
  const int c0 = 32 * p, l16 = lane & 15, l32 = lane & 31, hi = lane >> 5;
  const int bx = p + (part ? 2 + hi : 1);         // this lane's block (part 0: the upper half)
  const bool rows = part ? bx < 4 : hi && bx < 4;  // x is a row below
  float* xr = a + (32 * (bx < 4 ? bx : 3) + l32) * DLD + c0;
  PanelRows r;
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    if (k < 16) r.v[k & 15] = a[(c0 + l16) * DLD + c0 + k];
    r.u[k] = a[(c0 + 16 + l16) * DLD + c0 + k];
    const float x = xr[k];
    r.x[k] = rows ? x : (l32 == k ? 1.f : 0.f);
  }
  r.own = 1.f;
  panel_columns(std::make_integer_sequence<int, 32>{}, r, lane);
  if (rows) {
#pragma unroll
    for (int k = 0; k < 32; ++k) xr[k] = r.x[k];
  }
  if (part == 0) {
    if (!hi) {
#pragma unroll
      for (int k = 0; k < 32; ++k) y[(c0 + k) * DLD + c0 + l32] = r.x[k];
    }
    // the first non-positive (or NaN) pivot of the panel
    const uint32_t bad = uint32_t(__ballot(!(r.own > 0.f)));
    if (lane == 0 && bad != 0u) {
      const int f = __builtin_ctz(bad);
      if (kb + c0 + f < d) atomicCAS(info, 0, int(d - (kb + c0 + f)));
    }
  }
}

// A[bi][bj] -= L[bi][p] L[bj][p]^T for 32 x 32 blocks of the diagonal block, one wave
__device__ __forceinline__ void upd_block(float* a, int bi, int bj, int p, int lane) {
  mfma_block(a + 32 * bi * DLD + 32 * bj, DLD, a + 32 * bi * DLD + 32 * p, DLD,
             a + 32 * bj * DLD + 32 * p, DLD, true, 32, -1.f, 1.f, lane);
}

// Factor the diagonal block M[kb:kb+bs, kb:kb+bs] (lower) and invert the factor, one workgroup.
// The block is padded to 128 x 128 with the identity, so a partial block needs no special case.
// Four panels of 32 columns: two waves eliminate a panel in registers (factor_panel: all of its
// rows, and the inverse of its diagonal block), then the four waves update the next panel's block
// column on the fp32 matrix cores; while the next panel runs, the two other waves update the rest
// and build the inverse Y = L^-1 by inv([[A, 0], [B, C]]) = [[A^-1, 0], [-C^-1 B A^-1, C^-1]],
// first of the 64-column halves, then of the whole, as far as their parts exist.
// Writes Linv_kk, with exact zeros above the diagonal, to X (M itself is left as read).
// Bound: the chain of 128 columns, a reciprocal square root and the FMAs of one wave each, and a
// quarter of the time the block's way in and out of LDS: 53k cycles, 24 us. A single wave issues
// about one vector instruction in 6 cycles here, so the instruction count sets a panel's 8.3k
// cycles; running the next pivot's root beside a column's FMAs gained nothing. (Panels through an
// LDS buffer, one round
// trip a column: 30.5 us a block; the diagonal block alone with v_readlane broadcasts, 10k cycles
// a panel, and the rest by products with its inverse: 29 us.)
__global__ __launch_bounds__(256) void potrf_diag(const float* __restrict__ M, int64_t ldm,
                                                  int64_t kb, int bs, int64_t d,
                                                  float* __restrict__ X, int* __restrict__ info) {
  __shared__ __attribute__((aligned(16))) float lds[2 * NB * DLD + 64 * 68];
  float* const a = lds;                 // the block, becomes L (lower part meaningful)
  float* const y = lds + NB * DLD;      // Y = L^-1
  float* const tb = lds + 2 * NB * DLD; // product scratch
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: per-wave branches
  const bool full = bs == NB;
  if (full) {
    float4 q[NB * NB / 1024];
#pragma unroll
    for (int it = 0; it < NB * NB / 1024; ++it) {
      const int e = tid + 256 * it, i = e >> 5, j = (e & 31) * 4;
      q[it] = *reinterpret_cast<const float4*>(M + (kb + i) * ldm + kb + j);
    }
#pragma unroll
    for (int it = 0; it < NB * NB / 1024; ++it) {
      const int e = tid + 256 * it, i = e >> 5, j = (e & 31) * 4;
      a[i * DLD + j] = q[it].x, a[i * DLD + j + 1] = q[it].y;
      a[i * DLD + j + 2] = q[it].z, a[i * DLD + j + 3] = q[it].w;
    }
  } else {
    for (int e = tid; e < NB * NB; e += 256) {
      const int i = e >> 7, j = e & 127;
      a[i * DLD + j] = (i < bs && j < bs) ? M[(kb + i) * ldm + kb + j] : (i == j ? 1.f : 0.f);
    }
  }
  // upper 32-blocks of Y that the doubling reads as operands: (0, 1) and (2, 3)
  for (int e = tid; e < 2 * 32 * 32; e += 256) {
    const int o = (e >> 10) * 64, i = (e >> 5) & 31, j = e & 31;
    y[(o + i) * DLD + o + 32 + j] = 0.f;
  }
  __syncthreads();
  float* const t2 = tb;  // L10 Y00, then L[64:, :64] Y[:64, :64]
  auto half_product = [&](int bi, int bj) {
    mfma_block(t2 + 32 * bi * 68 + 32 * bj, 68, a + (64 + 32 * bi) * DLD, DLD, y + 32 * bj, DLD,
               false, 64, 1.f, 0.f, lane);
  };
  float* const t32 = a;  // L32 Y22 over the finished L00
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
    if (wave == 0 || (wave == 1 && p < 2)) {
      factor_panel(a, y, p, wave, kb, d, info, lane);
    } else if (p == 1) {
      if (wave == 2) {
        upd_block(a, 3, 2, 0, lane);
        upd_block(a, 3, 3, 0, lane);
      } else {
        mfma_block(t2, 33, a + 32 * DLD, DLD, y, DLD, false, 32, 1.f, 0.f, lane);  // L10 Y00
      }
    } else if (p == 2) {
      half_product(wave == 3, wave == 2);
      if (wave == 3) half_product(1, 1);
    } else if (p == 3) {
      if (wave == 1) {
        mfma_block(t32, DLD, a + 96 * DLD + 64, DLD, y + 64 * DLD + 64, DLD, false, 32, 1.f, 0.f,
                   lane);
      } else {  // rows 64 .. 95 of Y's lower left quarter need only Y22
        const int bj = wave - 2;
        mfma_block(y + 64 * DLD + 32 * bj, DLD, y + 64 * DLD + 64, DLD, t2 + 32 * bj, 68, false,
                   32, -1.f, 0.f, lane);
      }
    }
    __syncthreads();
    // the next panel's block column from panel p, and what else can be
    if (p == 0) {
      upd_block(a, wave < 3 ? 1 + wave : 2, wave < 3 ? 1 : 2, 0, lane);
    } else if (p == 1) {
      if (wave < 3)
        upd_block(a, wave == 0 ? 2 : 3, wave < 2 ? 2 : 3, 1, lane);
      else  // Y10 = -Y11 (L10 Y00)
        mfma_block(y + 32 * DLD, DLD, y + 32 * DLD + 32, DLD, t2, 33, false, 32, -1.f, 0.f, lane);
    } else if (wave == 0) {
      if (p == 2)
        upd_block(a, 3, 3, 2, lane);
      else  // Y32 = -Y33 (L32 Y22)
        mfma_block(y + 96 * DLD + 64, DLD, y + 96 * DLD + 96, DLD, t32, DLD, false, 32, -1.f, 0.f,
                   lane);
    }
    __syncthreads();
  }
  if (wave < 2)  // rows 96 .. 127: -[Y32 Y33] T2
    mfma_block(y + 96 * DLD + 32 * wave, DLD, y + 96 * DLD + 64, DLD, t2 + 32 * wave, 68, false,
               64, -1.f, 0.f, lane);
  __syncthreads();
  if (full) {
#pragma unroll 4
    for (int it = 0; it < NB * NB / 1024; ++it) {
      const int e = tid + 256 * it, i = e >> 5, j = (e & 31) * 4;
      float v[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = (j + c <= i) ? y[i * DLD + j + c] : 0.f;
      *reinterpret_cast<float4*>(X + (kb + i) * ldm + kb + j) = make_float4(v[0], v[1], v[2], v[3]);
    }
  } else {
    for (int e = tid; e < bs * NB; e += 256) {
      const int i = e >> 7, j = e & 127;
      if (j < bs) X[(kb + i) * ldm + kb + j] = (j <= i) ? y[i * DLD + j] : 0.f;
    }
  }
}

// U[i][j] = c_j X[d-1-i][d-1-j] for i <= j, else 0 (X the inverse factor of the normalised M)
__global__ void reverse_out(const float* __restrict__ X, int64_t ldm, int64_t d,
                            const float* __restrict__ cn, float* __restrict__ U, int64_t ldu) {
  const int64_t i = blockIdx.y;
  for (int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < d;
       j += int64_t(gridDim.x) * blockDim.x)
    U[i * ldu + j] = (j >= i) ? X[(d - 1 - i) * ldm + (d - 1 - j)] * cn[j] : 0.f;
}

// the same with four columns per thread (d divisible by 4; rows 16-byte aligned)
__global__ void reverse_out4(const float* __restrict__ X, int64_t ldm, int64_t d,
                             const float* __restrict__ cn, float* __restrict__ U, int64_t ldu) {
  const int64_t i = blockIdx.y;
  for (int64_t j = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * 4; j < d;
       j += int64_t(gridDim.x) * blockDim.x * 4) {
    float4 u = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j + 3 >= i) {
      const float4 x = *reinterpret_cast<const float4*>(X + (d - 1 - i) * ldm + (d - 4 - j));
      const float4 c = *reinterpret_cast<const float4*>(cn + j);
      u = make_float4(j >= i ? x.w * c.x : 0.f, j + 1 >= i ? x.z * c.y : 0.f,
                      j + 2 >= i ? x.y * c.z : 0.f, x.x * c.w);
    }
    *reinterpret_cast<float4*>(U + i * ldu + j) = u;
  }
}

int64_t ld_for(int64_t d) { return ((d + 63) / 64) * 64; }

// split of an n-column block: the first h columns, a multiple of NB, about half
int64_t split_at(int64_t n) { return (cdiv(n, NB) / 2) * NB; }

int64_t pad(int64_t n, int64_t m) { return cdiv(n, m) * m; }

// A node of n columns whose parts have at least this order runs its products on 16-bit planes: at
// 768 a factor of order 3000 takes 1.42 ms, 4096 1.93, 8192 4.85 and 14336 12.97; at 512 1.40, 2.06,
// 5.13 and 13.01, at 1024 1.44, 1.93, 4.86 and 13.15, at 2048 1.53, 1.99, 4.96 and 13.83. Below, the
// nine launches cost more than the products. (Beside H_G on the rest of the chip, 4096 x 4096 layers
// of 262144 and 65536 tokens: 9.10 and 4.48 ms with 768, 9.22 and 4.54 with 1536. Products on the
// fp32 matrix cores and, from order 3000, on six bf16 products a term split inside the kernel: 1.71
// ms at 3000, 2.47 at 4096 and 22.4 at 14336, with slower leaves; error of U against float64 5.5e-7
// and 8.6e-7 at 4096 and 14336, now 3.6e-7 and 6.3e-7.)
constexpr int64_t FRAG_MIN = 768;
bool frag_node(int64_t n) {
  const int64_t h = split_at(n);
  return h >= FRAG_MIN && n - h >= FRAG_MIN;
}

// floats of the two planes of a rows x k operand
int64_t planes(int64_t rows, int64_t k) { return pad(rows, 32) * pad(k, 16); }

// Scratch floats of an n-column block: a node keeps its product T (r x h; as planes of its
// transpose at a large node) until its last step, while the second child's recursion runs after
// it.
int64_t chol_scratch(int64_t n) {
  if (n <= NB) return 0;
  const int64_t h = split_at(n), r = n - h;
  const int64_t t = frag_node(n) ? planes(h, r) : r * h;
  return std::max(chol_scratch(h), t + chol_scratch(r));
}
// the planes a large node needs only while it runs (M21 or X22, X11, its transpose, L21)
int64_t chol_planes(int64_t n) {
  if (n <= NB || !frag_node(n)) return 0;
  const int64_t h = split_at(n), r = n - h;
  return std::max(planes(r, h), planes(r, r)) + 2 * planes(h, h) + planes(r, h);
}
// and the largest values of their rows, of each node its own: M21, L21, X22 (r rows), X11, its
// transpose, T^T (h)
int64_t chol_maxima(int64_t n) {
  if (n <= NB || !frag_node(n)) return 0;
  const int64_t h = split_at(n);
  return 3 * n + chol_maxima(h) + chol_maxima(n - h);
}

struct Chol {
  float *M, *X, *planes;
  int64_t ld, d;
  int* info;
  hipStream_t s;
};

// the two planes of an operand and the largest values of their rows
struct Planes {
  uint16_t *h, *l;
  int64_t ks;
  float* max;
};
Planes take_planes(float*& at, int64_t rows, int64_t k, float*& mx) {
  const int64_t n = planes(rows, k);
  Planes p{reinterpret_cast<uint16_t*>(at), reinterpret_cast<uint16_t*>(at) + n, pad(k, 16) / 16,
           mx};
  at += n;
  mx += rows;
  return p;
}
SplitJob split_job(const float* src, int64_t ld, int64_t rows, int64_t cols, int tri, bool trans,
                   const Planes& p) {
  return SplitJob{src, ld, rows, cols, tri, trans, p.max, p.h, p.l, p.ks, {}};
}
FragJob frag_job(const Planes& P, const Planes& Q, int64_t M, int64_t N, int64_t K, int flags,
                 float alpha, float* C, int64_t ldc) {
  FragJob j{};
  j.Ph = P.h, j.Pl = P.l, j.pks = P.ks, j.pmax = P.max;
  j.Qh = Q.h, j.Ql = Q.l, j.qks = Q.ks, j.qmax = Q.max;
  j.M = M, j.N = N, j.K = K, j.flags = flags, j.alpha = alpha, j.C = C, j.ldc = ldc;
  return j;
}

int chol_rec(const Chol& c, float* T, float*& mx, int64_t n0, int64_t n);

// The four products of a large node on fp16 planes (gemm_frag.hip). Every row of an operand is
// scaled by its own largest value: those of L21 and T = L21 X11 are small where the two parts
// hardly depend on each other, and X grows as the inverse square root of the smallest eigenvalue,
// which no fixed power of two covers. So L21 and T, whose largest values only the finished product
// knows, go through fp32 at X21's place, which nothing else uses before the last step. (A power of
// two per matrix, L21 and T leaving their products as planes: X overflowed from 4095 on, and a
// coupling of 1e-4 left X21 good to 4e-5 where it is now good to 4e-7. It took 1.85 ms at 4096 and
// 12.12 at 14336; twelve more launches of 5 to 8 us at 4096, and the reads for the largest values,
// are the difference to now.)
int chol_node_frag(const Chol& c, float* T, float*& mx, int64_t n0, int64_t n) {
  const int64_t h = split_at(n), r = n - h, ld = c.ld;
  KQ_TRY(chol_rec(c, T, mx, n0, h));
  const float* M21 = c.M + (n0 + h) * ld + n0;
  const float* X11 = c.X + n0 * ld + n0;
  float* X21 = c.X + (n0 + h) * ld + n0;
  const float* X22 = c.X + (n0 + h) * ld + n0 + h;
  float* M22 = c.M + (n0 + h) * ld + n0 + h;
  float* at = c.planes;
  const Planes pL = take_planes(at, r, h, mx), pX = take_planes(at, h, h, mx),
               pXt = take_planes(at, h, h, mx);
  float* at2 = at;
  const Planes pM = take_planes(at, r, h, mx), pY = take_planes(at2, r, r, mx);  // (the same place)
  const Planes pT = take_planes(T, h, r, mx);
  // tiles: the K ranges (or, for the lower triangle, the tiles themselves) make the work uneven,
  // so 256 x 256 tiles only where they come in several rounds of the chip
  auto tile = [](int64_t tiles256) { return tiles256 >= 2 * int64_t(device_cus()) ? 256 : 128; };
  const int64_t tr = cdiv(r, 256), th = cdiv(h, 256);
  const AbsMaxJob top[2] = {{M21, ld, r, h, TRI_FULL, pM.max, nullptr, {}},
                            {X11, ld, h, h, TRI_LOWER, pX.max, pXt.max, {}}};
  KQ_TRY(abs_max_launch(top, 2, c.s, "chol_split"));
  const SplitJob split[3] = {split_job(M21, ld, r, h, TRI_FULL, false, pM),
                             split_job(X11, ld, h, h, TRI_LOWER, false, pX),
                             split_job(X11, ld, h, h, TRI_LOWER, true, pXt)};
  KQ_TRY(split_planes_launch(split, 3, c.s, "chol_split"));
  // L21 = M21 X11^T
  FragJob l21 = frag_job(pM, pX, r, h, h, FRAG_Q_LOWER, 1.f, X21, ld);
  l21.rmax = pL.max;
  KQ_TRY(gemm_frag_f16(&l21, 1, tile(tr * th), c.s, "chol_trsm"));
  const SplitJob split_l = split_job(X21, ld, r, h, TRI_FULL, false, pL);
  KQ_TRY(split_planes_launch(&split_l, 1, c.s, "chol_split"));
  // M22 -= L21 L21^T (lower tiles) and T = L21 X11
  FragJob two[2] = {frag_job(pL, pL, r, r, h, FRAG_LOWER, -1.f, M22, ld),
                    frag_job(pL, pXt, r, h, h, FRAG_Q_UPPER, 1.f, X21, ld)};
  two[0].add = true;
  two[1].cmax = pT.max;
  KQ_TRY(gemm_frag_f16(two, 2, tile(tr * (tr + 1) / 2 + tr * th), c.s, "chol_syrk_trtri_row"));
  const SplitJob split_t = split_job(X21, ld, r, h, TRI_FULL, true, pT);
  KQ_TRY(split_planes_launch(&split_t, 1, c.s, "chol_split"));
  KQ_TRY(chol_rec(c, T, mx, n0 + h, r));
  const AbsMaxJob top22{X22, ld, r, r, TRI_LOWER, pY.max, nullptr, {}};
  KQ_TRY(abs_max_launch(&top22, 1, c.s, "chol_split"));
  const SplitJob split22 = split_job(X22, ld, r, r, TRI_LOWER, false, pY);
  KQ_TRY(split_planes_launch(&split22, 1, c.s, "chol_split"));
  // X21 = -X22 T
  const FragJob x21 = frag_job(pY, pT, r, h, r, FRAG_P_LOWER, -1.f, X21, ld);
  return gemm_frag_f16(&x21, 1, tile(tr * th), c.s, "trtri_update");
}

// L and L^-1 of the block [n0, n0 + n) of M; the lower part of the same block of X receives
// L^-1 (zeros on the upper part of the diagonal leaves). T: scratch of chol_scratch(n) floats; mx:
// the zeros that the large nodes take their maxima from.
int chol_rec(const Chol& c, float* T, float*& mx, int64_t n0, int64_t n) {
  float *M = c.M, *X = c.X;
  const int64_t ld = c.ld;
  hipStream_t s = c.s;
  if (n <= NB)
    return launch("chol_potrf_diag", potrf_diag, dim3(1), dim3(256), 0, s,
                  static_cast<const float*>(M), ld, n0, int(n), c.d, X, c.info);
  if (frag_node(n)) return chol_node_frag(c, T, mx, n0, n);
  const int64_t h = split_at(n), r = n - h;
  KQ_TRY(chol_rec(c, T, mx, n0, h));
  const float* M21 = M + (n0 + h) * ld + n0;
  const float* X11 = X + n0 * ld + n0;
  float* X21 = X + (n0 + h) * ld + n0;
  float* X22 = X + (n0 + h) * ld + n0 + h;
  float* M22 = M + (n0 + h) * ld + n0 + h;
  // L21 = M21 X11^T (op(B) = X11^T is upper triangular)
  KQ_TRY(gemm_f32(GEMM_TB | GEMM_OPB_UPPER, r, h, h, 1.f, M21, ld, X11, ld, 0.f, X21, ld, s,
                  "chol_trsm"));
  // M22 -= L21 L21^T (lower tiles only) and T = L21 X11 (X11 lower triangular), in one launch
  // (both need only L21 and X11)
  const GemmProb syrk{GEMM_TB | GEMM_LOWER_C, r, r, h, -1.f, X21, ld, X21, ld, 1.f, M22, ld};
  const GemmProb row{GEMM_B_LOWER, r, h, h, 1.f, X21, ld, X11, ld, 0.f, T, h};
  KQ_TRY(gemm_f32_dual(syrk, row, s, "chol_syrk_trtri_row"));
  KQ_TRY(chol_rec(c, T + r * h, mx, n0 + h, r));
  // X21 = -X22 T
  return gemm_f32(GEMM_A_LOWER, r, h, r, -1.f, X22, ld, T, h, 0.f, X21, ld, s, "trtri_update");
}

}  // namespace

size_t chol_ws_bytes(int64_t d) {
  if (d <= 0) return 0;
  const int64_t ld = ld_for(d);
  return 2 * align256(size_t(d) * ld * sizeof(float)) +
         align256(size_t(std::max<int64_t>(1, chol_scratch(d))) * sizeof(float)) +
         align256(size_t(chol_planes(d)) * sizeof(float)) +
         align256(size_t(chol_maxima(d)) * sizeof(float)) +
         align256(size_t(d) * sizeof(float)) + 512;
}

int chol_launch(float* H, int64_t d, int64_t ldh, float damp_rel, float* U, int64_t ldu,
                int* info, void* ws, hipStream_t s) {
  const int64_t ld = ld_for(d);
  Carver cv(ws);
  float* M = cv.take<float>(size_t(d) * ld);
  float* X = cv.take<float>(size_t(d) * ld);
  float* T = cv.take<float>(size_t(std::max<int64_t>(1, chol_scratch(d))));
  float* pl = cv.take<float>(size_t(chol_planes(d)));
  float* mx = cv.take<float>(size_t(chol_maxima(d)));
  float* cn = cv.take<float>(size_t(d));
  float* shift = cv.take<float>(1);

  KQ_TRY(launch("chol_diag_shift", diag_shift, dim3(1), dim3(1024), 0, s,
                static_cast<const float*>(H), d, ldh, damp_rel, shift, info));
  KQ_TRY(launch("chol_add_diag", add_diag, dim3(unsigned(cdiv(d, 256))), dim3(256), 0, s, H, d,
                ldh, static_cast<const float*>(shift), cn, mx, chol_maxima(d)));
  const unsigned gx = unsigned(cdiv(d, 256) < 64 ? cdiv(d, 256) : 64);
  const bool v4 = d % 4 == 0 && ldh % 4 == 0 && ldu % 4 == 0 && aligned(H, 16) && aligned(U, 16);
  const unsigned gx4 = unsigned(cdiv(d, 1024) < 64 ? cdiv(d, 1024) : 64);
  if (v4)
    KQ_TRY(launch("chol_reverse_copy", reverse_copy4, dim3(gx4, unsigned(d)), dim3(256), 0, s,
                  static_cast<const float*>(H), d, ldh, static_cast<const float*>(cn), M, ld));
  else
    KQ_TRY(launch("chol_reverse_copy", reverse_copy, dim3(gx, unsigned(d)), dim3(256), 0, s,
                  static_cast<const float*>(H), d, ldh, static_cast<const float*>(cn), M, ld));
  KQ_TRY(chol_rec(Chol{M, X, pl, ld, d, info, s}, T, mx, 0, d));
  if (v4)
    return launch("chol_reverse_out", reverse_out4, dim3(gx4, unsigned(d)), dim3(256), 0, s,
                  static_cast<const float*>(X), ld, d, static_cast<const float*>(cn), U, ldu);
  return launch("chol_reverse_out", reverse_out, dim3(gx, unsigned(d)), dim3(256), 0, s,
                static_cast<const float*>(X), ld, d, static_cast<const float*>(cn), U, ldu);
}

}  // namespace kq

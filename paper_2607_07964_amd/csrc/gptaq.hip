// The drift correction P = alpha ((D U^T) . M_U) U (Prop. 1; Alg. 2), M_U the strictly upper mask.
// Two triangular products, 2 d^3 / 3 flops together: T = D U^T on the tiles that touch the upper
// triangle (k from the column on), P = alpha T U there (k from the row to the column). From order
// PLANES_MIN both run on fp16 planes (gemm_frag.hip), every row of an operand (U's columns in the
// second product) divided by a power of two that brings its largest value below 2^14, so that a
// value keeps 22 bits or more down to 2^-28 of the largest; below, on the fp32 matrix cores.
// Measured (d = 4096): products 115 + 116 us on 128 x 128 tiles, bound by their operands' L2
// traffic and the uneven K ranges; units, splits and the cleared triangle 105 us. (Both products on
// the fp32 matrix cores: 374 + 287 us.)
#include "kq_common.hpp"

namespace kq {
namespace {

// P = 0 on and below the diagonal, four columns a thread (rows 16-byte aligned)
__global__ void clear_lower4(float* __restrict__ M, int64_t d, int64_t ld) {
  const int64_t i = blockIdx.y;
  for (int64_t j = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * 4; j <= i;
       j += int64_t(gridDim.x) * blockDim.x * 4) {
    float* m = M + i * ld + j;
    if (j + 3 <= i)
      *reinterpret_cast<float4*>(m) = make_float4(0.f, 0.f, 0.f, 0.f);
    else
      for (int k = 0; j + k <= i; ++k) m[k] = 0.f;
  }
}

// the power of two that divides mx (a largest absolute value) to below 2^14; 1 for none
__device__ float unit_of(float mx) {
  int e = mx > 0.f && mx <= 3.0e38f ? ilogbf(mx) - 13 : 0;
  if (e < -120) e = -120;
  return ldexpf(1.f, e);
}

// unit[i] of each row i, over its columns from the row's own on (strict: past it). Workgroup (row,
// matrix). cmax, if not NULL: its bits are cleared (clear) or turned into units.
__global__ __launch_bounds__(256) void row_units(const float* __restrict__ M0, int64_t ld0,
                                                 float* __restrict__ unit0, bool strict0,
                                                 const float* __restrict__ M1, int64_t ld1,
                                                 float* __restrict__ unit1, int64_t d,
                                                 float* __restrict__ cmax, bool clear) {
  __shared__ float red[4];
  const int64_t i = blockIdx.x;
  const bool second = blockIdx.y != 0;
  const float* m = second ? M1 + i * ld1 : M0 + i * ld0;
  const int64_t first = i + (!second && strict0);
  float mx = 0.f;
  for (int64_t j = (first & ~int64_t(3)) + 4 * threadIdx.x; j < d; j += 1024) {
    const float4 v = *reinterpret_cast<const float4*>(m + j);  // (within the padded row)
    const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (j + k >= first && j + k < d) mx = fmaxf(mx, fabsf(x[k]));
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    (second ? unit1 : unit0)[i] = unit_of(mx);
    if (!second) cmax[i] = clear ? 0.f : unit_of(cmax[i]);
  }
}

// cmax[column] = max(cmax, |U[rows][column]|) of the upper matrix U: 64 columns and a slab of rows
// a workgroup (non-negative floats compare as their bits; a NaN's are the largest: unit 1)
__global__ __launch_bounds__(256) void col_max(const float* __restrict__ U, int64_t ldu, int64_t d,
                                               float* __restrict__ cmax) {
  __shared__ float red[16][64];
  const int tid = threadIdx.x, q = (tid & 15) * 4, rr = tid >> 4;
  const int64_t c = int64_t(blockIdx.x) * 64 + q;
  float mx[4] = {};
  for (int64_t r = int64_t(blockIdx.y) * 16 + rr; r <= c + 3 && r < d && c < d;
       r += 16 * int64_t(gridDim.y)) {
    const float4 v = *reinterpret_cast<const float4*>(U + r * ldu + c);
    const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c + k >= r) mx[k] = fmaxf(mx[k], fabsf(x[k]));
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) red[rr][q + k] = mx[k];
  __syncthreads();
  if (tid < 64 && int64_t(blockIdx.x) * 64 + tid < d) {
    float m = 0.f;
    for (int r = 0; r < 16; ++r) m = fmaxf(m, red[r][tid]);
    atomicMax(reinterpret_cast<unsigned*>(cmax + int64_t(blockIdx.x) * 64 + tid),
              __float_as_uint(m));
  }
}

// (whole correction, fp32 matrix cores against planes: 74 against 82 us at d = 1024, 116 against
// 101 at 1536, 177 against 123 at 2048, 694 against 337 at 4096; the planes' error against 64 bits
// is the smaller one from 1024 on)
constexpr int64_t PLANES_MIN = 1280;

int64_t t_ld(int64_t d) { return cdiv(d, 64) * 64; }
// 16-bit values of one plane of a d x d operand
size_t plane(int64_t d) { return size_t(cdiv(d, 32) * 32) * size_t(cdiv(d, 16) * 16); }

}  // namespace

size_t gptaq_ws_bytes(int64_t d) {
  if (d <= 0) return 0;
  const size_t t = align256(size_t(d) * size_t(t_ld(d)) * sizeof(float)) + 256;
  if (d < PLANES_MIN) return t;
  return t + 4 * align256(plane(d) * sizeof(uint16_t)) + 3 * align256(size_t(d) * sizeof(float));
}

int gptaq_launch(const float* D, int64_t d, int64_t ldd, const float* U, int64_t ldu, float alpha,
                 float* P, int64_t ldp, void* ws, hipStream_t s) {
  Carver cv(ws);
  const int64_t ldt = t_ld(d);
  float* T = cv.take<float>(size_t(d) * size_t(ldt));
  const dim3 mgrid(unsigned(cdiv(d, 1024)), unsigned(d));
  if (d < PLANES_MIN) {
    KQ_TRY(gemm_f32(GEMM_TB | GEMM_B_LOWER | GEMM_UPPER_C, d, d, d, 1.f, D, ldd, U, ldu, 0.f, T,
                    ldt, s, "gptaq_d_ut"));
    KQ_TRY(launch("gptaq_mask", clear_lower4, mgrid, dim3(256), 0, s, T, d, ldt));
    KQ_TRY(gemm_f32(GEMM_A_UPPER | GEMM_OPB_UPPER | GEMM_UPPER_C, d, d, d, alpha, T, ldt, U, ldu,
                    0.f, P, ldp, s, "gptaq_t_u"));
    return launch("gptaq_mask", clear_lower4, mgrid, dim3(256), 0, s, P, d, ldp);
  }
  const int64_t ks = cdiv(d, 16), t256 = cdiv(d, 256) * (cdiv(d, 256) + 1) / 2;
  uint16_t* ah = cv.take<uint16_t>(plane(d));  // D, then T
  uint16_t* al = cv.take<uint16_t>(plane(d));
  uint16_t* bh = cv.take<uint16_t>(plane(d));  // U, then U^T
  uint16_t* bl = cv.take<uint16_t>(plane(d));
  float* ud = cv.take<float>(size_t(d));       // units of D's rows, then T's
  float* uu = cv.take<float>(size_t(d));       // U's rows
  float* uc = cv.take<float>(size_t(d));       // U's columns
  // the tiles' K ranges are uneven: 256 x 256 tiles only in two rounds of the chip (d = 4096: 393 us
  // with 128 x 128, 603 with 256 x 256)
  const int tile = t256 >= 2 * int64_t(device_cus()) ? 256 : 128;
  KQ_TRY(launch("gptaq_units", row_units, dim3(unsigned(d), 2), dim3(256), 0, s, D, ldd, ud, true,
                U, ldu, uu, d, uc, true));
  KQ_TRY(launch("gptaq_units", col_max, dim3(unsigned(cdiv(d, 64)), 16), dim3(256), 0, s, U, ldu,
                d, uc));
  const SplitJob s1[2] = {{D, ldd, d, d, SPLIT_STRICT_UPPER, false, 1.f, ud, ah, al, ks},
                          {U, ldu, d, d, SPLIT_UPPER, false, 1.f, uu, bh, bl, ks}};
  KQ_TRY(split_planes_launch(s1, 2, s, "gptaq_split"));
  FragJob j{};  // T[m][n] = sum_k D[m][k] U[n][k], n >= m (by tiles), so k > m for T's kept part
  j.Ph = ah, j.Pl = al, j.Qh = bh, j.Ql = bl, j.pks = j.qks = ks;
  j.M = j.N = j.K = d, j.flags = FRAG_Q_UPPER | FRAG_UPPER, j.alpha = 1.f;
  j.C = T, j.ldc = ldt, j.punit = ud, j.qunit = uu;
  KQ_TRY(gemm_frag_f16(&j, 1, tile, s, "gptaq_d_ut"));
  KQ_TRY(launch("gptaq_units", row_units, dim3(unsigned(d), 1), dim3(256), 0, s,
                static_cast<const float*>(T), ldt, ud, true, static_cast<const float*>(T), ldt, ud,
                d, uc, false));
  const SplitJob s2[2] = {{T, ldt, d, d, SPLIT_STRICT_UPPER, false, 1.f, ud, ah, al, ks},
                          {U, ldu, d, d, SPLIT_UPPER, true, 1.f, uc, bh, bl, ks}};
  KQ_TRY(split_planes_launch(s2, 2, s, "gptaq_split"));
  j.flags = FRAG_P_UPPER | FRAG_Q_LOWER | FRAG_UPPER, j.alpha = alpha;  // P[m][n], k in (m, n]
  j.C = P, j.ldc = ldp, j.punit = ud, j.qunit = uc;
  KQ_TRY(gemm_frag_f16(&j, 1, tile, s, "gptaq_t_u"));
  return launch("gptaq_mask", clear_lower4, mgrid, dim3(256), 0, s, P, d, ldp);
}

}  // namespace kq

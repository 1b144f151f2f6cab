// The drift correction P = alpha ((D U^T) . M_U) U (Prop. 1; Alg. 2), M_U the strictly upper mask.
// Two triangular products, 2 d^3 / 3 flops together: T = D U^T on the tiles that touch the upper
// triangle (k from the column on), P = alpha T U there (k from the row to the column). From order
// PLANES_MIN both run on fp16 planes (gemm_frag.hip), every row of an operand (U's columns in the
// second product) divided by a power of two that brings its largest value below 2^15: a value keeps
// 23 bits down to 2^-16 of its row's largest and is good to 2^-39 of that below (10 bits are left at
// 2^-29); for the first product U's columns are brought to one size first. Below that order, on the
// fp32 matrix cores.
// Measured (d = 4096): products 110 + 109 us on 128 x 128 tiles, bound by their operands' L2 traffic
// and the uneven K ranges; splits 49, largest values 28, the cleared triangle 10 us. (Both products
// on the fp32 matrix cores: 374 + 287 us.)
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

// (whole correction, fp32 matrix cores against planes: 92 and 92 us at d = 1280, 114 and 94 at 1536,
// 165 and 121 at 2048, 653 and 333 at 4096; error against 64 bits 5.4e-7 and 3.5e-7 at 1280, 9.7e-7
// and 6.2e-7 at 4096, the same with channels of sizes over eight decades)
constexpr int64_t PLANES_MIN = 1280;

int64_t t_ld(int64_t d) { return cdiv(d, 64) * 64; }
// 16-bit values of one plane of a d x d operand
size_t plane(int64_t d) { return size_t(cdiv(d, 32) * 32) * size_t(cdiv(d, 16) * 16); }

}  // namespace

size_t gptaq_ws_bytes(int64_t d) {
  if (d <= 0) return 0;
  const size_t t = align256(size_t(d) * size_t(t_ld(d)) * sizeof(float)) + 256;
  if (d < PLANES_MIN) return t;
  return t + 4 * align256(plane(d) * sizeof(uint16_t)) + align256(size_t(4 * d) * sizeof(float));
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
  // largest values of D's rows, T's, U's and U's columns
  float* md = cv.take<float>(size_t(4 * d));
  float *mt = md + d, *mu = mt + d, *mc = mu + d;
  // the tiles' K ranges are uneven: 256 x 256 tiles only in two rounds of the chip (d = 4096: 393 us
  // with 128 x 128, 603 with 256 x 256)
  const int tile = t256 >= 2 * int64_t(device_cus()) ? 256 : 128;
  KQ_TRY(clear_launch(md, 4 * d, s, "gptaq_split"));
  // T sums over channels k that D[m][k] grows with and U[n][k] falls with: U's columns are brought
  // to one size and D's take the inverse factors, or the small channels would drop out of the
  // planes of D's rows and the large ones out of U's. (T and U's rows are of one size over k.)
  const AbsMaxJob cols{U, ldu, d, d, TRI_UPPER, nullptr, mc, {}};
  KQ_TRY(abs_max_launch(&cols, 1, s, "gptaq_split"));
  const ColScale up{mc, false}, down{mc, true};
  const AbsMaxJob top[2] = {{D, ldd, d, d, TRI_STRICT_UPPER, md, nullptr, up},
                            {U, ldu, d, d, TRI_UPPER, mu, nullptr, down}};
  KQ_TRY(abs_max_launch(top, 2, s, "gptaq_split"));
  const SplitJob s1[2] = {{D, ldd, d, d, TRI_STRICT_UPPER, false, md, ah, al, ks, up},
                          {U, ldu, d, d, TRI_UPPER, false, mu, bh, bl, ks, down}};
  KQ_TRY(split_planes_launch(s1, 2, s, "gptaq_split"));
  FragJob j{};  // T[m][n] = sum_k D[m][k] U[n][k], n >= m (by tiles), so k > m for T's kept part
  j.Ph = ah, j.Pl = al, j.Qh = bh, j.Ql = bl, j.pks = j.qks = ks;
  j.M = j.N = j.K = d, j.flags = FRAG_Q_UPPER | FRAG_UPPER, j.alpha = 1.f;
  j.C = T, j.ldc = ldt, j.pmax = md, j.qmax = mu, j.rmax = mt;
  KQ_TRY(gemm_frag_f16(&j, 1, tile, s, "gptaq_d_ut"));
  const SplitJob s2[2] = {{T, ldt, d, d, TRI_STRICT_UPPER, false, mt, ah, al, ks, {}},
                          {U, ldu, d, d, TRI_UPPER, true, mc, bh, bl, ks, {}}};
  KQ_TRY(split_planes_launch(s2, 2, s, "gptaq_split"));
  j.flags = FRAG_P_UPPER | FRAG_Q_LOWER | FRAG_UPPER, j.alpha = alpha;  // P[m][n], k in (m, n]
  j.C = P, j.ldc = ldp, j.pmax = mt, j.qmax = mc, j.rmax = nullptr;
  KQ_TRY(gemm_frag_f16(&j, 1, tile, s, "gptaq_t_u"));
  return launch("gptaq_mask", clear_lower4, mgrid, dim3(256), 0, s, P, d, ldp);
}

}  // namespace kq

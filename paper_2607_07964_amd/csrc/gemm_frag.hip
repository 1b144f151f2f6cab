// Products of fp32 matrices split beforehand into two 16-bit planes, D = P Q^T with three matrix
// products per term, P Q ~ P_lo Q_hi + P_hi Q_lo + P_hi Q_hi (v_mfma_f32_32x32x16, fp32
// accumulators). Planes are kept in MFMA-fragment order (split_frag_index): 32 rows x 16 k form
// one kilobyte that a wave loads as it stands.
//   bf16 planes: x = bf16(x) + bf16(x - bf16(x)), the dropped parts ~2^-16 of each product. The
//     OBS trailing updates W += (-E) U (and, with the drift correction, + X P as a second K range
//     of the same product).
//   fp16 planes: 23 significant bits (what is left out is below 2^-23 of the value, the dropped
//     product of the low parts of the same order), so the accumulation in fp32 dominates the
//     error as it does in an fp32 GEMM. For values scaled into range: the large products of the
//     factorisation (normalised to a unit diagonal) and of the drift correction (a power of two
//     per row).
// Kernel: a (64 WT) x (64 WT) tile per workgroup of 4 waves (WT = 4: 256 x 256, one workgroup per
// CU; WT = 2: 128 x 128, two), each wave (32 WT) x (32 WT) in accumulators. K advances 16 at a
// time through a ring of four LDS stages filled by global_load_lds (a wave loads one plane of one
// operand, a kilobyte a load, which lands as the operand reads want it: no padding, no swizzle,
// no conflicts). Stage s + 4 is requested and the operands of stage s + 1 are read during the
// 12 / 48 products a wave runs on stage s, one barrier a stage.
// Bound: with 256 x 256 tiles the matrix cores (1536 cycles of products a stage against 32 KB of
// loads and 64 KB of LDS reads); with 128 x 128 tiles the L2 traffic of 16 KB per 384 cycles.
// Measured: 28672 x 4096 outputs, K = 4096, bf16 planes: 2.07 ms (1394 TFLOP/s computed), K = 512,
// N = 512: 74 us (610); 4096 x 2048, K = 2048 on 128 x 128 tiles 163 us (630). (128 x 128 tiles
// staged through registers with padded LDS rows, one product of K = 512 per lazy group, ran at 690
// at 28672 rows, bound by LDS traffic and by W read and written once a product: 7.7 ms of trailing
// products there, 4.8 ms now.)
// A triangular operand limits the tile's K range; tiles are then dealt longest range first.
// Tile order: the workgroups of an XCD (workgroup % 8) take whole tile columns (those past the
// last multiple of 8 tile by tile in turn), walked row by row, so that the 32 running together
// share their operands through its L2.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "kq_common.hpp"

namespace kq {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
#define KQ_LDS(p) ((__attribute__((address_space(3))) void*)(p))

template <int N>
__device__ __forceinline__ void wait_vm() {  // s_waitcnt vmcnt(N), the other counters free
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <bool F16>
__device__ __forceinline__ f32x16_t mfma16(u32x4_t a, u32x4_t b, f32x16_t c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// two values as fp16 high and low parts
__device__ __forceinline__ void split_f16(float a, float b, uint32_t& hi, uint32_t& lo) {
  const f16x2_t h = __builtin_convertvector(f32x2_t{a, b}, f16x2_t);
  const f16x2_t l = __builtin_convertvector(f32x2_t{a - float(h[0]), b - float(h[1])}, f16x2_t);
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, l);
}

struct Tiles {
  int nt_m, nt_n, blocks;
  bool by_n;  // walk along n (the tile rows of P are dealt to the XCDs) rather than along m
};

struct FragJobs {
  FragJob j[2];
  Tiles t[2];
};

// workgroups for nw walked x nd dealt tiles: per 8 walked tiles, an XCD has 8 (nd / 8) + nd % 8
__host__ __device__ inline int deal_blocks(int nw, int nd) {
  return 8 * ((nw + 7) / 8) * (8 * (nd / 8) + nd % 8);
}

// one 32 x 32 block of a tile at (m, n): C[m][n], or planes of D^T (row n, k = m: four
// consecutive m a lane and register quad)
__device__ __forceinline__ void store_block(const FragJob& J, const f32x16_t& acc, int64_t m,
                                            int64_t n, int lane) {
  const int64_t gm0 = m + 4 * (lane >> 5), gn = n + (lane & 31);
  if (J.Oh) {
    if (gn >= ((J.N + 31) & ~int64_t(31))) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t gm = gm0 + 8 * q;
      if (gm >= J.oks * 16) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gm + e < J.M ? J.alpha * acc[4 * q + e] : 0.f;
      uint32_t h[2], l[2];
      split_f16(v[0], v[1], h[0], l[0]);
      split_f16(v[2], v[3], h[1], l[1]);
      const int64_t f = split_frag_index(gn, gm, J.oks);
      *reinterpret_cast<uint2*>(J.Oh + f) = make_uint2(h[0], h[1]);
      *reinterpret_cast<uint2*>(J.Ol + f) = make_uint2(l[0], l[1]);
    }
    return;
  }
  if (gn >= J.N) return;
  const float an = J.qunit ? J.alpha * J.qunit[gn] : J.alpha;
  float* c = J.C + gm0 * J.ldc + gn;
  if (m + 32 <= J.M && !J.punit) {  // uniform: every row of the block exists
    float old[16];
    if (J.add) {
#pragma unroll
      for (int r = 0; r < 16; ++r) old[r] = c[(8 * (r >> 2) + (r & 3)) * J.ldc];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
      c[(8 * (r >> 2) + (r & 3)) * J.ldc] = J.add ? old[r] + an * acc[r] : an * acc[r];
    return;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t gm = gm0 + 8 * (r >> 2) + (r & 3);
    if (gm < J.M) {
      float* e = c + (8 * (r >> 2) + (r & 3)) * J.ldc;
      const float x = J.punit ? an * acc[r] * J.punit[gm] : an * acc[r];
      *e = J.add ? *e + x : x;
    }
  }
}

// the blocks one after another (an index sequence: a plain loop of this size is not unrolled, and
// the accumulators would go through scratch)
template <int WT, int... I>
__device__ __forceinline__ void store_all(std::integer_sequence<int, I...>, const FragJob& J,
                                          const f32x16_t (&acc)[WT][WT], int64_t m, int64_t n,
                                          int lane) {
  (store_block(J, acc[I / WT][I % WT], m + 32 * (I / WT), n + 32 * (I % WT), lane), ...);
}

template <bool F16, int WT>
__device__ __forceinline__ void frag_tile(const FragJob& J, const Tiles& T, int b,
                                          uint32_t* lds) {
  constexpr int TM = 64 * WT, G = TM / 32, R = 4;
  constexpr int PLANE = G * 256, STAGE = 4 * PLANE;  // dwords
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = T.by_n ? T.nt_n : T.nt_m, nd = T.by_n ? T.nt_m : T.nt_n;
  int tw, td;
  {
    const int x = b & 7, s = b >> 3, q = nd >> 3, rem = nd & 7, per = 8 * q + rem;
    const int blk = s / per, r = s % per;
    if (r < 8 * q) {
      tw = blk * 8 + r / q;
      // XCD x: columns x, 15 - x, 16 + x, 31 - x, ..., turned from row to row: an XCD hands its
      // workgroups to its four shader engines in strict turn and waits for the one that is full,
      // so each engine has to get long and short K ranges (with column c always on engine c % 4,
      // the triangular products of order 8192 took 1.06 ms each instead of 0.70)
      const int c = (r % q + (q < 4 ? (tw * q) >> 2 : tw)) % q;
      td = 16 * (c >> 1) + ((c & 1) ? 15 - x : x);
    } else {
      const int lin = x + 8 * (r - 8 * q);
      tw = blk * 8 + lin / rem;
      td = 8 * q + lin % rem;
    }
    if (tw >= nw) return;
    // longest K range first: it grows with the index of a lower operand
    if (J.flags & (T.by_n ? FRAG_Q_LOWER : FRAG_P_LOWER)) tw = nw - 1 - tw;
  }
  const int tm = T.by_n ? td : tw, tn = T.by_n ? tw : td;
  const int64_t m0 = int64_t(tm) * TM, n0 = int64_t(tn) * TM;
  if ((J.flags & FRAG_LOWER) && m0 + TM <= n0) return;
  if ((J.flags & FRAG_UPPER) && n0 + TM <= m0) return;
  int64_t kbeg = 0, kend = J.K;
  if (J.flags & FRAG_P_LOWER) kend = kend < m0 + TM ? kend : m0 + TM;  // P[m][k] = 0, k > m
  if (J.flags & FRAG_Q_LOWER) kend = kend < n0 + TM ? kend : n0 + TM;  // Q[n][k] = 0, k > n
  if (J.flags & FRAG_P_UPPER) kbeg = kbeg > m0 ? kbeg : m0;            // P[m][k] = 0, k < m
  if (J.flags & FRAG_Q_UPPER) kbeg = kbeg > n0 ? kbeg : n0;            // Q[n][k] = 0, k < n
  const int n1 = kend > kbeg ? int((kend - kbeg + 15) / 16) : 0;
  const int nst = n1 + int(J.K2 / 16);  // the second pair's K range follows the first's

  // this wave loads one plane of one operand
  const bool isq = wave >= 2;
  const int64_t ks = isq ? J.qks : J.pks, rows = isq ? J.N : J.M, r0 = isq ? n0 : m0;
  const int last = int((rows - 1 - r0) >> 5);  // last 32-row group of the tile
  const uint16_t* src1 = wave == 0 ? J.Ph : wave == 1 ? J.Pl : wave == 2 ? J.Qh : J.Ql;
  const uint16_t* src2 = wave == 0 ? J.P2h : wave == 1 ? J.P2l : wave == 2 ? J.Q2h : J.Q2l;
  const int64_t origin = (r0 >> 5) * ks * 512;
  src1 += origin + (kbeg >> 4) * 512;
  if (J.K2 > 0) src2 += origin;
  const uint32_t lo8 = uint32_t(lane) * 8;
  auto issue = [&](int st, int buf) {
    const int sc = st < nst ? st : nst - 1;  // past the end: the last stage again, never read
    const uint16_t* p = sc < n1 ? src1 + int64_t(sc) * 512 : src2 + int64_t(sc - n1) * 512;
    uint32_t* dst = lds + buf * STAGE + wave * PLANE;
#pragma unroll
    for (int g = 0; g < G; ++g)
      __builtin_amdgcn_global_load_lds(p + int64_t(g < last ? g : last) * ks * 512 + lo8,
                                       KQ_LDS(dst + g * 256), 16, 0, 0);
  };
  const int wm = wave & 1, wn = wave >> 1;
  u32x4_t fp[2][2][WT], fq[2][2][WT];  // [slot][plane][32-row group]
  auto frags = [&](int buf, int slot) {
    const uint32_t* s = lds + buf * STAGE + lane * 4;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        fp[slot][p][i] = *reinterpret_cast<const u32x4_t*>(s + p * PLANE + (wm * WT + i) * 256);
        fq[slot][p][i] =
            *reinterpret_cast<const u32x4_t*>(s + (2 + p) * PLANE + (wn * WT + i) * 256);
      }
  };
  f32x16_t acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f32x16_t{};
  auto mfmas = [&](int slot) {
    constexpr int pp[3] = {1, 0, 0}, qq[3] = {0, 1, 0};
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
          acc[i][j] = mfma16<F16>(fp[slot][pp[t]][i], fq[slot][qq[t]][j], acc[i][j]);
  };
  auto pattern = [&]() {  // reads over the first products, then the loads
#pragma unroll
    for (int i = 0; i < 4 * WT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, WT == 4 ? 2 : 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };
  auto body = [&](auto uc, int s) {
    constexpr int u = decltype(uc)::value;
    __builtin_amdgcn_sched_barrier(0);
    frags((u + 1) % R, (u + 1) & 1);
    // buffer u held stage s, whose operands every wave read before the last barrier
    issue(s + R, u);
    mfmas(u & 1);
    pattern();
    __builtin_amdgcn_sched_barrier(0);
    wait_vm<2 * G>();  // stage s + 2 has landed: only s + 3 and s + 4 are pending
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if (nst > 0) {
#pragma unroll
    for (int p = 0; p < R; ++p) issue(p, p);
    wait_vm<2 * G>();
    asm volatile("s_barrier" ::: "memory");
    frags(0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    int s = 0;
    for (; s + R <= nst; s += R) {
      body(std::integral_constant<int, 0>{}, s);
      body(std::integral_constant<int, 1>{}, s + 1);
      body(std::integral_constant<int, 2>{}, s + 2);
      body(std::integral_constant<int, 3>{}, s + 3);
    }
    if (s < nst) body(std::integral_constant<int, 0>{}, s);
    if (s + 1 < nst) body(std::integral_constant<int, 1>{}, s + 1);
    if (s + 2 < nst) body(std::integral_constant<int, 2>{}, s + 2);
    wait_vm<0>();
  }
  store_all<WT>(std::make_integer_sequence<int, WT * WT>{}, J, acc, m0 + wm * WT * 32,
                n0 + wn * WT * 32, lane);
}

// one or two independent products (the first one's workgroups first)
template <bool F16, int WT>
__global__ __launch_bounds__(256, WT == 4 ? 1 : 2) void gemm_frag(FragJobs a) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[4 * 4 * (2 * WT) * 256];
  const int i = int(blockIdx.x) < a.t[0].blocks ? 0 : 1;
  frag_tile<F16, WT>(a.j[i], a.t[i], int(blockIdx.x) - (i ? a.t[0].blocks : 0), lds);
}

Tiles deal(const FragJob& J, int tm) {
  Tiles t;
  t.nt_m = int(cdiv(J.M, tm));
  t.nt_n = int(cdiv(J.N, tm));
  // walk the index that sets the K range; else the longer one
  t.by_n = (J.flags & (FRAG_Q_UPPER | FRAG_Q_LOWER)) != 0 ||
           (!(J.flags & (FRAG_P_LOWER | FRAG_P_UPPER)) && t.nt_n > t.nt_m);
  t.blocks = t.by_n ? deal_blocks(t.nt_n, t.nt_m) : deal_blocks(t.nt_m, t.nt_n);
  return t;
}

// planes of src (or of its transpose): 64 x 64 tiles through LDS, 16-byte loads and stores
__global__ __launch_bounds__(256) void split_planes(SplitJob j0, SplitJob j1, SplitJob j2) {
  __shared__ float t[64][65];
  const SplitJob& J = blockIdx.z == 0 ? j0 : blockIdx.z == 1 ? j1 : j2;
  const int64_t r0 = int64_t(blockIdx.y) * 64, c0 = int64_t(blockIdx.x) * 64;
  if (r0 >= J.rows || c0 >= J.cols) {
    // (rows and k between the source's edge and the planes' last whole group lie in these tiles'
    // left or upper neighbours: 64 is a multiple of both 32 and 16)
    return;
  }
  // whole 256 x 256 blocks of zeros are outside every tile's K range
  if (J.tri == SPLIT_LOWER && c0 > (r0 | 255)) return;
  if ((J.tri == SPLIT_UPPER || J.tri == SPLIT_STRICT_UPPER) && r0 > (c0 | 255)) return;
  const int tid = threadIdx.x, q = (tid & 15) * 4, rr = tid >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + rr + 16 * i, c = c0 + q;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < J.rows && c < J.cols) v = *reinterpret_cast<const float4*>(J.src + r * J.ld + c);
    // the factor of the plane values: a constant, or the inverse of the row's (column's) unit
    const float fr = J.unit && !J.trans ? 1.f / J.unit[r < J.rows ? r : 0] : J.scale;
    float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = r < J.rows && c + k < J.cols && !(J.tri == SPLIT_LOWER && c + k > r) &&
                      !(J.tri == SPLIT_UPPER && c + k < r) &&
                      !(J.tri == SPLIT_STRICT_UPPER && c + k <= r);
      const float f = J.unit && J.trans ? 1.f / J.unit[c + k < J.cols ? c + k : 0] : fr;
      t[rr + 16 * i][q + k] = in ? x[k] * f : 0.f;
    }
  }
  __syncthreads();
  const int64_t n0 = J.trans ? c0 : r0, k0 = J.trans ? r0 : c0;
  const int64_t nrows = ((J.trans ? J.cols : J.rows) + 31) & ~int64_t(31);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = tid + 256 * i, nn = (e & 31) + 32 * (e >> 8), kk = ((e >> 5) & 7) * 8;
    if (n0 + nn >= nrows || k0 + kk >= J.ks * 16) continue;
    uint32_t h[4], l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float a = J.trans ? t[kk + 2 * c][nn] : t[nn][kk + 2 * c];
      const float b = J.trans ? t[kk + 2 * c + 1][nn] : t[nn][kk + 2 * c + 1];
      split_f16(a, b, h[c], l[c]);
    }
    const int64_t f = split_frag_index(n0 + nn, k0 + kk, J.ks);
    *reinterpret_cast<uint4*>(J.Oh + f) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint4*>(J.Ol + f) = make_uint4(l[0], l[1], l[2], l[3]);
  }
}

template <bool F16>
int frag_launch(const FragJob* jobs, int n, int tile, hipStream_t s, const char* name) {
  FragJobs a{};
  for (int i = 0; i < n; ++i) {
    const FragJob& J = a.j[i] = jobs[i];
    KQ_REQUIRE(J.K2 % 16 == 0 && (J.K2 == 0 || J.K % 16 == 0), KRONQ_ERR_INVALID_ARG,
               "gemm_frag: K ranges of a two-part product must be multiples of 16");
    a.t[i] = deal(J, tile);
  }
  const dim3 grid(unsigned(a.t[0].blocks + a.t[1].blocks));
  return launch(name, tile == 256 ? gemm_frag<F16, 4> : gemm_frag<F16, 2>, grid, dim3(256), 0, s,
                a);
}

}  // namespace

int gemm_frag_bf16(const FragJob& j, int tile, hipStream_t s, const char* name) {
  return frag_launch<false>(&j, 1, tile, s, name);
}
int gemm_frag_f16(const FragJob* jobs, int n, int tile, hipStream_t s, const char* name) {
  return frag_launch<true>(jobs, n, tile, s, name);
}

int split_planes_launch(const SplitJob* jobs, int n, hipStream_t s, const char* name) {
  int64_t r = 0, c = 0;
  for (int i = 0; i < n; ++i) {
    r = std::max(r, jobs[i].rows);
    c = std::max(c, jobs[i].cols);
  }
  return launch(name, split_planes, dim3(unsigned(cdiv(c, 64)), unsigned(cdiv(r, 64)), unsigned(n)),
                dim3(256), 0, s, jobs[0], jobs[n > 1 ? 1 : 0], jobs[n > 2 ? 2 : 0]);
}

}  // namespace kq

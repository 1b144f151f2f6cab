// Products of fp32 matrices split beforehand into two 16-bit planes, D = P Q^T with three matrix
// products per term, P Q ~ P_lo Q_hi + P_hi Q_lo + P_hi Q_hi (v_mfma_f32_32x32x16, fp32
// accumulators). Planes are kept in MFMA-fragment order (split_frag_index): 32 rows x 16 k form
// one kilobyte that a wave loads as it stands.
//   bf16 planes: x = bf16(x) + bf16(x - bf16(x)), the dropped parts ~2^-16 of each product. The
//     OBS trailing updates W += (-E) U (and, with the drift correction, + X P as a second K range
//     of the same product).
//   fp16 planes: each row of an operand divided by a power of two of its own that brings its
//     largest value into [2^14, 2^15) (plane_unit). 23 significant bits down to 2^-16 of that
//     (what is left out is below 2^-23 of the value, the dropped product of the low parts of the
//     same order), below it the row is good to 2^-39 of its largest value, so the accumulation in
//     fp32 dominates the error as it does in an fp32 GEMM. For the large products of the
//     factorisation and of the drift correction.
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
#include "kq_fwht.hpp"

namespace kq {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
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

// The power of two that divides mx (a largest absolute value) into [2^14, 2^15), the upper end of
// fp16; 1 for none, and never below 2^-120 (its inverse has to be finite).
__device__ __forceinline__ float plane_unit(float mx) {
  const int e = int(__float_as_uint(mx) >> 23);  // (mx >= 0)
  return mx > 0.f && e < 255 ? __uint_as_float(uint32_t(e > 21 ? e - 14 : 7) << 23) : 1.f;
}

// *p = max(*p, v) for v >= 0 (non-negative floats compare as their bits)
__device__ __forceinline__ void raise(float* p, float v) {
  atomicMax(reinterpret_cast<unsigned*>(p), __float_as_uint(v));
}

// Stores of a tile of fp16 planes: a wave brings 32 rows of its blocks into row order through LDS of
// its own (lw, rows of S floats) and then takes them in a loop, four columns a lane. Bound by the
// code's own way into the instruction cache, it being run once: with every value stored from its
// accumulator, units and maxima beside it, the loop-free form (5800 instructions at WT = 2, 18000 at
// WT = 4, here 900 and 3400) took 35 us for a product that takes 31.
template <int WT>
struct Stores {
  static constexpr int S = 32 * WT + 8;      // (rows r and r + 4 in different banks)
  static constexpr int LPR = 8 * WT;         // lanes per row
  static constexpr int RPI = 64 / LPR;       // rows at a time
};

// Rows [m, m + 32), columns [n, n + 32 WT), with the units of the planes' rows (pu, qu, in LDS, from
// the first row and column on); the rows' largest values go to rmax, this lane's columns' to cm.
template <int WT>
__device__ __forceinline__ void store_rows(const FragJob& J, const float* lw, int64_t m, int64_t n,
                                           int lane, const float* pu, const float* qu,
                                           float (&cm)[4]) {
  using L = Stores<WT>;
  const int c = 4 * (lane % L::LPR), sub = lane / L::LPR;
  const int64_t gn = n + c;
  const int left = int(J.N - gn < 4 ? (J.N > gn ? J.N - gn : 0) : 4);  // columns that exist
  const int rows = int(J.M - m < 32 ? (J.M > m ? J.M - m : 0) : 32);
  float4 q = *reinterpret_cast<const float4*>(qu + c);
  q.x *= J.alpha, q.y *= J.alpha, q.z *= J.alpha, q.w *= J.alpha;
  // (FRAG_UPPER: only columns past the row count for the maxima)
  const int diag = J.flags & FRAG_UPPER ? int(m - gn) : -64;
  const bool want = J.rmax || J.cmax;
  auto value = [&](int row) {
    float4 v = *reinterpret_cast<const float4*>(lw + row * L::S + c);
    const float p = pu[row];
    v.x = q.x * v.x * p, v.y = q.y * v.y * p, v.z = q.z * v.z * p, v.w = q.w * v.w * p;
    return v;
  };
  auto largest = [&](int row, const float4& v, int cols) {  // (every lane comes here)
    const int k = row < rows ? diag + row : 64;  // column k and those before do not count
    const float a0 = cols > 0 && k < 0 ? fabsf(v.x) : 0.f;
    const float a1 = cols > 1 && k < 1 ? fabsf(v.y) : 0.f;
    const float a2 = cols > 2 && k < 2 ? fabsf(v.z) : 0.f;
    const float a3 = cols > 3 && k < 3 ? fabsf(v.w) : 0.f;
    cm[0] = fmaxf(cm[0], a0), cm[1] = fmaxf(cm[1], a1);
    cm[2] = fmaxf(cm[2], a2), cm[3] = fmaxf(cm[3], a3);
    float r = fmaxf(fmaxf(a0, a1), fmaxf(a2, a3));
    r = fmaxf(r, dpp_mov<0xB1>(r));  // over each 16 lanes: within quads,
    r = fmaxf(r, dpp_mov<0x4E>(r));
    r = fmaxf(r, dpp_mov<0x141>(r));  // halves mirrored, rows mirrored
    r = fmaxf(r, dpp_mov<0x140>(r));
    if (J.rmax && (lane & 15) == 0 && row < rows) raise(J.rmax + m + row, r);
  };
  constexpr int U = 4;
#pragma unroll 1
  for (int i0 = 0; i0 < 32 / L::RPI; i0 += U) {
    float4 old[U];
    if (J.add) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int row = (i0 + u) * L::RPI + sub;
        if (row < rows && left == 4)
          old[u] = *reinterpret_cast<const float4*>(J.C + (m + row) * J.ldc + gn);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = (i0 + u) * L::RPI + sub;
      float4 v = value(row);
      if (J.add) v.x += old[u].x, v.y += old[u].y, v.z += old[u].z, v.w += old[u].w;
      if (row < rows && left == 4)
        *reinterpret_cast<float4*>(J.C + (m + row) * J.ldc + gn) = v;
      if (want) largest(row, v, left == 4 ? 4 : 0);
    }
  }
  if ((J.N & 3) && n + 32 * WT > J.N) {  // (uniform) the last one to three columns
#pragma unroll 1
    for (int i = 0; i < 32 / L::RPI; ++i) {
      const int row = i * L::RPI + sub;
      float4 v = value(row);
      float* o = J.C + (m + row) * J.ldc + gn;
      if (row < rows && left < 4) {
        if (left > 0) v.x = *o = J.add ? *o + v.x : v.x;
        if (left > 1) v.y = o[1] = J.add ? o[1] + v.y : v.y;
        if (left > 2) v.z = o[2] = J.add ? o[2] + v.z : v.z;
      }
      if (want) largest(row, v, left < 4 ? left : 0);
    }
  }
}

// the rows of blocks one after another (an index sequence: a plain loop of this size is not
// unrolled, and the accumulators would go through scratch)
template <int WT, int... I>
__device__ __forceinline__ void store_f16(std::integer_sequence<int, I...>, const FragJob& J,
                                          const f32x16_t (&acc)[WT][WT], float* lw, int64_t m,
                                          int64_t n, int lane, const float* pu, const float* qu) {
  using L = Stores<WT>;
  float cm[4] = {};
  auto rows = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (LDS of one wave: its accesses are
    __builtin_amdgcn_wave_barrier();                        // done in order)
    float* w = lw + 4 * (lane >> 5) * L::S + (lane & 31);
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) w[(8 * (r >> 2) + (r & 3)) * L::S + 32 * j] = acc[i][j][r];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    store_rows<WT>(J, lw, m + 32 * i, n, lane, pu + 32 * i, qu, cm);
  };
  (rows(std::integral_constant<int, I>{}), ...);
  if (J.cmax) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float v = cm[k];
#pragma unroll
      for (int o = L::LPR; o < 64; o <<= 1) v = fmaxf(v, __shfl_xor(v, o));
      const int64_t gn = n + 4 * (lane % L::LPR) + k;
      if (lane < L::LPR && gn < J.N) raise(J.cmax + gn, v);
    }
  }
}

// one 32 x 32 block of a tile of bf16 planes at (m, n), straight from the accumulators: the
// additions to C want many loads in flight
__device__ __forceinline__ void store_block(const FragJob& J, const f32x16_t& acc, int64_t m,
                                            int64_t n, int lane) {
  const int64_t gm0 = m + 4 * (lane >> 5), gn = n + (lane & 31);
  if (gn >= J.N) return;
  float* c = J.C + gm0 * J.ldc + gn;
  if (m + 32 <= J.M) {  // uniform: every row of the block exists
    float old[16];
    if (J.add) {
#pragma unroll
      for (int r = 0; r < 16; ++r) old[r] = c[(8 * (r >> 2) + (r & 3)) * J.ldc];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
      c[(8 * (r >> 2) + (r & 3)) * J.ldc] = J.add ? old[r] + J.alpha * acc[r] : J.alpha * acc[r];
    return;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (gm0 + 8 * (r >> 2) + (r & 3) < J.M) {
      float* e = c + (8 * (r >> 2) + (r & 3)) * J.ldc;
      *e = J.add ? *e + J.alpha * acc[r] : J.alpha * acc[r];
    }
  }
}

template <int WT, int... I>
__device__ __forceinline__ void store_bf16(std::integer_sequence<int, I...>, const FragJob& J,
                                           const f32x16_t (&acc)[WT][WT], int64_t m, int64_t n,
                                           int lane) {
  (store_block(J, acc[I / WT][I % WT], m + 32 * (I / WT), n + 32 * (I % WT), lane), ...);
}

template <bool F16, int WT>
__device__ __forceinline__ void frag_tile(const FragJob& J, const Tiles& T, int b,
                                          uint32_t* lds) {
  constexpr int TM = 64 * WT, G = TM / 32, R = 4;
  constexpr int PLANE = G * 256, STAGE = 4 * PLANE;  // dwords
  static_assert(4 * 32 * Stores<WT>::S + 2 * TM <= R * STAGE, "the stores' rows and units");
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
  // the second pair's K range follows the first's; there is a stage (see frag_launch)
  const int nst = n1 + int(J.K2 / 16);

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
  // the largest values behind the units of the tile's rows, then its columns (for the stores)
  const bool scaled = F16 && J.pmax;
  float top[TM / 128] = {};
  if (scaled) {
#pragma unroll
    for (int i = 0; i < TM / 128; ++i) {
      const int e = tid + 256 * i;
      const int64_t m = m0 + e < J.M ? m0 + e : J.M - 1;
      const int64_t n = n0 + e - TM < J.N ? n0 + e - TM : J.N - 1;
      top[i] = *(e < TM ? J.pmax + m : J.qmax + n);
    }
  }
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
  int el = threadIdx.x;
  asm volatile("" : "+v"(el));  // (the stores' addresses are formed here, not held over the loop)
  const int64_t mw = m0 + wm * WT * 32, nw0 = n0 + wn * WT * 32;
  if constexpr (F16) {
    asm volatile("s_barrier" ::: "memory");  // the ring is free: no wave's loads are on their way
    float* const rows32 = reinterpret_cast<float*>(lds);
    float* const units = rows32 + 4 * 32 * Stores<WT>::S;  // (in the ring: the compiler makes
    // every read of an LDS array wait for the loads into it once the kernel has a second array)
#pragma unroll
    for (int i = 0; i < TM / 128; ++i) units[el + 256 * i] = scaled ? plane_unit(top[i]) : 1.f;
    __syncthreads();
    store_f16<WT>(std::make_integer_sequence<int, WT>{}, J, acc,
                  rows32 + wave * 32 * Stores<WT>::S, mw, nw0, el & 63, units + wm * WT * 32,
                  units + TM + wn * WT * 32);
  } else {
    store_bf16<WT>(std::make_integer_sequence<int, WT * WT>{}, J, acc, mw, nw0, el & 63);
  }
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

// the differences r - c of the elements (r, c) that count
__device__ __forceinline__ void tri_range(int tri, int& lo, int& hi) {
  lo = tri == TRI_LOWER ? 0 : -0x40000000;
  hi = tri == TRI_UPPER ? 0 : tri == TRI_STRICT_UPPER ? -1 : 0x40000000;
}

// four values of row r from column c on (a whole vector, or what the row has left)
__device__ __forceinline__ void load4(const float* p, int64_t c, int64_t cols, float (&x)[4]) {
  if (c + 4 <= cols) {
    const float4 v = *reinterpret_cast<const float4*>(p + c);
    x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = c + k < cols ? p[c + k] : 0.f;
  }
}

// the factor of column c
__device__ __forceinline__ float col_factor(const ColScale& s, int64_t c) {
  const float u = plane_unit(s.max[c]);
  return s.inverse ? 1.f / u : u;
}

// Largest absolute values of the rows and columns: 32 x 256 tiles, a wave on 8 rows with all its
// loads in flight, one atomic per row and column of a tile. (Values compare as their bits; of a
// row with a NaN it is the NaN.)
__global__ __launch_bounds__(256) void abs_max(AbsMaxJob j0, AbsMaxJob j1) {
  constexpr int R = 8;
  __shared__ uint32_t red[4][256];
  const AbsMaxJob& J = blockIdx.z == 0 ? j0 : j1;
  const int64_t r0 = int64_t(blockIdx.y) * 4 * R, c0 = int64_t(blockIdx.x) * 256;
  if (r0 >= J.rows || c0 >= J.cols) return;
  const bool upper = J.tri == TRI_UPPER || J.tri == TRI_STRICT_UPPER;
  if (J.tri == TRI_LOWER && c0 > r0 + 4 * R - 1) return;
  if (upper && r0 > c0 + 255) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t rw = r0 + R * wave;
  const int left = int(J.rows - rw < R ? J.rows - rw : R);  // rows that exist (may be negative)
  // (a ragged last tile: lanes at and past the edge take the last four columns, some of them twice)
  const int64_t c = c0 + 4 * lane < J.cols - 4 ? c0 + 4 * lane : J.cols - 4;
  const float* p = J.src + (left > 0 ? rw : J.rows - 1) * J.ld + c;
  f32x4u_t x[R];
#pragma unroll
  for (int i = 0; i < R; ++i)
    x[i] = *reinterpret_cast<const f32x4u_t*>(p + int64_t(i < left ? i : left > 0 ? left - 1 : 0) *
                                                      J.ld);
  uint32_t v[R][4], cm[4] = {};
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) v[i][k] = __float_as_uint(x[i][k]) & 0x7FFFFFFFu;
  // the part that counts, where the tile is not all of it (uniform)
  if (J.tri != TRI_FULL && (upper ? r0 + 4 * R > c0 : c0 + 256 > r0)) {
    int lo, hi;
    tri_range(J.tri, lo, hi);
    const int d0 = int(rw - c);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (d0 + i - k < lo || d0 + i - k > hi) v[i][k] = 0;
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (i >= left) v[i][0] = v[i][1] = v[i][2] = v[i][3] = 0;  // (uniform)
#pragma unroll
    for (int k = 0; k < 4; ++k) cm[k] = max(cm[k], v[i][k]);
  }
  if (J.rmax) {
    // over the lanes: half of the rows change hands at each of three steps, then one row is left
    uint32_t m[R];
    float cf[4] = {};
    if (J.scale.max) {
#pragma unroll
      for (int k = 0; k < 4; ++k) cf[k] = col_factor(J.scale, c + k);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (J.scale.max) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          v[i][k] = __float_as_uint(__uint_as_float(v[i][k]) * cf[k]);
      }
      m[i] = max(max(v[i][0], v[i][1]), max(v[i][2], v[i][3]));
    }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) {
        const uint32_t keep = lane & o ? m[k + o] : m[k], give = lane & o ? m[k] : m[k + o];
        m[k] = max(keep, uint32_t(__shfl_xor(int(give), o)));
      }
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) m[0] = max(m[0], uint32_t(__shfl_xor(int(m[0]), o)));
    if (lane < left && lane < R) atomicMax(reinterpret_cast<unsigned*>(J.rmax + rw + lane), m[0]);
  }
  if (J.cmax) {  // (uniform over the workgroup)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c + k >= c0) red[wave][c + k - c0] = cm[k];  // (the same value where taken twice)
    __syncthreads();
    if (c0 + tid < J.cols)
      atomicMax(reinterpret_cast<unsigned*>(J.cmax + c0 + tid),
                max(max(red[0][tid], red[1][tid]), max(red[2][tid], red[3][tid])));
  }
}

__global__ void clear_floats(float* __restrict__ p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = 0.f;
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
  if (J.tri == TRI_LOWER && c0 > (r0 | 255)) return;
  if ((J.tri == TRI_UPPER || J.tri == TRI_STRICT_UPPER) && r0 > (c0 | 255)) return;
  const int tid = threadIdx.x, q = (tid & 15) * 4, rr = tid >> 4;
  int lo, hi;
  tri_range(J.tri, lo, hi);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + rr + 16 * i, c = c0 + q;
    float x[4] = {};
    if (r < J.rows) load4(J.src + r * J.ld, c, J.cols, x);
    if (J.scale.max) {
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] *= col_factor(J.scale, c + k < J.cols ? c + k : J.cols - 1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int d = int(r - c) - k;
      t[rr + 16 * i][q + k] = d >= lo && d <= hi ? x[k] : 0.f;
    }
  }
  __syncthreads();
  const int64_t n0 = J.trans ? c0 : r0, k0 = J.trans ? r0 : c0;
  const int64_t rows = J.trans ? J.cols : J.rows;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = tid + 256 * i, nn = (e & 31) + 32 * (e >> 8), kk = ((e >> 5) & 7) * 8;
    const int64_t n = n0 + nn;
    if (n >= ((rows + 31) & ~int64_t(31)) || k0 + kk >= J.ks * 16) continue;
    const float inv = 1.f / plane_unit(J.max[n < rows ? n : rows - 1]);
    uint32_t h[4], l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float a = J.trans ? t[kk + 2 * c][nn] : t[nn][kk + 2 * c];
      const float b = J.trans ? t[kk + 2 * c + 1][nn] : t[nn][kk + 2 * c + 1];
      split_f16(a * inv, b * inv, h[c], l[c]);
    }
    const int64_t f = split_frag_index(n, k0 + kk, J.ks);
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
    // every tile that is not skipped has a K range that is not empty
    KQ_REQUIRE(J.M > 0 && J.N > 0 && J.K + J.K2 > 0 && (!(J.flags & FRAG_P_UPPER) || J.M <= J.K) &&
                   (!(J.flags & FRAG_Q_UPPER) || J.N <= J.K),
               KRONQ_ERR_INVALID_ARG, "gemm_frag: empty product");
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

int abs_max_launch(const AbsMaxJob* jobs, int n, hipStream_t s, const char* name) {
  for (int i = 0; i < n; ++i)
    KQ_REQUIRE(jobs[i].cols >= 4, KRONQ_ERR_INVALID_ARG, "abs_max: fewer than four columns");
  const int64_t r = std::max(jobs[0].rows, jobs[n - 1].rows);
  const int64_t c = std::max(jobs[0].cols, jobs[n - 1].cols);
  return launch(name, abs_max, dim3(unsigned(cdiv(c, 256)), unsigned(cdiv(r, 32)), unsigned(n)),
                dim3(256), 0, s, jobs[0], jobs[n - 1]);
}

int clear_launch(float* p, int64_t n, hipStream_t s, const char* name) {
  const int64_t g = cdiv(n, 256);
  return launch(name, clear_floats, dim3(unsigned(g < 256 ? g : 256)), dim3(256), 0, s, p, n);
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

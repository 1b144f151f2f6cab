// Inference with a quantised layer: the rotations are applied online, O(d log d) per layer
// (Sec. 3.2 and 4.2; Limitations), around a matvec on the packed low-bit codes, so that
// y = S_G^-1 U^T W_hat' V S_X^-1 x (the original-space layer of Alg. 2's last line) is never
// formed as a dense matrix. For B <= 4 activation vectors:
//   1. x' = V S_X^-1 x and 3. y = S_G^-1 U^T y' by seg_transform: a transform of order
//      d = L m (m = 2^k <= 1024) is A (x) H_m with A = Q28 (or Q28^T) when d = 28 m and A = H_L
//      otherwise (Sylvester: H_d = H_L (x) H_m). Segment a of the output is H_m applied to
//      sum_k A[a][k] x_k over the L input segments, so workgroup (a, vector) mixes the segments,
//      runs one FWHT of m points in LDS and applies the multipliers: L workgroups per vector
//      instead of one.
//   2. y' = W_hat' x': the packed-code GEMV, bound by the HBM reads of the codes.
// Packed format: each run of 32 consecutive codes of a row is one 32 * bits-bit little-endian
// string held in `bits` uint32 words.
// GEMV (online_gemv_mfma, every code width and 1 to 4 vectors): the packed codes meet x' as bytes
// on the int8 matrix cores. x' is held as four signed byte digits per element, a 30-bit fixed
// point with one exponent per 128 columns, and the 4 x B digit vectors are the columns of the B
// operand of v_mfma_i32_16x16x64_i8, whose A operand is 16 rows of codes: two of them cover 128
// columns with exact integer sums, and one fp32 FMA per row, digit vector and 128 columns applies
// scale and exponent. The VALU only spreads the codes to bytes: 0.4 (4-bit) to 1.7 (3-bit)
// operations per code and lane, and about 0.4 for the sums, whatever the batch. (The dot4
// products of one vector at a time this replaces took 1.1 per code and vector with 2- and 4-bit
// codes, and an fp32 unpack-and-FMA 3.5 with 3- and 8-bit codes: a 14336 x 4096 3-bit matrix
// with four vectors took 168 us.) What bounds it now is its own short chain, one step after another:
// the first codes, the transform of x, the sums at the end (9.2 us at 4096 x 4096, of which an empty
// launch is 1.5 to 1.8).
#include <cmath>

#include "kq_common.hpp"
#include "kq_fwht.hpp"

namespace kq {
namespace {

__device__ __forceinline__ float ld_f32(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld_f32(const uint16_t* p, int64_t i) {
  return __uint_as_float(uint32_t(p[i]) << 16);
}

// one thread per (row, unit of 32 codes)
template <int BITS>
__global__ __launch_bounds__(256) void pack_codes(const uint8_t* __restrict__ codes,
                                                  int64_t d_out, int64_t units, int64_t ldq,
                                                  uint32_t* __restrict__ packed, int64_t ldp) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= d_out * units) return;
  const int64_t row = t / units, u = t % units;
  const uint8_t* c = codes + row * ldq + u * 32;
  uint32_t w[BITS];
#pragma unroll
  for (int k = 0; k < BITS; ++k) w[k] = 0u;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const uint32_t q = uint32_t(c[j]) & ((1u << BITS) - 1u);
    const int pos = j * BITS, wi = pos >> 5, off = pos & 31;
    w[wi] |= q << off;
    if (off + BITS > 32) w[wi + 1] |= q >> (32 - off);
  }
  uint32_t* o = packed + row * ldp + u * BITS;
#pragma unroll
  for (int k = 0; k < BITS; ++k) o[k] = w[k];
}

// Digits of x' for the integer GEMV. Per group of 128 columns, with |x'_j| < 2^e over the group,
// X_j = rint(x'_j 2^(30 - e)) = sum_k d_k 256^k with signed bytes d_k (so a value within 2^-6 of
// the group's largest is exact). A 32-column chunk's digits are 32 dwords [h][k][s], h = 0, 1,
// digit k = 0..3, s = 0..3: byte i is digit k of column digit_col(4 h + s, i) of the chunk,
// the order in which the GEMV spreads the codes of a packed chunk (code dword 4 h + s). Beside
// them, per group: the weight 2^(e - 30) and the sum of its x' (fp64, rounded once).
template <int BITS>
__device__ __forceinline__ int digit_col(int slot, int i) {
  if constexpr (BITS == 2) return 16 * (slot >> 2) + (slot & 3) + 4 * i;
  if constexpr (BITS == 8) return 4 * slot + i;
  return 8 * (slot >> 1) + (slot & 1) + 2 * i;  // 3 and 4 bits
}
__device__ __forceinline__ int digit_col(int bits, int slot, int i) {
  return bits == 2 ? digit_col<2>(slot, i) : bits == 8 ? digit_col<8>(slot, i)
                                                       : digit_col<4>(slot, i);
}
// exponent e of a group whose largest magnitude is mx (groups below 2^-96 keep that exponent)
__device__ __forceinline__ int group_exp(float mx) {
  return max(int((__float_as_uint(mx) >> 23) & 0xFFu) - 126, -96);
}
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float(uint32_t(127 + e) << 23); }
// the four digits of v as the bytes of a dword; up = 2^(30 - e)
__device__ __forceinline__ uint32_t digits_of(float v, float up) {
  return (uint32_t(int(rintf(v * up))) + 0x00808080u) ^ 0x00808080u;
}
// byte k of four digit dwords, in bytes 0..3
__device__ __forceinline__ uint32_t digit_bytes(uint32_t z0, uint32_t z1, uint32_t z2,
                                                uint32_t z3, int k) {
  const uint32_t sel = uint32_t(k) | (uint32_t(4 + k) << 8);  // byte k of each source
  const uint32_t lo = __builtin_amdgcn_perm(z1, z0, sel), hi = __builtin_amdgcn_perm(z3, z2, sel);
  return (lo & 0xFFFFu) | (hi << 16);
}

// The digits of the whole groups of 128 columns held one element per thread (tid < m, m a
// multiple of 128; every thread of the workgroup calls it): z (m dwords of LDS) and red (2 x 16
// doubles) are scratch; dig, gw and gs point at this vector's first group of the workgroup.
__device__ __forceinline__ void emit_digits(float v, int tid, int m, int bits,
                                            uint32_t* __restrict__ z, double* __restrict__ red,
                                            uint32_t* __restrict__ dig, float* __restrict__ gw,
                                            float* __restrict__ gs) {
  const bool in = tid < m;
  const int wave = tid >> 6;
  float mx = in ? fabsf(v) : 0.f;
  double sum = in ? double(v) : 0.0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, o));
    sum += __shfl_xor(sum, o);
  }
  if ((tid & 63) == 0) red[wave] = double(mx), red[16 + wave] = sum;
  __syncthreads();
  const int e = group_exp(fmaxf(float(red[wave & ~1]), float(red[wave | 1])));
  if (in) z[tid] = digits_of(v, pow2f(30 - e));
  if (in && (tid & 127) == 0) {
    gw[tid >> 7] = pow2f(e - 30);
    gs[tid >> 7] = float(red[16 + wave] + red[16 + (wave | 1)]);
  }
  __syncthreads();
  if (in) {
    const uint32_t* zc = z + (tid & ~31);
    const int w = tid & 31, k = (w >> 2) & 3, slot = 4 * (w >> 4) + (w & 3);
    dig[tid] = digit_bytes(zc[digit_col(bits, slot, 0)], zc[digit_col(bits, slot, 1)],
                           zc[digit_col(bits, slot, 2)], zc[digit_col(bits, slot, 3)], k);
  }
}

// 8 consecutive activations as loaded (16-byte loads), widened to fp32 later
template <typename T>
struct RawX;
template <>
struct RawX<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = reinterpret_cast<const float4*>(p)[0];
    b = reinterpret_cast<const float4*>(p)[1];
  }
  __device__ __forceinline__ void widen(float* v) const {
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  }
};
template <>
struct RawX<uint16_t> {
  uint4 a;
  __device__ __forceinline__ void load(const uint16_t* p) { a = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void widen(float* v) const {
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = __uint_as_float(w[k] << 16);
      v[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
    }
  }
};

// Transform of B vectors of order d = L m: out[b] = diag(post) (A (x) H_m) diag(pre) src[b] * norm
// (A = Q28 or Q28^T when has28, else the Sylvester H_L). Workgroup (a, b): segment a of vector b.
// With dig != nullptr (and m a multiple of 128) it writes the digits of the result instead.
template <typename T>
__global__ __launch_bounds__(1024) void seg_transform(
    const T* __restrict__ src, int64_t lds_, float* __restrict__ dst, int64_t ldd, int L, int m,
    const float* __restrict__ pre, const float* __restrict__ post, const float* __restrict__ q28,
    int q_trans, int has28, float norm, uint32_t* __restrict__ dig, float* __restrict__ gw,
    float* __restrict__ gs, int bits) {
  __shared__ float t[1024];
  __shared__ float arow[32];
  __shared__ double red[32];
  extern __shared__ __attribute__((aligned(16))) float xs[];  // L m floats: diag(pre) src[b]
  const int a = blockIdx.x, tid = threadIdx.x;
  const T* x = src + int64_t(blockIdx.y) * lds_;
  if (tid < L)
    arow[tid] = has28 ? (q_trans ? q28[tid * 28 + a] : q28[a * 28 + tid])
                      : ((__popc(unsigned(a & tid)) & 1) ? -1.f : 1.f);
  // the whole vector, scaled, into LDS with 16-byte loads (8 elements a thread and step), each
  // workgroup starting at its own offset: every workgroup reads all L segments, and in one
  // order, or with each thread's L loads in flight at once, their requests queued on the same
  // lines (a segment read straight from memory by each thread took about 10 us at 28 x 512)
  const int d = L * m;
  const bool vec = d % 8 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(pre) & 15) == 0;
  if (vec) {
    const int n8 = d / 8, rot = int((uint32_t(a) * 97u + uint32_t(blockIdx.y) * 31u) % uint32_t(n8));
    for (int i = tid; i < n8; i += 1024) {
      const int j = 8 * (i + rot < n8 ? i + rot : i + rot - n8);
      RawX<T> r;
      r.load(x + j);
      float v[8];
      r.widen(v);
      if (pre) {
        const float4 p0 = reinterpret_cast<const float4*>(pre + j)[0];
        const float4 p1 = reinterpret_cast<const float4*>(pre + j)[1];
        v[0] *= p0.x, v[1] *= p0.y, v[2] *= p0.z, v[3] *= p0.w;
        v[4] *= p1.x, v[5] *= p1.y, v[6] *= p1.z, v[7] *= p1.w;
      }
      float4* o = reinterpret_cast<float4*>(xs + j);
      o[0] = make_float4(v[0], v[1], v[2], v[3]);
      o[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
  } else {
    for (int i = tid; i < d; i += 1024) xs[i] = pre ? ld_f32(x, i) * pre[i] : ld_f32(x, i);
  }
  __syncthreads();
  if (tid < m) {
    float acc = 0.f;
    for (int k = 0; k < L; ++k) acc = fmaf(arow[k], xs[k * m + tid], acc);
    t[tid] = acc;
  }
  __syncthreads();
  fwht_lds(t, m, m, tid, 1024);  // radix-8 groups of stages; ends with a barrier
  const int64_t idx = int64_t(a) * m + tid;
  float v = 0.f;
  if (tid < m) {
    v = t[tid] * norm;
    if (post) v *= post[idx];
    if (!dig) dst[int64_t(blockIdx.y) * ldd + idx] = v;
  }
  if (dig) {  // (t is reused for the digits: emit_digits has a barrier before it writes there)
    const int64_t g0 = (int64_t(blockIdx.y) * d + int64_t(a) * m) >> 7;
    emit_digits(v, tid, m, bits, reinterpret_cast<uint32_t*>(t), red, dig + g0 * 128, gw + g0,
                gs + g0);
  }
}

// digits of B fp32 vectors of length d (a multiple of 128) that no transform produced, in place:
// workgroup (g, b) turns the 128 values of group g of vector b into their 128 digit dwords
__global__ __launch_bounds__(128) void digitize(float* x, int64_t d, int bits,
                                                float* __restrict__ gw, float* __restrict__ gs) {
  __shared__ uint32_t z[128];
  __shared__ double red[32];
  const int tid = threadIdx.x;
  const int64_t g = (int64_t(blockIdx.y) * d >> 7) + blockIdx.x;
  const float v = x[g * 128 + tid];  // read by every thread before emit_digits' first barrier
  emit_digits(v, tid, 128, bits, z, red, reinterpret_cast<uint32_t*>(x) + g * 128, gw + g,
              gs + g);
}

// lane (lane ^ 1) and (lane ^ 2) of each quad (DPP quad_perm [1,0,3,2] and [2,3,0,1])
__device__ __forceinline__ int quad_xor1(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
}
__device__ __forceinline__ int quad_xor2(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
}

typedef int i32x4_t __attribute__((ext_vector_type(4)));

// ---- the GEMV --------------------------------------------------------------------------------
// A workgroup of 8 waves takes blocks of 16 rows (blockIdx.x, + gridDim.x, ...); its waves share
// the columns, each a contiguous range of 128-column groups, walked in tiles of 4 groups: per tile
// a lane reads the codes of one row and one 32-column chunk of each group (lane = row + 16 chunk,
// the A operand's layout) and one scale and zero (row lane / 4, group lane % 4), unconditionally
// (indices clamped), two tiles ahead of their use. The waves' partial sums meet in LDS once per
// row block.
constexpr int GW = 8;  // waves
constexpr int GC = 4;  // groups of 128 columns per tile

template <int BITS>
struct Tile {
  uint32_t w[GC][BITS];
  float sc, ze;
};

template <int BITS>
__device__ __forceinline__ void load_tile(Tile<BITS>& T, int64_t row0, int g0, int ng, int lane,
                                          const uint32_t* __restrict__ packed, int64_t ldp,
                                          const float* __restrict__ scales,
                                          const float* __restrict__ zeros, int64_t ldsz,
                                          unsigned gpq, int64_t d_out) {
  const int64_t rs = row0 + (lane >> 2) < d_out ? row0 + (lane >> 2) : d_out - 1;
  const int gl = g0 + (lane & 3) < ng ? g0 + (lane & 3) : ng - 1;
  const int64_t at = rs * ldsz + unsigned(gl) / gpq;  // gpq groups of 128 per scale
  T.sc = scales[at];
  T.ze = zeros[at];
  const int64_t row = row0 + (lane & 15) < d_out ? row0 + (lane & 15) : d_out - 1;
  const uint32_t* p = packed + row * ldp + (lane >> 4) * BITS;
#pragma unroll
  for (int i = 0; i < GC; ++i) {
    const int g = g0 + i < ng ? g0 + i : ng - 1;
    const uint32_t* c = p + int64_t(g) * (4 * BITS);
    if constexpr (BITS == 2) {
      const uint2 v = *reinterpret_cast<const uint2*>(c);
      T.w[i][0] = v.x, T.w[i][1] = v.y;
    } else if constexpr (BITS == 3) {
      T.w[i][0] = c[0], T.w[i][1] = c[1], T.w[i][2] = c[2];
    } else {
#pragma unroll
      for (int k = 0; k < BITS; k += 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(c + k);
        T.w[i][k] = v.x, T.w[i][k + 1] = v.y, T.w[i][k + 2] = v.z, T.w[i][k + 3] = v.w;
      }
    }
  }
}

// 8 code dwords of a chunk in the digits' order (8-bit codes minus 128, as signed bytes)
template <int BITS>
__device__ __forceinline__ void spread_codes(const uint32_t (&w)[BITS], i32x4_t (&a)[2]) {
  uint32_t o[8];
  if constexpr (BITS == 2) {
#pragma unroll
    for (int s = 0; s < 8; ++s) o[s] = (w[s >> 2] >> (2 * (s & 3))) & 0x03030303u;
  } else if constexpr (BITS == 4) {
#pragma unroll
    for (int s = 0; s < 8; ++s) o[s] = (w[s >> 1] >> (4 * (s & 1))) & 0x0F0F0F0Fu;
  } else if constexpr (BITS == 8) {
#pragma unroll
    for (int s = 0; s < 8; ++s) o[s] = w[s] ^ 0x80808080u;
  } else {
    // eight 3-bit codes per 24 bits; the even (odd) ones sit 6 bits apart: the upper pair moves
    // up by 4, then the odd member of each pair by 2
    const uint32_t g[4] = {w[0], __builtin_amdgcn_alignbit(w[1], w[0], 24),
                           __builtin_amdgcn_alignbit(w[2], w[1], 16), w[2] >> 8};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint32_t t = g[s >> 1] >> (3 * (s & 1));
      const uint32_t u = (t & 0x1C7u) | ((t << 4) & 0x1C70000u);
      o[s] = (u & 0x00070007u) | ((u << 2) & 0x07000700u);
    }
  }
  a[0] = i32x4_t{int(o[0]), int(o[1]), int(o[2]), int(o[3])};
  a[1] = i32x4_t{int(o[4]), int(o[5]), int(o[6]), int(o[7])};
}

constexpr int FUSE_MAX_DIN = 8192;

// LDS slot of element j of the staged x': 4 floats of padding after every 128, so that the
// strided butterfly passes below hit distinct banks (a stride of 256 moves 8 banks)
__device__ __forceinline__ int xslot(int j) { return j + ((j >> 7) << 2); }

// the stages of strides 8 .. d/2 of the FWHT of d = 2^k staged elements (those of strides 1, 2, 4
// are applied in registers while staging), in groups of up to three stages per LDS round trip
template <int R>
__device__ __forceinline__ void stage_group_x(float* xt, int d, int lgh, int tid) {
  const int hm = (1 << lgh) - 1;
  for (int q = tid; q < d / R; q += 64 * GW) {
    const int base = ((q >> lgh) * (R << lgh)) + (q & hm);
    float v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = xt[xslot(base + (i << lgh))];
    hadamard_reg<R>(v);
#pragma unroll
    for (int i = 0; i < R; ++i) xt[xslot(base + (i << lgh))] = v[i];
  }
}
__device__ __forceinline__ void fwht_x(float* xt, int d, int tid) {
  for (int lgh = 3; (1 << lgh) < d;) {
    const int left = d >> lgh;
    if (left == 16 || left == 1024) {  // 4 stages, where that saves a round trip
      stage_group_x<16>(xt, d, lgh, tid);
      lgh += 4;
    } else if (left >= 8) {
      stage_group_x<8>(xt, d, lgh, tid);
      lgh += 3;
    } else if (left == 4) {
      stage_group_x<4>(xt, d, lgh, tid);
      lgh += 2;
    } else {
      stage_group_x<2>(xt, d, lgh, tid);
      lgh += 1;
    }
    __syncthreads();
  }
}

// With FUSE (one vector) the workgroup forms x' itself: x and the multipliers are requested before
// the tiles' codes, so the transform (the Sylvester FWHT of a power-of-two d_in, or the scaling
// alone) runs while the codes are in flight; it is repeated by every workgroup, which costs less
// than a separate launch at these sizes. Otherwise the digits come from dig, gw and gs.
template <int BITS, int NB, int FUSE, typename TX>
__global__ __launch_bounds__(64 * GW) void online_gemv_mfma(
    const uint32_t* __restrict__ packed, int64_t ldp, const float* __restrict__ scales,
    const float* __restrict__ zeros, int64_t ldsz, int group, int64_t d_out, int64_t d_in,
    const uint32_t* __restrict__ dig, const float* __restrict__ gw, const float* __restrict__ gs,
    const TX* __restrict__ x, const float* __restrict__ mul, int rotate, float norm,
    float* __restrict__ yr) {
  static_assert(!FUSE || NB == 1, "the fused transform takes one vector");
  extern __shared__ __attribute__((aligned(16))) uint32_t sm[];
  const int ng = int(d_in >> 7), nch = 4 * ng;
  uint32_t* sd = sm;  // digits [chunk][h][vector][k][4 dwords]
  float* sw = reinterpret_cast<float*>(sm + size_t(NB) * nch * 32);  // [vector][group] weights
  float* ss = sw + NB * ng;                                          // [vector][group] sums
  float* xt = ss + NB * ng;  // FUSE: d_in + d_in / 32 floats (slots xslot(j))
  // (2 NB ng floats are not always whole 16-byte units)
  float* sc = reinterpret_cast<float*>(
      sm + ((size_t(NB) * nch * 32 + 2 * NB * ng + (FUSE ? d_in + d_in / 32 : 0) + 3) & ~size_t(3)));
  if constexpr (FUSE) xt = sc - (d_in + d_in / 32);  // 16-byte aligned (both are whole units)
  float* red = sc + GW * 64;  // [2][GW][2][16][NB]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int64_t nblk = cdiv(d_out, 16);
  const int nrb = int((nblk - 1 - blockIdx.x) / gridDim.x + 1);  // row blocks (grid <= nblk)
  const int per = (ng + GW - 1) / GW;
  const int gbeg = wave * per < ng ? wave * per : ng, gend = gbeg + per < ng ? gbeg + per : ng;
  const int nt = (gend - gbeg + GC - 1) / GC;  // tiles per row block (0: this wave has no columns)
  const unsigned gpq = unsigned(group >> 7);
  RawX<TX> xr[FUSE ? 2 : 1];
  float4 mr[FUSE ? 4 : 1];
  if constexpr (FUSE) {  // indices clamped; a missing mul reads x's first bytes, unused
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int j0 = 8 * (tid + 64 * GW * k), j = j0 < d_in ? j0 : 0;
      xr[k].load(x + j);
      const float4* mp =
          reinterpret_cast<const float4*>(mul ? mul + j : reinterpret_cast<const float*>(x));
      mr[2 * k] = mp[0];
      mr[2 * k + 1] = mp[mul ? 1 : 0];
    }
  }
  // tiles in (row block, tile) order, clamped to the last one (loaded again, never used)
  auto load = [&](Tile<BITS>& T, int k, int t) {
    load_tile<BITS>(T, (int64_t(blockIdx.x) + int64_t(k) * gridDim.x) * 16, gbeg + t * GC, ng,
                    lane, packed, ldp, scales, zeros, ldsz, gpq, d_out);
  };
  auto next = [&](int& k, int& t) {
    if (++t >= nt) t = 0, ++k;
    if (k >= nrb) k = nrb - 1, t = nt > 0 ? nt - 1 : 0;
  };
  int k = 0, t = 0, k1 = 0, t1 = 0;
  next(k1, t1);
  Tile<BITS> A, B;
  load(A, k, t);
  load(B, k1, t1);
  if constexpr (FUSE) {
    // the butterflies of strides 1, 2, 4 on each thread's 8 consecutive values, in registers;
    // the other stages in LDS
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int j = 8 * (tid + 64 * GW * k);
      if (j < d_in) {
        float v[8];
        xr[k].widen(v);
        const float m[8] = {mr[2 * k].x, mr[2 * k].y, mr[2 * k].z, mr[2 * k].w,
                            mr[2 * k + 1].x, mr[2 * k + 1].y, mr[2 * k + 1].z, mr[2 * k + 1].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = mul ? v[e] * m[e] : v[e];
        if (rotate) hadamard_reg<8>(v);
        float4* dst = reinterpret_cast<float4*>(xt + xslot(j));  // 8 slots, no padding inside
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
      }
    }
    __syncthreads();
    if (rotate) fwht_x(xt, int(d_in), tid);  // each group ends with a barrier
    // digits: two threads per chunk (h = 0, 1), eight neighbours per group
    for (int u = tid; u < 2 * nch; u += 64 * GW) {  // whole groups: uniform over 8 lanes
      const int c = u >> 1, h = u & 1;
      float v[16], mx = 0.f;
      double sum = 0.0;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        v[e] = xt[xslot(32 * c + digit_col<BITS>(4 * h + (e >> 2), e & 3))] * norm;
        mx = fmaxf(mx, fabsf(v[e]));
        sum += double(v[e]);
      }
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, o));
        sum += __shfl_xor(sum, o);
      }
      const int e2 = group_exp(mx);
      const float up = pow2f(30 - e2);
      uint32_t z[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) z[e] = digits_of(v[e], up);
#pragma unroll
      for (int kd = 0; kd < 4; ++kd) {
        uint4 o;
        o.x = digit_bytes(z[0], z[1], z[2], z[3], kd);
        o.y = digit_bytes(z[4], z[5], z[6], z[7], kd);
        o.z = digit_bytes(z[8], z[9], z[10], z[11], kd);
        o.w = digit_bytes(z[12], z[13], z[14], z[15], kd);
        reinterpret_cast<uint4*>(sd)[u * 4 + kd] = o;
      }
      if ((u & 7) == 0) {
        sw[u >> 3] = pow2f(e2 - 30);
        ss[u >> 3] = float(sum);
      }
    }
  } else {
    // every workgroup copies the same digits: each starts at its own offset, so that their
    // requests spread over the L2 channels instead of queueing on one line at a time
    const int n16 = NB * nch * 8, r16 = int((uint32_t(blockIdx.x) * 97u) % uint32_t(n16));
    for (int i = tid; i < n16; i += 64 * GW) {
      const int ii = i + r16 < n16 ? i + r16 : i + r16 - n16;
      const int b = ii / (nch * 8), r = ii - b * (nch * 8);  // r = (chunk * 2 + h) * 4 + k
      reinterpret_cast<uint4*>(sd)[((r >> 2) * NB + b) * 4 + (r & 3)] =
          reinterpret_cast<const uint4*>(dig)[ii];
    }
    for (int i = tid; i < NB * ng; i += 64 * GW) sw[i] = gw[i], ss[i] = gs[i];
  }
  __syncthreads();
  // this lane's digit vector: digit n % 4 of vector n / 4 (columns past 4 NB repeat the last
  // vector; their sums are not used)
  const int bn = (n >> 2) < NB ? n >> 2 : NB - 1;
  const float wk = __uint_as_float(uint32_t(127 + 8 * (n & 3)) << 23);  // 256^k
  const uint32_t* db = sd + (bn * 4 + (n & 3)) * 4;
  const float* swb = sw + bn * ng;
  float* my = sc + wave * 64;
  float acc[4] = {}, zacc[NB] = {};
  auto tile = [&](const Tile<BITS>& T, int t) {
    const int g0 = gbeg + t * GC;
    // scales to the rows of the sums (rows 4 q .. 4 q + 3 of this lane); wave-private LDS
    __builtin_amdgcn_wave_barrier();
    my[(lane & 3) * 16 + (lane >> 2)] = T.sc;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (g0 + (lane & 3) < gend) {
      const float sz = T.sc * (BITS == 8 ? T.ze - 128.f : T.ze);
#pragma unroll
      for (int b = 0; b < NB; ++b) zacc[b] = fmaf(sz, ss[b * ng + g0 + (lane & 3)], zacc[b]);
    }
#pragma unroll
    for (int i = 0; i < GC; ++i) {
      if (g0 + i >= gend) break;  // uniform over the wave
      i32x4_t a[2];
      spread_codes<BITS>(T.w[i], a);
      const uint32_t* dp = db + ((g0 + i) * 4 + q) * (2 * NB * 16);
      i32x4_t D = {};
      D = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[0], *reinterpret_cast<const i32x4_t*>(dp), D, 0,
                                                0, 0);
      D = __builtin_amdgcn_mfma_i32_16x16x64_i8(
          a[1], *reinterpret_cast<const i32x4_t*>(dp + NB * 16), D, 0, 0, 0);
      const float ew = swb[g0 + i] * wk;
      const float4 s4 = *reinterpret_cast<const float4*>(my + i * 16 + 4 * q);
      acc[0] = fmaf(s4.x * ew, float(D[0]), acc[0]);
      acc[1] = fmaf(s4.y * ew, float(D[1]), acc[1]);
      acc[2] = fmaf(s4.z * ew, float(D[2]), acc[2]);
      acc[3] = fmaf(s4.w * ew, float(D[3]), acc[3]);
    }
  };
  auto quad = [](float v) {
    v += __int_as_float(quad_xor1(__float_as_int(v)));
    return v + __int_as_float(quad_xor2(__float_as_int(v)));
  };
  // end of row block k: the digits of each sum, then the waves'. The two halves of red take
  // turns, so one barrier per row block suffices.
  auto finish = [&](int k) {
    float* R = red + size_t((k & 1) * GW + wave) * 2 * 16 * NB;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = quad(acc[r]);
      if ((n & 3) == 0 && (n >> 2) < NB) R[(4 * q + r) * NB + (n >> 2)] = v;
      acc[r] = 0.f;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float v = quad(zacc[b]);
      if ((lane & 3) == 0) R[16 * NB + (lane >> 2) * NB + b] = v;
      zacc[b] = 0.f;
    }
    __syncthreads();
    if (tid < 16 * NB) {
      const float* P = red + size_t((k & 1) * GW) * 2 * 16 * NB + tid;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < GW; ++w) v += P[w * 2 * 16 * NB] - P[(w * 2 + 1) * 16 * NB];
      const int64_t row = (int64_t(blockIdx.x) + int64_t(k) * gridDim.x) * 16 + tid / NB;
      if (row < d_out) yr[int64_t(tid % NB) * d_out + row] = v;
    }
  };
  if (nt == 0) {  // no columns: join the sums
    for (int kk = 0; kk < nrb; ++kk) finish(kk);
    return;
  }
  // A holds tile (k, t), B the tile after it, (k1, t1); a buffer is refilled with the tile two
  // ahead as soon as its products are done
  for (;;) {
    tile(A, t);
    const bool end_a = t == nt - 1, last_a = end_a && k == nrb - 1;
    int k2 = k1, t2 = t1;
    next(k2, t2);
    if (!last_a) load(A, k2, t2);
    if (end_a) finish(k);
    if (last_a) break;
    tile(B, t1);
    const bool end_b = t1 == nt - 1, last_b = end_b && k1 == nrb - 1;
    const int kb = k1;
    k = k2, t = t2, k1 = k2, t1 = t2;
    next(k1, t1);
    if (!last_b) load(B, k1, t1);
    if (end_b) finish(kb);
    if (last_b) break;
  }
}

// LDS of the GEMV: digits, weights and sums, the staged vector, the scales' and the sums' scratch
size_t gemv_lds(int nb, int64_t d_in, bool fuse) {
  const size_t ng = size_t(d_in / 128);
  const size_t head = (size_t(nb) * size_t(d_in) + 2 * size_t(nb) * ng +
                       (fuse ? size_t(d_in + d_in / 32) : 0) + 3) & ~size_t(3);
  return (head + GW * 64 + size_t(2) * GW * 2 * 16 * size_t(nb)) * 4;
}

template <int BITS, int NB, int FUSE, typename TX>
int gemv_launch(const uint32_t* packed, int64_t ldp, const float* scales, const float* zeros,
                int64_t ldsz, int group, int64_t d_out, int64_t d_in, const uint32_t* dig,
                const float* gw, const float* gs, const void* x, const float* mul, bool rotate,
                float* yr, hipStream_t s) {
  const size_t lds = gemv_lds(NB, d_in, FUSE);
  // row blocks dealt to the workgroups the chip holds at once: two per CU where the LDS allows
  // (workgroups w and w + CUs, which share a CU, then hold together an equal share)
  const int64_t slots = int64_t(device_cus()) * (lds <= 80 * 1024 ? 2 : 1);
  const int64_t nblk = cdiv(d_out, 16);
  const float norm = rotate ? float(1.0 / std::sqrt(double(d_in))) : 1.f;
  return launch("online_gemv", online_gemv_mfma<BITS, NB, FUSE, TX>,
                dim3(static_cast<unsigned>(nblk < slots ? nblk : slots)), dim3(64 * GW), lds, s,
                packed, ldp, scales, zeros, ldsz, group, d_out, d_in, dig, gw, gs,
                static_cast<const TX*>(x), mul, int(rotate), norm, yr);
}

template <int BITS>
int gemv_bits(int nb, bool fuse, const uint32_t* packed, int64_t ldp, const float* scales,
              const float* zeros, int64_t ldsz, int group, int64_t d_out, int64_t d_in,
              const uint32_t* dig, const float* gw, const float* gs, const void* x, int x_dtype,
              const float* mul, bool rotate, float* yr, hipStream_t s) {
#define KQ_GEMV(NB_, FUSE_, TX_)                                                                 \
  gemv_launch<BITS, NB_, FUSE_, TX_>(packed, ldp, scales, zeros, ldsz, group, d_out, d_in, dig, \
                                     gw, gs, x, mul, rotate, yr, s)
  if (fuse) return x_dtype == KRONQ_BF16 ? KQ_GEMV(1, 1, uint16_t) : KQ_GEMV(1, 1, float);
  switch (nb) {
    case 1:
      return KQ_GEMV(1, 0, float);
    case 2:
      return KQ_GEMV(2, 0, float);
    case 3:
      return KQ_GEMV(3, 0, float);
    default:
      return KQ_GEMV(4, 0, float);
  }
#undef KQ_GEMV
}

// launch seg_transform for B rows of order d (identity scaling when !rotate); with gw, the digits
// of the result in place of its values (from the transform itself for segments of whole groups,
// else by a separate pass over dst)
int seg_transform_launch(const void* src, int dtype, int64_t lds_, float* dst, int64_t ldd,
                         int64_t batch, int64_t d, const float* pre, const float* post,
                         bool rotate, const float* q28, bool q_trans, hipStream_t s,
                         float* gw = nullptr, float* gs = nullptr, int bits = 0) {
  int L = 0, m = 0, has28 = 0;
  float norm = 1.f;
  const RotDim rd = rot_dim(d);
  if (rotate && rd.has28) {
    L = 28, m = int(rd.m), has28 = 1;
    norm = float(1.0 / std::sqrt(double(m)));
  } else if (rotate) {
    m = int(d < 1024 ? d : 1024), L = int(d / m);
    norm = float(1.0 / std::sqrt(double(d)));
  }
  const bool fused = gw && rotate && m % 128 == 0;
  if (!rotate) {
    KQ_TRY(rotate_vectors(src, dtype, lds_, dst, ldd, batch, d, pre, post, false, nullptr, false,
                          s));
  } else {
    const dim3 grid(static_cast<unsigned>(L), static_cast<unsigned>(batch));
    const size_t xs_bytes = size_t(L) * size_t(m) * sizeof(float);  // the staged vector
    uint32_t* dg = fused ? reinterpret_cast<uint32_t*>(dst) : nullptr;
    if (dtype == KRONQ_BF16)
      KQ_TRY(launch("online_transform", seg_transform<uint16_t>, grid, dim3(1024), xs_bytes, s,
                    static_cast<const uint16_t*>(src), lds_, dst, ldd, L, m, pre, post, q28,
                    int(q_trans), has28, norm, dg, gw, gs, bits));
    else
      KQ_TRY(launch("online_transform", seg_transform<float>, grid, dim3(1024), xs_bytes, s,
                    static_cast<const float*>(src), lds_, dst, ldd, L, m, pre, post, q28,
                    int(q_trans), has28, norm, dg, gw, gs, bits));
  }
  if (gw && !fused)
    KQ_TRY(launch("online_digitize", digitize,
                  dim3(static_cast<unsigned>(d / 128), static_cast<unsigned>(batch)), dim3(128),
                  0, s, dst, d, bits, gw, gs));
  return KRONQ_OK;
}

}  // namespace

int pack_codes_launch(const uint8_t* codes, int64_t d_out, int64_t d_in, int64_t ldq, int bits,
                      uint32_t* packed, int64_t ldp, hipStream_t s) {
  const int64_t units = d_in / 32;
  const dim3 grid(unsigned(cdiv(d_out * units, 256)));
  switch (bits) {
    case 2:
      return launch("pack_codes", pack_codes<2>, grid, dim3(256), 0, s, codes, d_out, units, ldq,
                    packed, ldp);
    case 3:
      return launch("pack_codes", pack_codes<3>, grid, dim3(256), 0, s, codes, d_out, units, ldq,
                    packed, ldp);
    case 4:
      return launch("pack_codes", pack_codes<4>, grid, dim3(256), 0, s, codes, d_out, units, ldq,
                    packed, ldp);
    default:
      return launch("pack_codes", pack_codes<8>, grid, dim3(256), 0, s, codes, d_out, units, ldq,
                    packed, ldp);
  }
}

// x' (or its digits, which take the same bytes), y', and the digits' weights and sums
size_t online_ws_bytes(int64_t d_out, int64_t d_in, int64_t batch) {
  if (d_out <= 0 || d_in <= 0 || batch <= 0) return 0;
  return align256(size_t(batch) * size_t(d_in) * sizeof(float)) +
         align256(size_t(batch) * size_t(d_out) * sizeof(float)) +
         2 * align256(size_t(batch) * size_t(d_in / 128) * sizeof(float)) + 256;
}

int online_matvec_launch(const uint32_t* packed, int64_t ldp, const float* scales,
                         const float* zeros, int64_t ldsz, int bits, int group, int64_t d_out,
                         int64_t d_in, const float* mul_in, const float* mul_out,
                         const float* q28_in, const float* q28_out, int flags, const void* x,
                         int x_dtype, int64_t ldx, int64_t batch, float* y, int64_t ldy, void* ws,
                         hipStream_t s) {
  Carver cv(ws);
  float* xr = cv.take<float>(size_t(batch) * size_t(d_in));
  float* yr = cv.take<float>(size_t(batch) * size_t(d_out));
  float* gw = cv.take<float>(size_t(batch) * size_t(d_in / 128));
  float* gs = cv.take<float>(size_t(batch) * size_t(d_in / 128));
  const int nb = int(batch);
  const bool rot_in = (flags & KRONQ_ROT_IN) != 0;
  // one vector whose transform the GEMV's workgroups can form themselves (16 values a thread)
  const bool fuse =
      nb == 1 && d_in <= FUSE_MAX_DIN && (!rot_in || (d_in & (d_in - 1)) == 0);
  // x' = V S_X^-1 x, as digits
  if (!fuse)
    KQ_TRY(seg_transform_launch(x, x_dtype, ldx, xr, d_in, batch, d_in, mul_in, nullptr, rot_in,
                                q28_in, false, s, gw, gs, bits));
  // y' = W_hat' x'
  const uint32_t* dig = reinterpret_cast<const uint32_t*>(xr);
#define KQ_GEMV_BITS(BITS_)                                                                      \
  gemv_bits<BITS_>(nb, fuse, packed, ldp, scales, zeros, ldsz, group, d_out, d_in, dig, gw, gs, x, \
                   x_dtype, mul_in, rot_in, yr, s)
  KQ_TRY(bits == 2   ? KQ_GEMV_BITS(2)
         : bits == 3 ? KQ_GEMV_BITS(3)
         : bits == 4 ? KQ_GEMV_BITS(4)
                     : KQ_GEMV_BITS(8));
#undef KQ_GEMV_BITS
  // y = S_G^-1 U^T y'
  return seg_transform_launch(yr, KRONQ_FP32, d_out, y, ldy, batch, d_out, nullptr, mul_out,
                              (flags & KRONQ_ROT_OUT) != 0, q28_out, true, s);
}

}  // namespace kq

// Append-time encoder: transform new keys/values and store the nearest
// codeword index of every group.
//
// Paper: Algorithm 1 (write step, Q+((k - k_bar) R_K)), Theorem 1 (key
// transform), Corollary 1 (s = v R_V), Sec. "Calibration" (each group gets
// the codeword at the smallest squared distance in the transform domain).
// The transform is evaluated in fp64, and the stored index is the argmin of the
// fp64 distances (smallest index among equal distances).
#include <math.h>

#include "encode_block.h"
#include "nova_kv_internal.h"

namespace novakv {

namespace {

// Sink-plus-recent band: a new token's element (bf16 bits) goes to the band
// when its position is there once the append is done (the sequence then ends
// at `end`): a sink slot, or the ring slot of the last n_rec positions.
__device__ __forceinline__ void store_band(const EncodeArgs &a, const int side, const int b, const int kv,
                                           const int pos, const int end, const int d, const uint16_t bits) {
  uint16_t *band = side == 0 ? a.band_k : a.band_v;
  if (!band || !position_in_pool(a.layout, pos)) return;
  if (!(pos < a.n_sink || (a.n_rec > 0 && pos >= end - a.n_rec))) return;
  const int nb = a.n_sink + a.n_rec;
  band[((static_cast<size_t>(b) * a.num_kv_heads + kv) * nb + band_slot(pos, a.n_sink, a.n_rec)) * a.head_dim + d] =
      bits;
}

// The same for elements d .. d + 3 (d a multiple of 4), given as fp32 bits (of
// bf16 values, or fp32 ones, rounded to nearest even).
__device__ __forceinline__ void store_band4(const EncodeArgs &a, const int side, const int b, const int kv,
                                            const int pos, const int end, const int d, const uint4 x) {
  uint16_t *band = side == 0 ? a.band_k : a.band_v;
  if (!band || !position_in_pool(a.layout, pos)) return;
  if (!(pos < a.n_sink || (a.n_rec > 0 && pos >= end - a.n_rec))) return;
  const int nb = a.n_sink + a.n_rec;
  auto bits = [](const uint32_t f) { return (f + 0x7fffu + ((f >> 16) & 1u)) >> 16; };
  *reinterpret_cast<uint2 *>(
      band + ((static_cast<size_t>(b) * a.num_kv_heads + kv) * nb + band_slot(pos, a.n_sink, a.n_rec)) * a.head_dim + d) =
      make_uint2(bits(x.x) | (bits(x.y) << 16), bits(x.z) | (bits(x.w) << 16));
}

// bf16 bits of an input element: as stored, or an fp32 value rounded to
// nearest even.
__device__ __forceinline__ uint16_t input_bf16_bits(const EncodeArgs &a, const void *src, const size_t idx) {
  if (a.in_bf16) return static_cast<const uint16_t *>(src)[idx];
  const uint32_t f = __float_as_uint(static_cast<const float *>(src)[idx]);
  return static_cast<uint16_t>((f + 0x7fffu + ((f >> 16) & 1u)) >> 16);
}

// Cross-lane steps on doubles without LDS traffic (each 32-bit half moves on
// its own).  row_dpp: DPP within 16-lane rows (quad_perm xor 1 = 0xB1, xor 2 =
// 0x4E, row_half_mirror = 0x141, row_mirror = 0x140).  swap_rows: the
// v_permlane{16,32}_swap of x (first operand) and y (second): R = 16
// exchanges the odd rows of x with the even rows of y, R = 32 the high half
// of x with the low half of y; the results are copied out of the returned
// vectors before any reinterpretation.
template <int CTRL>
__device__ __forceinline__ double row_dpp(const double x) {
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(x));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(u), CTRL, 0xf, 0xf, true));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(u >> 32), CTRL, 0xf, 0xf, true));
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}
template <int R>
__device__ __forceinline__ void swap_rows(double &x, double &y) {
  static_assert(R == 16 || R == 32, "row distance");
  const unsigned long long ux = static_cast<unsigned long long>(__double_as_longlong(x));
  const unsigned long long uy = static_cast<unsigned long long>(__double_as_longlong(y));
  const uint32_t xl = static_cast<uint32_t>(ux), xh = static_cast<uint32_t>(ux >> 32);
  const uint32_t yl = static_cast<uint32_t>(uy), yh = static_cast<uint32_t>(uy >> 32);
  uint32_t l0, l1, h0, h1;
  if constexpr (R == 16) {
    const auto sl = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto sh = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    l0 = sl[0], l1 = sl[1], h0 = sh[0], h1 = sh[1];
  } else {
    const auto sl = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
    const auto sh = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
    l0 = sl[0], l1 = sl[1], h0 = sh[0], h1 = sh[1];
  }
  x = __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(h0) << 32) | l0));
  y = __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(h1) << 32) | l1));
}
// Few new tokens (a decode step of a few sequences), plain formats: one workgroup
// per (token, sequence, KV head, side, block of 8 groups).  A block needs 32 transform
// columns (D x 32 fp32) and its 8 codebooks (16 KB), so each workgroup
// fetches a quarter (D=128) or half (D=64) of the parameters, all loads
// coalesced and issued before the first use; the launch costs about one
// memory latency.  The block itself is encode_block.h's team computation.
template <int D, bool FP8, bool TBF>
__global__ void __launch_bounds__(256) encode_small(EncodeArgs a) {
  constexpr int L = D / kGroupDim;
  constexpr int NB = L / encblk::kGroups;  // group blocks per token
  __shared__ encblk::Scratch<D> sc;
  const int blk = blockIdx.x % NB;
  const int side = (blockIdx.x / NB) & 1;
  const int t = blockIdx.x / (2 * NB);
  const int kv = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const void *tm = transform_of(side == 0 ? a.t_k : a.t_v, kv, D, TBF);
  const void *cb = side == 0 ? a.cb_k : a.cb_v;
  const size_t cw0 = static_cast<size_t>(kv) * L * kCodebookSize;
  const void *src = side == 0 ? a.k : a.v;
  uint8_t *pool = side == 0 ? a.k_codes : a.v_codes;
  const int pos = a.start_pos[b] + a.start_offset + t;
  if (!position_in_pool(a.layout, pos)) return;  // uniform: the workgroup stores nothing

  T4 trow[D / 32];
  uint2 cw[encblk::kPer];
  encblk::load_block<D>(tid, tm, TBF, cb, FP8, cw0, blk, trow, cw);
  if (tid < D) {
    const size_t idx = ((static_cast<size_t>(b) * a.n_new + t) * a.num_kv_heads + kv) * D + tid;
    double x = a.in_bf16 ? static_cast<double>(bf16_bits_to_float(static_cast<const uint16_t *>(src)[idx]))
                         : static_cast<double>(static_cast<const float *>(src)[idx]);
    if (side == 0) x -= static_cast<double>(a.kbar[kv * D + tid]);
    sc.xs[tid] = x;
    if (blk == 0 && a.band_k) {
      const int p0 = a.start_pos[b] + a.start_offset;
      store_band(a, side, b, kv, p0 + t, p0 + a.n_new, tid, input_bf16_bits(a, src, idx));
    }
  }
  __syncthreads();
  const size_t off = code_row_offset(a.layout, a.num_kv_heads, L, b, kv, pos);
  encblk::partial_block<D>(tid, sc, trow, TBF);
  __syncthreads();
  const int code = encblk::search_block<D>(tid, sc, cw, FP8);
  if ((tid & 31) == 0) pool[off + encblk::kGroups * blk + (tid >> 5)] = static_cast<uint8_t>(code);
}

// Tiles of tokens: one workgroup (8 waves) per (tile, KV head, side).  The
// tokens of all sequences are taken as one list, token i = b n_new + t, so a
// decode step's tokens share a tile as those of a prompt do.
//
//  * Transform: U^T = T^T (X - k_bar)^T with v_mfma_f64_16x16x4f64.  Wave
//    (ot, th) forms the 16 coefficients 16 ot .. +15, that is the groups
//    4 ot .. 4 ot + 3, of its 16 NTT tokens and keeps them in registers: register
//    k of lane (q, m) is coordinate q of group 4 ot + k, token 16 tt + m.
//    Operand layout (measured): A[m][k] in lane 16k + m, B[k][n] in lane
//    16k + n, D[m][n] in lane 16 (m mod 4) + n, register m / 4.
//  * Search, one group at a time, in three stages whose result is the fp64
//    argmin (smallest index among equal distances):
//    1. scores of all 256 codewords with v_mfma_f32_32x32x16_f16, 32 codewords
//       x 32 tokens in one instruction: the 16 slots of its contraction hold
//       4 coordinates x {hi, lo} of the token (the codeword is fp16 already),
//       |c|^2 as {hi, lo} and a constant per token that makes the score about
//       the squared distance.  A lane keeps the smallest block of 8 codewords
//       and the second smallest block's score: three min3-like instructions
//       for 8 scores and three for the block, under one per score.
//    2. the 8 scores of that block again in fp32, for the index and the
//       runner-up;
//    3. where the runner-up is nearer than the error bound of both (a few
//       tokens of 10^4), the wave searches that token's group in fp64; a group
//       with many such tokens is scored again first (kMany).
//    Group scale: codewords times a power of two, so that the largest
//    coordinate is in [32, 64); the token by a power of two of its own.  The
//    bound: an MFMA of this form errs by at most 2^-23.5 of the sum of its
//    products' magnitudes (measured, fp16 denormals included; 2^-21 allowed),
//    which is at most 8 (|u|^2 + d^2) for any codeword as near as d, and the
//    split operands by less; twice that is 2^-17, the test takes 2^-16.
//
// What bounds it: on this part a SIMD does not run VALU work of one wave while
// it runs matrix instructions of another, so the time is their sum.  Per token
// and group of head_dim 128: 32 cycles of fp64 transform, 8 of scores, 14 for
// the block minima, about 12 for operands, the block's 8 scores and the rest.
// (All scores in fp64 took 64 for the products and 48 for the argmin.)
// 4096 tokens of 32 sequences, 8 KV heads of 128: 4309 us with fp64 scores, 2352
// us like this, 2111 with the inputs loaded all at once (one element and one
// wait at a time before); 2 x 6001 tokens of head_dim 64 in the deployed format:
// 436 us (321 of them a workgroup per token for the scalar arm), 96, now 72 us.
constexpr int kTileWaves = 8;
// More undecided tokens of a group than this (of 64), and at the end it is scored
// once more without its repeated codewords (fp8 rounding of a group of little
// variance, empty clusters, zeros of either sign): scoring takes as long as three
// of the searches in fp64 that it spares.  8 x 2048 tokens, 8 KV heads of 128,
// every codeword twice: 3881 us token by token, 474 so (593 with all scores in
// fp64); keys with a scale 3279 and 540.  Well-spread codebooks: 2.5% slower at
// head_dim 128 for the registers that the end takes, the same at 64.
constexpr int kMany = 16;
constexpr int kSelPart = 8192;  // LDS bytes before the search's staging, for the per-token reductions

template <int D, int NTT>
struct TileShape {
  static constexpr int OT = D / 16;                  // coefficient tiles of 16
  static constexpr int TH = kTileWaves / OT;         // token runs: waves that share a coefficient tile
  static constexpr int TOKENS = 16 * NTT * TH;
  static constexpr int RS = D + 2;                   // LDS row stride of the inputs (doubles)
  static constexpr int BYTES_IN = TOKENS * RS * 8;
  static constexpr int BYTES_SEARCH = kSelPart + kTileWaves * 4096;
  // a quarter's transform (below): its coefficients, one copy per half of the
  // contraction, past the search's staging
  static constexpr int CT = OT / 4, RQ = 16 * CT + 2;
  static constexpr int BYTES_QUARTER = BYTES_SEARCH + 2 * TOKENS * RQ * 8;
  static constexpr int bytes(const bool split) {
    return split ? (BYTES_IN > BYTES_QUARTER ? BYTES_IN : BYTES_QUARTER) : (BYTES_IN > BYTES_SEARCH ? BYTES_IN : BYTES_SEARCH);
  }
};

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t pack_f16(const _Float16 a, const _Float16 b) {
  return __builtin_bit_cast(uint32_t, f16x2{a, b});
}
// x times 2^e, both halves, e in [-28, 29] (two factors: a power of two of fp16's range each)
__device__ __forceinline__ uint32_t scale_f16x2(const uint32_t x, const f16x2 s1, const f16x2 s2) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, x) * s1 * s2);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(const uint32_t x) {
  return max(x, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), CTRL, 0xf, 0xf, true)));
}
// The largest x of the wave, as a scalar.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  x = dpp_max<0xB1>(x);
  x = dpp_max<0x4E>(x);
  x = dpp_max<0x141>(x);
  x = dpp_max<0x140>(x);
  const auto s16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const uint32_t a = s16[0], b = s16[1];
  x = max(a, b);
  const auto s32 = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const uint32_t c = s32[0], d = s32[1];
  return __builtin_amdgcn_readfirstlane(max(c, d));
}
__device__ __forceinline__ double readlane_f64(const double x, const int l) {
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(x));
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), l);
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}
// v[i] of lane row q becomes v[q] of lane row i.
__device__ __forceinline__ void transpose_rows(double (&v)[4]) {
  swap_rows<16>(v[0], v[1]);
  swap_rows<16>(v[2], v[3]);
  swap_rows<32>(v[0], v[2]);
  swap_rows<32>(v[1], v[3]);
}

// Nearest codeword of the group at codeword cw to u (uniform), searched in
// fp64 by the whole wave; the smallest index among equal distances.
template <bool FP8>
__device__ int search_exact(const void *cb, const size_t cw, const int lane, const double (&u)[4]) {
  double best = INFINITY;
  int arg = 4 * lane;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma clang fp contract(off)
    const uint2 w = codeword(cb, FP8, cw + 4 * lane + j);
    const double e0 = u[0] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.x & 0xffff)));
    const double e1 = u[1] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.x >> 16)));
    const double e2 = u[2] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.y & 0xffff)));
    const double e3 = u[3] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.y >> 16)));
    double dist = e0 * e0;
    dist = dist + e1 * e1;
    dist = dist + e2 * e2;
    dist = dist + e3 * e3;
    if (dist < best) {
      best = dist;
      arg = 4 * lane + j;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ob < best || (ob == best && oa < arg)) {
      best = ob;
      arg = oa;
    }
  }
  return arg;
}

// Exponent of a group's largest coordinate (fp16 bits; denormals count as 2^-24 ..).
__device__ __forceinline__ int group_exponent(const uint32_t big) {
  return big == 0u ? 0 : __builtin_amdgcn_frexp_expf(half_bits_to_float(static_cast<uint16_t>(big))) - 1;
}

// Codewords 4 lane .. +3 of a group, as loaded (raw): scaled, with their norms,
// into the wave's staging.  Returns the largest magnitude's fp16 bits.  The
// codewords of `out` (bit j: 4 lane + j) get a norm that keeps them from being
// the nearest or the runner-up of any token.
template <bool FP8>
__device__ __forceinline__ uint32_t stage_group(const uint2 (&raw)[4], uint8_t *stage, const int lane,
                                                const uint32_t out = 0u) {
  uint2 w[4];
  uint32_t big = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    w[j] = codeword_f16(raw[j], FP8);
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 ax = __builtin_bit_cast(u16x2, w[j].x & 0x7fff7fffu), ay = __builtin_bit_cast(u16x2, w[j].y & 0x7fff7fffu);
    big = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, big), __builtin_elementwise_max(ax, ay)));
  }
  big = wave_max_u32(max(big & 0xffffu, big >> 16));
  const int ec = group_exponent(big);
  {
    const int e = 5 - ec, e1 = max(min(e, 14), -14), e2 = e - e1;  // e in [-10, 29]
    const _Float16 f1 = static_cast<_Float16>(ldexpf(1.f, e1)), f2 = static_cast<_Float16>(ldexpf(1.f, e2));
    const f16x2 s1 = {f1, f1}, s2 = {f2, f2};
    asm volatile("" ::: "memory");  // the group before is read; a wave's LDS operations run in order
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint2 c = make_uint2(scale_f16x2(w[j].x, s1, s2), scale_f16x2(w[j].y, s1, s2));
      const f16x2 cx = __builtin_bit_cast(f16x2, c.x), cy = __builtin_bit_cast(f16x2, c.y);
      const float c0 = cx[0], c1 = cx[1], c2 = cy[0], c3 = cy[1];
      float n = fmaf(c3, c3, fmaf(c2, c2, fmaf(c1, c1, c0 * c0)));
      if (out >> j & 1u) n = 60000.f;  // a norm is at most 4 * 64^2, and f at least 2^-14
      asm volatile("" : "+v"(n));  // hi is f16 of the rounded n everywhere (no product fused into the conversion)
      const _Float16 hi = static_cast<_Float16>(n);
      const _Float16 lo = static_cast<_Float16>(n - static_cast<float>(hi));
      reinterpret_cast<uint2 *>(stage)[4 * lane + j] = c;
      reinterpret_cast<uint2 *>(stage + 2048)[4 * lane + j] = make_uint2(pack_f16(hi, lo), 0x00003c00u);
    }
    asm volatile("" ::: "memory");
  }
  return big;
}

// Bit j: codeword 4 lane + j of the group (fp16) repeats one of a smaller index
// (zeros of either sign are the same), which is then never the answer.  Equal codewords meet in a hash table in the
// wave's staging; three tables, so that hardly one is missed (a missed one costs
// time: tokens near it are searched in fp64).
template <bool FP8>
__device__ __forceinline__ uint32_t repeated(const uint2 (&raw)[4], uint8_t *stage, const int lane) {
  const f16x2 zero = {0, 0};
  uint2 w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    w[j] = codeword_f16(raw[j], FP8);  // x + 0 is +0 for x = -0
    w[j] = make_uint2(__builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, w[j].x) + zero),
                      __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, w[j].y) + zero));
  }
  uint2 *all = reinterpret_cast<uint2 *>(stage);
  uint32_t *table = reinterpret_cast<uint32_t *>(stage + 2048);  // [512]: smallest index with this hash
  uint32_t out = 0u;
  asm volatile("" ::: "memory");  // the group before is read; a wave's LDS operations run in order
#pragma unroll
  for (int j = 0; j < 4; ++j) all[4 * lane + j] = w[j];
#pragma unroll 1
  for (int round = 0; round < 3; ++round) {
    const uint32_t mul = round == 0 ? 0x9e3779b1u : (round == 1 ? 0x85ebca77u : 0xc2b2ae3du);
#pragma unroll
    for (int i = 0; i < 8; ++i) table[64 * i + lane] = ~0u;
    asm volatile("" ::: "memory");
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[j] = ((w[j].x ^ (w[j].y * 0x27d4eb2fu)) * mul) >> 23;
      if (!(out >> j & 1u))
        __hip_atomic_fetch_min(table + h[j], static_cast<uint32_t>(4 * lane + j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t first = min(table[h[j]], 255u);
      const uint2 c = all[first];
      if (first < static_cast<uint32_t>(4 * lane + j) && c.x == w[j].x && c.y == w[j].y) out |= 1u << j;
    }
    asm volatile("" ::: "memory");
  }
  return out;
}

// The group at codeword cw staged again, its repeated codewords left out.
template <bool FP8>
__device__ __forceinline__ uint32_t stage_unrepeated(const void *cb, const size_t cw, uint8_t *stage, const int lane) {
  uint2 raw[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) raw[j] = codeword_raw(cb, FP8, cw + 4 * lane + j);
  return stage_group<FP8>(raw, stage, lane, repeated<FP8>(raw, stage, lane));
}

// Stages 1 and 2 of the search of a staged group: the code of each token (one
// per lane; NB 32-token tiles), and whether it has to be searched in fp64 (flag).
// big: stage_group's result; stage, arow: the wave's staging and the lane's
// operand rows in it; u: the token's coefficients, exact up to fp32 rounding,
// or each within err of its value (APPROX).
template <int NB, bool APPROX = false>
__device__ __forceinline__ int score_group(const uint32_t big, const uint8_t *stage, const uint8_t *arow, const int lane,
                                           const float (&u)[4], const float err, bool &flag) {
  const uint32_t half = lane >> 5;
  const int ec = group_exponent(big);
  // token operand: w = -2 u scaled to below 128, as hi and lo; f weighs the
  // norms, o makes the scores about squared distances
  float us[4], ws[4], f, o, a2;
  int eu;
  {
    const float um = fmaxf(fmaxf(fabsf(u[0]), fabsf(u[1])), fmaxf(fabsf(u[2]), fabsf(u[3])));
    eu = max(um > 0.f ? __builtin_amdgcn_frexp_expf(um) - 1 : ec, ec);
    flag = eu - ec > 14 || big >= 0x7c00u;  // f below fp16's normal range, or a codeword that is not finite
    a2 = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      us[i] = ldexpf(u[i], 5 - eu);
      a2 = fmaf(us[i], us[i], a2);
      ws[i] = -2.f * us[i];
    }
    f = ldexpf(1.f, max(ec - eu, -14));
    a2 = ldexpf(a2, min(eu - ec, 64));
    o = static_cast<float>(static_cast<_Float16>(fminf(a2, 16384.f)));
  }
  uint32_t b0[4], b1[4];  // B operands of the token tiles: lanes 0..31 {hi, lo} of w, lanes 32..63 {f, f, o, 0 ..}
  {
    _Float16 hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      hi[i] = static_cast<_Float16>(ws[i]);
      lo[i] = static_cast<_Float16>(ws[i] - static_cast<float>(hi[i]));
    }
    const uint32_t x[4] = {pack_f16(hi[0], hi[1]), pack_f16(hi[2], hi[3]), pack_f16(lo[0], lo[1]), pack_f16(lo[2], lo[3])};
    const _Float16 fh = static_cast<_Float16>(f);
    const uint32_t y[4] = {pack_f16(fh, fh), pack_f16(static_cast<_Float16>(o), static_cast<_Float16>(0.f)), 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto s = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
      b0[i] = s[0];
      b1[i] = s[1];
    }
  }
  const f16x8 bv0 = __builtin_bit_cast(f16x8, make_uint4(b0[0], b0[1], b0[2], b0[3]));
  const f16x8 bv1 = __builtin_bit_cast(f16x8, make_uint4(b1[0], b1[1], b1[2], b1[3]));

  // ---- 1: block minima.  The low 5 bits of a block's minimum hold the block
  // (its first codeword / 8): 4 t + b here, bit 1 (the lane half) below.
  float best[NB], second[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) best[c] = second[c] = INFINITY;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint2 av = *reinterpret_cast<const uint2 *>(arow + 256 * t);
    const f16x8 aop = __builtin_bit_cast(f16x8, make_uint4(av.x, av.y, half ? 0u : av.x, half ? 0u : av.y));
    const float16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float16_t d[NB];
    d[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, bv0, zero, 0, 0, 0);
    if constexpr (NB == 2) d[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, bv1, zero, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float *v = reinterpret_cast<const float *>(&d[c]) + 8 * b;
        float mn = fminf(fminf(v[0], v[1]), v[2]);
        mn = fminf(fminf(mn, v[3]), v[4]);
        mn = fminf(fminf(mn, v[5]), v[6]);
        mn = fminf(mn, v[7]);
        const float key = __uint_as_float((__float_as_uint(mn) & 0xffffffe0u) | static_cast<uint32_t>(4 * t + b));
        second[c] = __builtin_amdgcn_fmed3f(best[c], second[c], key);
        best[c] = fminf(best[c], key);
      }
  }
  // both lane halves of each tile; lane = token
  float kb, sb;
  {
#pragma unroll
    for (int c = 0; c < NB; ++c) best[c] = __uint_as_float(__float_as_uint(best[c]) | (half << 1));
    const float bl = best[0], bh = NB == 2 ? best[NB - 1] : best[0];
    const float sl = second[0], sh = NB == 2 ? second[NB - 1] : second[0];
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bl), __float_as_uint(bh), false, false);
    const auto s2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(sl), __float_as_uint(sh), false, false);
    const uint32_t x0 = sw[0], x1 = sw[1], y0 = s2[0], y1 = s2[1];
    const float p0 = __uint_as_float(x0), p1 = __uint_as_float(x1);
    kb = fminf(p0, p1);
    sb = fminf(fminf(fmaxf(p0, p1), __uint_as_float(y0)), __uint_as_float(y1));
  }
  const uint32_t blk = __float_as_uint(kb) & 31u;

  // ---- 2: the block's 8 scores in fp32
  float v1 = INFINITY, v2 = INFINITY;
  {
    const uint8_t *cp = stage + 64 * blk, *np = stage + 2048 + 64 * blk;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint4 c = reinterpret_cast<const uint4 *>(cp)[p], n = reinterpret_cast<const uint4 *>(np)[p];
      const uint32_t cw[2][2] = {{c.x, c.y}, {c.z, c.w}}, nn[2] = {n.x, n.z};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const f16x2 cx = __builtin_bit_cast(f16x2, cw[e][0]), cy = __builtin_bit_cast(f16x2, cw[e][1]);
        const f16x2 nx = __builtin_bit_cast(f16x2, nn[e]);
        float sc = fmaf(static_cast<float>(nx[0]), f, o);
        sc = fmaf(static_cast<float>(nx[1]), f, sc);
        sc = fmaf(static_cast<float>(cx[0]), ws[0], sc);
        sc = fmaf(static_cast<float>(cx[1]), ws[1], sc);
        sc = fmaf(static_cast<float>(cy[0]), ws[2], sc);
        sc = fmaf(static_cast<float>(cy[1]), ws[3], sc);
        const float key = __uint_as_float((__float_as_uint(sc) & 0xfffffff8u) | static_cast<uint32_t>(2 * p + e));
        v2 = __builtin_amdgcn_fmed3f(v1, v2, key);
        v1 = fminf(v1, key);
      }
    }
  }
  const float next = fminf(sb, v2), gap = next - v1;
  // (the terms of a score add up to at most 2^16, however large the token)
  float bound = 0x1p-16f * (fminf(2.f * a2, 65536.f) + fabsf(v1)) + 0x1p-14f;
  if constexpr (APPROX) {
    // two scores differ by 2 (c1 - c2) . u: an error of E in each coordinate
    // moves their gap by at most 4 E |c1 - c2|, where |c1 - c2| <= |u - c1| +
    // |u - c2| + 4 E, the distances about the runner-up's where the gap is
    // small, and <= 2 * 128 of the scaled codewords
    const float es = err * __builtin_amdgcn_exp2f(0.5f * static_cast<float>(10 - ec - eu));
    bound += 8.f * es * (__builtin_amdgcn_sqrtf(fminf(fmaxf(next + (a2 - o), 0.f), 16384.f * f)) + 2.f * es);
  }
  flag = flag || !(gap > bound);
  return static_cast<int>(8 * blk + (__float_as_uint(v1) & 7u));
}

// The inputs of a tile: NK vectors of four elements (index(k): the first one's
// index), as fp32 bits.  Every load is issued before the first is used: 8- or
// 16-byte loads where the inputs' address allows them, single elements
// otherwise.
template <int NK, class Index>
__device__ __forceinline__ void load_inputs(const int in_bf16, const int in_vec, const void *src, uint4 (&x)[NK], Index index) {
  if (in_bf16) {
    const uint16_t *p = static_cast<const uint16_t *>(src);
    uint2 h[NK];
    if (in_vec) {
#pragma unroll
      for (int k = 0; k < NK; ++k) h[k] = *reinterpret_cast<const uint2 *>(p + index(k));
    } else {
      uint16_t e[NK][4];
#pragma unroll
      for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) e[k][i] = p[index(k) + i];
#pragma unroll
      for (int k = 0; k < NK; ++k)
        h[k] = make_uint2(e[k][0] | (static_cast<uint32_t>(e[k][1]) << 16), e[k][2] | (static_cast<uint32_t>(e[k][3]) << 16));
    }
#pragma unroll
    for (int k = 0; k < NK; ++k)
      x[k] = make_uint4(h[k].x << 16, h[k].x & 0xffff0000u, h[k].y << 16, h[k].y & 0xffff0000u);
  } else if (in_vec) {
#pragma unroll
    for (int k = 0; k < NK; ++k) x[k] = *reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(src) + index(k));
  } else {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const uint32_t *p = static_cast<const uint32_t *>(src) + index(k);
      x[k] = make_uint4(p[0], p[1], p[2], p[3]);
    }
  }
}

// NTT: 16-token tiles per wave (2 or 4).  SPLIT: a workgroup searches a quarter
// of the groups (blockIdx.z >> 1 says which), one per wave, for launches whose
// tiles alone leave the chip idle.  It forms only the quarter's coefficients:
// four 16 x 16 tiles, the contraction in two halves, one per wave, added in LDS.
// A scaled key needs them all: there every workgroup runs the whole transform
// and wave ot searches group 4 ot + quarter.
template <int D, bool FP8, bool TBF, int NTT, bool SPLIT>
__global__ void __launch_bounds__(64 * kTileWaves) encode_tile(EncodeArgs a, const int first_side) {
  using T_ = TileShape<D, NTT>;
  constexpr int L = D / kGroupDim, NT = 64 * kTileWaves, TOK = T_::TOKENS, RS = T_::RS, KS = D / 4;
  constexpr int BYTES = T_::bytes(SPLIT);
  __shared__ __attribute__((aligned(16))) uint8_t smem[BYTES];
  double *xs = reinterpret_cast<double *>(smem);

  const int kv = blockIdx.y, side = first_side + (blockIdx.z & 1);
  const int only = SPLIT ? static_cast<int>(blockIdx.z >> 1) : 0;
  const bool scalar_arm = side == 1 && a.v_sq;
  if (SPLIT && scalar_arm && only != 0) return;  // its levels need every coefficient: one workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tok = a.batch * a.n_new;
  const int n0 = blockIdx.x * TOK;
  const void *tm = transform_of(side == 0 ? a.t_k : a.t_v, kv, D, TBF);
  const void *cb = side == 0 ? a.cb_k : a.cb_v;
  const size_t cw0 = static_cast<size_t>(kv) * L * kCodebookSize;
  const void *src = side == 0 ? a.k : a.v;
  uint8_t *pool = side == 0 ? a.k_codes : a.v_codes;

  // ---- transform operands first, so that their latency passes while the
  // inputs are staged: rows 4 ks + q, column 16 ot + m of T
  const int m = lane & 15, q = lane >> 4;
  const int ot = wave % T_::OT, th = wave / T_::OT;
  const bool quarter = SPLIT && !scalar_arm && !(side == 0 && a.k_scales);
  // a quarter's transform: wave = (half of the contraction, token tile, coefficient tile)
  const int qc = wave % T_::CT, qt = (wave & 3) / T_::CT, qh = wave >> 2;
  uint32_t tr[KS];  // as loaded (fp32 words, or zero-extended bf16)
  if (quarter) {
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
      tr[ks] = load_t1_raw(tm, (4 * (ks + KS / 2 * qh) + q) * D + 16 * (T_::CT * only + qc) + m, TBF);
  } else {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) tr[ks] = load_t1_raw(tm, (4 * ks + q) * D + 16 * ot + m, TBF);
  }

  // the token that this lane stores: its position is requested here, its cache
  // block after the barrier, so that neither is waited for where it is used
  const int tok = 16 * NTT * th + lane;  // of the tile
  bool stored = lane < 16 * NTT && n0 + tok < n_tok;
  const int tok_b = stored ? (n0 + tok) / a.n_new : 0, tok_t = n0 + tok - tok_b * a.n_new;
  const int tok_p0 = a.start_pos[tok_b];

  // inputs (minus k_bar for keys) to LDS in fp64: thread tid stages four
  // coordinates of tokens tid / (D / 4) + k * TP
  {
    constexpr int C4 = D / 4, TP = NT / C4, NK = TOK / TP;
    static_assert(NT % C4 == 0 && TOK % TP == 0, "a thread stages four coordinates of NK tokens");
    const int d = 4 * (tid % C4), s0 = tid / C4;
    const float4 kb = side == 0 ? *reinterpret_cast<const float4 *>(a.kbar + kv * D + d) : make_float4(0.f, 0.f, 0.f, 0.f);
    uint4 x[NK];  // fp32 bits
    load_inputs<NK>(a.in_bf16, a.in_vec, src, x, [&](const int k) {  // past the last token the last one is read again
      return (static_cast<size_t>(min(n0 + s0 + k * TP, n_tok - 1)) * a.num_kv_heads + kv) * D + d;
    });
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      double *row = xs + (s0 + k * TP) * RS + d;
      const bool in = n0 + s0 + k * TP < n_tok;
      const double2 lo = {static_cast<double>(__uint_as_float(x[k].x)) - static_cast<double>(kb.x),
                          static_cast<double>(__uint_as_float(x[k].y)) - static_cast<double>(kb.y)};
      const double2 hi = {static_cast<double>(__uint_as_float(x[k].z)) - static_cast<double>(kb.z),
                          static_cast<double>(__uint_as_float(x[k].w)) - static_cast<double>(kb.w)};
      *reinterpret_cast<double2 *>(row) = in ? lo : double2{0.0, 0.0};
      *reinterpret_cast<double2 *>(row + 2) = in ? hi : double2{0.0, 0.0};
    }
    if (a.band_k && (!SPLIT || only == 0)) {
      for (int k = 0; k < NK; ++k) {
        const int i = n0 + s0 + k * TP;
        if (i < n_tok) {
          const int b = i / a.n_new, t = i - b * a.n_new;
          const int p0 = a.start_pos[b] + a.start_offset;
          store_band4(a, side, b, kv, p0 + t, p0 + a.n_new, d, x[k]);
        }
      }
    }
  }
  __syncthreads();
  // the stored token's cache block, requested before the transform
  const int tok_pos = tok_p0 + a.start_offset + tok_t;
  stored = stored && position_in_pool(a.layout, tok_pos);
  const int tok_blk = stored ? tok_pos / a.layout.block_size : 0;
  int tok_phys = tok_b * a.layout.blocks_per_seq + tok_blk;
  if (a.layout.block_table) tok_phys = a.layout.block_table[tok_phys];

  double4_t acc[NTT];
#pragma unroll
  for (int j = 0; j < NTT; ++j) acc[j] = double4_t{0.0, 0.0, 0.0, 0.0};
  if (quarter) {
    const double *xr = xs + (16 * qt + m) * RS + q + 4 * (KS / 2) * qh;
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(t1_raw_value(tr[ks], TBF)), xr[4 * ks], acc[0], 0, 0, 0);
  } else {
    const double *xr = xs + (16 * NTT * th + m) * RS + q;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const double at = static_cast<double>(t1_raw_value(tr[ks], TBF));
#pragma unroll
      for (int j = 0; j < NTT; ++j)
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(at, xr[16 * j * RS + 4 * ks], acc[j], 0, 0, 0);
    }
  }
  __syncthreads();  // every wave has read its inputs; the region is free
  double *quad = reinterpret_cast<double *>(smem + T_::BYTES_SEARCH);  // [2][TOK][RQ]
  if (quarter) {
#pragma unroll
    for (int k = 0; k < 4; ++k) quad[(qh * TOK + 16 * qt + m) * T_::RQ + 16 * qc + 4 * k + q] = acc[0][k];
    __syncthreads();
  }
  // the stored token's code row
  const size_t off = ((static_cast<size_t>(tok_phys) * a.num_kv_heads + kv) * a.layout.block_size +
                      (tok_pos - tok_blk * a.layout.block_size)) * L;

  if (scalar_arm) {
    // Scalar value arm (paper: Sec. "Bit rate" and the implementation table):
    // offset = bf16(min), scale = bf16((max - min) / 3) over the token's
    // coefficients, level = clamp(round_half_even((s - offset) / scale), 0, 3)
    // with the stored values; coordinate 4g + j in bits 2j, 2j + 1 of byte g.
    double *red = reinterpret_cast<double *>(smem);  // [2][OT][TOK]: the coefficient tiles' min and max
#pragma unroll
    for (int j = 0; j < NTT; ++j) {
      double mn = fmin(fmin(acc[j][0], acc[j][1]), fmin(acc[j][2], acc[j][3]));
      double mx = fmax(fmax(acc[j][0], acc[j][1]), fmax(acc[j][2], acc[j][3]));
      double y = mn;
      swap_rows<16>(mn, y);
      mn = y = fmin(mn, y);
      swap_rows<32>(mn, y);
      mn = fmin(mn, y);
      y = mx;
      swap_rows<16>(mx, y);
      mx = y = fmax(mx, y);
      swap_rows<32>(mx, y);
      mx = fmax(mx, y);
      if (q == 0) {
        red[ot * TOK + 16 * NTT * th + 16 * j + m] = mn;
        red[(T_::OT + ot) * TOK + 16 * NTT * th + 16 * j + m] = mx;
      }
    }
    static_assert(2 * T_::OT * TOK * 8 <= BYTES, "the reductions fit");
    __syncthreads();
    uint32_t mine = 0u;  // the four code bytes of token `lane`
#pragma unroll
    for (int j = 0; j < NTT; ++j) {
      const int t = 16 * NTT * th + 16 * j + m;
      double mn = red[t], mx = red[T_::OT * TOK + t];
#pragma unroll
      for (int o = 1; o < T_::OT; ++o) {
        mn = fmin(mn, red[o * TOK + t]);
        mx = fmax(mx, red[(T_::OT + o) * TOK + t]);
      }
      const uint16_t zb = encblk::bf16_of(mn), sb = encblk::bf16_of((mx - mn) / 3.0);
      const double zero = bf16_bits_to_float(zb), scale = bf16_bits_to_float(sb);
      uint32_t w = 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t lev =
            scale > 0.0 ? static_cast<uint32_t>(fmin(fmax(rint((acc[j][k] - zero) / scale), 0.0), 3.0)) : 0u;
        w |= lev << (8 * k + 2 * q);
      }
      const auto s16 = __builtin_amdgcn_permlane16_swap(w, w, false, false);
      const uint32_t w0 = s16[0], w1 = s16[1];
      w = w0 | w1;
      const auto s32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
      const uint32_t w2 = s32[0], w3 = s32[1];
      w = w2 | w3;
      if (q == j) {
        mine = w;
        if (stored && ot == 0) {
          a.v_sq[(off / L) * 2] = sb;
          a.v_sq[(off / L) * 2 + 1] = zb;
        }
      }
    }
    if (stored) *reinterpret_cast<uint32_t *>(pool + off + 4 * ot) = mine;
    return;
  }

  if (side == 0 && a.k_scales) {
    // Key-scale format: rho of each key from its D coefficients (each square
    // rounded before it is added), stored as bf16; the coefficients are
    // divided by it (0 when rho = 0).
    double *part = reinterpret_cast<double *>(smem);  // [OT][TOK]
    static_assert(T_::OT * TOK * 8 <= kSelPart, "the partial sums fit before the search's staging");
#pragma unroll
    for (int j = 0; j < NTT; ++j) {
      double s;
      {
#pragma clang fp contract(off)
        s = acc[j][0] * acc[j][0];
        s = s + acc[j][1] * acc[j][1];
        s = s + acc[j][2] * acc[j][2];
        s = s + acc[j][3] * acc[j][3];
      }
      double y = s;
      swap_rows<16>(s, y);
      s = y = s + y;
      swap_rows<32>(s, y);
      s = s + y;
      if (q == 0) part[ot * TOK + 16 * NTT * th + 16 * j + m] = s;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NTT; ++j) {
      const int t = 16 * NTT * th + 16 * j + m;
      double s = 0.0;
#pragma unroll
      for (int o = 0; o < T_::OT; ++o) s += part[o * TOK + t];
      const double rho = sqrt(s) / sqrt(static_cast<double>(D));
      if (q == j && ot == 0 && stored && (!SPLIT || only == 0)) a.k_scales[off / L] = encblk::bf16_of(rho);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[j][k] = rho > 0.0 ? acc[j][k] / rho : 0.0;
    }
  }

  // ---- nearest codewords of the wave's groups
  // staging of a group: codewords (8 bytes, scaled) and {hi, lo, 1, 0} of their
  // squared norms, 2 KB each; written and read by this wave alone
  uint8_t *stage = smem + kSelPart + wave * 4096;
  const uint32_t half = lane >> 5;
  const int r = lane & 31;
  // the codeword in row r of an MFMA: register i of lane half h is row
  // 8 (i / 4) + 4 h + i mod 4, given to codeword 16 h + i of the tile, so that
  // registers 8 b .. 8 b + 7 are 8 consecutive codewords
  const int row_cw = 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
  const uint8_t *arow = stage + 2048 * half + 8 * row_cw;
  uint2 rn[4];  // codewords 4 lane .. 4 lane + 3 of the next group, as loaded
  const int g0 = !SPLIT ? 4 * ot : (quarter ? T_::OT * only + ot : 4 * ot + only);  // the wave's first group
  auto group_cw = [&](const int k) { return cw0 + static_cast<size_t>(g0 + k) * kCodebookSize; };
#pragma unroll
  for (int j = 0; j < 4; ++j) rn[j] = codeword_raw(cb, FP8, group_cw(0) + 4 * lane + j);
  // coefficients of the wave's group k, lane = token
  auto coefficients = [&](const int k, double (&u)[4]) {
    u[0] = u[1] = u[2] = u[3] = 0.0;
    if (quarter) {
      if (lane < 16 * NTT) {
        const double *ur = quad + tok * T_::RQ + 4 * ot;
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = ur[i] + ur[TOK * T_::RQ + i];
      }
    } else {
      const int c = SPLIT ? only : k;
#pragma unroll
      for (int j = 0; j < NTT; ++j) u[j] = c == 0 ? acc[j][0] : (c == 1 ? acc[j][1] : (c == 2 ? acc[j][2] : acc[j][3]));
      transpose_rows(u);  // u[i]: coordinate i of token `lane`
    }
  };
  // the undecided tokens (todo) of group k, in fp64
  auto decide = [&](unsigned long long todo, const int k, const double (&u)[4], int &code) {
    for (; todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const double uu[4] = {readlane_f64(u[0], l), readlane_f64(u[1], l), readlane_f64(u[2], l), readlane_f64(u[3], l)};
      const int c = search_exact<FP8>(cb, group_cw(k), lane, uu);
      if (lane == l) code = c;
    }
  };
  uint32_t code_acc = 0u, again = 0u;  // again: bit k, group k has many undecided tokens
#pragma unroll
  for (int k = 0; k < (SPLIT ? 1 : 4); ++k) {
    double u[4];
    coefficients(k, u);
    const uint2 cur[4] = {rn[0], rn[1], rn[2], rn[3]};
    if (k + 1 < (SPLIT ? 1 : 4)) {
#pragma unroll
      for (int j = 0; j < 4; ++j) rn[j] = codeword_raw(cb, FP8, group_cw(k + 1) + 4 * lane + j);
    }
    float us[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) us[i] = static_cast<float>(u[i]);
    bool flag;
    int code = score_group<NTT == 4 ? 2 : 1>(stage_group<FP8>(cur, stage, lane), stage, arow, lane, us, 0.f, flag);
    const unsigned long long todo = __ballot(flag && lane < 16 * NTT);
    if (__popcll(todo) > kMany)
      again |= 1u << k;
    else
      decide(todo, k, u, code);
    code_acc = SPLIT ? static_cast<uint32_t>(code) : (code_acc >> 8) | (static_cast<uint32_t>(code) << 24);
  }
  if (stored) {
    if constexpr (SPLIT)
      pool[off + g0] = static_cast<uint8_t>(code_acc);
    else
      *reinterpret_cast<uint32_t *>(pool + off + g0) = code_acc;
  }
#pragma unroll 1
  for (; again; again &= again - 1) {
    const int k = __builtin_ctz(again);
    double u[4];
    float us[4];
    coefficients(k, u);
#pragma unroll
    for (int i = 0; i < 4; ++i) us[i] = static_cast<float>(u[i]);
    bool flag;
    int code = score_group<NTT == 4 ? 2 : 1>(stage_unrepeated<FP8>(cb, group_cw(k), stage, lane), stage, arow, lane, us, 0.f, flag);
    decide(__ballot(flag && lane < 16 * NTT), k, u, code);
    if (stored) pool[off + g0 + k] = static_cast<uint8_t>(code);
  }
}

// The odd lane rows of x against the even ones of y, the high half of x against
// the low one of y.
__device__ __forceinline__ void swap16_f32(float &x, float &y) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const uint32_t a = s[0], b = s[1];
  x = __uint_as_float(a);
  y = __uint_as_float(b);
}
__device__ __forceinline__ void swap32_f32(float &x, float &y) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const uint32_t a = s[0], b = s[1];
  x = __uint_as_float(a);
  y = __uint_as_float(b);
}
__device__ __forceinline__ double wave_sum_f64(double x) {
  x += row_dpp<0xB1>(x);
  x += row_dpp<0x4E>(x);
  x += row_dpp<0x141>(x);
  x += row_dpp<0x140>(x);
  double y = x;
  swap_rows<16>(x, y);
  x += y;
  y = x;
  swap_rows<32>(x, y);
  return x + y;
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(const float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}

// The tiled encoder of a plain side (no key scale, no scalar arm), for launches
// that fill the chip: encode_tile's search on coefficients from the fp16 matrix
// cores.
//  * Transform: each token (minus k_bar, fp32) and the wave's 16 columns of T are
//    scaled by powers of two and split into hi = f16(x), lo = f16(x - hi); the
//    small products lo hi + hi lo are summed first, then hi hi, by
//    v_mfma_f32_16x16x32_f16.  Each coefficient is then within
//    E = 2^-18.5 |x| |T_j| of its value: an MFMA errs by at most 2^-21 of its
//    terms and its accumulator (2^-23.5 measured), four of them with sums up to
//    |x| |T_j|, 2^-19 together; the splits and the dropped lo lo add 2^-21.
//  * Search: as in encode_tile, the test of the runner-up widened by what E can
//    move a gap (score_group); a token that fails it has its group's four
//    coefficients formed and searched in fp64 (one of 10^3 token-groups), so
//    the codes are those of the fp64 transform.
// The fp64 transform took 32 of about 70 cycles per token and group on a SIMD,
// this one takes 3.
// A workgroup does NS tiles: T's split (25 of about 725 vector instructions per
// token and group and lane in single tiles) and the staging of a group's
// codewords (55) serve all of them.  One tile's coefficients are formed after
// the other's in the same LDS, and scored one after the other, so that two
// workgroups still share a CU (128 VGPRs, 50 KiB of LDS; pairs spill 39 registers,
// single tiles 6).  32 x 4096 tokens, 8 KV heads of 128: 2111 us with the fp64
// transform; single tiles and pairs side by side 1509 and 1476, with the groups
// that are scored again (kMany) 2.5% more.
template <int D, bool FP8, bool TBF, int NS>
__global__ void __launch_bounds__(64 * kTileWaves, 4) encode_fast(EncodeArgs a, const int first_side) {
  using T_ = TileShape<D, 4>;
  constexpr int L = D / kGroupDim, NT = 64 * kTileWaves, NTT = 4, TOK = T_::TOKENS;
  constexpr int RH = D + 8;                         // LDS row stride of the split inputs (halves)
  constexpr uint32_t kLo = TOK * RH * 2, kPlanes = 2 * kLo;
  constexpr uint32_t kTok = kPlanes > T_::BYTES_SEARCH ? kPlanes : T_::BYTES_SEARCH;  // per token: exponent, norm
  constexpr int KS = D / 32;                        // contraction steps of 32
  __shared__ __attribute__((aligned(16))) uint8_t smem[kTok + TOK * 8 + NS * NT * 8];
  const int kv = blockIdx.y, side = first_side + blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tok = a.batch * a.n_new;
  const int first = blockIdx.x * TOK * NS;
  const void *tm = transform_of(side == 0 ? a.t_k : a.t_v, kv, D, TBF);
  const void *cb = side == 0 ? a.cb_k : a.cb_v;
  const size_t cw0 = static_cast<size_t>(kv) * L * kCodebookSize;
  const void *src = side == 0 ? a.k : a.v;
  uint8_t *pool = side == 0 ? a.k_codes : a.v_codes;
  const int m = lane & 15, q = lane >> 4;
  const int ot = wave % T_::OT, th = wave / T_::OT;

  // ---- columns of T: rows 32 ks + 8 q + e, column 16 ot + m
  uint32_t tr[KS][8];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) tr[ks][e] = load_t1_raw(tm, (32 * ks + 8 * q + e) * D + 16 * ot + m, TBF);

  // ---- inputs: thread tid takes four coordinates of tokens tid / (D / 4) + k TP
  constexpr int C4 = D / 4, TP = NT / C4, NK = TOK / TP;
  const int d4 = 4 * (tid % C4), s0 = tid / C4;
  const float4 kb = side == 0 ? *reinterpret_cast<const float4 *>(a.kbar + kv * D + d4) : make_float4(0.f, 0.f, 0.f, 0.f);
  // the tokens that this lane stores (as in encode_tile)
  const int tok = 16 * NTT * th + lane;
  float uf[NS][4][4];  // [s][k][i]: coordinate i of group 4 ot + k, token `tok` of tile s
  float err[NS];
  // code rows of the lane's tokens (kNoRow: not stored), in LDS until the end
  constexpr size_t kNoRow = ~static_cast<size_t>(0);
  size_t *rows = reinterpret_cast<size_t *>(smem + kTok + TOK * 8) + wave * 64 * NS + lane;

  f16x8 thi[KS], tlo[KS];  // T split, with the wave's scale and its largest column norm
  float tnorm = 0.f;
  int et = 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int n0 = first + s * TOK;
    uint4 x[NK];  // fp32 bits
    load_inputs<NK>(a.in_bf16, a.in_vec, src, x, [&](const int k) {
      return (static_cast<size_t>(min(n0 + s0 + k * TP, n_tok - 1)) * a.num_kv_heads + kv) * D + d4;
    });
    bool stored = n0 + tok < n_tok;
    const int tok_b = stored ? (n0 + tok) / a.n_new : 0, tok_t = n0 + tok - tok_b * a.n_new;
    const int tok_p0 = a.start_pos[tok_b];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int t = s0 + k * TP;
      float v[4] = {__uint_as_float(x[k].x) - kb.x, __uint_as_float(x[k].y) - kb.y, __uint_as_float(x[k].z) - kb.z,
                    __uint_as_float(x[k].w) - kb.w};
      if (n0 + t >= n_tok) v[0] = v[1] = v[2] = v[3] = 0.f;
      // the token's largest element and its norm, over the C4 lanes that hold it
      float big = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
      big = fmaxf(big, dpp_f32<0xB1>(big));
      big = fmaxf(big, dpp_f32<0x4E>(big));
      big = fmaxf(big, dpp_f32<0x141>(big));
      big = fmaxf(big, dpp_f32<0x140>(big));
      if constexpr (C4 == 32) {
        float y = big;
        swap16_f32(big, y);
        big = fmaxf(big, y);
      }
      const int ex = big > 0.f ? __builtin_amdgcn_frexp_expf(big) : 0;
      float n2 = 0.f;
      _Float16 hi[4], lo[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float y = ldexpf(v[i], 5 - ex);
        n2 = fmaf(y, y, n2);
        hi[i] = static_cast<_Float16>(y);
        lo[i] = static_cast<_Float16>(y - static_cast<float>(hi[i]));
      }
      n2 += dpp_f32<0xB1>(n2);
      n2 += dpp_f32<0x4E>(n2);
      n2 += dpp_f32<0x141>(n2);
      n2 += dpp_f32<0x140>(n2);
      if constexpr (C4 == 32) {
        float y = n2;
        swap16_f32(n2, y);
        n2 += y;
      }
      uint8_t *row = smem + 2 * (t * RH + d4);
      *reinterpret_cast<uint2 *>(row) = make_uint2(pack_f16(hi[0], hi[1]), pack_f16(hi[2], hi[3]));
      *reinterpret_cast<uint2 *>(row + kLo) = make_uint2(pack_f16(lo[0], lo[1]), pack_f16(lo[2], lo[3]));
      if (d4 == 0)
        *reinterpret_cast<uint2 *>(smem + kTok + 8 * t) =
            make_uint2(static_cast<uint32_t>(ex), __float_as_uint(ldexpf(__builtin_amdgcn_sqrtf(n2), ex - 5)));
      if (a.band_k && n0 + t < n_tok) {
        const int b = (n0 + t) / a.n_new, p0 = a.start_pos[b] + a.start_offset;
        store_band4(a, side, b, kv, p0 + n0 + t - b * a.n_new, p0 + a.n_new, d4, x[k]);
      }
    }
    if (s == 0) {
      float big = 0.f, n2 = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) big = fmaxf(big, fabsf(t1_raw_value(tr[ks][e], TBF)));
      big = __uint_as_float(wave_max_u32(__float_as_uint(big)));
      et = big > 0.f ? __builtin_amdgcn_frexp_expf(big) : 0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float y = ldexpf(t1_raw_value(tr[ks][e], TBF), 5 - et);
          n2 = fmaf(y, y, n2);
          const _Float16 hi = static_cast<_Float16>(y);
          thi[ks][e] = hi;
          tlo[ks][e] = static_cast<_Float16>(y - static_cast<float>(hi));
        }
      float y = n2;  // over the lane rows, then the largest column
      swap16_f32(n2, y);
      n2 = y = n2 + y;
      swap32_f32(n2, y);
      n2 += y;
      tnorm = ldexpf(__builtin_amdgcn_sqrtf(__uint_as_float(wave_max_u32(__float_as_uint(n2)))), et - 5);
    }
    __syncthreads();
    const int tok_pos = tok_p0 + a.start_offset + tok_t;
    stored = stored && position_in_pool(a.layout, tok_pos);
    const int tok_blk = stored ? tok_pos / a.layout.block_size : 0;
    int tok_phys = tok_b * a.layout.blocks_per_seq + tok_blk;
    if (a.layout.block_table) tok_phys = a.layout.block_table[tok_phys];

#pragma unroll
    for (int j = 0; j < NTT; ++j) {
      typedef float float4_t __attribute__((ext_vector_type(4)));
      f16x8 xh[KS], xl[KS];
      const uint8_t *row = smem + 2 * ((16 * NTT * th + 16 * j + m) * RH + 8 * q);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        xh[ks] = *reinterpret_cast<const f16x8 *>(row + 64 * ks);
        xl[ks] = *reinterpret_cast<const f16x8 *>(row + kLo + 64 * ks);
      }
      float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) d = __builtin_amdgcn_mfma_f32_16x16x32_f16(tlo[ks], xh[ks], d, 0, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) d = __builtin_amdgcn_mfma_f32_16x16x32_f16(thi[ks], xl[ks], d, 0, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) d = __builtin_amdgcn_mfma_f32_16x16x32_f16(thi[ks], xh[ks], d, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) uf[s][j][i] = d[i];  // lane (q, m): coordinate i of group q, token 16 j + m
    }
    const uint2 tinfo = *reinterpret_cast<const uint2 *>(smem + kTok + 8 * tok);
    const int eu = static_cast<int>(tinfo.x) + et - 10;
    err[s] = 0x1.6a09e6p-19f * __uint_as_float(tinfo.y) * tnorm;  // 2^-18.5 |x| |T_j|
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      swap16_f32(uf[s][0][i], uf[s][1][i]);
      swap16_f32(uf[s][2][i], uf[s][3][i]);
      swap32_f32(uf[s][0][i], uf[s][2][i]);
      swap32_f32(uf[s][1][i], uf[s][3][i]);
#pragma unroll
      for (int k = 0; k < 4; ++k) uf[s][k][i] = ldexpf(uf[s][k][i], eu);
    }
    __syncthreads();  // every wave has read the inputs; the region is the next tile's or the search's
    rows[64 * s] = stored ? ((static_cast<size_t>(tok_phys) * a.num_kv_heads + kv) * a.layout.block_size +
                             (tok_pos - tok_blk * a.layout.block_size)) * L
                          : kNoRow;
  }

  uint8_t *stage = smem + kSelPart + wave * 4096;
  const int r = lane & 31;
  const uint8_t *arow = stage + 2048 * (lane >> 5) + 8 * (16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3));
  const int g0 = 4 * ot;
  uint2 rn[4];
  auto group_cw = [&](const int k) { return cw0 + static_cast<size_t>(g0 + k) * kCodebookSize; };
#pragma unroll
  for (int j = 0; j < 4; ++j) rn[j] = codeword_raw(cb, FP8, group_cw(0) + 4 * lane + j);
  // the undecided tokens (todo) of group k, tile s, in fp64: a token's four
  // coefficients, a lane adds D / 64 rows, then the search
  auto decide = [&](unsigned long long todo, const int k, const int n0, int &code) {
    for (; todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const size_t idx = (static_cast<size_t>(n0 + 16 * NTT * th + l) * a.num_kv_heads + kv) * D;
      double uu[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < D / 64; ++i) {
        const int row = lane + 64 * i;
        double x = a.in_bf16 ? static_cast<double>(bf16_bits_to_float(static_cast<const uint16_t *>(src)[idx + row]))
                             : static_cast<double>(static_cast<const float *>(src)[idx + row]);
        if (side == 0) x -= static_cast<double>(a.kbar[kv * D + row]);
        const float4 t = t4_value(load_t4(tm, static_cast<size_t>(row) * D + 4 * (g0 + k), TBF), TBF);
        uu[0] = fma(x, static_cast<double>(t.x), uu[0]);
        uu[1] = fma(x, static_cast<double>(t.y), uu[1]);
        uu[2] = fma(x, static_cast<double>(t.z), uu[2]);
        uu[3] = fma(x, static_cast<double>(t.w), uu[3]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) uu[i] = wave_sum_f64(uu[i]);
      const int c = search_exact<FP8>(cb, group_cw(k), lane, uu);
      if (lane == l) code = c;
    }
  };
  uint32_t code_acc[NS] = {}, again = 0u;  // again: bit 4 s + k, group k of tile s has many undecided tokens
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint2 cur[4] = {rn[0], rn[1], rn[2], rn[3]};
    const uint32_t big = stage_group<FP8>(cur, stage, lane);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int n0 = first + s * TOK;
      if (k < 3 && s == NS - 1) {  // the next group's codewords, in flight while the last tile is scored
#pragma unroll
        for (int j = 0; j < 4; ++j) rn[j] = codeword_raw(cb, FP8, group_cw(k + 1) + 4 * lane + j);
      }
      bool flag;
      int code = score_group<2, true>(big, stage, arow, lane, uf[s][k], err[s], flag);
      const unsigned long long todo = __ballot(flag && n0 + tok < n_tok);
      if (__popcll(todo) > kMany)
        again |= 1u << (4 * s + k);
      else
        decide(todo, k, n0, code);
      code_acc[s] = (code_acc[s] >> 8) | (static_cast<uint32_t>(code) << 24);
      __builtin_amdgcn_sched_barrier(0);  // one tile's scores in registers at a time
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const size_t row = rows[64 * s];
    if (row != kNoRow) *reinterpret_cast<uint32_t *>(pool + row + g0) = code_acc[s];
  }
#pragma unroll 1
  for (; again; again &= again - 1) {
    const int e = __builtin_ctz(again), k = e & 3;
    float u[4] = {0.f, 0.f, 0.f, 0.f}, er = err[0];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (e >> 2 == s) er = err[s];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        if (e == 4 * s + kk)
#pragma unroll
          for (int i = 0; i < 4; ++i) u[i] = uf[s][kk][i];
    }
    const int n0 = first + (e >> 2) * TOK;
    bool flag;
    int code = score_group<2, true>(stage_unrepeated<FP8>(cb, group_cw(k), stage, lane), stage, arow, lane, u, er, flag);
    decide(__ballot(flag && n0 + tok < n_tok), k, n0, code);
    const size_t row = rows[64 * (e >> 2)];
    if (row != kNoRow) pool[row + g0 + k] = static_cast<uint8_t>(code);
  }
}

// Two tiles per workgroup of encode_fast (its T split and its staged codewords
// serve both) once that leaves two launch rounds of two workgroups per CU; below
// that one tile, which ends sooner: 2 x 1024 tokens, 8 KV heads of 128, 34.6 us in
// single tiles.  Larger ones, single tiles and pairs: 2 x 4096 tokens 116.4 and
// 112.7, 32 x 4096 1509 and 1476, 4 x 12000 of head_dim 64 275 and 252.
constexpr int kPairWorkgroups = 1024;

// TBF: the transforms are stored as bf16 (a compile-time choice, so that the
// fp32 kernels carry no branch on it).
// Whole groups per wave once the tiles give every CU a workgroup; below that one
// group per wave and tiles of half the tokens, eight times the workgroups: 8
// sequences of 24 tokens, 8 KV heads of 128, took 38.7 us in 64-token tiles,
// 18.4 us so with the whole transform in each, 12.9 us with a quarter each.
template <int D, bool FP8, bool TBF>
void launch_tiles(const EncodeArgs &a, hipStream_t stream) {
  const long long n = static_cast<long long>(a.batch) * a.n_new;
  auto blocks = [&](const int tokens) { return static_cast<unsigned>((n + tokens - 1) / tokens); };
  const dim3 block(64 * kTileWaves);
  const unsigned tiles = blocks(TileShape<D, 4>::TOKENS);
  if (static_cast<long long>(tiles) * 2 * a.num_kv_heads < 256) {
    encode_tile<D, FP8, TBF, 2, true>
        <<<dim3(blocks(TileShape<D, 2>::TOKENS), a.num_kv_heads, 8), block, 0, stream>>>(a, 0);
    return;
  }
  // a scaled key and the scalar arm store values of the coefficients themselves
  // and take the fp64 transform; the other sides encode_fast
  const bool slow_k = a.k_scales, slow_v = a.v_sq;
  if (!slow_k || !slow_v) {
    const int sides = slow_k == slow_v ? 2 : 1;
    const unsigned pairs = (tiles + 1) / 2;
    if (static_cast<long long>(pairs) * sides * a.num_kv_heads >= kPairWorkgroups)
      encode_fast<D, FP8, TBF, 2><<<dim3(pairs, a.num_kv_heads, sides), block, 0, stream>>>(a, slow_k ? 1 : 0);
    else
      encode_fast<D, FP8, TBF, 1><<<dim3(tiles, a.num_kv_heads, sides), block, 0, stream>>>(a, slow_k ? 1 : 0);
  }
  if (slow_k || slow_v)
    encode_tile<D, FP8, TBF, 4, false>
        <<<dim3(tiles, a.num_kv_heads, slow_k == slow_v ? 2 : 1), block, 0, stream>>>(a, slow_k ? 0 : 1);
}

// Few tokens in the plain formats: encode_small, a workgroup per token, side and
// eight groups, as long as its workgroups stay below four per CU (8 KV
// heads of 128, one token per sequence: 5.6 us against 7.5 us in tiles for 8
// sequences, 7.5 both for 16, 12.6 against 8.1 for 32).  The key scale and the scalar arm need
// a token's whole transform, which the tiles form once (one sequence, both
// formats: 10.8 us against 13.8 with a workgroup per token and block).
template <int D, bool TBF>
hipError_t launch_encode_t(const EncodeArgs &a, hipStream_t stream) {
  const long long blocks = 2ll * (D / kGroupDim / encblk::kGroups) * a.n_new;
  if (!a.k_scales && !a.v_sq && blocks * a.batch * a.num_kv_heads < 1024) {
    const dim3 grid(static_cast<unsigned>(blocks), a.num_kv_heads, a.batch);
    if (a.cb_fp8)
      encode_small<D, true, TBF><<<grid, dim3(256), 0, stream>>>(a);
    else
      encode_small<D, false, TBF><<<grid, dim3(256), 0, stream>>>(a);
  } else {
    a.cb_fp8 ? launch_tiles<D, true, TBF>(a, stream) : launch_tiles<D, false, TBF>(a, stream);
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_encode_d(const EncodeArgs &a, hipStream_t stream) {
  return a.t_bf16 ? launch_encode_t<D, true>(a, stream) : launch_encode_t<D, false>(a, stream);
}

}  // namespace

hipError_t launch_encode(const EncodeArgs &args, hipStream_t stream) {
  EncodeArgs a = args;
  const uintptr_t addr = reinterpret_cast<uintptr_t>(a.k) | reinterpret_cast<uintptr_t>(a.v);
  a.in_vec = addr % (a.in_bf16 ? 8 : 16) == 0 ? 1 : 0;
  switch (a.head_dim) {
    case 64: return launch_encode_d<64>(a, stream);
    case 128: return launch_encode_d<128>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace novakv

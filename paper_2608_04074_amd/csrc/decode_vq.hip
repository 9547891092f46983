// Decode attention with fp32 precision throughout, for every layout: any
// block size, up to 8 query heads per KV head, head_dim 64 or 128, in one
// launch (query transform, split pass, band, combine of the splits).  It takes
// the calls that the table kernels (decode_lut.hip, decode_lut64.hip) do not:
// more than 4 query heads per KV head at head_dim 128, and caches whose
// 16-token runs are not contiguous.
//
// Paper: Algorithm 1 (attention step); Sec. "Decoding kernel and read path"
// (q' = q R_K^{-T} once per step, one codeword lookup per group, k_bar dropped
// by Lemma S1, split-KV decode); Corollary 1 (v_hat = s_hat R_V^T); Sec.
// "Sink-plus-recent band"; the sinks appendix (sink added once after the
// combine, shifted by -(q . k_bar) * scale).
//
// Both contractions run on the matrix cores with fp32 accumulation.  The
// codewords are fp16 and enter exactly; the other operand (q', then the
// probabilities) is fp32 and enters as two fp16 parts, hi = f16(x) and
// lo = f16((x - hi) 2^11), which carry it to half an fp32 ulp.  A 16x16x32
// MFMA has 16 columns: 8 heads x {hi, lo}, so the split costs nothing.
//  * K: lane (kg, m) gathers the codewords of token m, groups GP kg .. +GP-1,
//    from the key codebook in LDS (8 bytes each); they are the A operand as
//    they come.  B holds q' (each head scaled by a power of two to [1, 2)).
//  * softmax: columns h and h + 8 are added (one DPP rotation) and hold the
//    same logits; lane (tau, column) has tokens 16 a + 4 tau + i of the round.
//  * V: transposing gathers of the value codebook give coordinates as rows
//    and tokens as the contraction; the column's lane already holds the
//    probabilities of just these tokens, hi in columns 0..7, lo in 8..15.
//
// What bounds it: LDS.  Per token and KV head 64 (D = 128) 8-byte gathers at
// random codes: 4 cycles of a CU, and 5.2 of bank conflicts (counted), of the
// 9.6 that a token takes (4.0 ns).  Beside them 8 MFMA cycles and about 20 VALU
// cycles per SIMD, i.e. 7 per CU.  The scalar arm at head_dim 128 spills 25 to 31
// registers, some of them in the token loop.  A step of 16 sequences of up to 12000
// tokens, 64 query and 8 KV heads of 128, 32-token pages: 51.8 us with the
// encode of its token (74 MB of codes); three launches that gathered and
// multiplied one coordinate at a time on the VALU took 2798 us.  Its error
// against fp64 is 2.1e-7 of the result there (theirs was 5.1e-7).
#include <math.h>

#include "lut_common.h"
#include "nova_kv_internal.h"

namespace novakv {

namespace {

using namespace lut;

constexpr int kH = kMaxGqa;         // head columns
constexpr int kWaves = 12;          // 3 waves per SIMD within 168 VGPRs
constexpr int kNT = 64 * kWaves;
constexpr int kRound = 64;          // tokens per round and wave: four tiles of 16
constexpr float kLoUp = 2048.f, kLoDown = 1.f / 2048.f;
constexpr float kLazyLog2 = 8.f;    // reference lag allowed in the online softmax (log2 units)
constexpr float kLog2e = 1.44269504088896341f;

// LDS layout (bytes).
template <int D>
struct Lds {
  static constexpr int L = D / kGroupDim;
  static constexpr uint32_t kK = 0;                          // key codebook [L][256] codewords
  static constexpr uint32_t kV = L * 2048;                   // value codebook, in planes (below)
  static constexpr uint32_t kQ = 2 * L * 2048;               // query [8][D] f32, later s_hat
  static constexpr uint32_t kQB = kQ + kH * D * 4;           // q' parts [2][8][D] f16
  static constexpr uint32_t kOwn = kQB + 2 * kH * D * 2;     // own partial: codes [8][D], band [8][D] f32
  static constexpr uint32_t kStat = kOwn + 2 * kH * D * 4;   // f32 words: m [8], l [8], sink [8], q.k_bar [8], 2^e [8]
  static constexpr uint32_t kCtl = kStat + 5 * kH * 4;
  static constexpr uint32_t kBytes = kCtl + 16;
  // the codebook region is reused: partial sums of q' in the setup (key half),
  // the waves' partials and the combine's partial outputs after the loop
  static constexpr int kWaveFloats = 2 * kH + kH * (D + 4);
  static_assert(2 * kWaves * kWaveFloats * 4 <= 2 * L * 2048, "the waves' partials fit in the codebook region");
  static_assert(8 * kH * D * 4 <= L * 2048 || D == 64, "q' parts fit in the key codebook region");
  static_assert(kBytes <= 160 * 1024, "LDS budget of a workgroup");
};

template <int N>
struct Bytes;  // N code bytes in one load
template <>
struct Bytes<8> { typedef uint2 type; };
template <>
struct Bytes<4> { typedef uint32_t type; };
__device__ __forceinline__ uint32_t code_byte(const uint2 w, const int i) { return ((i < 4 ? w.x : w.y) >> (8 * (i & 3))) & 0xffu; }
__device__ __forceinline__ uint32_t code_byte(const uint32_t w, const int i) { return (w >> (8 * i)) & 0xffu; }

__device__ __forceinline__ float wave_maxf(float x) {
  x = fmaxf(x, row_ror<8>(x));
  x = fmaxf(x, row_ror<4>(x));
  x = fmaxf(x, row_ror<2>(x));
  x = fmaxf(x, row_ror<1>(x));
  return max_rows32(max_rows16(x));
}

__device__ __forceinline__ float input_value(const void *p, const size_t i, const int bf16) {
  return bf16 ? bf16_bits_to_float(static_cast<const uint16_t *>(p)[i]) : static_cast<const float *>(p)[i];
}

// hi and lo parts of an fp32 value (|x| below the fp16 range).  x is made
// opaque: a product fused into one of the conversions of hi but not the other
// would leave two different roundings of it.
__device__ __forceinline__ void split_f16(float x, _Float16 &hi, _Float16 &lo) {
  asm volatile("" : "+v"(x));
  hi = static_cast<_Float16>(x);
  lo = static_cast<_Float16>((x - static_cast<float>(hi)) * kLoUp);
}

// Scalar value arm: a code byte's four levels minus 1.5 (exact in fp16).
__device__ __forceinline__ uint2 centred_levels(const uint32_t c) {
  const uint2 q = sq_unpack_f16(c);
  const half2_t half3 = {static_cast<_Float16>(1.5f), static_cast<_Float16>(1.5f)};
  return make_uint2(__builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, q.x) - half3),
                    __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, q.y) - half3));
}

// Running reference of a softmax column.
struct Lag {
  float m;
  __device__ __forceinline__ bool move(const float zmax, float &alpha) {  // true where the reference moves off a finite one
    const float mn = fmaxf(m, zmax);
    const bool bump = mn > m + kLazyLog2;
    alpha = bump ? __builtin_amdgcn_exp2f(m - mn) : 1.f;
    const bool rescale = bump && m != -INFINITY;
    m = bump ? mn : m;
    return rescale;
  }
  __device__ __forceinline__ float base() const { return m == -INFINITY ? 0.f : m; }
};

// One workgroup per (sequence, KV head, split).  The splits tile the span that
// is read from the pools, and the band's rows; the last split to count in
// merges the partials (plain words with device-coherent stores, completed
// before the count, as in decode_lut64.hip).
template <int D, bool KS, bool SQ, bool FP8, bool TBF>
__global__ void __launch_bounds__(kNT) decode_vq(DecodeArgs a) {
  using S_ = Lds<D>;
  constexpr int L = D / kGroupDim;
  constexpr int GP = L / 4;                 // groups per lane quarter
  constexpr int NX = GP;                    // coordinate tiles of 16
  using Codes = typename Bytes<GP>::type;
  __shared__ __attribute__((aligned(16))) uint8_t smem[S_::kBytes];
  const uint32_t sbase = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_u8_ptr)smem));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int kv, b, split;
  unit_of_workgroup(xcd_contiguous(blockIdx.x, gridDim.x), a.n_split, a.b_chunk, a.num_kv_heads, kv, b, split);
  const int G = a.gqa;
  const int bk = b * a.num_kv_heads + kv;
  const size_t row0 = static_cast<size_t>(b) * a.num_q_heads + kv * G;

  const int S = a.seq_lens[b];
  const int att_lo = a.window > 0 ? max(0, S - a.window) : 0;
  const AttendedSpans spn = attended_spans(att_lo, S, a.n_sink, a.n_rec);
  const int t0 = spn.code_lo + split * a.chunk;
  const int t1 = min(spn.code_hi, t0 + a.chunk);
  const bool act = t0 < t1;
  const int ns = max(0, spn.sink_end - att_lo);
  const int nband = a.band_k ? ns + (S - spn.code_hi) : 0;
  const int bper = (nband + a.n_split - 1) / a.n_split;
  const int bfirst = min(nband, split * bper), bcount = min(nband, bfirst + bper) - bfirst;

  float *qs = reinterpret_cast<float *>(smem + S_::kQ);
  float *stat = reinterpret_cast<float *>(smem + S_::kStat);
  int *ctl = reinterpret_cast<int *>(smem + S_::kCtl);

  // ---- lane roles
  const int n = lane & 15, tau = lane >> 4;      // column (head n & 7, part n >> 3) / K row m = n, and lane row
  const int vi = (lane >> 2) & 3, vu = lane & 3;  // value gathers: token 4 tau + vi of a tile, group quarter vu

  // ---- round addressing: lane l owns token R + l (the last one past the end)
  const int bs = a.layout.block_size;
  const int bs_shift = (bs & (bs - 1)) == 0 ? __builtin_ctz(bs) : -1;
  const bool contig = a.layout.block_table == nullptr && a.layout.blocks_per_seq == 1;
  struct Owner {
    int phys, row;
  };
  auto owner = [&](const int R) -> Owner {
    const int t = min(R + lane, t1 - 1);
    if (contig) return Owner{b, t};
    const int blk = bs_shift >= 0 ? t >> bs_shift : t / bs;
    const int logical = b * a.layout.blocks_per_seq + blk;
    return Owner{a.layout.block_table ? a.layout.block_table[logical] : logical, t - blk * bs};
  };
  struct Round {
    Codes k[4], v[4];
    uint32_t ks, vq;
  };
  auto load_round = [&](const Owner o, Round &r) {
    const size_t row = (static_cast<size_t>(o.phys) * a.num_kv_heads + kv) * bs + o.row;
    const size_t off = row * L;
    const int lo = static_cast<int>(off), hi = static_cast<int>(off >> 32);
    auto of = [&](const int src) -> size_t {
      return (static_cast<size_t>(static_cast<uint32_t>(__shfl(hi, src))) << 32) | static_cast<uint32_t>(__shfl(lo, src));
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) r.k[t] = *reinterpret_cast<const Codes *>(a.k_codes + of(16 * t + n) + GP * tau);
#pragma unroll
    for (int t = 0; t < 4; ++t) r.v[t] = *reinterpret_cast<const Codes *>(a.v_codes + of(16 * t + 4 * tau + vi) + GP * vu);
    if constexpr (KS) r.ks = a.k_scales[row];
    if constexpr (SQ) r.vq = reinterpret_cast<const uint32_t *>(a.v_sq)[row];
  };
  const int nrounds = act ? (t1 - t0 + kRound - 1) / kRound : 0;
  Round rb[2];
  Owner own_next{0, 0};
  if (wave < nrounds) load_round(owner(t0 + kRound * wave), rb[0]);
  if (wave + kWaves < nrounds) own_next = owner(t0 + kRound * (wave + kWaves));

  // ---- setup: query, q' and its parts, sink logits, codebooks into LDS.
  // Every load is issued before the first use.
  {
    constexpr int QPER = (kH * D + kNT - 1) / kNT;
    float qv[QPER];
#pragma unroll
    for (int k = 0; k < QPER; ++k) {
      const int e = tid + k * kNT;
      qv[k] = e < G * D ? input_value(a.q, row0 * D + e, a.q_bf16) : 0.f;
    }
    constexpr int C4 = D / 4, RPT = D / 16;  // column quads; rows of t_k_inv_t per thread
    constexpr int QT = 16 * C4;              // threads that hold them
    constexpr int PARTS = QT / 64;
    const int e4 = tid % C4, jq = tid / C4;
    T4 trow[RPT];
    constexpr int CPER = (L * 256 + kNT - 1) / kNT;
    uint2 kst[CPER], vst[CPER];
    const void *cbk = codebook_from(a.cb_k, FP8, static_cast<size_t>(kv) * L * 256);
    const void *cbv = codebook_from(a.cb_v, FP8, static_cast<size_t>(kv) * L * 256);
    if (act) {
      if (tid < QT) {
        const size_t tk = (static_cast<size_t>(kv) * D + RPT * jq) * D + 4 * e4;
#pragma unroll
        for (int r = 0; r < RPT; ++r) trow[r] = load_t4(a.t_k_inv_t, tk + r * D, TBF);
      }
#pragma unroll
      for (int k = 0; k < CPER; ++k) kst[k] = codeword_raw(cbk, FP8, min(tid + k * kNT, L * 256 - 1));
      if constexpr (!SQ) {
#pragma unroll
        for (int k = 0; k < CPER; ++k) vst[k] = codeword_raw(cbv, FP8, min(tid + k * kNT, L * 256 - 1));
      }
    }
#pragma unroll
    for (int k = 0; k < QPER; ++k)
      if (tid + k * kNT < kH * D) qs[tid + k * kNT] = qv[k];
    if (act) {
      // value entry (g, c): plane g mod GP (8 KB), line c of 32 bytes, slot
      // g / GP, so that the 4 lanes of a token read one line's 4 slots
#pragma unroll
      for (int k = 0; k < CPER; ++k) {
        const int e = min(tid + k * kNT, L * 256 - 1), g = e >> 8, c = e & 255;
        *reinterpret_cast<uint2 *>(smem + S_::kV + (g % GP) * 8192 + 32 * c + 8 * (g / GP)) =
            SQ ? centred_levels(c) : codeword_f16(vst[k], FP8);
      }
    }
    __syncthreads();
    // q . k_bar and the shifted sink logit of head w (log2 units): the last
    // waves, two heads each
    if (wave >= 8) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int h = 2 * (wave - 8) + k;
        float dot = 0.f;
        for (int i = lane; i < D; i += 64) dot = fmaf(qs[h * D + i], a.kbar[static_cast<size_t>(kv) * D + i], dot);
        dot = wave_sum(dot);
        if (lane == 0) {
          stat[2 * kH + h] = a.sinks && h < G ? (a.sinks[kv * G + h] - a.scale * dot) * kLog2e : -INFINITY;
          stat[3 * kH + h] = dot;
        }
      }
    }
    if (act) {
      float *qsum = reinterpret_cast<float *>(smem + S_::kK);  // [PARTS][8][D]
      if (tid < QT) {
#pragma unroll
        for (int h = 0; h < kH; ++h) {
          float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int r = 0; r < RPT; ++r) {
            const float x = qs[h * D + RPT * jq + r];
            const float4 t = t4_value(trow[r], TBF);
            acc.x = fmaf(x, t.x, acc.x);
            acc.y = fmaf(x, t.y, acc.y);
            acc.z = fmaf(x, t.z, acc.z);
            acc.w = fmaf(x, t.w, acc.w);
          }
          // the wave's row groups of the same columns
          if constexpr (C4 == 16) {
            acc.x = add_rows16(acc.x); acc.y = add_rows16(acc.y); acc.z = add_rows16(acc.z); acc.w = add_rows16(acc.w);
          }
          acc.x = add_rows32(acc.x); acc.y = add_rows32(acc.y); acc.z = add_rows32(acc.z); acc.w = add_rows32(acc.w);
          if (lane < C4) *reinterpret_cast<float4 *>(qsum + (wave * kH + h) * D + 4 * e4) = acc;
        }
      }
      __syncthreads();
      if (wave < kH) {  // head `wave`: sum the parts, scale to [1, 2) and split
        constexpr int PL = D / 64;
        float x[PL], big = 0.f;
#pragma unroll
        for (int k = 0; k < PL; ++k) {
          x[k] = 0.f;
#pragma unroll
          for (int p = 0; p < PARTS; ++p) x[k] += qsum[(p * kH + wave) * D + lane + 64 * k];
          x[k] *= a.qscale;
          big = fmaxf(big, fabsf(x[k]));
        }
        big = wave_maxf(big);
        const int e = big > 0.f ? __builtin_amdgcn_frexp_expf(big) - 1 : 0;
        _Float16 *qb = reinterpret_cast<_Float16 *>(smem + S_::kQB);
#pragma unroll
        for (int k = 0; k < PL; ++k) {
          _Float16 hi, lo;
          split_f16(ldexpf(x[k], -e), hi, lo);
          qb[wave * D + lane + 64 * k] = hi;
          qb[(kH + wave) * D + lane + 64 * k] = lo;
        }
        if (lane == 0) stat[4 * kH + wave] = ldexpf(1.f, e);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < CPER; ++k)
        *reinterpret_cast<uint2 *>(smem + S_::kK + 8 * min(tid + k * kNT, L * 256 - 1)) = codeword_f16(kst[k], FP8);
    }
    __syncthreads();
  }

  // ---- token loop
  Lag ref{-INFINITY}, ref2{-INFINITY};  // ref2 (scalar value arm): of the probabilities times the token's scale
  float l_run = 0.f, z_run = 0.f;       // z_run: sum of p * (offset + 1.5 scale)
  float4_t acc[NX];
#pragma unroll
  for (int X = 0; X < NX; ++X) acc[X] = float4_t{0.f, 0.f, 0.f, 0.f};
  if (act) {
    const uint32_t kbase = sbase + S_::kK + GP * tau * 2048;
    const uint32_t vbase = sbase + S_::kV + 8 * vu;
    half8_t qb[GP / 2];  // B operands: coordinates of groups GP tau + 2 s, + 2 s + 1
#pragma unroll
    for (int s = 0; s < GP / 2; ++s)
      qb[s] = *reinterpret_cast<const half8_t *>(smem + S_::kQB + 2 * (n * D + 4 * (GP * tau + 2 * s)));
    const bool lo_col = n >= kH;
    const float fs = stat[4 * kH + (n & 7)] * (lo_col ? kLoDown : 1.f);
    typedef __attribute__((address_space(3))) const half4_t *lds_half4_ptr;

    auto process = [&](const int R, const Round &r) {
      float z[16];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < GP / 2; ++s) {
          const half4_t c0 = *(lds_half4_ptr)(uintptr_t)(kbase + (2 * s) * 2048 + 8 * code_byte(r.k[t], 2 * s));
          const half4_t c1 = *(lds_half4_ptr)(uintptr_t)(kbase + (2 * s + 1) * 2048 + 8 * code_byte(r.k[t], 2 * s + 1));
          const half8_t av = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
          d = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, qb[s], d, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x = d[i] * fs;
          z[4 * t + i] = x + row_ror<8>(x);
        }
      }
      if constexpr (KS) {
#pragma unroll
        for (int j = 0; j < 16; ++j)
          z[j] *= __uint_as_float(static_cast<uint32_t>(__shfl(static_cast<int>(r.ks), 16 * (j >> 2) + 4 * tau + (j & 3))) << 16);
      }
      const bool ragged = R + kRound > t1;
      if (ragged) {
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (R + 16 * (j >> 2) + 4 * tau + (j & 3) >= t1) z[j] = -INFINITY;
      }
      float zmax = z[0];
#pragma unroll
      for (int j = 1; j < 16; ++j) zmax = fmaxf(zmax, z[j]);
      zmax = max_rows32(max_rows16(zmax));
      float alpha;
      bool rescale = ref.move(zmax, alpha);
      const float base = ref.base();
      float w[16], lsum = 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        w[j] = __builtin_amdgcn_exp2f(z[j] - base);
        lsum += w[j];
      }
      l_run = fmaf(l_run, alpha, lsum);
      if constexpr (SQ) {
        // value = (offset + 1.5 scale) + scale (level - 1.5): the two sums are
        // small, where offset and scale * level would cancel.  The first is
        // formed in fp32; the levels' weights p * scale have a reference of
        // their own, so that any scale stays in fp16 range
        float zs = 0.f, ymax = -INFINITY, mant[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          uint32_t g = static_cast<uint32_t>(__shfl(static_cast<int>(r.vq), 16 * (j >> 2) + 4 * tau + (j & 3)));
          if (ragged && z[j] == -INFINITY) g = 0u;  // rows past the tokens may hold anything
          const float scale = __uint_as_float(g << 16);
          zs = fmaf(w[j], fmaf(1.5f, scale, __uint_as_float(g & 0xffff0000u)), zs);
          mant[j] = __builtin_amdgcn_frexp_mantf(scale);
          z[j] += static_cast<float>(__builtin_amdgcn_frexp_expf(scale));
          ymax = fmaxf(ymax, z[j]);
        }
        z_run = fmaf(z_run, alpha, zs);
        ymax = max_rows32(max_rows16(ymax));
        rescale = ref2.move(ymax, alpha);
        const float base2 = ref2.base();
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = __builtin_amdgcn_exp2f(z[j] - base2) * mant[j];
      }
      if (__any(rescale)) {
#pragma unroll
        for (int X = 0; X < NX; ++X) acc[X] *= alpha;
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        half8_t pb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          _Float16 hi, lo;
          split_f16(w[8 * hf + e], hi, lo);
          pb[e] = lo_col ? lo : hi;
        }
#pragma unroll
        for (int X = 0; X < NX; ++X) {
          const half4_t va = tr16_read(vbase + X * 8192 + 32 * code_byte(r.v[2 * hf], X));
          const half4_t vb = tr16_read(vbase + X * 8192 + 32 * code_byte(r.v[2 * hf + 1], X));
          const half8_t av = __builtin_shufflevector(va, vb, 0, 1, 2, 3, 4, 5, 6, 7);
          acc[X] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, pb, acc[X], 0, 0, 0);
        }
      }
    };
    // one round in flight while one is processed, the block-table entry of the
    // round after requested with it
    for (int rd = wave; rd < nrounds; rd += 2 * kWaves) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int cur = rd + k * kWaves;
        if (cur >= nrounds) break;
        const int nxt = cur + kWaves, nxt2 = nxt + kWaves;
        if (nxt < nrounds) load_round(own_next, rb[k ^ 1]);
        if (nxt2 < nrounds) own_next = owner(t0 + kRound * nxt2);
        process(t0 + kRound * cur, rb[k]);
      }
    }
    // columns hi and lo of a head, then the denominators over the lane rows
    const float fa = lo_col ? kLoDown : 1.f;
    float f2 = 1.f, z_tot = 0.f;
    if constexpr (SQ) {
      f2 = ref2.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ref2.m - ref.base());
      z_tot = add_rows32(add_rows16(z_run));
    }
#pragma unroll
    for (int X = 0; X < NX; ++X)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float y = acc[X][i] * fa;
        acc[X][i] = fmaf(y + row_ror<8>(y), f2, z_tot);
      }
    l_run = add_rows32(add_rows16(l_run));
  }

  // ---- band share: exact bf16 rows on the fp32 matrix cores (products and
  // sums in fp32), 16 rows per wave and step, columns = heads.  Contraction
  // slot (step t, lane row tau) of the logits is coordinate (D / 4) tau + t.
  constexpr int CP = D / 16;  // value coordinates per lane: CP m + X
  Lag bref{-INFINITY};
  float bl = 0.f;
  float4_t bacc[CP];
#pragma unroll
  for (int X = 0; X < CP; ++X) bacc[X] = float4_t{0.f, 0.f, 0.f, 0.f};
  if (bcount > 0) {
    const size_t hb = static_cast<size_t>(bk) * (a.n_sink + a.n_rec);
    auto row_of = [&](const int r) -> size_t {
      const int i = bfirst + min(r, bcount - 1);
      const int p = i < ns ? att_lo + i : spn.code_hi + (i - ns);
      return (hb + band_slot(p, a.n_sink, a.n_rec)) * D;
    };
    const float qk = stat[3 * kH + (n & 7)];
    for (int tile = wave; 16 * tile < bcount; tile += kWaves) {
      const uint16_t *kr = a.band_k + row_of(16 * tile + n) + (D / 4) * tau;
      uint4 kw[D / 32];
#pragma unroll
      for (int c = 0; c < D / 32; ++c) kw[c] = reinterpret_cast<const uint4 *>(kr)[c];
      uint32_t vw[4][CP / 2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t *vr = reinterpret_cast<const uint32_t *>(a.band_v + row_of(16 * tile + 4 * tau + i) + CP * n);
#pragma unroll
        for (int c = 0; c < CP / 2; ++c) vw[i][c] = vr[c];
      }
      float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < D / 32; ++c) {
        const uint32_t ws[4] = {kw[c].x, kw[c].y, kw[c].z, kw[c].w};
        const float *qr = qs + (n & 7) * D + (D / 4) * tau + 8 * c;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float kx = __uint_as_float((e & 1) ? (ws[e >> 1] & 0xffff0000u) : (ws[e >> 1] << 16));
          d = __builtin_amdgcn_mfma_f32_16x16x4f32(kx, qr[e], d, 0, 0, 0);
        }
      }
      float z[4], zmax = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[i] = 16 * tile + 4 * tau + i < bcount ? (d[i] - qk) * a.qscale : -INFINITY;
        zmax = fmaxf(zmax, z[i]);
      }
      zmax = max_rows32(max_rows16(zmax));
      float alpha;
      if (__any(bref.move(zmax, alpha))) {
#pragma unroll
        for (int X = 0; X < CP; ++X) bacc[X] *= alpha;
      }
      const float base = bref.base();
      float lsum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[i] = __builtin_amdgcn_exp2f(z[i] - base);
        lsum += z[i];
      }
      bl = fmaf(bl, alpha, lsum);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int X = 0; X < CP; ++X) {
          const uint32_t w = vw[i][X >> 1];
          const float v = __uint_as_float((X & 1) ? (w & 0xffff0000u) : (w << 16));
          bacc[X] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, z[i], bacc[X], 0, 0, 0);
        }
    }
    bl = add_rows32(add_rows16(bl));
  }

  // ---- rows of t_v for the combine, requested before the merge: thread
  // t < 4 D holds row t mod D, columns (D / 4) (t / D) ..
  const int od = tid % D, oj = tid / D;
  T4 tv[D / 16];
  if (tid < 4 * D) {
    const size_t row = (static_cast<size_t>(kv) * D + od) * D + (D / 4) * oj;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) tv[i] = load_t4(a.t_v, row + 4 * i, TBF);
  }

  __syncthreads();  // every wave is done with the codebooks
  float *merge = reinterpret_cast<float *>(smem);
  constexpr int WF = S_::kWaveFloats;
  const int nmerge = nband > 0 ? 2 * kWaves : kWaves;  // partials: the waves' codes, then the waves' band rows
  if (n < kH) {
    float *mw = merge + wave * WF, *mb = mw + kWaves * WF;
    if (tau == 0) {
      mw[n] = ref.m;
      mw[kH + n] = l_run;
    }
#pragma unroll
    for (int X = 0; X < NX; ++X) *reinterpret_cast<float4_t *>(mw + 2 * kH + n * (D + 4) + 4 * (GP * tau + X)) = acc[X];
    if (nband > 0) {
      if (tau == 0) {
        mb[n] = bref.m;
        mb[kH + n] = bl;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int X = 0; X < CP; ++X) mb[2 * kH + n * (D + 4) + CP * (4 * tau + i) + X] = bacc[X][i];
    }
  }
  __syncthreads();
  float *ownc = reinterpret_cast<float *>(smem + S_::kOwn), *ownb = ownc + kH * D;
  const size_t prow = row0 * a.n_split + split;  // row of head 0 in the exchange, heads n_split apart
  const size_t brow = static_cast<size_t>(a.batch) * a.num_q_heads * a.n_split;  // the band's rows follow
  for (int i = tid; i < G * D; i += kNT) {
    const int h = i / D, d = i % D;
    float big = -INFINITY;
    for (int w = 0; w < nmerge; ++w) big = fmaxf(big, merge[w * WF + h]);
    float num = 0.f, den = 0.f, bnum = 0.f;
    if (big != -INFINITY) {
#pragma unroll 4
      for (int w = 0; w < kWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(merge[w * WF + h] - big);
        num = fmaf(f, merge[w * WF + 2 * kH + h * (D + 4) + d], num);
        den = fmaf(f, merge[w * WF + kH + h], den);
      }
#pragma unroll 4
      for (int w = kWaves; w < nmerge; ++w) {
        const float f = __builtin_amdgcn_exp2f(merge[w * WF + h] - big);
        bnum = fmaf(f, merge[w * WF + 2 * kH + h * (D + 4) + d], bnum);
        den = fmaf(f, merge[w * WF + kH + h], den);
      }
    }
    ownc[i] = num;
    ownb[i] = bnum;
    if (d == 0) {
      stat[h] = big;
      stat[kH + h] = den;
    }
    if (a.n_split > 1) {
      const size_t r = prow + static_cast<size_t>(h) * a.n_split;
      store_dev(a.part_acc + r * D + d, num);
      if (nband > 0) store_dev(a.part_acc + (brow + r) * D + d, bnum);
      if (d == 0) {
        store_dev(a.part_ml + 2 * r, big);
        store_dev(a.part_ml + 2 * r + 1, den);
      }
    }
  }
  if (a.n_split > 1) {
    __builtin_amdgcn_s_waitcnt(0);  // this thread's stores have completed
    __syncthreads();
    if (tid == 0) {
      const int last = __hip_atomic_fetch_add(a.counters + bk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.n_split - 1;
      if (last) __hip_atomic_store(a.counters + bk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ctl[0] = last;
    }
    __syncthreads();
    if (ctl[0] == 0) return;
  } else {
    __syncthreads();
  }

  // ---- combine: the splits in index order, the sink once, then the inverse
  // value transform; the band's value term is in the original domain
  float *shat = qs, *bout = ownb;
  for (int i = tid; i < kH * D; i += kNT) {
    const int h = i / D, d = i % D;
    float s_out = 0.f, b_out = 0.f;
    if (h < G) {
      const size_t r0 = (row0 + h) * a.n_split;
      const float sink = stat[2 * kH + h];
      float big = sink, num = 0.f, bnum = 0.f, den = sink == -INFINITY ? 0.f : 1.f;
      auto take = [&](const float ms, const float ls, const float as, const float ab) {
        if (ms == -INFINITY) return;
        if (ms > big) {
          const float f = big == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(big - ms);
          num *= f;
          bnum *= f;
          den *= f;
          big = ms;
        }
        const float f = __builtin_amdgcn_exp2f(ms - big);
        num = fmaf(f, as, num);
        bnum = fmaf(f, ab, bnum);
        den = fmaf(f, ls, den);
      };
      if (a.n_split == 1) {
        take(stat[h], stat[kH + h], ownc[i], nband > 0 ? ownb[i] : 0.f);
      } else {
        // eight splits' words (this split's own among them) are requested
        // before any is used: one round trip for each eight, not two for each
        // split (one sequence of 32000 tokens, 64 query heads: 34.2 us, now 28.0
        // in more splits; 2000 tokens 18.9, now 17.8)
        constexpr int BATCH = 8;
        for (int s0 = 0; s0 < a.n_split; s0 += BATCH) {
          float ms[BATCH], ls[BATCH], as[BATCH], ab[BATCH];
#pragma unroll
          for (int j = 0; j < BATCH; ++j) {
            const size_t r = r0 + min(s0 + j, a.n_split - 1);
            ms[j] = load_dev(a.part_ml + 2 * r);
            ls[j] = load_dev(a.part_ml + 2 * r + 1);
            as[j] = load_dev(a.part_acc + r * D + d);
          }
          if (nband > 0) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j)
              ab[j] = load_dev(a.part_acc + (brow + r0 + min(s0 + j, a.n_split - 1)) * D + d);
          } else {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) ab[j] = 0.f;
          }
#pragma unroll
          for (int j = 0; j < BATCH; ++j)
            if (s0 + j < a.n_split) take(ms[j], ls[j], as[j], ab[j]);
        }
      }
      s_out = den > 0.f ? num / den : 0.f;
      b_out = den > 0.f ? bnum / den : 0.f;
    }
    shat[i] = s_out;
    if (h < G) bout[i] = b_out;
  }
  __syncthreads();
  float *outp = reinterpret_cast<float *>(smem);  // [4][8][D]
  if (tid < 4 * D) {
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      float x = 0.f;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) {
        const float4 s4 = *reinterpret_cast<const float4 *>(shat + h * D + (D / 4) * oj + 4 * i);
        const float4 t = t4_value(tv[i], TBF);
        x = fmaf(s4.x, t.x, x);
        x = fmaf(s4.y, t.y, x);
        x = fmaf(s4.z, t.z, x);
        x = fmaf(s4.w, t.w, x);
      }
      outp[(oj * kH + h) * D + od] = x;
    }
  }
  __syncthreads();
  for (int i = tid; i < G * D; i += kNT) {
    const float o = (outp[i] + outp[kH * D + i]) + (outp[2 * kH * D + i] + outp[3 * kH * D + i]);
    a.out[row0 * D + i] = nband > 0 ? o + bout[i] : o;
  }
}

template <int D, bool KS, bool SQ>
void launch_vq_format(const DecodeArgs &a, const dim3 grid, hipStream_t stream) {
  if (a.t_bf16)
    a.cb_fp8 ? decode_vq<D, KS, SQ, true, true><<<grid, dim3(kNT), 0, stream>>>(a)
             : decode_vq<D, KS, SQ, false, true><<<grid, dim3(kNT), 0, stream>>>(a);
  else
    a.cb_fp8 ? decode_vq<D, KS, SQ, true, false><<<grid, dim3(kNT), 0, stream>>>(a)
             : decode_vq<D, KS, SQ, false, false><<<grid, dim3(kNT), 0, stream>>>(a);
}

template <int D>
void launch_vq_d(const DecodeArgs &a, const dim3 grid, hipStream_t stream) {
  if (a.v_sq)
    a.k_scales ? launch_vq_format<D, true, true>(a, grid, stream) : launch_vq_format<D, false, true>(a, grid, stream);
  else
    a.k_scales ? launch_vq_format<D, true, false>(a, grid, stream) : launch_vq_format<D, false, false>(a, grid, stream);
}

}  // namespace

hipError_t launch_decode_vq(const DecodeArgs &a, hipStream_t stream) {
  if (a.append || a.gqa > kH) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(a.batch) * a.num_kv_heads * a.n_split);
  switch (a.head_dim) {
    case 64: launch_vq_d<64>(a, grid, stream); break;
    case 128: launch_vq_d<128>(a, grid, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace novakv

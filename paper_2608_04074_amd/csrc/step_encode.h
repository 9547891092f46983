// The new token's encode inside the one-launch decode step when the call
// has a sink-plus-recent band whose recent part holds that token.
//
// Paper: Algorithm 1 (the write of the new token, then the attention), Sec.
// "Sink-plus-recent band" (the newest positions are held in BF16 and
// attended exactly), Sec. "Bit rate" (keys as VQ codes with a per-token BF16
// scale, values as per-token affine INT2).
//
// The new token is the band's last row, so the attention needs none of its
// codes: the encode only stores them (codes, and in the key-scale format the
// scale, in the scalar value arm the levels and (scale, offset)), exactly as
// the one-token encoder does.  Its work is a list of tasks, run by teams of
// 256 threads (4 whole waves) that meet through an LDS arrival counter:
//   keys:   one block item per 8 groups, or with the key scale one task (all
//           D coefficients, rho, then every block's codes of u / rho);
//   values: one block item per 8 groups, or in the scalar arm one task (all
//           D coefficients, min and max, levels).
// Every task does the one-token encoder's arithmetic (encode_block.h), so
// both paths store the same bytes.
#pragma once

#include "encode_block.h"
#include "lut_common.h"
#include "nova_kv_internal.h"

namespace novakv {
namespace step {

// All four waves of a team arrive, then each continues once the counter has
// reached 4 * phase: LDS writes before the call are visible after it.
__device__ __forceinline__ void team_meet(int *ctr, const int phase) {
  if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  while (__hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < 4 * phase)
    __builtin_amdgcn_s_sleep(1);
}

template <int D, bool KS, bool SQ>
struct Tasks {
  static constexpr int kBlocks = D / kGroupDim / encblk::kGroups;
  static constexpr int kKey = KS ? 1 : kBlocks;
  static constexpr int kAll = kKey + (SQ ? 1 : kBlocks);
  // meetings of task j: its x, then two per block of coefficients and one for
  // rho (key scale) or two for the levels (scalar arm); a block item meets twice
  __device__ static int phases(const int j) {
    if (j < kKey) return KS ? 2 + 2 * kBlocks : 2;
    return SQ ? 3 + 2 * kBlocks : 2;
  }
  // a team's meetings for tasks first, first + stride, ..., with the last one
  // after its last task
  __device__ static int phases_of(const int first, const int stride) {
    int n = 1;
    for (int j = first; j < kAll; j += stride) n += phases(j);
    return n;
  }
};

// LDS of one team: two sets of scratch that successive tasks alternate
// between, so no meeting guards their reuse.
template <int D>
struct Scratch {
  encblk::Scratch<D> sc[2];
  double u[2][D];              // a whole-token task's coefficients
  double red[2][2 * D / 64];   // its min and max words
  uint8_t q[2][D];             // its scalar-arm levels
};

// Words of a new token handed to the split that attends it (DecodeArgs::xnew):
// key code of group g, value code of group g, key scale, scalar-arm word.
constexpr int kWordK = 0, kWordV = 32, kWordScale = 64, kWordSq = 65, kWords = 66;
constexpr int kWordCount = 127;  // who has finished with them, in a captured call
struct NoPublish {
  __device__ __forceinline__ void operator()(int, uint32_t) const {}
};

// Tasks first, first + stride, ... of the new token at code row offset tokoff
// of the pools, by team thread t (0..255); meet() is the team's meeting, and
// publish(word, value) gets every stored value.
// TBF: the transforms are stored as bf16.
// wide: 8 KB of LDS for whole-token tasks that request the transform at once
// (encoder workgroups; nullptr: block after block, in the registers that a
// decoding workgroup leaves).
template <int D, bool KS, bool SQ, bool TBF, class Meet, class Publish = NoPublish>
__device__ __forceinline__ void encode_token(const DecodeArgs &a, Scratch<D> &ls, const int b, const int kv,
                                             const int first, const int stride, const size_t tokoff, const int t,
                                             const bool fp8, Meet meet, Publish publish = NoPublish(),
                                             double *wide = nullptr) {
  using T = Tasks<D, KS, SQ>;
  constexpr int L = D / kGroupDim;
  const size_t elem = (static_cast<size_t>(b) * a.num_kv_heads + kv) * D + (t & (D - 1));
  auto element = [&](const bool key) {  // element t of the token minus k_bar (keys) or of the token (values)
    const void *src = key ? a.k_new : a.v_new;
    double x = a.new_bf16 ? static_cast<double>(bf16_bits_to_float(static_cast<const uint16_t *>(src)[elem]))
                          : static_cast<double>(static_cast<const float *>(src)[elem]);
    if (key) x -= static_cast<double>(a.kbar[kv * D + t]);
    return x;
  };
  const size_t cw0 = static_cast<size_t>(kv) * L * kCodebookSize;
  int k = 0;
  for (int j = first; j < T::kAll; j += stride, ++k) {
    encblk::Scratch<D> &s = ls.sc[k & 1];
    double *u = ls.u[k & 1];
    const bool key = j < T::kKey;
    const void *tm = transform_of(key ? a.t_k : a.t_v, kv, D, TBF);
    const void *cb = key ? a.cb_k : a.cb_v;
    T4 rows[D / 32];
    uint2 cw[encblk::kPer];
    if ((key && KS) || (!key && SQ)) {
      if (wide) {
        T4 all[encblk::WideRows<D>::RPT];
        encblk::load_wide_rows<D>(t, tm, TBF, all);
        if (key) encblk::load_codewords(t, cb, fp8, cw0, 0, cw);
        if (t < D) s.xs[t] = element(key);
        meet();
        encblk::wide_coefficients<D>(t, s.xs, TBF, all, wide, u, meet);
      } else {
        encblk::load_rows<D>(t, tm, TBF, 0, rows);
        if (key) encblk::load_codewords(t, cb, fp8, cw0, 0, cw);
        if (t < D) s.xs[t] = element(key);
        meet();
        encblk::token_coefficients<D>(t, s, tm, TBF, rows, u, meet);
      }
      if (key) {
        // rho, then the blocks' codes of the coefficients divided by it (the
        // next block's codewords requested while one block is searched)
        if (t == 0) s.wpart[0][0] = encblk::key_scale<D>(u);
        meet();
        const double rho = s.wpart[0][0];
#pragma unroll
        for (int bb = 0; bb < T::kBlocks; ++bb) {
          uint2 nx[encblk::kPer];
          if (bb + 1 < T::kBlocks) encblk::load_codewords(t, cb, fp8, cw0, bb + 1, nx);
          double uu[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double v = u[encblk::kCols * bb + 4 * (t >> 5) + i];
            uu[i] = rho > 0.0 ? v / rho : 0.0;
          }
          const int code = encblk::search_codes(t, uu, cw, fp8);
          if ((t & 31) == 0) {
            const int g = encblk::kGroups * bb + (t >> 5);
            a.k_codes_w[tokoff + g] = static_cast<uint8_t>(code);
            publish(kWordK + g, static_cast<uint32_t>(code));
          }
          if (bb + 1 < T::kBlocks) {
#pragma unroll
            for (int i = 0; i < encblk::kPer; ++i) cw[i] = nx[i];
          }
        }
        if (t == 0) {
          a.k_scales_w[tokoff / L] = encblk::bf16_of(rho);
          publish(kWordScale, encblk::bf16_of(rho));
        }
      } else {
        uint16_t sbits, zbits;
        encblk::sq_levels<D>(t, u, ls.red[k & 1], ls.q[k & 1], meet, sbits, zbits);
        if (t < L) {
          const uint8_t levels = encblk::sq_byte(ls.q[k & 1], t);
          a.v_codes_w[tokoff + t] = levels;
          publish(kWordV + t, levels);
        }
        if (t == 0) {
          a.v_sq_w[(tokoff / L) * 2] = sbits;
          a.v_sq_w[(tokoff / L) * 2 + 1] = zbits;
          publish(kWordSq, sbits | (static_cast<uint32_t>(zbits) << 16));
        }
      }
    } else {
      const int blk = key ? j : j - T::kKey;
      encblk::load_block<D>(t, tm, TBF, cb, fp8, cw0, blk, rows, cw);
      if (t < D) s.xs[t] = element(key);
      meet();
      encblk::partial_block<D>(t, s, rows, TBF);
      meet();
      const int code = encblk::search_block<D>(t, s, cw, fp8);
      if ((t & 31) == 0) {
        const int g = encblk::kGroups * blk + (t >> 5);
        (key ? a.k_codes_w : a.v_codes_w)[tokoff + g] = static_cast<uint8_t>(code);
        publish((key ? kWordK : kWordV) + g, static_cast<uint32_t>(code));
      }
    }
  }
  meet();  // every read of the scratch is done
}

// The new token's key and value rows (bf16: as given, or an fp32 element
// rounded to nearest even) into its band slot, by threads 0 .. 2D-1.
template <int D>
__device__ __forceinline__ void store_band_rows(const DecodeArgs &a, const int b, const int kv, const int pos) {
  const int tid = threadIdx.x;
  if (tid >= 2 * D || !position_in_pool(a.layout, pos)) return;
  const int side = tid / D, d = tid % D;
  const void *src = side ? a.v_new : a.k_new;
  const size_t idx = (static_cast<size_t>(b) * a.num_kv_heads + kv) * D + d;
  uint16_t bits;
  if (a.new_bf16) {
    bits = static_cast<const uint16_t *>(src)[idx];
  } else {
    const uint32_t f = __float_as_uint(static_cast<const float *>(src)[idx]);
    bits = static_cast<uint16_t>((f + 0x7fffu + ((f >> 16) & 1u)) >> 16);
  }
  const int nb = a.n_sink + a.n_rec;
  (side ? a.band_v_w : a.band_k_w)[((static_cast<size_t>(b) * a.num_kv_heads + kv) * nb +
                                    band_slot(pos, a.n_sink, a.n_rec)) * D + d] = bits;
}

// ---- the step's encode in workgroups of its own
//
// Where the step's launch leaves CUs idle, n_enc workgroups of it do nothing
// else than encode its token: enc_per_unit for each (sequence, KV head), each
// with TEAMS teams.
//  * Without a band they hand the token's values to the split that holds its
//    position as tagged words (HAND), while that split is still in its setup
//    or token loop.  They come first in the dispatch order, so within one
//    launch each XCD starts them before its decoding workgroups.  That says
//    nothing of launches on other streams, whose workgroups may hold the CUs
//    that an encoder needs: the split therefore looks for the words only
//    new_polls times, then forms them itself (form_new_token), and no workgroup
//    ever waits for one that may not have started.
//  * With the token in the band nothing waits for them, and they come last.
//    (In a full launch they would follow the decode: 32 sequences of 8192
//    tokens in the deployed format took 75 us so, 63 in two launches.)
constexpr int kNewNone = 0, kNewCodes = 1, kNewBand = 2;  // what a decoding workgroup does about the token

constexpr int kWide = 8192;  // LDS bytes of a team's whole-token sums

// Replays of a captured call repeat its tag, so the words of a unit are emptied
// by the last of those who use them: its encoder workgroups, once their stores
// have completed, and its reader, once it has the words or has given up on
// them.  (Emptied by a reader that gave up, a word that comes later would be
// taken for the next replay's.)  The count travels with the tag, as whatever a
// call of another shape left in its word must not be taken for one.
__device__ __forceinline__ void retire_new_token(const DecodeArgs &a, const int unit) {  // one thread
  uint64_t *xn = a.xnew + static_cast<size_t>(unit) * 8 * 32;
  const uint32_t all = static_cast<uint32_t>(a.enc_per_unit) + 1;
  uint64_t old = lut::get_word(xn + kWordCount);
  uint32_t count;
  uint64_t now;
  do {  // a failed exchange means that another of the `all` has counted in
    count = lut::word_ready(a.epoch, old) ? static_cast<uint32_t>(old) + 1 : 1;
    now = count == all ? 0 : (static_cast<uint64_t>(a.epoch) << 32) | count;
  } while (!__hip_atomic_compare_exchange_strong(xn + kWordCount, &old, now, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT));
  if (count == all)
    for (int w = 0; w < kWords; ++w) lut::clear_word(xn + w);
}

// An encoder workgroup's work (number wg < n_enc).
template <int D, int TEAMS, bool KS, bool FP8, bool SQ, bool TBF, bool HAND, class RowOf>
__device__ __forceinline__ void encode_workgroup(const DecodeArgs &a, uint8_t *smem, const int wg, RowOf row_of) {
  const int unit = wg / a.enc_per_unit, e = wg - unit * a.enc_per_unit;
  if (unit >= a.batch * a.num_kv_heads) return;  // n_enc is rounded up
  const int b = unit / a.num_kv_heads, kv = unit - b * a.num_kv_heads;
  const int S = a.seq_lens[b];
  if (!position_in_pool(a.layout, S - 1)) return;  // (an empty sequence; its reader tests the same)
  const int tid = threadIdx.x, team = tid >> 8;
  Scratch<D> *ls = reinterpret_cast<Scratch<D> *>(smem);
  double *wide = reinterpret_cast<double *>(smem + TEAMS * sizeof(Scratch<D>));
  int *ctr = reinterpret_cast<int *>(smem + TEAMS * (sizeof(Scratch<D>) + kWide));
  if (tid < TEAMS) ctr[tid] = 0;
  __syncthreads();
  uint64_t *xn = a.xnew + static_cast<size_t>(unit) * 8 * 32;
  int phase = 0;  // shared by every copy of the meeting
  auto meet = [&] { team_meet(ctr + team, ++phase); };
  auto publish = [&](const int w, const uint32_t v) {
    if (HAND && a.new_polls > 0) lut::put_word(a.epoch, xn + w, __uint_as_float(v));
  };
  encode_token<D, KS, SQ, TBF>(a, ls[team], b, kv, e * TEAMS + team, TEAMS * a.enc_per_unit, row_of(b, kv, S - 1),
                               tid & 255, FP8, meet, publish, wide + team * (kWide / 8));
  if (HAND && a.clear_xch) {
    __builtin_amdgcn_s_waitcnt(0);  // this thread's words have landed
    __syncthreads();
    if (tid == 0) retire_new_token(a, unit);
  }
}

// The handed-over words of a unit's new token, read by one whole wave: lane l
// gets words l (key codes in lanes 0 .., value codes in lanes 32 ..), and
// every lane the scale and the scalar-arm word in their formats.  False if
// some are not there yet.
template <int L, bool KS, bool SQ>
__device__ __forceinline__ bool take_new_token(const DecodeArgs &a, const int unit, const int lane, uint32_t &code,
                                               uint32_t &scale, uint32_t &sq) {
  const uint64_t *xn = a.xnew + static_cast<size_t>(unit) * 8 * 32;
  const int w = (lane & 32) + (lane & (L - 1));
  for (int n = 1;; ++n) {
    const uint64_t c = lut::get_word(xn + w);
    uint64_t ks = 0, vq = 0;
    bool ready = lut::word_ready(a.epoch, c);
    if constexpr (KS) {
      ks = lut::get_word(xn + kWordScale);
      ready = ready && lut::word_ready(a.epoch, ks);
    }
    if constexpr (SQ) {
      vq = lut::get_word(xn + kWordSq);
      ready = ready && lut::word_ready(a.epoch, vq);
    }
    if (__all(ready)) {
      code = static_cast<uint32_t>(c) & 0xffu;
      scale = static_cast<uint32_t>(ks);
      sq = static_cast<uint32_t>(vq);
      return true;
    }
    if (n >= a.new_polls) return false;
    __builtin_amdgcn_s_sleep(2);
  }
}

// The same values formed by the reading wave itself, where its encoder has not
// delivered them: fp64 sums and distances as in encode_block.h, one group after
// the other.  It stores nothing; the encoder workgroup does, before the launch
// ends.
__device__ __forceinline__ double lane_f64(const double x, const int l) {  // uniform l
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(x));
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), l);
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}
struct TokenInputs {  // of one (sequence, KV head)
  const void *x[2], *t[2], *cb[2];  // key and value: row, transform, codebook of the KV head
  const float *kbar;
  int bf16;
};
struct TokenValues {  // as take_new_token hands them out
  uint32_t code, scale, sq;
};
template <int D, bool KS, bool FP8, bool SQ, bool TBF>
__device__ __forceinline__ TokenValues form_new_token(const TokenInputs in, const int lane) {
  constexpr int L = D / kGroupDim;
  uint32_t code = 0, scale = 0, sq = 0;
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    const bool key = side == 0;
    const void *src = key ? in.x[0] : in.x[1], *tm = key ? in.t[0] : in.t[1], *cb = key ? in.cb[0] : in.cb[1];
    auto element = [&](const int d) {  // element lane + d, minus k_bar for keys
      const double x = in.bf16 ? static_cast<double>(bf16_bits_to_float(static_cast<const uint16_t *>(src)[lane + d]))
                               : static_cast<double>(static_cast<const float *>(src)[lane + d]);
      return key ? x - static_cast<double>(in.kbar[lane + d]) : x;
    };
    // coefficients lane and, at head_dim 128, lane + 64 (else u1 = u0)
    double u0 = 0.0, u1 = 0.0;
    auto rows = [&](const double x, const int first) {
#pragma unroll 4
      for (int r = 0; r < 64; ++r) {
        const double xr = lane_f64(x, r);
        const size_t row = static_cast<size_t>(first + r) * D + lane;
        u0 = fma(xr, static_cast<double>(t1_value(tm, row, TBF)), u0);
        if constexpr (D == 128) u1 = fma(xr, static_cast<double>(t1_value(tm, row + 64, TBF)), u1);
      }
    };
    rows(element(0), 0);
    if constexpr (D == 128) rows(element(64), 64);
    else u1 = u0;
    if (!key && SQ) {
      double mn = fmin(u0, u1), mx = fmax(u0, u1);
      for (int o = 32; o > 0; o >>= 1) {
        mn = fmin(mn, __shfl_xor(mn, o, 64));
        mx = fmax(mx, __shfl_xor(mx, o, 64));
      }
      const uint16_t zb = encblk::bf16_of(mn), sb = encblk::bf16_of((mx - mn) / 3.0);
      const double zero = bf16_bits_to_float(zb), sc = bf16_bits_to_float(sb);
      sq = sb | (static_cast<uint32_t>(zb) << 16);
      auto level = [&](const double u) {
        return sc > 0.0 ? static_cast<uint32_t>(fmin(fmax(rint((u - zero) / sc), 0.0), 3.0)) : 0u;
      };
      const uint32_t q0 = level(u0), q1 = level(u1);
      uint32_t byte = 0u;  // of group lane mod L
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = 4 * (lane & (L - 1)) + j;
        const uint32_t l0 = __shfl(q0, c & 63, 64), l1 = __shfl(q1, c & 63, 64);
        byte |= (c < 64 ? l0 : l1) << (2 * j);
      }
      if (lane >= 32) code = byte;
      continue;
    }
    if (key && KS) {
      double n2 = D == 128 ? u0 * u0 + u1 * u1 : u0 * u0;
      for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o, 64);
      const double rho = sqrt(n2) / sqrt(static_cast<double>(D));
      scale = encblk::bf16_of(rho);
      u0 = rho > 0.0 ? u0 / rho : 0.0;
      u1 = rho > 0.0 ? u1 / rho : 0.0;
    }
    // nearest codeword of each group: lane l takes codewords 4 l .. 4 l + 3
#pragma unroll 1
    for (int g = 0; g < L; ++g) {
      double v[4], best = INFINITY;
      int arg = 4 * lane;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = lane_f64(g >= 16 ? u1 : u0, (4 * g + i) & 63);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma clang fp contract(off)
        const uint2 w = codeword(cb, FP8, static_cast<size_t>(g) * kCodebookSize + 4 * lane + j);
        const double e0 = v[0] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.x & 0xffff)));
        const double e1 = v[1] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.x >> 16)));
        const double e2 = v[2] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.y & 0xffff)));
        const double e3 = v[3] - static_cast<double>(half_bits_to_float(static_cast<uint16_t>(w.y >> 16)));
        const double dist = e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
        if (dist < best) {
          best = dist;
          arg = 4 * lane + j;
        }
      }
      for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o, 64);
        const int oa = __shfl_xor(arg, o, 64);
        if (ob < best || (ob == best && oa < arg)) {
          best = ob;
          arg = oa;
        }
      }
      if ((lane & (L - 1)) == g && (lane >= 32) == !key) code = static_cast<uint32_t>(arg);
    }
  }
  return TokenValues{code, scale, sq};
}
template <int D, bool TBF>
__device__ __forceinline__ TokenInputs token_inputs(const DecodeArgs &a, const int b, const int kv) {
  const size_t row = (static_cast<size_t>(b) * a.num_kv_heads + kv) * D * (a.new_bf16 ? 2 : 4);
  const size_t cw = static_cast<size_t>(kv) * (D / kGroupDim) * kCodebookSize;
  return TokenInputs{{static_cast<const uint8_t *>(a.k_new) + row, static_cast<const uint8_t *>(a.v_new) + row},
                     {transform_of(a.t_k, kv, D, TBF), transform_of(a.t_v, kv, D, TBF)},
                     {codebook_from(a.cb_k, a.cb_fp8, cw), codebook_from(a.cb_v, a.cb_fp8, cw)},
                     a.kbar + kv * D, a.new_bf16};
}

}  // namespace step
}  // namespace novakv

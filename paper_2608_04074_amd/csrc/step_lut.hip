// The head_dim-128 table kernel (decode_lut_d128.h) as a step whose token is
// encoded by workgroups of the launch.
#include "decode_lut_d128.h"

namespace novakv {

namespace {

// The step with its encoder in n_enc workgroups of the launch: without a band
// the first ones (a multiple of 8, so the others keep their XCDs), which a
// decoding workgroup may wait for; with one the last ones.
template <int WAVES, bool KS, bool FP8, bool SQ, bool TBF, bool BAND>
__global__ void __launch_bounds__(WAVES * 64) step_lut_d128(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes<WAVES, false>()];
  constexpr int TEAMS = WAVES / 4;
  static_assert(TEAMS * (sizeof(step::Scratch<kD>) + step::kWide + 4) <= lds_bytes<WAVES, false>(), "team scratch");
  const int n_main = static_cast<int>(gridDim.x) - a.n_enc;
  const int wg = static_cast<int>(blockIdx.x);
  if (BAND ? wg >= n_main : wg < a.n_enc) {
    const int bsz = a.layout.block_size;
    const int bs_shift = (bsz & (bsz - 1)) == 0 ? __builtin_ctz(bsz) : -1;
    step::encode_workgroup<kD, TEAMS, KS, FP8, SQ, TBF, !BAND>(
        a, smem, BAND ? wg - n_main : wg, [&](const int b, const int kv, const int p) {
          return subtile_offset(a, b, kv, p & ~15, bs_shift) + static_cast<size_t>(p & 15) * kL;
        });
    return;
  }
  unit_pass<WAVES, false, KS, FP8, SQ, false, TBF, BAND ? step::kNewBand : step::kNewCodes>(
      a, smem, BAND ? wg : wg - a.n_enc, n_main);
}

template <bool KS, bool SQ, bool TBF>
void launch_step_d128(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  if (a.band_k)
    a.cb_fp8 ? step_lut_d128<12, KS, true, SQ, TBF, true><<<grid, block, 0, stream>>>(a)
             : step_lut_d128<12, KS, false, SQ, TBF, true><<<grid, block, 0, stream>>>(a);
  else
    a.cb_fp8 ? step_lut_d128<12, KS, true, SQ, TBF, false><<<grid, block, 0, stream>>>(a)
             : step_lut_d128<12, KS, false, SQ, TBF, false><<<grid, block, 0, stream>>>(a);
}

template <bool TBF>
void launch_step_storage(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  if (a.v_sq)
    a.k_scales ? launch_step_d128<true, true, TBF>(a, grid, block, stream)
               : launch_step_d128<false, true, TBF>(a, grid, block, stream);
  else
    a.k_scales ? launch_step_d128<true, false, TBF>(a, grid, block, stream)
               : launch_step_d128<false, false, TBF>(a, grid, block, stream);
}

}  // namespace

hipError_t launch_step_lut(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  a.t_bf16 ? launch_step_storage<true>(a, grid, block, stream) : launch_step_storage<false>(a, grid, block, stream);
  return hipGetLastError();
}

}  // namespace novakv

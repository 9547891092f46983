// The head_dim-64 table kernel (decode_lut_d64.h): the decode, and the step with
// a band whose token the first split to arrive encodes.
#include "decode_lut_d64.h"

namespace novakv {

namespace {

template <int WAVES, bool KS, bool FP8, bool SQ, bool BSTEP, bool TBF>
__global__ void __launch_bounds__(WAVES * 64) decode_lut_d64(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes<WAVES>()];
  unit_pass<WAVES, KS, FP8, SQ, BSTEP, TBF, step::kNewNone>(a, smem, blockIdx.x, gridDim.x);
}

}  // namespace

template <bool BSTEP, bool TBF>
void launch_d64(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  constexpr int W = 16;
  if (a.v_sq) {  // the scalar value arm (keys in either codebook format)
    if (a.k_scales)
      a.cb_fp8 ? decode_lut_d64<W, true, true, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a)
               : decode_lut_d64<W, true, false, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
    else
      a.cb_fp8 ? decode_lut_d64<W, false, true, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a)
               : decode_lut_d64<W, false, false, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
  } else if (a.k_scales) {
    a.cb_fp8 ? decode_lut_d64<W, true, true, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a)
             : decode_lut_d64<W, true, false, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
  } else {
    a.cb_fp8 ? decode_lut_d64<W, false, true, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a)
             : decode_lut_d64<W, false, false, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
  }
}

hipError_t launch_decode_lut64(const DecodeArgs &a, hipStream_t stream) {
  // 16 waves, 4 per SIMD: the kernel fits in 128 VGPRs.  A step (append) runs
  // here only with a band whose recent part holds the new token (its encoder then
  // in the first split to arrive), or with encoder workgroups.
  if (a.n_enc > 0 ? (!a.append || a.n_enc % 8 != 0 || (a.band_k && a.n_rec < 1))
                  : (a.append && !(a.band_k && a.n_rec >= 1)))
    return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(a.batch * a.num_kv_heads * a.n_split + a.n_enc));
  const dim3 block(16 * 64);
  if (a.n_enc > 0) return launch_step_lut64(a, grid, block, stream);
  if (a.t_bf16)
    a.append ? launch_d64<true, true>(a, grid, block, stream) : launch_d64<false, true>(a, grid, block, stream);
  else
    a.append ? launch_d64<true, false>(a, grid, block, stream) : launch_d64<false, false>(a, grid, block, stream);
  return hipGetLastError();
}

}  // namespace novakv

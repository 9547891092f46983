// The head_dim-128 table kernel (decode_lut_d128.h): the decode, and the step
// whose token the splits' teams encode.
#include "decode_lut_d128.h"

namespace novakv {

namespace {

template <int WAVES, bool APPEND, bool KS, bool FP8, bool SQ, bool BSTEP, bool TBF>
__global__ void __launch_bounds__(WAVES * 64) decode_lut_d128(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[lds_bytes<WAVES, APPEND>()];
  unit_pass<WAVES, APPEND, KS, FP8, SQ, BSTEP, TBF, step::kNewNone>(a, smem, blockIdx.x, gridDim.x);
}

}  // namespace

template <bool APPEND, bool KS, bool BSTEP, bool TBF>
void launch_d128(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  constexpr int W = 12;
  if (a.v_sq) {
    if (a.cb_fp8)
      decode_lut_d128<W, APPEND, KS, true, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
    else
      decode_lut_d128<W, APPEND, KS, false, true, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
  } else {
    if (a.cb_fp8)
      decode_lut_d128<W, APPEND, KS, true, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
    else
      decode_lut_d128<W, APPEND, KS, false, false, BSTEP, TBF><<<grid, block, 0, stream>>>(a);
  }
}

template <bool TBF>
void launch_d128_storage(const DecodeArgs &a, const dim3 grid, const dim3 block, hipStream_t stream) {
  if (a.append && a.band_k)
    a.k_scales ? launch_d128<true, true, true, TBF>(a, grid, block, stream)
               : launch_d128<true, false, true, TBF>(a, grid, block, stream);
  else if (a.append)  // plain or fp8 codebooks (checked by the caller)
    a.cb_fp8 ? decode_lut_d128<12, true, false, true, false, false, TBF><<<grid, block, 0, stream>>>(a)
             : decode_lut_d128<12, true, false, false, false, false, TBF><<<grid, block, 0, stream>>>(a);
  else
    a.k_scales ? launch_d128<false, true, false, TBF>(a, grid, block, stream)
               : launch_d128<false, false, false, TBF>(a, grid, block, stream);
}

hipError_t launch_decode_lut(const DecodeArgs &a, hipStream_t stream) {
  // A fused step in the key-scale or scalar value format, or with a band,
  // attends its new token as the band's last row: it needs a recent band.
  // Encoder workgroups serve any format, without a band or with such a one.
  if (a.n_enc > 0 ? (!a.append || a.n_enc % 8 != 0 || (a.band_k && a.n_rec < 1))
                  : (a.append && (a.k_scales || a.v_sq || a.band_k) && !(a.band_k && a.n_rec >= 1)))
    return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(a.batch * a.num_kv_heads * a.n_split + a.n_enc));
  const dim3 block(12 * 64);
  if (a.n_enc > 0) return launch_step_lut(a, grid, block, stream);
  a.t_bf16 ? launch_d128_storage<true>(a, grid, block, stream) : launch_d128_storage<false>(a, grid, block, stream);
  return hipGetLastError();
}

}  // namespace novakv

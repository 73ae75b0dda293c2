// The gated form of the stream GEMM (gemm_stream.h): silu(gate) * up of a fused gate / up projection, in BF16.
#include "gemm_stream.h"

namespace amx {

hipError_t launch_gemm_stream_glu(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                                  const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                                  const uint8_t* B_scales, void* out_bf16, int64_t ld_out, hipStream_t s,
                                  const KernelTimer& timer) {
  if (N % 64 != 0) return hipErrorInvalidValue;
  return stream_launch<true>(scale_kind, asym, group_size, M, N, K, A_codes, A_scales, B_codes, B_scales, nullptr, nullptr,
                             reinterpret_cast<float*>(out_bf16), ld_out, 1, s, timer);
}

}  // namespace amx

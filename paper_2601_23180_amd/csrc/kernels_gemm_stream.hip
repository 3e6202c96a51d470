// Streaming kernel (gemm_stream.hpp): residual products, the adapter's plain product and the LM head of odd widths.
#include "gemm_stream.hpp"

namespace ts {

void launch_gemm_stream_qkv(hipStream_t st, const GemmArgs &a);      // kernels_gemm_stream_qkv.hip
void launch_gemm_stream_swiglu(hipStream_t st, const GemmArgs &a);   // kernels_gemm_stream_swiglu.hip

void launch_gemm_stream(hipStream_t st, const GemmArgs &a) {
  switch (a.epi) {
    case EPI_QKV: launch_gemm_stream_qkv(st, a); break;
    case EPI_SWIGLU: launch_gemm_stream_swiglu(st, a); break;
    case EPI_RESID: dispatch_rows<EPI_RESID>(st, a); break;
    case EPI_PLAIN: dispatch_rows<EPI_PLAIN>(st, a); break;
    default: dispatch_rows<EPI_HEAD>(st, a); break;
  }
}

}  // namespace ts

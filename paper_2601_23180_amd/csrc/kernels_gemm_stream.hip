// Streaming kernel (gemm_stream.hpp): residual products, the adapter's plain product and the LM head of odd widths.
#include "gemm_stream.hpp"

namespace ts {

bool launch_gemm_stream_qkv(hipStream_t st, const GemmArgs &a);      // kernels_gemm_stream_qkv.hip
bool launch_gemm_stream_swiglu(hipStream_t st, const GemmArgs &a);   // kernels_gemm_stream_swiglu.hip

bool launch_gemm_stream(hipStream_t st, const GemmArgs &a) {
  switch (a.epi) {
    case EPI_QKV: return launch_gemm_stream_qkv(st, a);
    case EPI_SWIGLU: return launch_gemm_stream_swiglu(st, a);
    case EPI_RESID: return dispatch_rows<EPI_RESID>(st, a);
    case EPI_PLAIN: return dispatch_rows<EPI_PLAIN>(st, a);
    default: return dispatch_rows<EPI_HEAD>(st, a);
  }
}

}  // namespace ts

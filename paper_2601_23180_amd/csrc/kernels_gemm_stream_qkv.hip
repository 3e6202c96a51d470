// Streaming kernel (gemm_stream.hpp): QKV projections.
#include "gemm_stream.hpp"

namespace ts {

bool launch_gemm_stream_qkv(hipStream_t st, const GemmArgs &a) { return dispatch_rows<EPI_QKV>(st, a); }

}  // namespace ts

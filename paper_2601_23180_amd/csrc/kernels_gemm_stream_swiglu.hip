// Streaming kernel (gemm_stream.hpp): gate + up products.
#include "gemm_stream.hpp"

namespace ts {

bool launch_gemm_stream_swiglu(hipStream_t st, const GemmArgs &a) { return dispatch_rows<EPI_SWIGLU>(st, a); }

}  // namespace ts

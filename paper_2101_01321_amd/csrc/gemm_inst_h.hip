// Persistent MatMul (gemm_stream.h): 256 x 192 tiles.
#include "gemm_stream.h"

namespace ibert {
template int launch_stream<256, 192, 8, false>(GemmArgs&, bool, hipStream_t);
template int launch_stream<256, 192, 8, true>(GemmArgs&, bool, hipStream_t);
}  // namespace ibert

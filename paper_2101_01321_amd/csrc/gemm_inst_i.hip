// Few-token MatMul (gemm_few.h).
#include "gemm_few.h"

namespace ibert {
template int launch_few<1, 1, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<1, 1, true>(const GemmArgs&, bool, hipStream_t);
template int launch_few<1, 2, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<1, 2, true>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 2, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 2, true>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 4, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 4, true>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 6, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<2, 6, true>(const GemmArgs&, bool, hipStream_t);
template int launch_few<4, 4, false>(const GemmArgs&, bool, hipStream_t);
template int launch_few<4, 4, true>(const GemmArgs&, bool, hipStream_t);
}  // namespace ibert

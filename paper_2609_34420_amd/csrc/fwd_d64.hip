// bf16 forward at head dim 64.
#include "fwd_mfma.hpp"

namespace gt {
template hipError_t launch_fwd_mfma<64, 64, false>(const FwdArgs&, hipStream_t);
template hipError_t launch_fwd_mfma<64, 64, true>(const FwdArgs&, hipStream_t);
}  // namespace gt

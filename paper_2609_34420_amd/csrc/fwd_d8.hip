// bf16 forward at head dim 8, on 32-wide tiles whose extra features are zero.
#include "fwd_mfma.hpp"

namespace gt {
template hipError_t launch_fwd_mfma<32, 8, false>(const FwdArgs&, hipStream_t);
template hipError_t launch_fwd_mfma<32, 8, true>(const FwdArgs&, hipStream_t);
}  // namespace gt

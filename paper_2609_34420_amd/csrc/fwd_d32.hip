// bf16 forward at head dim 32.
#include "fwd_mfma.hpp"

namespace gt {
template hipError_t launch_fwd_mfma<32, 32, false>(const FwdArgs&, hipStream_t);
template hipError_t launch_fwd_mfma<32, 32, true>(const FwdArgs&, hipStream_t);
}  // namespace gt

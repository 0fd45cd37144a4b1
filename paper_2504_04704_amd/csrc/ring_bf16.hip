// The ring kernel for bf16 (see ring_pass.hpp).
#include "ring_pass.hpp"

namespace lagkv {

hipError_t launch_ring_bf16(const PassArgs& a, hipStream_t s) { return launch_ring_t<BF16>(a, s); }
hipError_t launch_direct_bf16(const PassArgs& a, hipStream_t s) { return launch_direct_t<BF16>(a, s); }

}  // namespace lagkv

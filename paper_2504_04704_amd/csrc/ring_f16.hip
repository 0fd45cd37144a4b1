// The ring kernel for f16 (see ring_pass.hpp).
#include "ring_pass.hpp"

namespace lagkv {

hipError_t launch_ring_f16(const PassArgs& a, hipStream_t s) { return launch_ring_t<F16>(a, s); }
hipError_t launch_direct_f16(const PassArgs& a, hipStream_t s) { return launch_direct_t<F16>(a, s); }

}  // namespace lagkv

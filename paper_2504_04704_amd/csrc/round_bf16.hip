// The single-round append kernel for one element type (a file each, so that they compile side by side).
#include "round_pass.hpp"

namespace lagkv {

hipError_t launch_round_bf16(const AppendArgs& a, hipStream_t s) { return launch_round_t<BF16>(a, s); }

}  // namespace lagkv

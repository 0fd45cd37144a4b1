// The chunk-at-a-time kernel for one element type (a file each, so that they compile side by side).
#include "chunk_pass.hpp"

namespace lagkv {

hipError_t launch_chunk_f16(const PassArgs& a, hipStream_t s) { return launch_chunk_t<F16>(a, s); }

}  // namespace lagkv

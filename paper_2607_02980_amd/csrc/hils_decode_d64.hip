// The decode kernels of head dim 64 (one source per head dim, compiled side by side).
#include "hils_decode.hpp"

namespace hils {

hipError_t launch_decode_d64(const FwdArgs& a, hipStream_t s) { return dispatch_decode<64>(a, s); }

}  // namespace hils

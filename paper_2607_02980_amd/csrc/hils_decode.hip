// Host side of the decode forward: workspace size and dispatch over the head dim.
#include "hils_decode_layout.hpp"

namespace hils {

// Compute units of the current device (a host-side attribute query; nothing cached).
int device_cus() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
        return 256;
    return n;
}


size_t decode_workspace_bytes(int B, int N, int Hkv, int G, int d, int L, int K, int W, int head_norm) {
    return dec_layout(B, N, Hkv, G, d, L, K, W, head_norm).total;
}

hipError_t launch_decode_fwd(const FwdArgs& a, hipStream_t s) {
    if (a.d == 64) return launch_decode_d64(a, s);
    if (a.d == 128) return launch_decode_d128(a, s);
    return hipErrorInvalidValue;
}

}  // namespace hils

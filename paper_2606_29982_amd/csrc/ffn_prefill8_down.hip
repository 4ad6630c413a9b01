// The down kernel of the 8-bit prefill products (ffn_prefill8.h).
#include "ffn_prefill8.h"

namespace caee {

hipError_t launch_prefill8_down(const FfnParams& p, unsigned workgroups, hipStream_t s) {
    ffn_launch(k_prefill8<false>, dim3(workgroups), dim3(kP8Threads), s, p);
    return hipGetLastError();
}

}  // namespace caee

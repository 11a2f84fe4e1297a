// Decode kernels: shift-accumulate scores, fp16 values.
#include "decode_kernel.hpp"

namespace potattn {

template hipError_t launch_mode_vf<kScorePot, 0>(int, int, bool, const DecodeArgs&, hipStream_t,
                                                 hipEvent_t, hipEvent_t);

}  // namespace potattn

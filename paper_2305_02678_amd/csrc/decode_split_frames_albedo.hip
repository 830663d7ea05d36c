// The split FP32 decode (decode_split.h): variants with learned frames and the albedo head.
#include "decode_split.h"

namespace nam {

hipError_t dispatch_split_frames_albedo(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s) {
    return dispatch_split_filter<true, true>(sh, a, cu, s);
}

}  // namespace nam

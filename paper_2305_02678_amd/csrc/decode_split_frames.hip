// The split FP32 decode (decode_split.h): variants with learned frames.
#include "decode_split.h"

namespace nam {

hipError_t dispatch_split_frames(const MlpShape& sh, SplitArgs& a, int cu, hipStream_t s) {
    return dispatch_split_filter<true, false>(sh, a, cu, s);
}

}  // namespace nam

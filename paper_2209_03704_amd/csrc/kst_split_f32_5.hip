// The 5 x 5 kernels of kst_split_f32.h (a file per kernel edge: they compile side by side).
#include "kst_split_f32.h"

namespace kst {

hipError_t launch_split_f32_5(const float *in, const float *w_seg, float *out, void *ws, const Shape &s, hipStream_t stream)
{
    const SplitPlan r = split_plan(s);
    return r.ok ? split_f32_launch_n<5>(in, w_seg, out, (char *)ws, r, stream) : hipErrorInvalidValue;
}

}  // namespace kst

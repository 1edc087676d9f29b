// The 3 x 3 kernels of kst_fwd_packed.h (a file per kernel edge: they compile side by side).
#include "kst_fwd_packed.h"

namespace kst {

hipError_t launch_packed_f32_3(const float *in, const float *w_seg, float *out, void *ws, const Shape &s, hipStream_t stream)
{
    const FwdPackedPlan r = fwd_packed_plan(s);
    return r.ok ? fwd_packed_launch_any<3>(in, w_seg, out, ws, r, stream) : hipErrorInvalidValue;
}

}  // namespace kst

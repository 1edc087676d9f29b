// The 3 x 3 kernels of kst_din_packed.h (a file per kernel edge: they compile side by side).
#include "kst_din_packed.h"

namespace kst {

hipError_t launch_din_packed_3(const float *g, const void *w, float *din, void *ws, const Shape &s, bool odd, kst_dtype dt,
                               hipStream_t stream)
{
    const DinPackedPlan r = din_packed_plan(s, odd, dt);
    return r.ok ? din_packed_launch_any<3>(g, w, din, ws, r, dt, stream) : hipErrorInvalidValue;
}

}  // namespace kst

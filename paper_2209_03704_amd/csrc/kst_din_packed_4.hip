// The 4 x 4 kernels of kst_din_packed.h (a file per kernel edge: they compile side by side).
#include "kst_din_packed.h"

namespace kst {

hipError_t launch_din_packed_4(const float *g, const void *w, float *din, void *ws, const Shape &s, bool odd, kst_dtype dt,
                               hipStream_t stream)
{
    const DinPackedPlan r = din_packed_plan(s, odd, dt);
    return r.ok ? din_packed_launch_any<4>(g, w, din, ws, r, dt, stream) : hipErrorInvalidValue;
}

// Which layers (those of kst_split_din.hip come first): either side timed on 150 random layers of 0.005 to 1.3 G products.
// Two exceptions lost: the pipelined fp32 kernel (fp32 weights, maps and channels of whole groups of four, even padding
// factor) is 3 to 12 % faster where its tiles of 128 input channels are mostly real (1 x 768 x 96 x 12 x 12, n = 4, P = 2:
// 21.7 us there, 24.5 here; with 64 of 128 channels real this one gains 1.4), and few channels on both sides leave
// little besides the launches (2 x 33 x 3 x 44 x 44, n = 5: 10.0 us there, 12.3 here).
bool din_packed_applies(const Shape &s, bool odd, kst_dtype dt)
{
    if (s.n < 3 || s.n > 5 || s.Cin < 8) return false;
    const double edge = s.N - 2 * s.frame;
    const double products = (double)s.B * edge * edge * s.n * s.n * s.Cin * s.Cout;
    if (products < 0.005e9 || (s.Cout <= 4 && s.Cin < 64 && products < 0.05e9)) return false;
    const bool pipelined = dt == KST_F32 && !odd && (s.M & 3) == 0 && (s.Cin & 3) == 0 && (s.Cout & 3) == 0;
    if (pipelined && 2 * ((s.Cin + 127) / 128 * 128) < 3 * s.Cin) return false;
    return din_packed_plan(s, odd, dt).ok;
}

// (0 for a layer these kernels do not take)
size_t din_packed_workspace_bytes(const Shape &s, bool odd, kst_dtype dt)
{
    const DinPackedPlan r = din_packed_plan(s, odd, dt);
    return r.ok ? r.g_bytes + r.w_bytes + r.part_bytes : 0;
}

hipError_t launch_din_packed(const float *g, const void *w, float *din, void *ws, const Shape &s, bool odd, kst_dtype dt,
                             hipStream_t stream)
{
    switch (s.n) {
        case 3: return launch_din_packed_3(g, w, din, ws, s, odd, dt, stream);
        case 4: return launch_din_packed_4(g, w, din, ws, s, odd, dt, stream);
        case 5: return launch_din_packed_5(g, w, din, ws, s, odd, dt, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kst

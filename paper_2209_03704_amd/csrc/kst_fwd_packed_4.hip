// The 4 x 4 kernels of kst_fwd_packed.h (a file per kernel edge: they compile side by side).
#include "kst_fwd_packed.h"

namespace kst {

hipError_t launch_packed_f32_4(const float *in, const float *w_seg, float *out, void *ws, const Shape &s, hipStream_t stream)
{
    const FwdPackedPlan r = fwd_packed_plan(s);
    return r.ok ? fwd_packed_launch_any<4>(in, w_seg, out, ws, r, stream) : hipErrorInvalidValue;
}

// Which layers (those of kst_split_f32.hip come first): either side timed on 110 random layers of up to 4 G products.  Layers
// of few positions below 0.2 G products stay with the position-block kernel, which reads everything once (9 x 304 x 56 x 6 x
// 6, n = 4, P = 2: 17 us there, 24 here).  With up to four output channels the passes over the input are what counts: what
// they write is six bytes a value where the other kernels read four, and on large inputs that is not won back (121 x 189 x
// 3 x 41 x 41, n = 4, P = 3: 180 us there, 247 here); the direct kernel takes about 100 us per G products and at least 0.01 us
// per kernel element and input channel, which it walks one after the other (141 x 440 x 3 x 7 x 7, n = 5, P = 3, 0.2 G
// products: 227 us there).  Fewer than 128 input channels are few such steps (61 x 23 x 3 x 34 x 34: 14 us there, 23 here).
bool packed_f32_applies(const Shape &s)
{
    if (s.lean || s.n < 3 || s.n > 5 || s.Cin < 8 || split_f32_applies(s)) return false;
    const double products = (double)s.B * s.E * s.E * s.n * s.n * s.Cin * s.Cout;
    if (products < (s.Cout > 4 ? 0.02e9 : 0.01e9) || (products < 0.2e9 && igemm_f32_small_supported(s))) return false;
    if (s.Cout <= 4 && (s.Cin < 128 || tapmajor_f32_supported(s))) return false;
    const FwdPackedPlan r = fwd_packed_plan(s);
    if (!r.ok || s.Cout > 4) return r.ok;
    const double walk = 6.0 + 0.01 * s.n * s.n * s.Cin, there = 10.0 + products * 1.0e-7;
    return r.us < 0.9 * (there > walk ? there : walk);
}

size_t packed_f32_workspace_bytes(const Shape &s)
{
    const FwdPackedPlan r = fwd_packed_plan(s);
    return r.ok ? r.x_bytes + r.w_bytes + r.part_bytes : 0;
}

hipError_t launch_packed_f32(const float *in, const float *w_seg, float *out, void *ws, const Shape &s, hipStream_t stream)
{
    switch (s.n) {
        case 3: return launch_packed_f32_3(in, w_seg, out, ws, s, stream);
        case 4: return launch_packed_f32_4(in, w_seg, out, ws, s, stream);
        case 5: return launch_packed_f32_5(in, w_seg, out, ws, s, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kst

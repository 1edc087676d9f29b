// Which layers the kernels of kst_split_f32.h run, their workspace and their launch.
#include "kst_split_f32.h"

namespace kst {

bool split_f32_applies(const Shape &s)
{
    if (s.lean || s.n < 3 || s.n > 5 || s.Cout < 16 || s.Cin <= S_KC) return false;   // (a plan's integers hold such kernels)
    const double products = (double)s.B * s.E * s.E * s.n * s.n * s.Cin * s.Cout;
    if (products < 1.5e9) return false;
    // Both sides timed on 1650 random layers of 1.5 to 12 G products (n = 3 .. 5, maps of 4 to 64, 17 to 1024 channels).
    // Where the plain fp32 kernel is the other one (channels no whole groups of four or, unframed, columns) this one was
    // at least 1.4 times as fast on all 730 of them.
    const SplitPlan r = split_plan(s);
    const bool pipelined = (s.Cin & 3) == 0 && (s.Cout & 3) == 0 && (s.frame > 0 || (s.N & 3) == 0);
    if (!pipelined || !r.ok) return r.ok;
    // The pipelined fp32 kernel is another matter.  Passes of fewer than eight channel chunks keep their first and last
    // ones in view: 23 of 67 such layers lost, at any size (10 x 96 x 192 x 64 x 64, n = 3, P = 2, 7 G products: 180 us
    // here against 145): not for this kernel.  With eight and more, none of 200 layers from 4 G products lost.  Below that both
    // times are known well enough to compare: here (within 5 % on 561 layers) a launch chain of 13 us, 0.5 per kernel
    // tap and chunk of a workgroup's share, 0.9 per million weights to split, 17.6 per piece of its share (filling the
    // pipeline, storing) and 0.6 per workgroup that adds to a pass; there 22 and 17.2 per G products of whole tiles.
    // From 1.5 G products 58 of 495 were slower here than there, by up to a third; of those this keeps 11 are, by up to 9 %.
    // (The times here are those of three parts.  Layers planned for two take 0.75 to 0.97 of them, the ranges' pass included: of
    // 120 such layers of 1.5 to 5 G products all ran 1.8 to 2.4 times as fast as there, and the rule takes every one.)
    if (s.Cin < 8 * S_KC) return false;
    if (products >= 4.0e9) return true;
    const EvenShares &k = r.k;
    const double shares = (double)k.rounds * k.grid + k.passes;                  // passes of both parities
    const double units = shares * r.p.chunks * (s.n * s.n) / 2 / S_GRID;
    const double pieces = k.rounds + (k.passes ? (double)k.passes / S_GRID + 1.0 : 0.0);
    const double here = 13.0 + 0.5 * units + 0.9e-6 * (r.p.w_bytes / 6) + 17.6 * pieces +
                        (k.passes ? 0.6 * S_GRID / k.passes : 0.0);
    const double tiles = (double)((r.p.Mtot + 127) / 128) * 128 * ((s.Cout + 63) / 64 * 64);
    const double there = 22.0 + 17.2e-9 * tiles * s.n * s.n * s.Cin + (s.frame > 0 && (r.p.N0 & 3) != 0 ? 4.0 : 0.0);
    return there > 1.02 * here;
}

size_t split_f32_workspace_bytes(const Shape &s)
{
    const SplitPlan r = split_plan(s);
    return split_weight_bytes(r) + (size_t)r.k.slots() * S_SLOT * sizeof(float);
}

hipError_t launch_split_f32(const float *in, const float *w_seg, float *out, void *ws, const Shape &s, hipStream_t stream)
{
    switch (s.n) {
        case 3: return launch_split_f32_3(in, w_seg, out, ws, s, stream);
        case 4: return launch_split_f32_4(in, w_seg, out, ws, s, stream);
        case 5: return launch_split_f32_5(in, w_seg, out, ws, s, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kst

// fp32 products on the bf16 matrix cores: pieces shared by the forward and the gradient kernels
// that split their fp32 operands into three bfloat16 parts.
//
// v_mfma_f32_32x32x16_bf16 multiplies sixteen times what v_mfma_f32_32x32x2_f32 does in the same time
// (2.24 against 0.15 PFLOP/s measured on this chip with nothing but multiplies).  An fp32 value is the
// exact sum of three bfloat16 parts, x = x0 + x1 + x2 (rounded to nearest: |x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|),
// and a product of two such sums needs six of the nine partial products:
//     x w ~ x0 w0 + (x0 w1 + x1 w0) + (x0 w2 + x1 w1 + x2 w0)
// What is left out, x1 w2 + x2 w1 + x2 w2, is at most 2^-24 of the product, what one fp32 addition may
// be off by; every partial product is exact in fp32 and all sums are fp32 sums.
//
// bfloat16 has fp32's exponents but 16 bits less below the point, so the low parts of a small value would fall below
// its smallest step (2^-133: an operand of 1e-36 would keep 14 bits, one of 3e-38 five).  All operands are therefore
// multiplied by 2^24 before they are split, which makes every part of every fp32 value, subnormal ones too, a normal
// bfloat16 number, and the sums by 2^-48 before anything else is done with them.
//
// A value that is infinite, not a number, or rounds to infinity in bfloat16 has no such parts.  Each of them makes
// every sum it enters infinite or not a number, and so does a sum beyond fp32's largest value over 2^48; the stores
// look for sums that are not finite and take those elements from fp32 MFMAs instead: a wave multiplies a whole
// block of them again, straight from memory, in lanes that together read whole lines.  (One lane per element and one
// multiply-add at a time took up to a quarter of a million dependent steps for an element of the kernel gradient.)
#pragma once
#include "kst_igemm_common.h"

namespace kst {

constexpr float SPLIT_SCALE = 0x1p24f;                       // of both operands
constexpr float SPLIT_UNSCALE = 0x1p-48f;                    // of their products' sums

// Eight values times SPLIT_SCALE -> their three bfloat16 parts.
__device__ __forceinline__ void split3(const float (&v)[8], bf16x8 &p0, bf16x8 &p1, bf16x8 &p2)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        p0[j] = (__bf16)(v[j] * SPLIT_SCALE);
        const float r1 = fmaf(v[j], SPLIT_SCALE, -(float)p0[j]);
        p1[j] = (__bf16)r1;
        p2[j] = (__bf16)(r1 - (float)p1[j]);
    }
}

// A value that is the same in all lanes, where the compiler cannot know (arguments of a function that is not inlined).
__device__ __forceinline__ int same(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A tensor below 2 GB as a buffer: loads past its end return zero instead of touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *ptr, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(ptr), 0, (int)bytes, 0x00027000);
}
// lane_bytes: this lane's offset; wave_bytes: the same in all lanes and inside the buffer.
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, unsigned wave_bytes)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_bytes, (int)wave_bytes, 0));
}
__device__ __forceinline__ bf16x8 load_bf16x8(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, unsigned wave_bytes)
{
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, (int)wave_bytes, 0));
}

// Even shares.  The work is a list of passes (tile-major, row parity r = pass & 1) of `chunks` channel chunks, a chunk
// of parity r costing tapsr.  Workgroup g of `grid` does passes g * rounds .. + rounds - 1 whole; the (pass, chunk)
// units of the remaining passes are cut into `grid` ranges of equal cost.  A piece of a range that covers a whole pass
// is stored; any other goes to a slot and a second kernel adds a pass's slots in workgroup order.  Slots are numbered
// along the list, workgroup + shared pass (each piece is a workgroup or a pass further than the one before it), where
// that makes fewer of them than two per workgroup: 2 g for the first piece of workgroup g's range, 2 g + 1 for a later.
constexpr int S_GRID = 256;                                  // CUs of the chip
struct EvenShares {
    int chunks;                // channel chunks per pass
    int grid;                  // workgroups (<= S_GRID)
    int rounds;                // whole passes per workgroup (none unless grid == S_GRID; even where taps0 != taps1)
    int passes;                // passes that are shared
    int taps0, taps1;
    int per, more;             // cost of the list: per * grid + more, below 2^30
    __host__ __device__ int listed() const { return rounds * grid; }        // first shared pass
    __host__ __device__ bool along_list() const { return passes < grid; }
    int slots() const { return passes == 0 ? 0 : along_list() ? grid + passes - 1 : 2 * grid; }
    // Slot of workgroup g's piece of shared pass `rel`; first: its range begins in that pass.
    __device__ int slot(int g, int rel, bool first) const { return along_list() ? g + rel : 2 * g + (first ? 0 : 1); }
    // First unit of workgroup g's range.
    __host__ __device__ int begin(int g) const
    {
        const unsigned cost = (unsigned)g * per + (unsigned)g * more / (unsigned)grid;
        const unsigned pass0 = (unsigned)chunks * taps0, pair = pass0 + (unsigned)chunks * taps1;
        const unsigned both = cost / pair, rest = cost - both * pair;
        const unsigned unit = rest < pass0 ? rest / (unsigned)taps0 : (unsigned)chunks + (rest - pass0) / (unsigned)taps1;
        return (int)(both * 2u * (unsigned)chunks + unit);
    }
    // The workgroup whose range holds `unit` (begin(g) <= unit < begin(g + 1)).
    __device__ int owner(int unit) const
    {
        const int pass = unit / chunks, c = unit - pass * chunks;
        const float cost = (float)chunks * ((pass >> 1) * (taps0 + taps1) + (pass & 1) * taps0) + (float)c * (pass & 1 ? taps1 : taps0);
        int g = min((int)(cost * (float)grid / ((float)per * (float)grid + (float)more)), grid - 1);
        while (g > 0 && begin(g) > unit) --g;
        while (g + 1 < grid && begin(g + 1) <= unit) ++g;
        return g;
    }
};

}  // namespace kst

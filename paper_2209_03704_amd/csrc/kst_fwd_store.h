// Where the fp32 forward kernels on the bf16 matrix cores leave their sums: stores of finite ones, and the blocks that hold
// others again in fp32 multiplies (see kst_split_common.h).
#pragma once
#include "kst_split_common.h"

namespace kst {

namespace {

struct FwdShape {
    int B, Cin, Cout, N, M, E, EE;   // N: framed map's edge; M: edge of the planes written
    int q, N0;             // zero frame supplied here; edge of the tensor in memory (N = N0 + 2 q)
    int Mtot;
    unsigned off[4];       // element offset of W_p
    int crop;              // 1: quad members land one row and one column earlier (M is then the cropped map's edge)
    Epilogue epi;
};

// Where this lane's column of position block `blk` of the tile lies.
struct Column {
    int mb, mi, mj;
    bool valid;
};
__device__ __forceinline__ Column column_of(const FwdShape &p, int m0, int blk, int l32)
{
    Column c;
    int m = m0 + blk * 32 + l32;
    c.valid = m < p.Mtot;
    m = min(m, p.Mtot - 1);
    c.mb = m / p.EE;
    const int mrem = m - c.mb * p.EE;
    c.mi = mrem / p.E;
    c.mj = mrem - c.mi * p.E;
    return c;
}

// 32 output channels x 32 positions of one class in fp32 MFMAs, by a whole wave, where split sums are not finite.
// x: the input of the batch item of this lane's position (lane % 32); w: the class's weights (Ta x Tb taps) at this
// lane's output channel (live: there is one); (iy, ix): the window's corner in the unframed input.
__device__ __forceinline__ floatx16 fp32_block_here(const float *x, const float *w, bool live, int Cin, int Cout, int N0, int Ta,
                                                    int Tb, int iy, int ix)
{
    const int kk = (threadIdx.x >> 5) & 1;                   // an MFMA's two reduction steps: two input channels
    const size_t plane = (size_t)N0 * N0, w_plane = (size_t)Ta * Tb * Cout;
    floatx16 sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.0f;
#pragma unroll 1
    for (int t = 0; t < Ta * Tb; ++t) {
        const int y = iy + t / Tb, c = ix + t % Tb;
        const bool inside = y >= 0 && y < N0 && c >= 0 && c < N0;
        const float *px = x + (inside ? (size_t)y * N0 + c : 0) + kk * plane, *pw = w + (size_t)t * Cout + kk * w_plane;
#pragma unroll 1
        for (int c0 = 0; c0 < Cin; c0 += 8) {                // four MFMAs' operands in flight together
            float wv[4], xv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = c0 + 2 * j + kk < Cin;
                wv[j] = live && ok ? *pw : 0.0f;
                xv[j] = inside && ok ? *px : 0.0f;
                pw += 2 * w_plane;
                px += 2 * plane;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[j], xv[j], sum, 0, 0, 0);
        }
    }
    return sum;
}

// (the main kernel, whose registers are full, calls it)
__device__ __attribute__((noinline)) floatx16 fp32_block(const float *x, const float *w, bool live, int Cin, int Cout, int N0,
                                                         int Ta, int Tb, int iy, int ix)
{
    return fp32_block_here(x, w, live, same(Cin), same(Cout), same(N0), same(Ta), same(Tb), iy, ix);
}

// Class (r, s) at position c; co: this lane's output channel as a row (lane % 32) of the block.
template <int n, bool CALL>
__device__ __forceinline__ floatx16 fp32_class_block(const float *in, const float *w_seg, const FwdShape &p, const Column &c,
                                                     int r, int s, int co)
{
    const unsigned off = r ? (s ? p.off[3] : p.off[2]) : (s ? p.off[1] : p.off[0]);
    const float *x = in + (size_t)c.mb * p.Cin * p.N0 * p.N0, *w = w_seg + off + min(co, p.Cout - 1);
    const int Ta = taps_for_parity(n, r), Tb = taps_for_parity(n, s), iy = c.mi + r - p.q, ix = c.mj + s - p.q;
    if constexpr (CALL) return fp32_block(x, w, co < p.Cout, p.Cin, p.Cout, p.N0, Ta, Tb, iy, ix);
    else return fp32_block_here(x, w, co < p.Cout, p.Cin, p.Cout, p.N0, Ta, Tb, iy, ix);
}

// Store one output channel's two elements (column parities) of a lane: final values, after the epilogue.
__device__ __forceinline__ void store_pair(float *__restrict__ out, const FwdShape &p, float v0, float v1, int r, int co,
                                           const Column &c)
{
    if (epi_on(p.epi)) {
        const float bias = epi_bias(p.epi, co);
        v0 = epi_apply(v0, bias, p.epi.act);
        v1 = epi_apply(v1, bias, p.epi.act);
    }
    const int y = 2 * c.mi + r - p.crop, x = 2 * c.mj - p.crop;
    if (y < 0 || y >= p.M) return;
    float *q = out + (((size_t)c.mb * p.Cout + co) * p.M + y) * p.M + x;
    if (x >= 0 && x + 1 < p.M && (reinterpret_cast<uintptr_t>(q) & 7u) == 0) {
        *reinterpret_cast<float2 *>(q) = make_float2(v0, v1);
    } else {
        if (x >= 0 && x < p.M) q[0] = v0;
        if (x + 1 < p.M) q[1] = v1;
    }
}

}  // namespace

}  // namespace kst

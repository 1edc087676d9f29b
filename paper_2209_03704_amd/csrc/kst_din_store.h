// Where the input gradient's kernels on the bf16 matrix cores leave their sums: stores of finite ones, and the blocks that
// hold others again in fp32 multiplies (see kst_split_common.h).
#pragma once
#include "kst_split_common.h"

namespace kst {

namespace {

struct DinShape {
    int B, Cin, Cout;
    int N, M, shift;       // edges of din and g; g row of image row h: h + shift
    int Mtot;              // positions: B N N
};

__device__ __forceinline__ float weight_of(const float *w, size_t i) { return w[i]; }
__device__ __forceinline__ float weight_of(const uint16_t *w, size_t i) { return to_f32(w[i]); }
__device__ __forceinline__ float weight_of(const half_bits *w, size_t i) { return to_f32(w[i]); }

// 32 input channels x 32 positions in fp32 MFMAs, by a whole wave, where split sums are not finite.  g: of the batch
// item of this lane's position (lane % 32); w: of this lane's input channel (live: there is one); (y, x): row and column
// of g for tap (0, 0).
template <class T>
__device__ __forceinline__ floatx16 din_fp32_block_here(const float *g, const T *w, bool live, int n, int Cin, int Cout, int M,
                                                        int y, int x)
{
    const int kk = (threadIdx.x >> 5) & 1;            // an MFMA's two reduction steps: two output channels
    const size_t plane = (size_t)M * M, w_plane = (size_t)Cin * n * n;
    floatx16 sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.0f;
#pragma unroll 1
    for (int t = 0; t < n * n; ++t) {
        const int gy = y - t / n, gx = x - t % n;
        const bool inside = gy >= 0 && gy < M && gx >= 0 && gx < M;
        const float *pg = g + (inside ? (size_t)gy * M + gx : 0) + kk * plane;
        const T *pw = w + t + kk * w_plane;
#pragma unroll 1
        for (int c0 = 0; c0 < Cout; c0 += 8) {        // four MFMAs' operands in flight together
            float wv[4], gv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = c0 + 2 * j + kk < Cout;
                wv[j] = live && ok ? weight_of(pw, 0) : 0.0f;
                gv[j] = inside && ok ? *pg : 0.0f;
                pw += 2 * w_plane;
                pg += 2 * plane;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[j], gv[j], sum, 0, 0, 0);
        }
    }
    return sum;
}

// (the main kernel, whose registers are full, calls it)
template <class T>
__device__ __attribute__((noinline)) floatx16 din_fp32_block(const float *g, const T *w, bool live, int n, int Cin, int Cout,
                                                             int M, int y, int x)
{
    return din_fp32_block_here(g, w, live, same(n), same(Cin), same(Cout), same(M), y, x);
}

struct DinColumn {
    int mb, ma, mc;
    bool valid;
};
__device__ __forceinline__ DinColumn din_column(const DinShape &p, int m)
{
    DinColumn c;
    c.valid = m < p.Mtot;
    m = min(m, p.Mtot - 1);
    c.mb = m / (p.N * p.N);
    const int rem = m - c.mb * p.N * p.N;
    c.ma = rem / p.N;
    c.mc = rem - c.ma * p.N;
    return c;
}

// The 16 sums of one block (channels ci0 + 8 (v / 4) + v % 4) at this lane's position.
template <int n, bool CALL, class T>
__device__ __forceinline__ void din_store(const float *__restrict__ g, const T *__restrict__ w, float *__restrict__ din,
                                          const DinShape &p, const float (&a)[16], int ci0, const DinColumn &c)
{
    const size_t plane = (size_t)p.N * p.N;
    float *o = din + ((size_t)c.mb * p.Cin + ci0) * plane + c.ma * p.N + c.mc;
    float zero = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int d = 8 * (v >> 2) + (v & 3);
        if (c.valid && ci0 + d < p.Cin) o[d * plane] = a[v];
        zero = fmaf(a[v], 0.0f, zero);
    }
    if (__builtin_expect(__ballot(zero != 0.0f) != 0, 0)) {  // (all lanes of the wave, also those past the last position)
        const int ci = (ci0 & ~31) + (int)(threadIdx.x & 31);
        const float *gb = g + (size_t)c.mb * p.Cout * p.M * p.M;
        const T *wb = w + (size_t)min(ci, p.Cin - 1) * n * n;
        const int y = 2 * c.ma + n - 1 + p.shift, x = 2 * c.mc + n - 1 + p.shift;
        floatx16 f;
        if constexpr (CALL) f = din_fp32_block(gb, wb, ci < p.Cin, n, p.Cin, p.Cout, p.M, y, x);
        else f = din_fp32_block_here(gb, wb, ci < p.Cin, n, p.Cin, p.Cout, p.M, y, x);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int d = 8 * (v >> 2) + (v & 3);
            if (c.valid && ci0 + d < p.Cin && a[v] * 0.0f != 0.0f) o[d * plane] = f[v];
        }
    }
}

}  // namespace

}  // namespace kst

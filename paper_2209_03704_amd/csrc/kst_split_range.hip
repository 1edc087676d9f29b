// Largest and smallest magnitude of two operands and how many of their values are not zero: the scales of two half-precision
// parts, and whether the operands have them (see kst_split_common.h).
//
// What bounds it: memory, each operand read once.  256 workgroups of 512 threads, a fixed share of a tensor each, four
// 16-byte loads of a lane in flight.  128 x 512 x 16 x 16 and 256 x 512 x 4 x 4, 75 MB: 13 us (5.8 TB/s).
#include "kst_split_common.h"

namespace kst {

namespace {

__global__ void __launch_bounds__(RANGE_THREADS) split_range_kernel(RangeOperand a, RangeOperand b, int wgs_a,
                                                                    RangePart *__restrict__ to)
{
    constexpr int AT_ONCE = 4;
    const bool first = (int)blockIdx.x < wgs_a;
    const RangeOperand &o = first ? a : b;
    const size_t groups = o.count / (o.half ? 8 : 4);             // of sixteen bytes
    const int wg = first ? (int)blockIdx.x : (int)blockIdx.x - wgs_a, wgs = first ? wgs_a : RANGE_WGS - wgs_a;
    const size_t mine = (size_t)wg * RANGE_THREADS + threadIdx.x, step = (size_t)wgs * RANGE_THREADS;
    unsigned most = 0u, least = ~0u, real = 0u;
    auto take = [&](unsigned bits) {
        bits &= 0x7fffffffu;
        most = max(most, bits);
        least = min(least, bits - 1u);                            // (a zero: all ones)
        real += bits != 0u ? 1u : 0u;
    };
    auto count_two = [&](unsigned bits) { real += ((bits & 0x7fffu) != 0u ? 1u : 0u) + ((bits & 0x7fff0000u) != 0u ? 1u : 0u); };
    for (size_t g = mine; g < groups; g += AT_ONCE * step) {
        uint4 v[AT_ONCE];
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const size_t at = g + i * step;
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            if (at < groups) v[i] = static_cast<const uint4 *>(o.p)[at];
        }
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            if (o.half) {
                count_two(v[i].x);
                count_two(v[i].y);
                count_two(v[i].z);
                count_two(v[i].w);
            } else {
                take(v[i].x);
                take(v[i].y);
                take(v[i].z);
                take(v[i].w);
            }
        }
    }
    const size_t rest = groups * (o.half ? 8 : 4) + mine;         // the last few
    if (rest < o.count) {
        if (o.half) count_two(static_cast<const uint16_t *>(o.p)[rest]);
        else take(static_cast<const unsigned *>(o.p)[rest]);
    }
    __shared__ RangePart waves[RANGE_THREADS / 64];
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        most = max(most, (unsigned)__shfl_xor((int)most, d));
        least = min(least, (unsigned)__shfl_xor((int)least, d));
        real += (unsigned)__shfl_xor((int)real, d);
    }
    if ((threadIdx.x & 63) == 0) waves[threadIdx.x >> 6] = {most, least, real, 0u};
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < RANGE_THREADS / 64; ++i) {
            most = max(most, waves[i].most);
            least = min(least, waves[i].least);
            real += waves[i].real;
        }
        to[blockIdx.x] = {most, least, real, 0u};
    }
}

}  // namespace

int split_range_share(size_t bytes_a, size_t bytes_b)
{
    const int share = (int)(RANGE_WGS * ((double)bytes_a / ((double)bytes_a + (double)bytes_b)) + 0.5);
    return share < 1 ? 1 : share > RANGE_WGS - 1 ? RANGE_WGS - 1 : share;
}

hipError_t launch_split_range(const RangeOperand &a, const RangeOperand &b, void *to, hipStream_t stream)
{
    const size_t bytes_a = a.count * (a.half ? 2 : 4), bytes_b = b.count * (b.half ? 2 : 4);
    hipLaunchKernelGGL(split_range_kernel, dim3(RANGE_WGS), dim3(RANGE_THREADS), 0, stream, a, b, split_range_share(bytes_a, bytes_b),
                       (RangePart *)to);
    return hipGetLastError();
}

}  // namespace kst

// Largest and smallest magnitude of two operands: the scales of two half-precision parts, and whether they have them (see
// kst_split_common.h).
//
// What bounds it: memory, each operand read once.  256 workgroups of 512 threads, a fixed share of a tensor each, four
// 16-byte loads of a lane in flight.
#include "kst_split_common.h"

namespace kst {

namespace {

__global__ void __launch_bounds__(RANGE_THREADS) split_range_kernel(RangeOperand a, RangeOperand b, int wgs_a,
                                                                    RangePart *__restrict__ to)
{
    constexpr int AT_ONCE = 4;
    const bool first = (int)blockIdx.x < wgs_a;
    const float *__restrict__ p = first ? a.p : b.p;
    const size_t count = first ? a.count : b.count, groups = count / 4;
    const int wg = first ? (int)blockIdx.x : (int)blockIdx.x - wgs_a, wgs = first ? wgs_a : RANGE_WGS - wgs_a;
    const size_t mine = (size_t)wg * RANGE_THREADS + threadIdx.x, step = (size_t)wgs * RANGE_THREADS;
    unsigned most = 0u, least = ~0u;
    auto take = [&](unsigned bits) {
        bits &= 0x7fffffffu;
        most = max(most, bits);
        least = min(least, bits - 1u);                            // (a zero: all ones)
    };
    for (size_t g = mine; g < groups; g += AT_ONCE * step) {
        uint4 v[AT_ONCE];
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {                       // (past the last: the last one again)
            const size_t at = g + i * step;
            v[i] = *reinterpret_cast<const uint4 *>(p + 4 * (at < groups ? at : groups - 1));
        }
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            take(v[i].x);
            take(v[i].y);
            take(v[i].z);
            take(v[i].w);
        }
    }
    if (4 * groups + mine < count) take(__float_as_uint(p[4 * groups + mine]));        // the last one to three
    __shared__ RangePart waves[RANGE_THREADS / 64];
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        most = max(most, (unsigned)__shfl_xor((int)most, d));
        least = min(least, (unsigned)__shfl_xor((int)least, d));
    }
    if ((threadIdx.x & 63) == 0) waves[threadIdx.x >> 6] = {most, least};
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < RANGE_THREADS / 64; ++i) {
            most = max(most, waves[i].most);
            least = min(least, waves[i].least);
        }
        to[blockIdx.x] = {most, least};
    }
}

}  // namespace

int split_range_share(size_t count_a, size_t count_b)
{
    if (count_a == 0) return 0;
    const int share = (int)(RANGE_WGS * ((double)count_a / ((double)count_a + (double)count_b)) + 0.5);
    return share < 1 ? 1 : share > RANGE_WGS - 1 ? RANGE_WGS - 1 : share;
}

hipError_t launch_split_range(const RangeOperand &a, const RangeOperand &b, void *to, hipStream_t stream)
{
    hipLaunchKernelGGL(split_range_kernel, dim3(RANGE_WGS), dim3(RANGE_THREADS), 0, stream, a, b, split_range_share(a.count, b.count),
                       (RangePart *)to);
    return hipGetLastError();
}

}  // namespace kst

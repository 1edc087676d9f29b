// Largest magnitude of two operands and of the smallest of their blocks: the scales of two half-precision parts (see
// kst_split_common.h).
//
// A block is what a result that another tensor's values do not dwarf may consist of: 64 neighbours of an operand whose batch items and
// positions are the result's; for weights, and for both operands of a kernel gradient, at least sixteen values of one of
// the channels that are the result's (values a whole number of periods apart).
//
// What bounds it: memory, each operand read once.  256 workgroups of 512 threads, a fixed share of a tensor each, four
// 16-byte loads of a lane in flight; a block's largest magnitude is taken over the sixteen lanes of a row, or by a lane over
// its own values.  128 x 512 x 16 x 16 and 256 x 512 x 4 x 4, 75 MB: 16 us (4.8 TB/s).
#include "kst_split_common.h"

namespace kst {

namespace {

struct Share {
    const float *p;
    size_t count, step;    // step: groups of four from one of a lane's loads to its next, 0: blocks are neighbours
    int apart;
};

__device__ __forceinline__ unsigned row_max(unsigned v)            // over the 16 lanes of a row
{
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));    // row_ror:8, 4, 2, 1
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
}

// Magnitude bits of a tensor's four elements at group g of `count` elements (past the last: zeros).
__device__ __forceinline__ uint4 group_of(const float *__restrict__ p, size_t g, size_t count)
{
    uint4 t = make_uint4(0u, 0u, 0u, 0u);
    if ((g + 1) * 4 <= count) {
        t = *reinterpret_cast<const uint4 *>(p + g * 4);
    } else {
        if (g * 4 < count) t.x = __float_as_uint(p[g * 4]);
        if (g * 4 + 1 < count) t.y = __float_as_uint(p[g * 4 + 1]);
        if (g * 4 + 2 < count) t.z = __float_as_uint(p[g * 4 + 2]);
    }
    return make_uint4(t.x & 0x7fffffffu, t.y & 0x7fffffffu, t.z & 0x7fffffffu, t.w & 0x7fffffffu);
}
__device__ __forceinline__ unsigned most_of(const uint4 &t) { return max(max(t.x, t.y), max(t.z, t.w)); }

__global__ void __launch_bounds__(RANGE_THREADS) split_range_kernel(Share a, Share b, int wgs_a, RangePart *__restrict__ to)
{
    constexpr int AT_ONCE = 4;
    const bool first = (int)blockIdx.x < wgs_a;
    const Share s = first ? a : b;
    const float *__restrict__ p = s.p;
    const size_t groups = (s.count + 3) / 4;
    const int wg = first ? (int)blockIdx.x : (int)blockIdx.x - wgs_a, wgs = first ? wgs_a : RANGE_WGS - wgs_a;
    const size_t mine = (size_t)wg * RANGE_THREADS + threadIdx.x;
    unsigned most = 0u, least = ~0u;
    if (s.step == 0) {
        // (a row of sixteen lanes takes sixteen neighbouring groups; lanes past the last group hold zero)
        const size_t step = (size_t)wgs * RANGE_THREADS;
        for (size_t g = mine; g - threadIdx.x % 16u < groups; g += AT_ONCE * step) {
            unsigned v[AT_ONCE];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) v[i] = most_of(group_of(p, g + i * step, s.count));
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) {
                const unsigned block = row_max(v[i]);
                most = max(most, block);
                least = min(least, block - 1u);                   // (nothing but zeros: all ones)
            }
        }
    } else if (mine < s.step) {
        uint4 m = make_uint4(0u, 0u, 0u, 0u);
        for (size_t g = mine; g < groups; g += AT_ONCE * s.step) {
            uint4 v[AT_ONCE];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) v[i] = group_of(p, g + i * s.step, s.count);
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) m = make_uint4(max(m.x, v[i].x), max(m.y, v[i].y), max(m.z, v[i].z), max(m.w, v[i].w));
        }
        most = most_of(m);
        least = s.apart ? min(min(m.x - 1u, m.y - 1u), min(m.z - 1u, m.w - 1u)) : most - 1u;
    }
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

// A lane's loads a whole number of periods apart, sixteen of them or more, by as many lanes as that leaves; neighbours
// where a period has more groups than the share has lanes, or comes round less often.
Share share_of(const RangeOperand &o, int wgs)
{
    Share s = {o.p, o.count, 0, o.apart ? 1 : 0};
    if (o.period == 0) return s;
    const size_t lanes = (size_t)wgs * RANGE_THREADS, groups = (o.count + 3) / 4;
    const size_t period = (o.period & 3) == 0 ? o.period / 4 : (o.period & 1) == 0 ? o.period / 2 : o.period;   // in groups
    const size_t most = groups / 16 < lanes ? groups / 16 : lanes;
    s.step = most / period * period;
    return s;
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
    const int wgs_a = split_range_share(a.count, b.count);
    hipLaunchKernelGGL(split_range_kernel, dim3(RANGE_WGS), dim3(RANGE_THREADS), 0, stream, share_of(a, wgs_a),
                       share_of(b, RANGE_WGS - wgs_a), wgs_a, (RangePart *)to);
    return hipGetLastError();
}

}  // namespace kst

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

// ---- two half-precision parts ----
//
// Where the reduction is long, fp32 operands are split into two half-precision parts instead, x = x0 + 2^-12 x1 (rounded to
// nearest: |x - x0| <= 2^-11 |x|, what is left over at most 2^-23 |x|), and a product is x0 w0 + 2^-12 (x0 w1 + x1 w0): three
// partial products of six.  22 to 23 bits of each operand and the product x1 w1 left out are an error of 7.6e-8 of a sum of
// products of random sign, beside which the sums' own roundings are made smaller than with three parts: the largest products'
// sums are added to a total every few steps instead of running through the whole reduction.
//
// Half precision has five bits of exponent, so both tensors are scaled by a power of two that brings their largest
// magnitude to [2^14, 2^15), and the second part is held 2^12 times its size (its products have sums of their own for that):
// every value down to 2^-15, 2^-29 to 2^-30 of the tensor's largest, then has its two parts to within 2^-22 of itself (2^-23 from 2^-14
// on), and a product is formed to within 2^-20 of itself at worst, whatever else is in the tensors.  A tensor that has
// a smaller value, zeros aside, or one that is not finite goes through the three-part kernels, in the same launches: a pass of its own
// over both tensors (kst_split_range.hip) finds the largest and the smallest magnitude.  Nothing less will do.  A result is a sum of
// products, so one operand's zeros and small values choose which values of the other count, and a few small values, in
// whatever company, can be all there is of some result.  (Of 60 tensors of 8 and of 16 million normal random values one each had a smaller one.  Layers
// planned for two parts that go through three take 1.26 to 1.45 times as long.)
//
// Zeros matter too: what an addition of nothing does not round.  The error of three parts falls with the share of the products
// that are not zero, that of two does not: its square is 0.2e-14 + 6e-16 for each step of a chain times that share, against 1.0e-14 to
// 2.4e-14.  The pass counts the values that are not zero; a plan says which share of the products it wants (so many steps of a chain without zeros, over its steps).
constexpr int RANGE_WGS = 256, RANGE_THREADS = 512;
constexpr int RANGE_APART = 29;              // powers of two from the smallest value to the largest
constexpr float LOW_SCALE = 0x1p12f;

// Of one workgroup's share of a tensor: bits of the largest magnitude; of the smallest but zero, less one (none: all ones); values
// that are not zero.
struct RangePart {
    unsigned most, least, real, pad;
};
static_assert(RANGE_WGS * sizeof(RangePart) == SPLIT_RANGE_BYTES, "");
// What a launch reads in front of its operands: `two` where they have two half-precision parts, scaled by 2^ea and 2^eb.
struct SplitHead {
    unsigned two;
    int ea, eb;
    unsigned pad;
};
constexpr unsigned SPLIT_TWO = 0xffffffffu;  // (two bfloat16 NaNs that no third part is: see quiet())

// Eight values times 2^e -> their two half-precision parts.
__device__ __forceinline__ void split2(const float (&v)[8], int e, bf16x8 &p0, bf16x8 &p1)
{
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    halfx8 h, l;
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const floatx2 t = {__builtin_amdgcn_ldexpf(v[j], e), __builtin_amdgcn_ldexpf(v[j + 1], e)};
        const halfx2 r = __builtin_convertvector(t, halfx2);
        h[j] = r[0];
        h[j + 1] = r[1];
        l[j] = (_Float16)fmaf((float)r[0], -LOW_SCALE, t[0] * LOW_SCALE);      // (exact: one rounding, to half precision)
        l[j + 1] = (_Float16)fmaf((float)r[1], -LOW_SCALE, t[1] * LOW_SCALE);
    }
    p0 = __builtin_bit_cast(bf16x8, h);
    p1 = __builtin_bit_cast(bf16x8, l);
}

// NaNs of third parts -> one that is not part of SPLIT_TWO.
__device__ __forceinline__ bf16x8 quiet(bf16x8 p)
{
    typedef unsigned short shortx8 __attribute__((ext_vector_type(8)));
    shortx8 b = __builtin_bit_cast(shortx8, p);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = (b[j] & 0x7fffu) > 0x7f80u ? (unsigned short)0x7fc0u : b[j];
    return __builtin_bit_cast(bf16x8, b);
}

// The scales of two tensors from the shares that split_range wrote, by a whole workgroup of 256.  from: least product of the
// tensors' numbers of values that are not zero.
__device__ __forceinline__ SplitHead split_head(const RangePart *__restrict__ part, int wgs_a, float from)
{
    static_assert(RANGE_WGS == 256, "one share per thread");
    __shared__ RangePart waves[2][4];
    const int tid = threadIdx.x;
    const RangePart mine = part[tid];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const bool in = (tid < wgs_a) == (t == 0);
        unsigned most = in ? mine.most : 0u, least = in ? mine.least : ~0u, real = in ? mine.real : 0u;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            most = max(most, (unsigned)__shfl_xor((int)most, d));
            least = min(least, (unsigned)__shfl_xor((int)least, d));
            real += (unsigned)__shfl_xor((int)real, d);
        }
        if ((tid & 63) == 0) waves[t][tid >> 6] = {most, least, real, 0u};
    }
    __syncthreads();
    SplitHead h = {SPLIT_TWO, 0, 0, 0u};
    float products = 1.0f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        unsigned most = 0u, least = ~0u, real = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            most = max(most, waves[t][i].most);
            least = min(least, waves[t][i].least);
            real += waves[t][i].real;
        }
        products *= (float)real;
        if (most >= 0x7f800000u) h.two = 0u;
        if (most == 0u || most >= 0x7f800000u) continue;
        const int top = __builtin_amdgcn_frexp_expf(__uint_as_float(most));
        if (top - __builtin_amdgcn_frexp_expf(__uint_as_float(least + 1u)) > RANGE_APART) h.two = 0u;
        (t == 0 ? h.ea : h.eb) = 15 - top;
    }
    if (products < from) h.two = 0u;
    return h;
}
// ... and what the launch that wrote the operands left of them at `end` - 16.
__device__ __forceinline__ SplitHead read_head(const char *__restrict__ end)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(end - 16);
    return {(unsigned)__builtin_amdgcn_readfirstlane((int)v.x), __builtin_amdgcn_readfirstlane((int)v.y),
            __builtin_amdgcn_readfirstlane((int)v.z), 0u};
}

// Totals of accumulator blocks that a kernel's registers have no room for, in LDS: a lane's own cells, 16 bytes at a time.  (Not
// by LDS atomics: those took the forward kernel from 300 to 1240 us on 128 x 512 x 256 x 16 x 16, n = 4.)
template <int THREADS>
struct LdsTotals {
    float4 *cells;                           // this lane's first
    __device__ __forceinline__ void clear(int block) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) cells[(block * 4 + q) * THREADS] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __device__ __forceinline__ void add(int block, const floatx16 &v) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 t = cells[(block * 4 + q) * THREADS];
            t.x += v[4 * q];
            t.y += v[4 * q + 1];
            t.z += v[4 * q + 2];
            t.w += v[4 * q + 3];
            cells[(block * 4 + q) * THREADS] = t;
        }
    }
    __device__ __forceinline__ void add_to(int block, floatx16 &v) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 t = cells[(block * 4 + q) * THREADS];
            v[4 * q] += t.x;
            v[4 * q + 1] += t.y;
            v[4 * q + 2] += t.z;
            v[4 * q + 3] += t.w;
        }
    }
};

// Positions of an unframed map of edge N that meet each tap of one axis inside a map of edge M, padding factor P, all taps.
inline double taps_inside(int N, int n, int P, int M)
{
    int hits = 0;
    for (int u = 0; u < n; ++u) {
        const int lo = P >= u ? 0 : (u - P + 1) / 2, hi = M - 1 + u - P < 0 ? -1 : (M - 1 + u - P) / 2;
        const int last = hi < N - 1 ? hi : N - 1;
        hits += last >= lo ? last - lo + 1 : 0;
    }
    return hits;
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

// The workgroups whose ranges meet shared pass `rel`, all lanes of a wave together: a lane finds where one range begins.  (One
// after the other the divisions of eight such beginnings, and slots asked for in turn, were up to a third of a sum's launch:
// 128 x 512 x 256 x 16 x 16, n = 4: 16.0 -> 11.2 us; input gradient of 64 x 512 x 256 x 8 x 8, n = 4, P = 2: 11.0 -> 9.4.)
struct PassOwners {
    int g0, g1, base;
    bool near;                           // the masks hold (a bit per workgroup from base)
    unsigned long long empty, first;     // its range is empty; begins in this pass
    __device__ PassOwners(const EvenShares &k, int rel)
    {
        const int u0 = rel * k.chunks, u1 = u0 + k.chunks - 1, lane = threadIdx.x & 63;
        const float cost = (float)k.chunks * ((rel >> 1) * (k.taps0 + k.taps1) + (rel & 1) * k.taps0);
        base = __builtin_amdgcn_readfirstlane(max((int)(cost * (float)k.grid / ((float)k.per * (float)k.grid + (float)k.more)) - 2, 0));
        const int g = min(base + lane, k.grid), b = k.begin(g), next = __shfl_down(b, 1);
        const unsigned long long from = __ballot(g < k.grid && b <= u0), to = __ballot(g < k.grid && b <= u1);
        near = from != 0 && to != ~0ull;
        g0 = near ? base + __popcll(from) - 1 : k.owner(u0);
        g1 = near ? base + __popcll(to) - 1 : k.owner(u1);
        empty = __ballot(b == next);
        first = __ballot(b >= u0);
    }
    __device__ bool holds(const EvenShares &k, int g) const
    {
        return near ? !((empty >> (g - base)) & 1) : k.begin(g) != k.begin(g + 1);
    }
    __device__ bool begins(const EvenShares &k, int g, int rel) const
    {
        return near ? ((first >> (g - base)) & 1) != 0 : k.begin(g) >= rel * k.chunks;
    }
};

// a += this thread's 16 sums (four groups THREADS apart) of every slot of pass `rel`, in workgroup order, two slots' loads at a time.
template <int THREADS>
__device__ __forceinline__ void add_slots(const float *__restrict__ ws, size_t slot_floats, const EvenShares &k, const PassOwners &o,
                                          int rel, float4 (&a)[4])
{
    int held = 0;                                     // (a slot that can be read where there is nothing to add)
    for (int g = o.g0; g <= o.g1; g += 2) {
        float4 v[2][4];
        bool ok[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ok[i] = g + i <= o.g1 && o.holds(k, g + i);
            if (ok[i]) held = k.slot(g + i, rel, o.begins(k, g + i, rel));
            const float4 *d = reinterpret_cast<const float4 *>(ws + (size_t)held * slot_floats) + threadIdx.x;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[i][q] = d[q * THREADS];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (ok[i])
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[q].x += v[i][q].x;
                    a[q].y += v[i][q].y;
                    a[q].z += v[i][q].z;
                    a[q].w += v[i][q].w;
                }
    }
}

// An operand's value, whatever its type.
__device__ __forceinline__ float value_of(const float *p) { return *p; }
__device__ __forceinline__ float value_of(const uint16_t *p) { return to_f32(*p); }
__device__ __forceinline__ float value_of(const half_bits *p) { return to_f32(*p); }

// Forward: taps in the order they are walked, by window offset, in the classes form the up to four classes that meet it.
template <int n, bool ROWS>
struct FwdTaps {
    static constexpr int side = n / 2 + 1, offsets = side * side, taps = ROWS ? offsets : n * n;
    int cls[taps] = {}, local[taps] = {}, offset[taps] = {};
    constexpr FwdTaps()
    {
        int q = 0;
        for (int o = 0; o < offsets; ++o) {
            if (ROWS) {
                offset[o] = o;
                continue;
            }
            for (int c = 0; c < 4; ++c) {
                const int a = o / side - (c >> 1), b = o % side - (c & 1);
                if (a < 0 || a >= taps_for_parity(n, c >> 1) || b < 0 || b >= taps_for_parity(n, c & 1)) continue;
                cls[q] = c;
                local[q] = a * taps_for_parity(n, c & 1) + b;
                offset[q] = o;
                ++q;
            }
        }
    }
};

}  // namespace kst

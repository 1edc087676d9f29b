// Kernel gradient on the bf16 matrix cores (in and g split into three bfloat16 parts, see kst_split_common.h; bfloat16
// input is its own only part).
//
//   dw[co][ci][u][v] = sum_b sum_a sum_c in[b][ci][a][c] * g[b][co][2 (a + q) - u][2 (c + q) - v]
//
// (q: the zero frame of the padding factor; for an odd one g starts a row and a column later).  As n * n GEMMs: rows =
// output channels, columns = input channels, reduction over batch items and positions.  An MFMA's sixteen reduction
// steps are sixteen batch items at one position: the shift a kernel tap asks of g is then one of whole operands, where
// neighbouring positions in a lane's eight values would have to be moved by single elements.
//
// Two passes over memory bring both operands into that form ([block of 32 channels][row][column][16 items][part][lane]
// [8 items]), then every operand is one contiguous 1 KB load into registers.  A workgroup of four waves owns 128 x 128
// channels and two taps, a wave 64 x 64 of them: 8 blocks, the largest partial products' sums apart from the others',
// 256 accumulator registers; 48 MFMAs per step for 18 loads, one step ahead.  What bounds it is the rate at which the
// cache of a CU hands over those operands (18 KB per wave and 1536 cycles; each is wanted by two waves).
// 64 x 512 x 256 x 8 x 8, n = 4, P = 2: 15 us for the two passes, 83 us here and 9 us for the sums, where framing g, the
// fp32 multiplies and their sums took 202; with bfloat16 input 64 x 256 x 128 x 16 x 16: 21 + 57 + 9 against 212.
#include "kst_split_common.h"

namespace kst {

namespace {

constexpr int E_THREADS = 256;
constexpr int E_TC = 128;                // channels per workgroup, both kinds

struct DwParams {
    int B, Cin, Cout, N, M;              // edges of in and g
    int q2;                              // position (a, c) meets g rows 2 a + q2 - u
    int groups, steps;                   // groups of 16 items; positions x groups
    int tiles_co, tiles_ci, pairs;
    int splits, per_split;               // steps per split, even
    unsigned x_bytes, g_bytes;           // of the operands
};

__device__ __forceinline__ float value_of(const float *p) { return *p; }
__device__ __forceinline__ float value_of(const uint16_t *p) { return to_f32(*p); }
__device__ __forceinline__ float value_of(const half_bits *p) { return to_f32(*p); }

// Four neighbours at p, of which `count` exist; VEC: all four in one aligned load.
template <bool VEC, class T>
__device__ __forceinline__ void load_four(const T *p, int count, float (&v)[4])
{
    if constexpr (VEC) {
        T t[4];
        __builtin_memcpy(t, __builtin_assume_aligned(p, 4 * sizeof(T)), sizeof(t));
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = count > 0 ? value_of(t + i) : 0.0f;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = i < count ? value_of(p + i) : 0.0f;
    }
}

// src[B][C][edge][edge] -> operands of PARTS parts, zeros past the last item and channel.  One wave per (channel block,
// group of items, row, eight columns): a lane reads eight neighbours of eight items, in two loads each where the rows
// are whole groups of four (VEC).  Lanes of a wave read different rows, so what a lane leaves of its line has to come
// from the cache again: a float g of 64 x 128 x 32 x 32 takes 15 us (5.6 TB/s of
// the 33 MB read and 50 MB written), 27 with four columns and one element per load.
constexpr int E_COLS = 8;

template <int PARTS, bool VEC, class T>
__global__ void __launch_bounds__(256) split_items_kernel(const T *__restrict__ src, char *__restrict__ dst, int B, int C,
                                                          int edge, int groups, unsigned tasks)
{
    unsigned t = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (t >= tasks) return;
    const unsigned runs = (unsigned)(edge + E_COLS - 1) / E_COLS;
    const int x0 = E_COLS * (int)(t % runs);
    t /= runs;
    const int y = (int)(t % (unsigned)edge);
    t /= (unsigned)edge;
    const int group = (int)(t % (unsigned)groups), blk = (int)(t / (unsigned)groups);
    const int lane = threadIdx.x & 63, c = blk * 32 + (lane & 31), b = group * 16 + 8 * (lane >> 5);
    float v[8][E_COLS / 4][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool ok = c < C && b + j < B;
        const T *row = src + ((ok ? (size_t)(b + j) * C + c : 0) * edge + y) * edge;
#pragma unroll
        for (int h = 0; h < E_COLS / 4; ++h) {
            const int x = x0 + 4 * h, count = ok ? edge - x : 0;
            load_four<VEC>(row + (x < edge ? x : 0), count, v[j][h]);
        }
    }
#pragma unroll
    for (int i = 0; i < E_COLS; ++i) {
        if (x0 + i >= edge) break;
        float eight[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) eight[j] = v[j][i >> 2][i & 3];
        bf16x8 part[3];
        split3(eight, part[0], part[1], part[2]);
        char *d = dst + ((((size_t)blk * edge + y) * edge + x0 + i) * groups + group) * (PARTS * 1024) + lane * 16;
#pragma unroll
        for (int k = 0; k < PARTS; ++k) *reinterpret_cast<bf16x8 *>(d + k * 1024) = part[k];
    }
}

template <int PARTS, class T>
hipError_t split_items(const T *src, char *dst, int B, int C, int edge, int groups, hipStream_t stream)
{
    const unsigned tasks = (unsigned)((C + 31) / 32) * groups * edge * ((edge + E_COLS - 1) / E_COLS);
    const dim3 grid((tasks + 3) / 4), block(256);
    if (edge % 4 == 0)
        hipLaunchKernelGGL((split_items_kernel<PARTS, true, T>), grid, block, 0, stream, src, dst, B, C, edge, groups, tasks);
    else
        hipLaunchKernelGGL((split_items_kernel<PARTS, false, T>), grid, block, 0, stream, src, dst, B, C, edge, groups, tasks);
    return hipGetLastError();
}

// Partial sums part[split][tap][co][ci].
template <int n, int XP>
__global__ void __launch_bounds__(E_THREADS, 1) split_dw_kernel(const void *__restrict__ xf, const void *__restrict__ gf,
                                                               float *__restrict__ part, DwParams p)
{
    constexpr int NN = n * n;
    // The split index runs fastest: workgroups that read the same positions share an XCD where the splits are a
    // multiple of eight.
    unsigned id = blockIdx.x;
    const int split = (int)(id % (unsigned)p.splits);
    id /= (unsigned)p.splits;
    const int tile_co = (int)(id % (unsigned)p.tiles_co);
    id /= (unsigned)p.tiles_co;
    const int pair = (int)(id % (unsigned)p.pairs), tile_ci = (int)(id / (unsigned)p.pairs);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cob = __builtin_amdgcn_readfirstlane(tile_co * 4 + (wave & 1) * 2);        // first blocks of 32 channels
    const int cib = __builtin_amdgcn_readfirstlane(tile_ci * 4 + (wave >> 1) * 2);
    const int last_co = (p.Cout - 1) / 32, last_ci = (p.Cin - 1) / 32;
    int u[2], v[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int tap = min(2 * pair + t, NN - 1);            // (the last pair of an odd number: twice the same tap)
        u[t] = __builtin_amdgcn_readfirstlane(tap / n);
        v[t] = __builtin_amdgcn_readfirstlane(tap % n);
    }

    // (the same in all lanes: the operands' addresses stay scalar)
    const int s_begin = __builtin_amdgcn_readfirstlane(split * p.per_split);
    const int s_end = __builtin_amdgcn_readfirstlane(min(p.steps, s_begin + p.per_split));
    int group = __builtin_amdgcn_readfirstlane(s_begin % p.groups), s = s_begin;
    int c = __builtin_amdgcn_readfirstlane(s_begin / p.groups % p.N), a = __builtin_amdgcn_readfirstlane(s_begin / p.groups / p.N);

    bf16x8 xr[2][2][XP], gr[2][2][2][3];
    // Operands of the next step (zeros past the last one) -> register set.
    auto fetch = [&](auto setc) {
        constexpr int set = decltype(setc)::value;
        const bool live = s < s_end;
        const __amdgpu_buffer_rsrc_t xb = buffer_of(xf, live ? p.x_bytes : 0u);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const unsigned at = live ? (unsigned)((min(cib + i, last_ci) * p.N + a) * p.N + c) * p.groups + group : 0u;
#pragma unroll
            for (int k = 0; k < XP; ++k) xr[set][i][k] = load_bf16x8(xb, lane * 16 + k * 1024, at * (XP * 1024));
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int y = 2 * a + p.q2 - u[t], x = 2 * c + p.q2 - v[t];
            const bool inside = live && y >= 0 && y < p.M && x >= 0 && x < p.M;
            const __amdgpu_buffer_rsrc_t gb = buffer_of(gf, inside ? p.g_bytes : 0u);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned at = inside ? (unsigned)((min(cob + i, last_co) * p.M + y) * p.M + x) * p.groups + group : 0u;
#pragma unroll
                for (int k = 0; k < 3; ++k) gr[set][t][i][k] = load_bf16x8(gb, lane * 16 + k * 1024, at * 3072u);
            }
        }
        ++s;
        if (++group == p.groups) {
            group = 0;
            if (++c == p.N) {
                c = 0;
                ++a;
            }
        }
    };

    floatx16 acc[2][2][2], low[2][2][2];              // [tap][output channels][input channels]
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][i][j][r] = low[t][i][j][r] = 0.0f;

    auto multiply = [&](auto setc) {
        constexpr int set = decltype(setc)::value;
        static_for<3>([&](auto wc) {                  // partial products, smallest first: gp + xp = 2, 1, 0
            constexpr int sum = 2 - decltype(wc)::value;
            static_for<3>([&](auto gc) {
                constexpr int gp = decltype(gc)::value, xp = sum - gp;
                if constexpr (xp >= 0 && xp < XP) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                floatx16 &d = sum == 0 ? acc[t][i][j] : low[t][i][j];
                                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gr[set][t][i][gp], xr[set][j][xp], d, 0, 0, 0);
                            }
                }
            });
        });
        // the loads of the next step spread over the MFMAs of this one
        static_for<8 * (XP == 1 ? 3 : 6)>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // global read
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);      // vector arithmetic
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    using std::integral_constant;
    fetch(integral_constant<int, 0>{});
    for (int k = s_begin; k < s_end; k += 2) {
        fetch(integral_constant<int, 1>{});
        multiply(integral_constant<int, 0>{});
        fetch(integral_constant<int, 0>{});
        multiply(integral_constant<int, 1>{});
    }

    const size_t plane = (size_t)p.Cout * p.Cin;
    static_for<2>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if (2 * pair + t >= NN) return;
        float *o = part + ((size_t)split * NN + 2 * pair + t) * plane;
        static_for<4>([&](auto bc) {
            constexpr int i = decltype(bc)::value >> 1, j = decltype(bc)::value & 1;
            const int ci = (cib + j) * 32 + (lane & 31), co0 = (cob + i) * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int co = co0 + 8 * (r >> 2) + (r & 3);
                if (co < p.Cout && ci < p.Cin) o[(size_t)co * p.Cin + ci] = (acc[t][i][j][r] + low[t][i][j][r]) * SPLIT_UNSCALE;
            }
        });
    });
}

// The elements of 64 neighbouring (co, ci) pairs whose split sums are not finite, in fp32 MFMAs, by a whole wave.  `bad`:
// the taps of this lane's pair e0 + lane that have to be done again.  For one output channel and up to 32 input channels
// at a time, all taps are the rows of one product over batch items and positions: the g values of a channel's taps are
// neighbours, and 16384 positions take 0.25 ms of multiplies.
template <int n, class T>
__device__ __forceinline__ void dw_fp32_pairs(const T *in, const float *g, float *dw, const DwParams &p, size_t e0,
                                                        unsigned bad)
{
    constexpr int NN = n * n;
    const int lane = threadIdx.x & 63, kk = lane >> 5, row = lane & 31;
    const int B = p.B, Cin = p.Cin, Cout = p.Cout, N = p.N, M = p.M, q2 = p.q2;
    const size_t last = (size_t)Cout * Cin - 1, x_plane = (size_t)N * N, g_plane = (size_t)M * M;
    const int u = row / n, v = row % n;               // this lane's tap as a row (row < NN)
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        const size_t e = e0 + half * 32 + row < last ? e0 + half * 32 + row : last;
        const unsigned wanted = (unsigned)__shfl((int)bad, half * 32 + row);
        const int co = (int)(e / (unsigned)Cin), ci = (int)(e - (size_t)co * (unsigned)Cin);
        const int co_end = same(__shfl(co, 31));
        for (int o = same(__shfl(co, 0)); o <= co_end; ++o) {
            if (__ballot(co == o && wanted != 0) == 0) continue;
            floatx16 sum;
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[r] = 0.0f;
            const T *x = in + (size_t)ci * x_plane;
            const float *gb = g + (size_t)o * g_plane;
            for (int b = 0; b < B; ++b) {
                for (int a = 0; a < N; ++a) {
                    const int y = 2 * a + q2 - u;
                    const bool y_in = row < NN && y >= 0 && y < M;
#pragma unroll 1
                    for (int c0 = 0; c0 < N; c0 += 8) {       // four MFMAs' operands in flight together
                        float gv[4], xv[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {         // an MFMA's two reduction steps: two columns
                            const int c = c0 + 2 * j + kk, gx = 2 * c + q2 - v;
                            gv[j] = y_in && c < N && gx >= 0 && gx < M ? gb[(size_t)y * M + gx] : 0.0f;
                            xv[j] = c < N ? value_of(x + a * N + c) : 0.0f;
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            sum = __builtin_amdgcn_mfma_f32_32x32x2f32(gv[j], xv[j], sum, 0, 0, 0);
                    }
                }
                x += (size_t)Cin * x_plane;
                gb += (size_t)Cout * g_plane;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tap = 8 * (r >> 2) + 4 * kk + (r & 3);
                if (tap < NN && co == o && ((wanted >> tap) & 1u)) dw[e * NN + tap] = sum[r];
            }
        }
    }
}

// dw[co][ci][tap] = the splits' partial sums in split order.  One thread per (co, ci).
template <int n, class T>
__global__ void __launch_bounds__(256, n == 5 ? 6 : 8) split_dw_sum_kernel(const float *__restrict__ part, const T *__restrict__ in,
                                                           const float *__restrict__ g, float *__restrict__ dw, DwParams p)
{
    constexpr int NN = n * n;
    const size_t plane = (size_t)p.Cout * p.Cin, mine = (size_t)blockIdx.x * 256u + threadIdx.x;
    const size_t e = mine < plane ? mine : plane - 1;  // (no lane leaves early: a wave does some elements together)
    float t[NN];
#pragma unroll
    for (int i = 0; i < NN; ++i) t[i] = part[(size_t)i * plane + e];
    for (int s = 1; s < p.splits; ++s)
#pragma unroll
        for (int i = 0; i < NN; ++i) t[i] += part[((size_t)s * NN + i) * plane + e];
    float zero = 0.0f;
#pragma unroll
    for (int i = 0; i < NN; ++i) zero = fmaf(t[i], 0.0f, zero);
    unsigned bad = 0;
    if (mine < plane) {
        if (zero == 0.0f) {
#pragma unroll
            for (int i = 0; i < NN; ++i) dw[e * NN + i] = t[i];
        } else {
#pragma unroll
            for (int i = 0; i < NN; ++i) {
                if (t[i] * 0.0f == 0.0f) dw[e * NN + i] = t[i];
                else bad |= 1u << i;
            }
        }
    }
    if (__builtin_expect(__ballot(bad != 0) != 0, 0)) dw_fp32_pairs<n>(in, g, dw, p, mine - (threadIdx.x & 63), bad);
}

struct DwPlan {
    bool ok;
    DwParams p;
    size_t x_bytes, g_bytes, part_bytes;      // multiples of 1 KB
};

// s: the framed problem with Shape::frame = q; odd: the padding factor is odd; parts: of the input.
DwPlan dw_plan(const Shape &s, bool odd, int parts)
{
    DwPlan r;
    DwParams &p = r.p;
    const int NN = s.n * s.n;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout;
    p.N = s.N - 2 * s.frame;
    p.M = s.M - (odd ? 2 : 0);
    p.q2 = 2 * s.frame - (odd ? 1 : 0);
    p.groups = (s.B + 15) / 16;
    const double steps = (double)p.N * p.N * p.groups;
    p.steps = (int)(steps < 1e9 ? steps : 1e9);
    p.tiles_co = (s.Cout + E_TC - 1) / E_TC;
    p.tiles_ci = (s.Cin + E_TC - 1) / E_TC;
    p.pairs = (NN + 1) / 2;
    // As many splits as give every CU one workgroup, with at least 16 steps each.
    const double tiles = (double)p.tiles_co * p.tiles_ci * p.pairs;
    int splits = tiles < 256.0 ? (int)(256.0 / tiles) : 1;
    if (splits > p.steps / 16) splits = p.steps / 16 > 0 ? p.steps / 16 : 1;
    p.per_split = ((p.steps + splits - 1) / splits + 1) & ~1;
    p.splits = (p.steps + p.per_split - 1) / p.per_split;
    r.x_bytes = (size_t)((s.Cin + 31) / 32) * p.N * p.N * p.groups * parts * 1024;
    r.g_bytes = (size_t)((s.Cout + 31) / 32) * p.M * p.M * p.groups * 3 * 1024;
    r.part_bytes = ((size_t)p.splits * NN * s.Cout * s.Cin * sizeof(float) + 255) & ~(size_t)255;
    p.x_bytes = (unsigned)r.x_bytes;
    p.g_bytes = (unsigned)r.g_bytes;
    r.ok = s.n >= 3 && s.n <= 5 && steps < 1e9 && tiles < 1e6 && r.x_bytes < (1u << 31) && r.g_bytes < (1u << 31);
    return r;
}

template <int n, int XP, class T>
hipError_t dw_launch(const T *in, const float *g, float *dw, char *ws, const DwPlan &pl, hipStream_t stream)
{
    const DwParams &p = pl.p;
    char *xf = ws, *gf = ws + pl.x_bytes;
    float *part = (float *)(gf + pl.g_bytes);
    hipError_t e = split_items<XP>(in, xf, p.B, p.Cin, p.N, p.groups, stream);
    if (e != hipSuccess) return e;
    e = split_items<3>(g, gf, p.B, p.Cout, p.M, p.groups, stream);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)p.splits * p.tiles_co * p.tiles_ci * p.pairs;
    hipLaunchKernelGGL((split_dw_kernel<n, XP>), dim3(blocks), dim3(E_THREADS), 0, stream, (const void *)xf, (const void *)gf,
                       part, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t pairs = (size_t)p.Cout * p.Cin;
    hipLaunchKernelGGL((split_dw_sum_kernel<n, T>), dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, stream,
                       (const float *)part, in, g, dw, p);
    return hipGetLastError();
}

template <int XP, class T>
hipError_t dw_launch_n(const T *in, const float *g, float *dw, char *ws, const DwPlan &pl, int n, hipStream_t stream)
{
    if (n == 3) return dw_launch<3, XP>(in, g, dw, ws, pl, stream);
    if (n == 4) return dw_launch<4, XP>(in, g, dw, ws, pl, stream);
    return dw_launch<5, XP>(in, g, dw, ws, pl, stream);
}

}  // namespace

bool split_dw_applies(const Shape &s, bool odd, kst_dtype dt)
{
    if (s.n < 3 || s.n > 5) return false;
    const double edge = s.N - 2 * s.frame, nn = s.n * s.n;
    const double products = (double)s.B * edge * edge * nn * s.Cin * s.Cout;
    const double padded = (double)((s.B + 15) / 16 * 16) * edge * edge * nn * ((s.Cin + 127) / 128 * 128) *
                          ((s.Cout + 127) / 128 * 128);
    // What fills items and channels up to whole blocks is multiplied too.  Both sides timed on 1014 random layers from 3
    // to 16 G products: 1.5 times as fast on average, with 1.8 to 2.2 times the products multiplied 25 of 121 layers
    // lost.  One kind did not gain: with 9 products per value of g and input channel and at most one tile of those, the
    // passes over g (four times the positions) show, and on maps of whole groups of four columns the fp32 multiplies
    // are at their best: of 32 such layers 15 lost (68 x 128 x 128 x 24 x 24, P = 3: 220 us here against 181).  bfloat16
    // input halves the multiplies and gained there too.
    const bool g_bound = s.n == 3 && s.Cin <= E_TC && dt != KST_BF16 && edge > 8 && ((int)edge & 3) == 0;
    return products >= 3.0e9 && padded <= 1.5 * products && !g_bound && dw_plan(s, odd, 3).ok;
}

static int parts_of(kst_dtype dt) { return dt == KST_BF16 ? 1 : 3; }

// (0 for a layer this kernel does not take)
size_t split_dw_workspace_bytes(const Shape &s, bool odd, kst_dtype dt)
{
    const DwPlan r = dw_plan(s, odd, parts_of(dt));
    if (!r.ok) return 0;
    return r.x_bytes + r.g_bytes + r.part_bytes;
}

hipError_t launch_split_dw(const void *in, const float *g, float *dw, void *ws, const Shape &s, bool odd, kst_dtype dt,
                           hipStream_t stream)
{
    const DwPlan r = dw_plan(s, odd, parts_of(dt));
    if (!r.ok) return hipErrorInvalidValue;
    if (dt == KST_BF16) return dw_launch_n<1>((const uint16_t *)in, g, dw, (char *)ws, r, s.n, stream);
    if (dt == KST_F16) return dw_launch_n<3>((const half_bits *)in, g, dw, (char *)ws, r, s.n, stream);
    return dw_launch_n<3>((const float *)in, g, dw, (char *)ws, r, s.n, stream);
}

}  // namespace kst

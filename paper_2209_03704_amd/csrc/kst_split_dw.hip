// Kernel gradient on the bf16 matrix cores (in and g split into three bfloat16 parts, see kst_split_common.h; bfloat16
// input is its own only part; large layers: two parts of half precision, one where the input has that type).
//
//   dw[co][ci][u][v] = sum_b sum_a sum_c in[b][ci][a][c] * g[b][co][2 (a + q) - u][2 (c + q) - v]
//
// (q: the zero frame of the padding factor; for an odd one g starts a row and a column later).  As n * n GEMMs: rows =
// output channels, columns = input channels, reduction over batch items and positions.  An MFMA's sixteen reduction
// steps are sixteen batch items at one position: the shift a kernel tap asks of g is then one of whole operands, where
// neighbouring positions in a lane's eight values would have to be moved by single elements.
//
// With few batch items an "item" is a strip of rows of one: its rows of g, those it shares with the next strip included,
// are laid out on their own, so that a tap's shift stays one of whole operands.
//
// Two passes over memory bring both operands into that form ([block of 32 channels][row][column][16 items][part][lane]
// [8 items]), then every operand is one contiguous 1 KB load into registers.  A workgroup of four waves owns 128 x 128
// channels and two taps on large layers, a wave 64 x 64 of them (or 32 x 64, or 64 x 32, and four taps): 8 blocks, the largest partial products' sums apart from the others',
// 256 accumulator registers; 48 MFMAs per step for 18 loads, one step ahead.  What bounds it is the rate at which the
// cache of a CU hands over those operands (18 KB per wave and 1536 cycles; each is wanted by two waves).
// With two parts half the MFMAs want two thirds of the operands, three steps ahead.
// 64 x 512 x 256 x 8 x 8, n = 4, P = 2: 6 us for the ranges, 13 for the operands, 53 here (81 with three parts) and 9 for
// the sums, where framing g, the fp32 multiplies and their sums took 202; with bfloat16 input 64 x 256 x 128 x 16 x 16: 19 + 46 + 9
// against 212.
#include "kst_split_common.h"

namespace kst {

namespace {

constexpr int E_THREADS = 256;
constexpr int E_TOTALS = 2;
constexpr int E_SEGMENT = 8;             // two parts: steps after which each of the accumulators has been added to the total

struct DwParams {
    int B, Cin, Cout, N, M;              // edges of in and g
    int q2;                              // position (a, c) meets g rows 2 a + q2 - u
    int strips, R, GR;                   // strips per batch item; rows of in and rows of g (with the halo) of a strip
    int yo;                              // row a of a strip meets its rows 2 a + yo - u of g
    int groups, steps;                   // groups of 16 items (strips); positions of a strip x groups
    int wave_co, wave_ci;                // waves of a workgroup along the channels; the others along the taps
    int tiles_co, tiles_ci, tiles_taps;
    int splits, per_split;               // steps per split, even
    unsigned x_bytes, g_bytes;           // of the operands
    int two;                             // g of two half-precision parts (input: two, or half precision itself) where the ranges allow
    int range_share;                     // workgroups of the ranges' launch that took the input
    float from;                          // ... and of all pairs of an input value and one of g, how many at least have no zero
};

// Four neighbours at p, of which `count` exist.  (Four at once whatever their alignment: aligned to their own size only.)
template <class T>
__device__ __forceinline__ void load_four(const T *p, int count, float (&v)[4])
{
    T t[4] = {};
    if (count >= 4) {
        __builtin_memcpy(t, p, sizeof(t));
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < count) t[i] = p[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < count ? value_of(t + i) : 0.0f;
}

// src[B][C][edge][edge] -> operands of PARTS parts, zeros past the last item and channel.  An item is a strip of `rows`
// rows, of which strip k of a batch item starts at row k * pitch + first (rows outside the map: zeros).  One wave per
// (channel block, group of items, row, eight columns): a lane reads eight neighbours of eight items, in two loads each.
// Lanes of a wave read different rows, so what a lane leaves of its line has to come from the cache again: a float g of
// 64 x 128 x 32 x 32 takes 15 us (5.6 TB/s of the 33 MB read and 50 MB written), 27 with four columns and one element
// per load.
constexpr int E_COLS = 8;

template <class T>
struct Items {
    const T *src;
    char *dst;
    int C, edge, rows, pitch, first;
    unsigned tasks;                      // waves
    unsigned blocks() const { return (tasks + 3) / 4; }
};

template <class T>
Items<T> items_of(const T *src, char *dst, int C, int edge, int rows, int pitch, int first, const DwParams &p)
{
    return {src, dst, C, edge, rows, pitch, first,
            (unsigned)((C + 31) / 32) * p.groups * rows * ((edge + E_COLS - 1) / E_COLS)};
}

// The share of one workgroup.  Two half-precision parts (one of half precision) where `range` is given and allows; SECOND: src is
// the tensor whose third parts leave room for the head.
template <int PARTS, bool SECOND, class T>
__device__ __forceinline__ void split_items(const Items<T> &q, unsigned block, char *__restrict__ head_end,
                                            const RangePart *__restrict__ range, const DwParams &p)
{
    const T *__restrict__ src = q.src;
    char *__restrict__ dst = q.dst;
    const int B = p.B, C = q.C, edge = q.edge, strips = p.strips, rows = q.rows, pitch = q.pitch, first = q.first, groups = p.groups;
    SplitHead head = {0u, 0, 0, 0u};
    if (range) {
        head = split_head(range, p.range_share, p.from);
        if (SECOND && head.two && block == 0 && threadIdx.x == 0)
            *reinterpret_cast<uint4 *>(head_end - 16) = make_uint4(head.two, (unsigned)head.ea, (unsigned)head.eb, 0u);
    }
    const int parts = !head.two ? PARTS : PARTS == 3 ? 2 : 1, exponent = SECOND ? head.eb : head.ea;
    unsigned t = block * 4u + (threadIdx.x >> 6);
    if (t >= q.tasks) return;
    const unsigned runs = (unsigned)(edge + E_COLS - 1) / E_COLS;
    const int x0 = E_COLS * (int)(t % runs);
    t /= runs;
    const int y = (int)(t % (unsigned)rows);
    t /= (unsigned)rows;
    const int group = (int)(t % (unsigned)groups), blk = (int)(t / (unsigned)groups);
    const int lane = threadIdx.x & 63, c = blk * 32 + (lane & 31), item = group * 16 + 8 * (lane >> 5);
    int b = item / strips, k = item - b * strips;
    float v[8][E_COLS / 4][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int at = k * pitch + first + y;
        const bool ok = c < C && b < B && at >= 0 && at < edge;
        const T *row = src + ((ok ? (size_t)b * C + c : 0) * edge + (ok ? at : 0)) * edge;
#pragma unroll
        for (int h = 0; h < E_COLS / 4; ++h) {
            const int x = x0 + 4 * h, count = ok ? edge - x : 0;
            load_four(row + (x < edge ? x : 0), count, v[j][h]);
        }
        if (++k == strips) {
            k = 0;
            ++b;
        }
    }
#pragma unroll
    for (int i = 0; i < E_COLS; ++i) {
        if (x0 + i >= edge) break;
        float eight[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) eight[j] = v[j][i >> 2][i & 3];
        bf16x8 part[3];
        if (head.two) {
            split2(eight, exponent, part[0], part[1]);
        } else {
            split3(eight, part[0], part[1], part[2]);
            if (SECOND) part[2] = quiet(part[2]);
        }
        char *d = dst + ((((size_t)blk * rows + y) * edge + x0 + i) * groups + group) * (size_t)(parts * 1024) + lane * 16;
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
            if (p < parts) *reinterpret_cast<bf16x8 *>(d + p * 1024) = part[p];
    }
}

// Both tensors in one launch, g's workgroups, which have more to do, first: one after the other they left the chip idle at the
// end of the first (64 x 512 x 256 x 8 x 8, n = 4, P = 2: 18.1 -> 12.6 us; bfloat16, 64 x 256 x 128 x 16 x 16: 22 -> 19).
template <int XP, class T>
__global__ void __launch_bounds__(256) split_items_kernel(Items<T> x, Items<float> g, unsigned g_blocks, char *__restrict__ head_end,
                                                          const RangePart *__restrict__ range, DwParams p)
{
    if (blockIdx.x < g_blocks) split_items<3, true>(g, blockIdx.x, head_end, range, p);
    else split_items<XP, false>(x, blockIdx.x - g_blocks, head_end, range, p);
}

// Partial sums part[split][tap][co][ci].  A wave: TB taps x CB x IB blocks of 32 channels.  XP, GP: parts of the operands (GP =
// 3: bfloat16 ones, 2: of half precision, scaled as the head says).
template <int n, int XP, int GP, int CB, int IB, int TB>
__device__ __forceinline__ void split_dw_work(const void *__restrict__ xf, const void *__restrict__ gf,
                                              float *__restrict__ part, const DwParams &p, const SplitHead &head)
{
    constexpr int NN = n * n;
    // The split index runs fastest: workgroups that read the same positions share an XCD where the splits are a
    // multiple of eight.
    unsigned id = blockIdx.x;
    const int split = (int)(id % (unsigned)p.splits);
    id /= (unsigned)p.splits;
    const int tile_co = (int)(id % (unsigned)p.tiles_co);
    id /= (unsigned)p.tiles_co;
    const int tile_taps = (int)(id % (unsigned)p.tiles_taps), tile_ci = (int)(id / (unsigned)p.tiles_taps);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_co = wave % p.wave_co, wave_ci = wave / p.wave_co % p.wave_ci, wave_taps = wave / (p.wave_co * p.wave_ci);
    // first blocks of 32 channels, first tap
    const int cob = __builtin_amdgcn_readfirstlane((tile_co * p.wave_co + wave_co) * CB);
    const int cib = __builtin_amdgcn_readfirstlane((tile_ci * p.wave_ci + wave_ci) * IB);
    const int tap0 = __builtin_amdgcn_readfirstlane((tile_taps * (4 / (p.wave_co * p.wave_ci)) + wave_taps) * TB);
    const int last_co = (p.Cout - 1) / 32, last_ci = (p.Cin - 1) / 32;
    if (cob > last_co || cib > last_ci || tap0 >= NN) return;    // (a wave of its own: nothing waits for it)
    int u[TB], v[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const int tap = min(tap0 + t, NN - 1);                // (past the last: the last one again)
        u[t] = __builtin_amdgcn_readfirstlane(tap / n);
        v[t] = __builtin_amdgcn_readfirstlane(tap % n);
    }

    // (the same in all lanes: the operands' addresses stay scalar)
    const int s_begin = __builtin_amdgcn_readfirstlane(split * p.per_split);
    const int s_end = __builtin_amdgcn_readfirstlane(min(p.steps, s_begin + p.per_split));
    int group = __builtin_amdgcn_readfirstlane(s_begin % p.groups), s = s_begin;
    int c = __builtin_amdgcn_readfirstlane(s_begin / p.groups % p.N), a = __builtin_amdgcn_readfirstlane(s_begin / p.groups / p.N);

    // Operand numbers: a step's number is its place in x's list, g's follows from the position less a tap's shift.
    unsigned x_at[IB], g_at[CB];
    int shift[TB];
#pragma unroll
    for (int i = 0; i < IB; ++i) x_at[i] = (unsigned)min(cib + i, last_ci) * p.R * p.N * p.groups;
#pragma unroll
    for (int i = 0; i < CB; ++i) g_at[i] = (unsigned)min(cob + i, last_co) * p.GR * p.M * p.groups;
#pragma unroll
    for (int t = 0; t < TB; ++t) shift[t] = (u[t] * p.M + v[t]) * p.groups;
    constexpr int SETS = GP == 2 && TB * CB * GP + IB * XP <= 12 ? 4 : 2;
    bf16x8 xr[SETS][IB][XP], gr[SETS][TB][CB][GP];
    // Operands of the next step (zeros past the last one) -> register set.
    auto fetch = [&](auto setc) {
        constexpr int set = decltype(setc)::value;
        // (a mask the compiler cannot see through: no branches here)
        const unsigned live = (unsigned)__builtin_amdgcn_readfirstlane(s < s_end ? -1 : 0);
        const __amdgpu_buffer_rsrc_t xb = buffer_of(xf, p.x_bytes & live);
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const unsigned at = (x_at[i] + s) & live;
#pragma unroll
            for (int k = 0; k < XP; ++k) xr[set][i][k] = load_bf16x8(xb, lane * 16 + k * 1024, at * (XP * 1024));
        }
        const int here = ((2 * a + p.yo) * p.M + 2 * c + p.q2) * p.groups + group;
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int y = 2 * a + p.yo - u[t], x = 2 * c + p.q2 - v[t];        // (a row of the strip, a column of the map)
            const unsigned inside = (unsigned)y < (unsigned)p.GR && (unsigned)x < (unsigned)p.M ? live : 0u;
            const __amdgpu_buffer_rsrc_t gb = buffer_of(gf, p.g_bytes & inside);
#pragma unroll
            for (int i = 0; i < CB; ++i) {
                const unsigned at = (g_at[i] + (unsigned)(here - shift[t])) & inside;
#pragma unroll
                for (int k = 0; k < GP; ++k) gr[set][t][i][k] = load_bf16x8(gb, lane * 16 + k * 1024, at * (GP * 1024u));
            }
        }
        // (carries as arithmetic: a branch in front of each step would end the block its instructions are dealt out in)
        ++s;
        const int column = ++group == p.groups ? 1 : 0;
        group -= column * p.groups;
        c += column;
        const int row = c == p.N ? 1 : 0;
        c -= row * p.N;
        a += row;
    };

    // (two parts: the total to which the largest products' sums are added, a block per step, before they start again)
    // (all but TR blocks' totals are in LDS: the operands of three steps ahead want the registers)
    constexpr int BLOCKS = TB * CB * IB, TR = E_TOTALS;
    __shared__ float4 totals[(BLOCKS - TR) * 4 * E_THREADS];
    const LdsTotals<E_THREADS> spare = {totals + tid};
    floatx16 acc[TB][CB][IB], low[TB][CB][IB], total[TR > 0 ? TR : 1], zeros;   // [tap][output channels][input channels]
#pragma unroll
    for (int r = 0; r < 16; ++r) zeros[r] = 0.0f;
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int j = 0; j < IB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int b = (t * CB + i) * IB + j;
                    acc[t][i][j][r] = low[t][i][j][r] = 0.0f;
                    if (b < TR) total[b][r] = 0.0f;
                }
    if constexpr (GP == 2)
        static_for<BLOCKS - TR>([&](auto bc) { spare.clear(decltype(bc)::value); });

    auto multiply = [&](auto setc, auto stepc) {
        constexpr int set = decltype(setc)::value, PER = BLOCKS / E_SEGMENT, first = decltype(stepc)::value * PER;
        constexpr auto flushed = [](int b) { return GP == 2 && b >= first && b < first + PER; };
        static_for<BLOCKS>([&](auto bc) {
            constexpr int b = decltype(bc)::value, t = b / (CB * IB), i = b / IB % CB, j = b % IB;
            if constexpr (flushed(b)) {
                if constexpr (b < TR) total[b] += acc[t][i][j];
                else spare.add(b - TR, acc[t][i][j]);
            }
        });
        static_for<GP>([&](auto wc) {                 // partial products, smallest first: gp + xp = GP - 1 ... 0
            constexpr int sum = GP - 1 - decltype(wc)::value;
            static_for<GP>([&](auto gc) {
                constexpr int gp = decltype(gc)::value, xp = sum - gp;
                if constexpr (xp >= 0 && xp < XP)
                    static_for<BLOCKS>([&](auto bc) {
                        constexpr int b = decltype(bc)::value, t = b / (CB * IB), i = b / IB % CB, j = b % IB;
                        if constexpr (flushed(b) && sum == 0) {
                            acc[t][i][j] = mfma16<true>(gr[set][t][i][gp], xr[set][j][xp], zeros);
                        } else {
                            floatx16 &d = sum == 0 ? acc[t][i][j] : low[t][i][j];
                            d = mfma16<GP == 2>(gr[set][t][i][gp], xr[set][j][xp], d);
                        }
                    });
            });
        });
        // the loads of the next step spread over the MFMAs of this one
        static_for<BLOCKS * (GP == 2 ? 1 + XP : XP == 1 ? 3 : XP == 2 ? 5 : 6)>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // global read
            __builtin_amdgcn_sched_group_barrier(0x002, GP == 2 ? 3 : 2, 0);   // vector arithmetic
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    using std::integral_constant;
    static_for<SETS - 1>([&](auto setc) { fetch(setc); });
    if constexpr (GP == 3) {
        for (int k = s_begin; k < s_end; k += 2) {
            fetch(integral_constant<int, 1>{});
            multiply(integral_constant<int, 0>{}, integral_constant<int, 0>{});
            fetch(integral_constant<int, 0>{});
            multiply(integral_constant<int, 1>{}, integral_constant<int, 0>{});
        }
    } else {
        for (int k = s_begin; k < s_end; k += E_SEGMENT)             // (steps past the last one: zeros)
            static_for<E_SEGMENT>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                fetch(integral_constant<int, (i + SETS - 1) % SETS>{});
                multiply(integral_constant<int, i % SETS>{}, ic);
            });
    }

    const size_t plane = (size_t)p.Cout * p.Cin;
    static_for<TB>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if (tap0 + t >= NN) return;
        float *o = part + ((size_t)split * NN + tap0 + t) * plane;
        static_for<CB * IB>([&](auto bc) {
            constexpr int i = decltype(bc)::value / IB, j = decltype(bc)::value % IB;
            const int ci = (cib + j) * 32 + (lane & 31), co0 = (cob + i) * 32 + 4 * (lane >> 5);
            floatx16 sum = acc[t][i][j];
            if constexpr (GP == 2) {
                sum += low[t][i][j] * (1.0f / LOW_SCALE);
                constexpr int b = (t * CB + i) * IB + j;
                if constexpr (b < TR) sum += total[b];
                else spare.add_to(b - TR, sum);
            } else {
                sum += low[t][i][j];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int co = co0 + 8 * (r >> 2) + (r & 3);
                if (co < p.Cout && ci < p.Cin)
                    o[(size_t)co * p.Cin + ci] = GP == 2 ? __builtin_amdgcn_ldexpf(sum[r], -(head.ea + head.eb)) : sum[r] * SPLIT_UNSCALE;
            }
        });
    });
}

// TWO: both kinds of parts in one launch, told apart by the head.
template <int n, int XP, int CB, int IB, int TB, bool TWO>
__global__ void __launch_bounds__(E_THREADS, 1) split_dw_kernel(const void *__restrict__ xf, const void *__restrict__ gf,
                                                               float *__restrict__ part, DwParams p)
{
    if constexpr (TWO) {
        const SplitHead head = read_head((const char *)gf + p.g_bytes);
        if (head.two == SPLIT_TWO) {
            split_dw_work<n, XP - 1, 2, CB, IB, TB>(xf, gf, part, p, head);
            return;
        }
    }
    split_dw_work<n, XP, 3, CB, IB, TB>(xf, gf, part, p, {0u, 0, 0, 0u});
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
    int form;                                 // 0: 2 x 2 channel blocks x 2 taps per wave, 1: 1 x 2 x 4, 2: 2 x 1 x 4
    double us;                                // what the plan's cost model says
    DwParams p;
    size_t x_bytes, g_bytes, part_bytes;      // multiples of 1 KB
};

// Large layers with whole tiles of 128 channels and whole groups of items.
// What fills items and channels up to whole blocks is multiplied too.  Both sides timed on 1014 random layers from 3
// to 16 G products: 1.5 times as fast on average, with 1.8 to 2.2 times the products multiplied 25 of 121 layers
// lost.  One kind did not gain: with 9 products per value of g and input channel and at most one tile of those, the
// passes over g (four times the positions) show, and on maps of whole groups of four columns the fp32 multiplies
// are at their best: of 32 such layers 15 lost (68 x 128 x 128 x 24 x 24, P = 3: 220 us here against 181).  bfloat16
// input halves the multiplies and gained there too.
bool whole_items(const Shape &s, kst_dtype dt)
{
    const double edge = s.N - 2 * s.frame, nn = s.n * s.n;
    const double products = (double)s.B * edge * edge * nn * s.Cin * s.Cout;
    const double padded = (double)((s.B + 15) / 16 * 16) * edge * edge * nn * ((s.Cin + 127) / 128 * 128) *
                          ((s.Cout + 127) / 128 * 128);
    const bool g_bound = s.n == 3 && s.Cin <= 128 && dt != KST_BF16 && edge > 8 && ((int)edge & 3) == 0;
    return products >= 3.0e9 && padded <= 1.5 * products && !g_bound;
}

// s: the framed problem with Shape::frame = q; odd: the padding factor is odd.  The scratch is laid out for `parts` parts
// of the input; everything else is chosen without a look at them.  whole: batch items are not cut into strips, a workgroup
// has 128 x 128 channels.
DwPlan dw_plan(const Shape &s, bool odd, int parts, bool whole, bool half = false)
{
    DwPlan r;
    DwParams &p = r.p;
    const int NN = s.n * s.n;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout;
    p.N = s.N - 2 * s.frame;
    p.M = s.M - (odd ? 2 : 0);
    p.q2 = 2 * s.frame - (odd ? 1 : 0);
    r.ok = false;
    r.us = 1e30;
    if (s.n < 3 || s.n > 5) return r;
    const int blocks_co = (s.Cout + 31) / 32, blocks_ci = (s.Cin + 31) / 32;
    if ((double)s.B * p.N * p.N >= 1e9 || (double)blocks_co * blocks_ci * NN >= 1e6) return r;
    // A wave's shape: the one that multiplies least for padding, two taps where that is the same (with one block of input
    // channels a wave loads 27 operands per 48 MFMAs, otherwise 18, where the caches hand over 24 in that time).
    double best = 1e30;
    int waves_co = 1, waves_ci = 1, waves_taps = 1;
    for (int form = 0; form < (whole ? 1 : 3); ++form) {
        const int cb = form == 1 ? 1 : 2, ib = form == 2 ? 1 : 2, tb = form == 0 ? 2 : 4;
        const int co = (blocks_co + cb - 1) / cb, ci = (blocks_ci + ib - 1) / ib, taps = (NN + tb - 1) / tb;
        const double cost = (double)co * ci * taps * (form == 2 ? 1.2 : 1.0);
        if (cost < 0.99 * best) {
            best = cost;
            r.form = form;
            waves_co = co;
            waves_ci = ci;
            waves_taps = taps;
        }
    }
    p.wave_co = whole || waves_co > 1 ? 2 : 1;
    p.wave_ci = whole || waves_ci > 1 ? 2 : 1;
    const int wave_taps = 4 / (p.wave_co * p.wave_ci);
    p.tiles_co = (waves_co + p.wave_co - 1) / p.wave_co;
    p.tiles_ci = (waves_ci + p.wave_ci - 1) / p.wave_ci;
    p.tiles_taps = (waves_taps + wave_taps - 1) / wave_taps;
    const double tiles = (double)p.tiles_co * p.tiles_ci * p.tiles_taps;
    // Strips per batch item: what fills the groups of sixteen against the rows of g that two strips both need.  Times: 48
    // MFMAs of a wave and step in 1.4 us / 256 steps of a CU, operands at 4 TB/s, partial sums at 3.
    const size_t plane = (size_t)s.Cout * s.Cin;
    for (int strips = 1; strips <= (whole ? 1 : p.N); strips = strips < 4 ? strips + 1 : strips + strips / 2) {
        const int R = (p.N + strips - 1) / strips, real = (p.N + R - 1) / R;
        if (real != strips) continue;
        const int GR = whole ? p.M : 2 * R + s.n - 2, groups = (s.B * strips + 15) / 16;
        const double x_bytes = (double)blocks_ci * R * p.N * groups * 3072.0, g_bytes = (double)blocks_co * GR * p.M * groups * 3072.0;
        const int steps = R * p.N * groups;
        // As many splits as give every CU one workgroup, with at least 8 (16) steps each.
        const int least = whole ? 16 : 8;
        int splits = tiles < 256.0 ? (int)(256.0 / tiles) : 1;
        if (splits > steps / least) splits = steps / least > 0 ? steps / least : 1;
        const int per = ((steps + splits - 1) / splits + 1) & ~1;
        splits = (steps + per - 1) / per;
        const double rounds = (double)(long long)((tiles * splits + 255.0) / 256.0);
        const double us = 16.0 + rounds * per * 1.25 + (x_bytes + g_bytes) * 1.7 / 4.0e6 + (splits + 1.0) * plane * NN * 4.0 / 3.0e6;
        if (x_bytes >= 2147483648.0 || g_bytes >= 2147483648.0 || us >= 0.97 * r.us) continue;
        r.us = us;
        r.ok = true;
        p.strips = strips;
        p.R = R;
        p.GR = GR;
        p.yo = whole ? p.q2 : s.n - 1;
        p.groups = groups;
        p.steps = steps;
        p.per_split = per;
        p.splits = splits;
        r.x_bytes = (size_t)blocks_ci * R * p.N * groups * parts * 1024;
        r.g_bytes = (size_t)blocks_co * GR * p.M * groups * 3 * 1024;
        r.part_bytes = ((size_t)splits * NN * plane * sizeof(float) + 255) & ~(size_t)255;
        p.x_bytes = (unsigned)r.x_bytes;
        p.g_bytes = (unsigned)r.g_bytes;
    }
    // Two half-precision parts where that is no less exact than three bfloat16 ones, as in the forward kernel: from 48 steps of
    // a chain (half precision 40), without empty items and taps that meet no g, the error was at most 0.99 of the other's on
    // 442 random layers, below 24 up to 2 times it.  Times as fast on them: 1.30 and 1.21 in the mean, at least 1.05 and 0.99
    // (64 x 512 x 256 x 8 x 8, n = 4, P = 2: 53 us, 81 with three parts).  bfloat16 input: two partial products for three, which
    // the ranges' pass outweighs (0.98).  Steps of products that are not zero: from 22 and 18 (50 layers, 1 to 0.06 of the input not
    // zero: no less exact from 20 to 26 and 15 to 23, at most 1.03 times the other's error from these lines).
    const double values = (double)s.B * s.Cin * p.N * p.N, g_values = (double)s.B * s.Cout * p.M * p.M;
    p.two = 0;
    p.from = 0.0f;
    if (r.ok && parts > 1) {
        const double inside = taps_inside(p.N, s.n, p.q2, p.M) / ((double)p.N * s.n);
        const double steps = p.per_split * inside * inside * s.B * p.N / (16.0 * p.groups * p.R);
        p.from = (float)((half ? 18.0 : 22.0) / steps * values * g_values);
        p.two = steps >= (half ? 40.0 : 48.0) && plane * NN * sizeof(float) >= SPLIT_RANGE_BYTES;
    }
    p.range_share = split_range_share((size_t)(values * (half ? 2 : 4)), (size_t)(g_values * 4));
    return r;
}

template <int n, int XP, class T>
hipError_t dw_launch(const T *in, const float *g, float *dw, char *ws, const DwPlan &pl, hipStream_t stream)
{
    const DwParams &p = pl.p;
    char *xf = ws, *gf = ws + pl.x_bytes;
    float *part = (float *)(gf + pl.g_bytes);
    hipError_t e;
    const RangePart *range = nullptr;
    char *head_end = gf + p.g_bytes;
    if (p.two) {                                      // (the shares lie in the result until both operands are split)
        // (half precision needs no scale: what is infinite or not a number in it is found in the sums)
        e = launch_split_range({in, (size_t)p.B * p.Cin * p.N * p.N, !std::is_same_v<T, float>},
                               {g, (size_t)p.B * p.Cout * p.M * p.M, false}, dw, stream);
        if (e != hipSuccess) return e;
        range = (const RangePart *)dw;
    }
    const Items<T> x_items = items_of(in, xf, p.Cin, p.N, p.R, p.R, 0, p);
    const Items<float> g_items = items_of(g, gf, p.Cout, p.M, p.GR, 2 * p.R, p.q2 - p.yo, p);
    hipLaunchKernelGGL((split_items_kernel<XP, T>), dim3(x_items.blocks() + g_items.blocks()), dim3(256), 0, stream, x_items,
                       g_items, g_items.blocks(), head_end, range, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 blocks((unsigned)p.splits * p.tiles_co * p.tiles_ci * p.tiles_taps), threads(E_THREADS);
    const void *x = xf, *gp = gf;
    auto kernel = pl.form == 0   ? &split_dw_kernel<n, XP, 2, 2, 2, false>
                  : pl.form == 1 ? &split_dw_kernel<n, XP, 1, 2, 4, false>
                                 : &split_dw_kernel<n, XP, 2, 1, 4, false>;
    if constexpr (XP > 1)
        if (p.two)
            kernel = pl.form == 0   ? &split_dw_kernel<n, XP, 2, 2, 2, true>
                     : pl.form == 1 ? &split_dw_kernel<n, XP, 1, 2, 4, true>
                                    : &split_dw_kernel<n, XP, 2, 1, 4, true>;
    hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, x, gp, part, p);
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

// Other layers: batch items cut into strips, a wave's shape by the channels.  Both sides timed on 200 random layers of 0.03
// to 1.3 G products: from 48 input and 32 output channels 1.1 to 1.9 times as fast (2 x 268 x 396 x 17 x 17, n = 5, P = 1,
// bfloat16: 133 -> 70 us), 5 x 5 kernels, where the fp32 multiplies' kernel has no second channel block, from 0.03 G,
// others from 0.25 G: below that, four launches cost what the multiplies save.  Two things did not gain: fp32 input with 3 x
// 3 kernels (0.76 to 1.2, passes over g as above), and one or two batch items in fp32, whose fp32 kernel runs at its best
// on maps of whole groups of four (2 x 778 x 96 x 20 x 20, n = 4: 50 us there against 62).  Fewer channels are mostly padding (3
// output channels of 32: 2 to 2.5 times slower).  Of 614 more layers 27 were slower: 8 of 22 whose only split is three tenths
// and more empty items (1 x 928 x 288 x 10 x 10, n = 5, P = 2, bfloat16: 60 us there, 84 here; strips are few and channels
// many), and with kernels of up to 4 x 4 layers of few channels on both sides, whose sums go round in a hundred splits (32 x 50
// x 64 x 18 x 18, n = 4, half precision: 58 there, 72 here).  Without those the others are 1.39 times as fast, 7 slower by 5 to 13 %.
bool split_dw_applies(const Shape &s, bool odd, kst_dtype dt)
{
    if (s.n < 3 || s.n > 5) return false;
    if (whole_items(s, dt)) return dw_plan(s, odd, 3, true).ok;
    const double edge = s.N - 2 * s.frame;
    const double products = (double)s.B * edge * edge * s.n * s.n * s.Cin * s.Cout;
    if (s.Cout < 32 || s.Cin < 48) return false;
    if (s.n == 5 ? products < 0.03e9 || (dt == KST_F32 && s.B < 2) : products < 0.25e9 || s.B < 2) return false;
    if (dt == KST_F32 && (s.n == 3 || (s.n == 4 && s.B < 4 && ((int)edge & 3) == 0))) return false;
    if (s.n < 5 && s.Cin * s.Cout < 5000) return false;
    const DwPlan r = dw_plan(s, odd, 3, false);
    const double items = (double)s.B * edge / (16.0 * r.p.groups * r.p.R);           // share of the items that are real
    return r.ok && (r.p.splits > 1 || items >= 0.7);
}

// (Eleven bits of half precision are two parts.)
static int parts_of(kst_dtype dt) { return dt == KST_BF16 ? 1 : dt == KST_F16 ? 2 : 3; }

// widest: with room for three parts of the input whatever its type.  (0 for a layer this kernel does not take.)
size_t split_dw_workspace_bytes(const Shape &s, bool odd, kst_dtype dt, bool widest)
{
    if (s.n < 3 || s.n > 5) return 0;
    const DwPlan r = dw_plan(s, odd, widest ? 3 : parts_of(dt), whole_items(s, dt));
    if (!r.ok) return 0;
    return r.x_bytes + r.g_bytes + r.part_bytes;
}

hipError_t launch_split_dw(const void *in, const float *g, float *dw, void *ws, const Shape &s, bool odd, kst_dtype dt,
                           hipStream_t stream)
{
    const DwPlan r = dw_plan(s, odd, parts_of(dt), whole_items(s, dt), dt == KST_F16);
    if (!r.ok) return hipErrorInvalidValue;
    if (dt == KST_BF16) return dw_launch_n<1>((const uint16_t *)in, g, dw, (char *)ws, r, s.n, stream);
    if (dt == KST_F16) return dw_launch_n<2>((const half_bits *)in, g, dw, (char *)ws, r, s.n, stream);
    return dw_launch_n<3>((const float *)in, g, dw, (char *)ws, r, s.n, stream);
}

}  // namespace kst

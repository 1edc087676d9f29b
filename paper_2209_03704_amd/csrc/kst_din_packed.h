// Input gradient on the bf16 matrix cores, g repacked once: any map edge, padding factor and channel counts, kernels of
// 3 x 3 to 5 x 5.  (kst_split_din.hip, which splits g while staging, holds the rows that 128 positions touch of all four
// parities of g at once: only some maps fit, and each block of input channels splits g again.)
//
//   din[b][ci][a][c] = sum_co sum_u sum_v g[b][co][2 (a + q) - u][2 (c + q) - v] * w[co][ci][u][v]
//
// As a GEMM: rows = input channels, columns = positions m = (b, a, c) of the unframed map, reduction over (co, u, v).
// Image row h = 2 a + t (t = n - 1 - u) of g framed by what the taps reach: the rows of one parity, and the columns, make a
// plane in which a tap's positions are shifted by whole cells.  The first launch writes g's three bfloat16 parts as
//   [batch][chunk][parity][part][row][column][16 channels]
// with the frame's zeros, and the weights' parts in MFMA operand order.  The second walks (chunk, parity): the rows of one
// plane that a tile's positions touch go through LDS (two stages, a barrier per step, 16-byte groups as they lie), weights
// straight into registers some taps ahead.
//
// Few output channels (at most four, S2D): the sixteen values of a chunk are four channels times the four parities, so a
// window of ceil(n / 2)^2 cells has all taps (those past the kernel's edge: zero weights) and no MFMA multiplies twelve
// empty channels.
//
// What bounds it: small layers by the launches and a step's latency (0.5 us: g's planes are asked for two steps ahead), large
// ones by the multiplies and the first launch's traffic (4.9 TB/s of 4 bytes read and 6 and the frame written per value).
// Against the fp32 multiplies' kernels on 150 random layers of up to 1.3 G products: 1.43 times as fast in the mean
// (4 x 192 x 456 x 12 x 12, n = 5, P = 3, half precision: 92 -> 37 us; 173 x 32 x 104 x 12 x 12, n = 5: 224 -> 62; one step
// ahead instead of two: 1.36 in the mean); 64 x 128 x 3 x 32 x 32, n = 4, P = 2: 33 -> 29.  Error against 64 bits: 0.3 to
// 1 of before.  One block per wave where workgroups are few (two per CU), 2 x 2 blocks, which read half as much from LDS
// and the caches per multiply, where the cost model says so.
#pragma once
#include "kst_din_store.h"

namespace kst {

namespace {

constexpr int F_THREADS = 256;
constexpr unsigned F_OUTSIDE = 0x80000000u;   // byte offset past every buffer here (all below 2 GB)

struct DinPackedParams : DinShape {
    int Hp, Wp;                               // rows and columns of a plane
    int tiles_m, tiles_ci, splits;
    int chunks, chunks_per_split;
    int groups;                               // 16-byte groups of a tile's rows of one part: 2 per cell
    unsigned g_bytes, w_bytes;                // of the operands
    unsigned plane;                           // bytes of one part of a plane
    unsigned g_blocks, w_tasks;               // of the first launch
};

// Steps of a chunk (parities), taps of a step.
template <int n, bool S2D>
struct DinSteps {
    static constexpr int side = (n + 1) / 2, steps = S2D ? 1 : 4, taps = S2D ? side * side : n * n;
    static constexpr int width(int step) { return S2D ? side : taps_for_parity(n, step & 1); }
    static constexpr int count(int step) { return S2D ? taps : class_taps(n, step); }
    static constexpr int first(int step) { return S2D ? 0 : class_tap_base(n, step); }
};

// Two neighbouring values of a row of g, zero outside the map.
__device__ __forceinline__ void g_pair(const float *row, bool inside, int x, int M, float &a, float &b)
{
    a = inside && x >= 0 && x < M ? row[x] : 0.0f;
    b = inside && x + 1 >= 0 && x + 1 < M ? row[x + 1] : 0.0f;
}

// The first p.g_blocks workgroups: g -> its parts, a lane one cell and eight of the chunk's sixteen values (both column
// parities of one row parity, or all four parities).  The others: w -> its parts, a wave (block of 32 input channels, chunk,
// u): [block][chunk][tap][part][lane][8 values].
template <int n, int WP, bool S2D, class T>
__global__ void __launch_bounds__(F_THREADS) din_pack_kernel(const float *__restrict__ g, const T *__restrict__ w,
                                                             char *__restrict__ gx, char *__restrict__ wx, DinPackedParams p)
{
    using Steps = DinSteps<n, S2D>;
    if (blockIdx.x < p.g_blocks) {
        const size_t i = (size_t)blockIdx.x * F_THREADS + threadIdx.x;
        const int kk = (int)(i & 1);
        size_t t = i >> 1;
        const int c = (int)(t % (unsigned)p.Wp);
        t /= (unsigned)p.Wp;
        const int r = (int)(t % (unsigned)p.Hp);
        t /= (unsigned)p.Hp;
        int py = 0;
        if (!S2D) {
            py = (int)(t & 1);
            t >>= 1;
        }
        const int chunk = (int)(t % (unsigned)p.chunks), b = (int)(t / (unsigned)p.chunks);
        if (b >= p.B) return;
        const int x = 2 * c + p.shift;
        const size_t map = (size_t)p.M * p.M;
        char *cell = gx + (((size_t)b * p.chunks + chunk) * Steps::steps * 3) * p.plane + ((size_t)r * p.Wp + c) * 32 + kk * 16;
        float v[2][8];
        if constexpr (S2D) {
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int co = chunk * 4 + kk * 2 + o;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int y = 2 * r + h + p.shift;
                    const bool inside = co < p.Cout && y >= 0 && y < p.M;
                    g_pair(g + ((size_t)b * p.Cout + (inside ? co : 0)) * map + (inside ? (size_t)y * p.M : 0), inside, x, p.M,
                           v[0][4 * o + 2 * h], v[0][4 * o + 2 * h + 1]);
                }
            }
        } else {
            const int y = 2 * r + py + p.shift;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int co = chunk * 16 + kk * 8 + j;
                const bool inside = co < p.Cout && y >= 0 && y < p.M;
                g_pair(g + ((size_t)b * p.Cout + (inside ? co : 0)) * map + (inside ? (size_t)y * p.M : 0), inside, x, p.M, v[0][j],
                       v[1][j]);
            }
        }
#pragma unroll
        for (int px = 0; px < (S2D ? 1 : 2); ++px) {
            bf16x8 part[3];
            split3(v[px], part[0], part[1], part[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *reinterpret_cast<bf16x8 *>(cell + (size_t)((2 * py + px) * 3 + k) * p.plane) = part[k];
        }
        return;
    }
    const unsigned task = (blockIdx.x - p.g_blocks) * 4u + (threadIdx.x >> 6);
    if (task >= p.w_tasks) return;
    constexpr int ROWS = S2D ? Steps::side : n;               // tasks per block and chunk: rows of cells, or u
    const unsigned block = task / ROWS;
    const int rowt = (int)(task - block * ROWS);
    const int blk = (int)(block / (unsigned)p.chunks), chunk = (int)(block - (unsigned)blk * p.chunks);
    const int lane = threadIdx.x & 63, ci = blk * 32 + (lane & 31), kk = lane >> 5;
    char *d = wx + (size_t)block * Steps::taps * (WP * 1024) + lane * 16;
    auto put = [&](int tap, const float (&v)[8]) {
        bf16x8 part[3];
        split3(v, part[0], part[1], part[2]);
#pragma unroll
        for (int k = 0; k < WP; ++k) *reinterpret_cast<bf16x8 *>(d + (tap * WP + k) * 1024) = part[k];
    };
    if constexpr (S2D) {
#pragma unroll
        for (int dx = 0; dx < Steps::side; ++dx) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int co = chunk * 4 + kk * 2 + (j >> 2), u = n - 1 - (2 * rowt + ((j >> 1) & 1)), x = n - 1 - (2 * dx + (j & 1));
                v[j] = ci < p.Cin && co < p.Cout && u >= 0 && x >= 0
                           ? weight_of(w, (((size_t)co * p.Cin + ci) * n + u) * n + x)
                           : 0.0f;
            }
            put(rowt * Steps::side + dx, v);
        }
    } else {
        float t[8][n];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < n; ++v) {
                const int co = chunk * 16 + kk * 8 + j;
                t[j][v] = ci < p.Cin && co < p.Cout ? weight_of(w, (((size_t)co * p.Cin + ci) * n + rowt) * n + v) : 0.0f;
            }
        const int ty = n - 1 - rowt, py = ty & 1;
#pragma unroll
        for (int v = 0; v < n; ++v) {
            const int tx = n - 1 - v, px = tx & 1;
            float eight[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) eight[j] = t[j][v];
            put((py ? class_tap_base(n, 2 + px) : class_tap_base(n, px)) + (ty >> 1) * taps_for_parity(n, px) + (tx >> 1), eight);
        }
    }
}

// Four waves along the positions, PB blocks of 32 each, RB blocks of 32 input channels; the largest partial products' sums
// apart from the others'.
template <int n, int WP, bool S2D, int PB, int RB, int NT, class T>
__global__ void __launch_bounds__(F_THREADS, PB * RB == 1 && (S2D || NT == 3) ? 2 : 1)
    din_packed_kernel(const float *__restrict__ g, const T *__restrict__ w, const char *__restrict__ gx, const char *__restrict__ wx,
                      float *__restrict__ din, float *__restrict__ ws, DinPackedParams p)
{
    using Steps = DinSteps<n, S2D>;
    constexpr int TAPS = Steps::taps, TM = 128 * PB, PART = NT * F_THREADS * 16, STAGE = 3 * PART;
    constexpr int SETS = TAPS % 4 == 0 ? 4 : TAPS % 3 == 0 ? 3 : 5, AHEAD = SETS - 1;     // (divides the taps)
    constexpr int TAP = WP * 1024;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    unsigned id = blockIdx.x;
    const int tile_ci = (int)(id % (unsigned)p.tiles_ci);
    id /= (unsigned)p.tiles_ci;
    const int tile_m = (int)(id % (unsigned)p.tiles_m), split = (int)(id / (unsigned)p.tiles_m);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NN = p.N * p.N, m0 = tile_m * TM, b0 = m0 / NN;
    const int R0 = b0 * p.Hp + (m0 - b0 * NN) / p.N;           // first row of the tile, rows stacked over batch items

    int xa[PB];                                                // LDS byte address of the window's first cell
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const DinColumn c = din_column(p, m0 + (wave * PB + pb) * 32 + l32);
        xa[pb] = ((c.mb * p.Hp + c.ma - R0) * p.Wp + c.mc) * 32 + kk * 16;
    }
    const __amdgpu_buffer_rsrc_t gbuf = buffer_of(gx, p.g_bytes), wbuf = buffer_of(wx, p.w_bytes);
    unsigned x_off[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int group = tid + F_THREADS * k, cell = group >> 1;
        const int lr = cell / p.Wp, c = cell - lr * p.Wp, R = R0 + lr, b = R / p.Hp;
        x_off[k] = group < p.groups && b < p.B ? (unsigned)b * p.chunks * (Steps::steps * 3) * p.plane +
                                                     ((unsigned)(R - b * p.Hp) * p.Wp + c) * 32u + (group & 1) * 16u
                                               : F_OUTSIDE;
    }
    // The planes of the next DEPTH steps are on their way (a step of few taps is over before memory has answered).
    constexpr int DEPTH = S2D ? 1 : 2;
    bf16x8 x_reg[DEPTH][3][NT];
    auto fetch_x = [&](auto setc, int step) {                  // step: chunk * steps + parity
        constexpr int set = decltype(setc)::value;
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int k = 0; k < NT; ++k) x_reg[set][part][k] = load_bf16x8(gbuf, x_off[k], (unsigned)(step * 3 + part) * p.plane);
    };
    auto write_x = [&](auto setc, int stage) {
        constexpr int set = decltype(setc)::value;
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int k = 0; k < NT; ++k)
                *reinterpret_cast<bf16x8 *>(lds + stage + part * PART + (tid + F_THREADS * k) * 16) = x_reg[set][part][k];
    };
    bf16x8 wf[SETS][RB][WP];
    unsigned w_base[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
        w_base[rb] = (unsigned)min(tile_ci * RB + rb, (p.Cin - 1) / 32) * p.chunks * (TAPS * TAP);
    auto fetch_w = [&](auto qc, int chunk) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int part = 0; part < WP; ++part)
                wf[q % SETS][rb][part] = load_bf16x8(wbuf, lane * 16 + part * 1024, w_base[rb] + (unsigned)(chunk * TAPS + q) * TAP);
    };
    floatx16 acc[RB][PB], low[RB][PB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[rb][pb][v] = low[rb][pb][v] = 0.0f;

    using std::integral_constant;
    const int k0 = split * p.chunks_per_split, k1 = min(p.chunks, k0 + p.chunks_per_split), last_step = k1 * Steps::steps - 1;
    fetch_x(integral_constant<int, 0>{}, k0 * Steps::steps);
    if constexpr (DEPTH == 2) fetch_x(integral_constant<int, 1>{}, k0 * Steps::steps + 1);
    static_for<AHEAD>([&](auto qc) { fetch_w(qc, k0); });
    write_x(integral_constant<int, 0>{}, 0);
    int stage = 0;
    for (int chunk = k0; chunk < k1; ++chunk) {
        const int next = min(chunk + 1, k1 - 1);               // (past the last chunk: read again, never multiplied)
        static_for<Steps::steps>([&](auto sc) {
            constexpr int step = decltype(sc)::value, q0 = Steps::first(step), COUNT = Steps::count(step), W = Steps::width(step);
            __syncthreads();                                   // this step's stage is written, the other one is free
            fetch_x(integral_constant<int, step % DEPTH>{}, min(chunk * Steps::steps + step + DEPTH, last_step));
            bf16x8 xf[2][PB][3];
            auto read_x = [&](auto ic) {
                constexpr int i = decltype(ic)::value;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int part = 0; part < 3; ++part)
                        xf[i & 1][pb][part] = *reinterpret_cast<const bf16x8 *>(lds + stage + part * PART + xa[pb] +
                                                                                ((i / W) * p.Wp + i % W) * 32);
            };
            read_x(integral_constant<int, 0>{});
            static_for<COUNT>([&](auto ic) {
                constexpr int i = decltype(ic)::value, q = q0 + i;
                if constexpr (i + 1 < COUNT) read_x(integral_constant<int, i + 1>{});
                fetch_w(integral_constant<int, (q + AHEAD) % TAPS>{}, q + AHEAD < TAPS ? chunk : next);
                static_for<3>([&](auto sumc) {                 // partial products, smallest first: xp + wp = 2, 1, 0
                    constexpr int sum = 2 - decltype(sumc)::value;
                    static_for<WP>([&](auto wc) {
                        constexpr int wp = decltype(wc)::value, xp = sum - wp;
                        if constexpr (xp >= 0) {
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                                for (int pb = 0; pb < PB; ++pb) {
                                    floatx16 &to = sum == 0 ? acc[rb][pb] : low[rb][pb];
                                    to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q % SETS][rb][wp], xf[i & 1][pb][xp], to, 0, 0, 0);
                                }
                        }
                    });
                });
                __builtin_amdgcn_sched_barrier(0);             // (left alone, every load is moved down to its use)
            });
            stage = STAGE - stage;
            if (step + 1 < Steps::steps || chunk + 1 < k1) write_x(integral_constant<int, (step + 1) % DEPTH>{}, stage);
        });
    }
    const bool whole = p.splits == 1;
    static_for<PB * RB>([&](auto ic) {
        constexpr int i = decltype(ic)::value, pb = i / RB, rb = i % RB;
        float a[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = (acc[rb][pb][v] + low[rb][pb][v]) * SPLIT_UNSCALE;
        if (whole) {
            din_store<n, true>(g, w, din, p, a, (tile_ci * RB + rb) * 32 + 4 * kk, din_column(p, m0 + (wave * PB + pb) * 32 + l32));
        } else {
            // [split][position block][channel block][4 values of a lane]
            const size_t blk = ((size_t)split * (p.tiles_m * 4 * PB) + (tile_m * 4 + wave) * PB + pb) * (p.tiles_ci * RB) +
                               tile_ci * RB + rb;
            float4 *d = reinterpret_cast<float4 *>(ws + blk * 1024) + lane;
#pragma unroll
            for (int v = 0; v < 4; ++v) d[v * 64] = make_float4(a[4 * v], a[4 * v + 1], a[4 * v + 2], a[4 * v + 3]);
        }
    });
}

// One wave per block of 32 positions and 32 input channels: its partial sums in split order.
template <int n, class T>
__global__ void __launch_bounds__(F_THREADS) din_packed_sum_kernel(const float *__restrict__ g, const T *__restrict__ w,
                                                                   float *__restrict__ din, const float *__restrict__ ws,
                                                                   DinPackedParams p, unsigned blocks, unsigned ci_blocks)
{
    const unsigned blk = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (blk >= blocks) return;
    const int lane = threadIdx.x & 63, pos = (int)(blk / ci_blocks), ci = (int)(blk % ci_blocks);
    float a[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] = 0.0f;
#pragma unroll 2
    for (int s = 0; s < p.splits; ++s) {
        const float4 *d = reinterpret_cast<const float4 *>(ws + ((size_t)s * blocks + blk) * 1024) + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = d[q * 64];
            a[4 * q] += v.x;
            a[4 * q + 1] += v.y;
            a[4 * q + 2] += v.z;
            a[4 * q + 3] += v.w;
        }
    }
    din_store<n, false>(g, w, din, p, a, ci * 32 + 4 * (lane >> 5), din_column(p, pos * 32 + (lane & 31)));
}

struct DinPackedPlan {
    bool ok, s2d;
    int pb, rb, nt;
    double us;                                // what the cost model says
    DinPackedParams p;
    size_t g_bytes, w_bytes, part_bytes;      // multiples of 256
};

inline DinPackedPlan din_packed_plan_for(const Shape &s, bool odd, int wp, int block)
{
    DinPackedPlan r;
    DinPackedParams &p = r.p;
    const int n = s.n;
    r.ok = false;
    r.us = 1e30;
    r.pb = r.rb = block;
    if (n < 3 || n > 5) return r;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout;
    p.N = s.N - 2 * s.frame;
    p.M = s.M - (odd ? 2 : 0);
    p.shift = 2 * s.frame - (odd ? 1 : 0) - (n - 1);
    r.s2d = s.Cout <= 4;
    p.Hp = p.Wp = p.N + (n - 1) / 2;
    if ((double)s.B * p.Hp * p.Hp >= 1e9 || (r.s2d && block > 1)) return r;
    p.Mtot = s.B * p.N * p.N;
    const int tm = 128 * block, tci = 32 * block, side = (n + 1) / 2;
    const int steps = r.s2d ? 1 : 4, taps = r.s2d ? side * side : n * n;
    p.tiles_m = (p.Mtot + tm - 1) / tm;
    p.tiles_ci = (s.Cin + tci - 1) / tci;
    p.chunks = (s.Cout + (r.s2d ? 3 : 15)) / (r.s2d ? 4 : 16);
    const int dg = (tm - 2) / p.N + 1, crossings = (dg + p.N - 1) / p.N;   // rows tm positions can step over, items they enter
    const size_t groups = (size_t)(dg + crossings * (p.Hp - p.N) + (n - 1) / 2 + 1) * p.Wp * 2;
    const size_t plane = (size_t)p.Hp * p.Wp * 32;
    const size_t g_bytes = (size_t)s.B * p.chunks * steps * 3 * plane;
    const size_t blocks_ci = (size_t)(s.Cin + 31) / 32, w_bytes = blocks_ci * p.chunks * taps * wp * 1024;
    const unsigned long long tiles = (unsigned long long)p.tiles_m * p.tiles_ci;
    if (groups > 5 * F_THREADS || g_bytes >= F_OUTSIDE || w_bytes >= F_OUTSIDE || tiles > (1u << 20)) return r;
    r.nt = block == 1 && groups <= 3 * F_THREADS ? 3 : 5;
    p.groups = (int)groups;
    p.plane = (unsigned)plane;
    p.g_bytes = (unsigned)g_bytes;
    p.w_bytes = (unsigned)w_bytes;
    r.g_bytes = (g_bytes + 255) & ~(size_t)255;
    r.w_bytes = (w_bytes + 255) & ~(size_t)255;
    const size_t lanes = (size_t)s.B * p.chunks * (r.s2d ? 1 : 2) * p.Hp * p.Wp * 2;
    p.g_blocks = (unsigned)((lanes + F_THREADS - 1) / F_THREADS);
    p.w_tasks = (unsigned)(blocks_ci * p.chunks * (r.s2d ? side : n));
    // Splits of the reduction by the time they would take: rounds of as many workgroups as fit the chip (two per CU where
    // their stages do), 3 us each beside the multiplies; a step takes 0.5 us however few its taps are; a split adds its
    // partial sums.
    const double tap = 0.016 * block * block * (wp == 1 ? 3 : wp == 2 ? 5 : 6) * taps;         // us per chunk
    const double at_once = r.nt == 3 ? 512.0 : 256.0, floor = 0.5 * steps;
    const double sums = (double)tiles * tm * tci * 4.0;
    p.splits = 1;
    p.chunks_per_split = p.chunks;
    for (int c = 1; c <= 16 && c <= p.chunks; ++c) {
        const int cps = (p.chunks + c - 1) / c;
        if ((p.chunks + cps - 1) / cps != c) continue;
        const double wgs = (double)tiles * c, rounds = (double)(long long)((wgs + at_once - 1.0) / at_once);
        const double shared = wgs > 256.0 ? at_once / 256.0 : 1.0, chunk = tap * shared > floor ? tap * shared : floor;
        const double us = rounds * (cps * chunk + 3.0) + (c > 1 ? 4.0 + (c + 1) * sums / 4.0e6 : 0.0);
        if (us < 0.95 * r.us) {
            r.us = us;
            p.splits = c;
            p.chunks_per_split = cps;
        }
    }
    r.part_bytes = p.splits > 1 ? (size_t)p.splits * tiles * tm * tci * sizeof(float) : 0;
    r.us += 4.0 + (g_bytes * 1.7 + w_bytes * 1.7) / 4.0e6;
    r.ok = true;
    return r;
}

inline int din_packed_parts(kst_dtype dt) { return dt == KST_BF16 ? 1 : dt == KST_F16 ? 2 : 3; }   // (eleven bits are two parts)

inline DinPackedPlan din_packed_plan(const Shape &s, bool odd, kst_dtype dt)
{
    const DinPackedPlan one = din_packed_plan_for(s, odd, din_packed_parts(dt), 1);
    const DinPackedPlan two = din_packed_plan_for(s, odd, din_packed_parts(dt), 2);
    if (!two.ok || (one.ok && one.us <= two.us)) return one;
    return two;
}

template <int n, int WP, bool S2D, int BLOCK, int NT, class T>
hipError_t din_packed_launch_tile(const float *g, const T *w, float *din, char *ws, const DinPackedPlan &pl, hipStream_t stream)
{
    const DinPackedParams &p = pl.p;
    char *gx = ws, *wx = ws + pl.g_bytes;
    float *part = (float *)(wx + pl.w_bytes);
    hipLaunchKernelGGL((din_pack_kernel<n, WP, S2D, T>), dim3(p.g_blocks + (p.w_tasks + 3) / 4), dim3(F_THREADS), 0, stream, g, w,
                       gx, wx, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int stage = 3 * NT * F_THREADS * 16;
    const int lds = S2D && p.chunks == 1 ? stage : 2 * stage;  // (a single step has no next one)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&din_packed_kernel<n, WP, S2D, BLOCK, BLOCK, NT, T>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 2 * stage);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((din_packed_kernel<n, WP, S2D, BLOCK, BLOCK, NT, T>), dim3((unsigned)p.tiles_m * p.tiles_ci * p.splits),
                       dim3(F_THREADS), lds, stream, g, w, (const char *)gx, (const char *)wx, din, part, p);
    e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    const unsigned ci_blocks = (unsigned)p.tiles_ci * BLOCK, blocks = (unsigned)p.tiles_m * 4 * BLOCK * ci_blocks;
    hipLaunchKernelGGL((din_packed_sum_kernel<n, T>), dim3((blocks + 3) / 4), dim3(F_THREADS), 0, stream, g, w, din,
                       (const float *)part, p, blocks, ci_blocks);
    return hipGetLastError();
}

template <int n, int WP, class T>
hipError_t din_packed_launch(const float *g, const T *w, float *din, char *ws, const DinPackedPlan &pl, hipStream_t stream)
{
    if (pl.s2d)
        return pl.nt == 3 ? din_packed_launch_tile<n, WP, true, 1, 3>(g, w, din, ws, pl, stream)
                          : din_packed_launch_tile<n, WP, true, 1, 5>(g, w, din, ws, pl, stream);
    if (pl.pb == 2) return din_packed_launch_tile<n, WP, false, 2, 5>(g, w, din, ws, pl, stream);
    return pl.nt == 3 ? din_packed_launch_tile<n, WP, false, 1, 3>(g, w, din, ws, pl, stream)
                      : din_packed_launch_tile<n, WP, false, 1, 5>(g, w, din, ws, pl, stream);
}

template <int n>
hipError_t din_packed_launch_any(const float *g, const void *w, float *din, void *ws, const DinPackedPlan &pl, kst_dtype dt,
                                 hipStream_t stream)
{
    if (dt == KST_BF16) return din_packed_launch<n, 1>(g, (const uint16_t *)w, din, (char *)ws, pl, stream);
    if (dt == KST_F16) return din_packed_launch<n, 2>(g, (const half_bits *)w, din, (char *)ws, pl, stream);
    return din_packed_launch<n, 3>(g, (const float *)w, din, (char *)ws, pl, stream);
}

}  // namespace

}  // namespace kst

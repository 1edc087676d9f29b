// fp32 forward layers on the bf16 matrix cores, the input repacked once: any channel counts, map edges and padding factors,
// kernels of 3 x 3 to 5 x 5.  (kst_split_f32.h, for large layers, splits the input while staging, once per block of 128
// output channels and row parity; its tiles and shared passes want 1.5 G products and many channels to pay.  Which layers come
// here: kst_fwd_packed.hip.)
//
// Section 3.3, Eqs. 7-10: quad positions m = (b * E + i) * E + j across the columns of the MFMAs, input channels 16 at a
// time.  The first launch writes the input's three bfloat16 parts as [batch][chunk][part][row][column][16 channels], the
// zero frame of a padded layer included, and the weights' parts in MFMA operand order.  The second stages the rows that a
// tile's positions touch in 16-byte groups (two stages, one barrier per chunk) and multiplies them in one of two forms:
//   classes   rows = 32 output channels, four accumulators, the taps of the four classes one after the other;
//   rows      rows = 8 output channels x four classes, one accumulator: at a window offset the rows of a class that has no
//             tap there are zero weights.  ceil(n / 2 + 1/2)^2 MFMAs instead of n^2, for few output channels.  One or two
//             blocks of positions a wave; in the classes form two would be 256 accumulators, and the rest spilled (16 x 20 x
//             288 x 100 x 100, n = 3, P = 1: 665 us, one block 597).
//
// What bounds it: small layers by three launches and a chunk's latency, large ones by the multiplies and the first launch's
// traffic (4 bytes read and 6 and the frame written per value).  Against the kernels that ran them before, 538
// random layers that come here: 2.2 times as fast in the mean, 2.9 where the plain fp32 kernel was the other one (5 x 26 x 288 x
// 40 x 40, n = 5: 156 -> 45 us; 5 x 160 x 67 x 37 x 37, n = 4, P = 2: 169 -> 44); rows form: 46 x 248 x 3 x 11 x 11, n = 4, P = 2:
// 46 -> 27.  Error against 64 bits on 2598 random layers: 0.10 to 0.95 of before.
#pragma once
#include "kst_fwd_store.h"

namespace kst {

namespace {

constexpr int P_THREADS = 256;
constexpr unsigned P_OUTSIDE = 0x80000000u;   // byte offset past every buffer here (all below 2 GB)

struct FwdPackedParams : FwdShape {
    int tiles_m, co_blocks, splits;           // co_blocks: of 32 (classes) or 8 (rows) output channels
    int chunks, chunks_per_split;
    int groups;                               // 16-byte groups of a tile's rows of one part: 2 per position
    unsigned x_bytes, w_bytes;                // of the operands
    unsigned plane;                           // bytes of one part of a chunk's framed map
    unsigned x_blocks, w_tasks;               // of the first launch
};

// The first p.x_blocks workgroups: the input, a lane one position of the framed map and eight channels.  The others: weights,
// a wave (block of output channels, chunk, tap): [block][chunk][tap][part][lane][8 channels].
template <int n, bool ROWS>
__global__ void __launch_bounds__(P_THREADS) fwd_pack_kernel(const float *__restrict__ in, const float *__restrict__ w_seg,
                                                             char *__restrict__ x, char *__restrict__ wx, FwdPackedParams p)
{
    static constexpr FwdTaps<n, ROWS> order{};
    constexpr int TAPS = FwdTaps<n, ROWS>::taps, side = FwdTaps<n, ROWS>::side;
    float v[8];
    bf16x8 part[3];
    if (blockIdx.x < p.x_blocks) {
        const size_t i = (size_t)blockIdx.x * P_THREADS + threadIdx.x;
        const int kk = (int)(i & 1);
        size_t t = i >> 1;
        const int c = (int)(t % (unsigned)p.N);
        t /= (unsigned)p.N;
        const int r = (int)(t % (unsigned)p.N);
        t /= (unsigned)p.N;
        const int chunk = (int)(t % (unsigned)p.chunks), b = (int)(t / (unsigned)p.chunks);
        if (b >= p.B) return;
        const int y = r - p.q, col = c - p.q, ci = chunk * 16 + kk * 8;
        const bool inside = y >= 0 && y < p.N0 && col >= 0 && col < p.N0;
        const size_t map = (size_t)p.N0 * p.N0;
        const float *src = in + ((size_t)b * p.Cin + min(ci, p.Cin - 1)) * map + (inside ? (size_t)y * p.N0 + col : 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = inside && ci + j < p.Cin ? src[j * map] : 0.0f;
        split3(v, part[0], part[1], part[2]);
        char *d = x + ((size_t)b * p.chunks + chunk) * 3 * p.plane + ((size_t)r * p.N + c) * 32 + kk * 16;
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<bf16x8 *>(d + (size_t)k * p.plane) = part[k];
        return;
    }
    const unsigned task = (blockIdx.x - p.x_blocks) * 4u + (threadIdx.x >> 6);
    if (task >= p.w_tasks) return;
    const unsigned block = task / TAPS, q = task - block * TAPS;
    const int blk = (int)(block / (unsigned)p.chunks), chunk = (int)(block - (unsigned)blk * p.chunks);
    const int lane = threadIdx.x & 63, l32 = lane & 31, ci = chunk * 16 + 8 * (lane >> 5);
    int cls, local, co;
    bool real;
    if constexpr (ROWS) {
        cls = l32 & 3;
        co = blk * 8 + (l32 >> 2);
        const int a = (int)q / side - (cls >> 1), b = (int)q % side - (cls & 1), Tb = taps_for_parity(n, cls & 1);
        real = a >= 0 && a < taps_for_parity(n, cls >> 1) && b >= 0 && b < Tb;
        local = a * Tb + b;
    } else {
        cls = order.cls[q];
        local = order.local[q];
        co = blk * 32 + l32;
        real = true;
    }
    const int Tp = taps_for_parity(n, cls >> 1) * taps_for_parity(n, cls & 1);
    const unsigned off = cls == 0 ? p.off[0] : cls == 1 ? p.off[1] : cls == 2 ? p.off[2] : p.off[3];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = real && co < p.Cout && ci + j < p.Cin ? w_seg[off + ((size_t)(ci + j) * Tp + local) * p.Cout + co] : 0.0f;
    split3(v, part[0], part[1], part[2]);
    char *d = wx + ((size_t)block * TAPS + q) * 3072 + lane * 16;
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<bf16x8 *>(d + k * 1024) = part[k];
}

// A block's sums, in LDS as own[(item * 4 + class) * 64 + lane], to the output: items are a lane's 16 output channels
// (classes) or its four (rows).  Sums that are not finite are taken from fp32 multiplies first.
template <int n, bool ROWS>
__device__ __forceinline__ void fwd_finish(const float *__restrict__ in, const float *__restrict__ w_seg, float *__restrict__ out,
                                           const FwdPackedParams &p, float *own, int blk, const Column &c)
{
    constexpr int ITEMS = ROWS ? 4 : 16;
    const int lane = threadIdx.x & 63, l32 = lane & 31, kk = lane >> 5;
    float zero = 0.0f;
#pragma unroll 4
    for (int i = 0; i < ITEMS * 4; ++i) zero = fmaf(own[i * 64], 0.0f, zero);
    if (__builtin_expect(__ballot(zero != 0.0f) != 0, 0)) {    // (all lanes of the wave, also those past the last position)
#pragma unroll 1
        for (int cls = 0; cls < 4; ++cls) {
            const floatx16 f = fp32_class_block<n, true>(in, w_seg, p, c, cls >> 1, cls & 1, blk * (ROWS ? 8 : 32) + l32);
            static_for<ITEMS>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                float again;
                if constexpr (ROWS) {                          // row 2 i + kk of the block's first eight
                    const int from = l32 + 32 * (i >> 1);
                    const float even = __shfl(f[2 * (i & 1)], from), odd = __shfl(f[2 * (i & 1) + 1], from);
                    again = kk ? odd : even;
                } else {
                    again = f[i];
                }
                float *mine = own + (i * 4 + cls) * 64;
                if (*mine * 0.0f != 0.0f) *mine = again;
            });
        }
    }
    if (!c.valid) return;
#pragma unroll 4
    for (int i = 0; i < ITEMS; ++i) {
        const int co = ROWS ? blk * 8 + 2 * i + kk : blk * 32 + 8 * (i >> 2) + 4 * kk + (i & 3);
        const float *mine = own + i * 256;
        if (co < p.Cout) {
            store_pair(out, p, mine[0], mine[64], 0, co, c);
            store_pair(out, p, mine[128], mine[192], 1, co, c);
        }
    }
}

// Four waves along the positions, PB blocks of 32 each (two: rows form), one block of output channels; the largest partial
// products' sums apart from the others'.
template <int n, bool ROWS, int PB, int NT>
__global__ void __launch_bounds__(P_THREADS, PB == 1 && (ROWS || NT == 3) ? 2 : 1)
    fwd_packed_kernel(const float *__restrict__ in, const float *__restrict__ w_seg, const char *__restrict__ x,
                      const char *__restrict__ wx, float *__restrict__ out, float *__restrict__ ws, FwdPackedParams p)
{
    constexpr FwdTaps<n, ROWS> order{};
    constexpr int TAPS = FwdTaps<n, ROWS>::taps, side = FwdTaps<n, ROWS>::side, OFFSETS = side * side;
    constexpr int TM = 128 * PB, PART = NT * P_THREADS * 16, STAGE = 3 * PART, NA = ROWS ? 1 : 4;
    constexpr int SETS = TAPS % 4 == 0 ? 4 : TAPS % 3 == 0 ? 3 : 5, AHEAD = SETS - 1;     // (divides the taps)
    constexpr int ITEMS = ROWS ? 4 : 16;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    unsigned id = blockIdx.x;
    const int blk = (int)(id % (unsigned)p.co_blocks);
    id /= (unsigned)p.co_blocks;
    const int tile_m = (int)(id % (unsigned)p.tiles_m), split = (int)(id / (unsigned)p.tiles_m);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = tile_m * TM, b0 = m0 / p.EE;
    const int R0 = b0 * p.N + (m0 - b0 * p.EE) / p.E;          // first row of the tile, rows stacked over batch items

    int xa[PB];                                                // LDS byte address of the window's first position
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const Column c = column_of(p, m0, wave * PB + pb, l32);
        xa[pb] = ((c.mb * p.N + c.mi - R0) * p.N + c.mj) * 32 + kk * 16;
    }
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(x, p.x_bytes), wbuf = buffer_of(wx, p.w_bytes);
    unsigned x_off[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int group = tid + P_THREADS * k, pos = group >> 1;
        const int lr = pos / p.N, c = pos - lr * p.N, R = R0 + lr, b = R / p.N;
        x_off[k] = group < p.groups && b < p.B ? (unsigned)b * p.chunks * 3u * p.plane + ((unsigned)(R - b * p.N) * p.N + c) * 32u +
                                                     (group & 1) * 16u
                                               : P_OUTSIDE;
    }
    bf16x8 x_reg[3][NT];
    auto fetch_x = [&](int chunk) {
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int k = 0; k < NT; ++k) x_reg[part][k] = load_bf16x8(xbuf, x_off[k], (unsigned)(chunk * 3 + part) * p.plane);
    };
    auto write_x = [&](int stage) {
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int k = 0; k < NT; ++k)
                *reinterpret_cast<bf16x8 *>(lds + stage + part * PART + (tid + P_THREADS * k) * 16) = x_reg[part][k];
    };
    bf16x8 wf[SETS][3];
    const unsigned w_base = (unsigned)blk * p.chunks * (TAPS * 3072);
    auto fetch_w = [&](auto qc, int chunk) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int part = 0; part < 3; ++part)
            wf[q % SETS][part] = load_bf16x8(wbuf, lane * 16 + part * 1024, w_base + (unsigned)(chunk * TAPS + q) * 3072u);
    };
    floatx16 acc[NA][PB], low[NA][PB];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][pb][v] = low[a][pb][v] = 0.0f;
    // Rows form, whose layers are cut into few splits: every fourth chunk the largest products' sums go to a total and start
    // again, for an error that does not grow with all of a long reduction's roundings (2 x 195 x 104 x 24 x 24, n = 5: 2.2e-7 as
    // one chain, 1.6e-7 on the kernel before).
    floatx16 total[ROWS ? PB : 1];
#pragma unroll
    for (int pb = 0; pb < (ROWS ? PB : 1); ++pb)
#pragma unroll
        for (int v = 0; v < 16; ++v) total[pb][v] = 0.0f;

    using std::integral_constant;
    const int k0 = split * p.chunks_per_split, k1 = min(p.chunks, k0 + p.chunks_per_split);
    fetch_x(k0);
    static_for<AHEAD>([&](auto qc) { fetch_w(qc, k0); });
    write_x(0);
    int stage = 0;
    for (int chunk = k0; chunk < k1; ++chunk) {
        const int next = min(chunk + 1, k1 - 1);               // (past the last chunk: read again, never multiplied)
        __syncthreads();                                       // this chunk's stage is written, the other one is free
        fetch_x(next);
        bf16x8 xf[2][PB][3];
        auto read_x = [&](auto oc) {
            constexpr int o = decltype(oc)::value;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int part = 0; part < 3; ++part)
                    xf[o & 1][pb][part] = *reinterpret_cast<const bf16x8 *>(lds + stage + part * PART + xa[pb] +
                                                                            ((o / side) * p.N + o % side) * 32);
        };
        read_x(integral_constant<int, 0>{});
        static_for<TAPS>([&](auto qc) {
            constexpr int q = decltype(qc)::value, o = order.offset[q], a = ROWS ? 0 : order.cls[q];
            if constexpr ((q == 0 || order.offset[q == 0 ? 0 : q - 1] != o) && o + 1 < OFFSETS) read_x(integral_constant<int, o + 1>{});
            fetch_w(integral_constant<int, (q + AHEAD) % TAPS>{}, q + AHEAD < TAPS ? chunk : next);
            static_for<3>([&](auto sumc) {                     // partial products, smallest first: xp + wp = 2, 1, 0
                constexpr int sum = 2 - decltype(sumc)::value;
                static_for<sum + 1>([&](auto wc) {
                    constexpr int wp = decltype(wc)::value, xp = sum - wp;
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) {
                        floatx16 &to = sum == 0 ? acc[a][pb] : low[a][pb];
                        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q % SETS][wp], xf[o & 1][pb][xp], to, 0, 0, 0);
                    }
                });
            });
            __builtin_amdgcn_sched_barrier(0);                 // (left alone, every load is moved down to its use)
        });
        stage = STAGE - stage;
        if (chunk + 1 < k1) write_x(stage);
        if constexpr (ROWS) {
            if (((chunk - k0) & 3) == 3) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        total[pb][v] += acc[0][pb][v];
                        acc[0][pb][v] = 0.0f;
                    }
            }
        }
    }
    // A wave's own part of LDS takes the sums: the stores are a loop then and not a copy of their code per register.
    __syncthreads();
    float *own = reinterpret_cast<float *>(lds) + wave * (ITEMS * 256) + lane;
    static_for<PB>([&](auto pbc) {
        constexpr int pb = decltype(pbc)::value;
        const Column c = column_of(p, m0, wave * PB + pb, l32);
        auto sum = [&](auto ic) {
            constexpr int i = decltype(ic)::value, a = ROWS ? 0 : i & 3, v = ROWS ? i : i >> 2;
            if constexpr (ROWS) return (total[pb][v] + (acc[a][pb][v] + low[a][pb][v])) * SPLIT_UNSCALE;
            return (acc[a][pb][v] + low[a][pb][v]) * SPLIT_UNSCALE;
        };
        if (p.splits == 1) {
            static_for<ITEMS * 4>([&](auto ic) { own[decltype(ic)::value * 64] = sum(ic); });
            fwd_finish<n, ROWS>(in, w_seg, out, p, own, blk, c);
        } else {
            float *d = ws + (((size_t)split * (p.tiles_m * 4 * PB) + (tile_m * 4 + wave) * PB + pb) * p.co_blocks + blk) * (ITEMS * 256) +
                       lane;
            static_for<ITEMS * 4>([&](auto ic) { d[decltype(ic)::value * 64] = sum(ic); });
        }
    });
}

// One wave per block of 32 positions and of output channels: its partial sums in split order.
template <int n, bool ROWS>
__global__ void __launch_bounds__(P_THREADS) fwd_packed_sum_kernel(const float *__restrict__ in, const float *__restrict__ w_seg,
                                                                   float *__restrict__ out, const float *__restrict__ ws,
                                                                   FwdPackedParams p, unsigned blocks)
{
    constexpr int ITEMS = ROWS ? 4 : 16;
    __shared__ float lds[4 * ITEMS * 256];
    const unsigned at = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (at >= blocks) return;
    const int lane = threadIdx.x & 63;
    float a[ITEMS * 4];
#pragma unroll
    for (int i = 0; i < ITEMS * 4; ++i) a[i] = 0.0f;
    for (int s = 0; s < p.splits; ++s) {
        const float *d = ws + ((size_t)s * blocks + at) * (ITEMS * 256) + lane;
#pragma unroll
        for (int i = 0; i < ITEMS * 4; ++i) a[i] += d[i * 64];
    }
    float *own = lds + (threadIdx.x >> 6) * (ITEMS * 256) + lane;
#pragma unroll
    for (int i = 0; i < ITEMS * 4; ++i) own[i * 64] = a[i];
    fwd_finish<n, ROWS>(in, w_seg, out, p, own, (int)(at % (unsigned)p.co_blocks),
                        column_of(p, 0, (int)(at / (unsigned)p.co_blocks), lane & 31));
}

struct FwdPackedPlan {
    bool ok, rows;
    int pb, nt;
    double us;                                // what the cost model says
    FwdPackedParams p;
    size_t x_bytes, w_bytes, part_bytes;      // multiples of 256
};

inline FwdPackedPlan fwd_packed_plan_for(const Shape &s, bool rows, int pb)
{
    FwdPackedPlan r;
    FwdPackedParams &p = r.p;
    const int n = s.n;
    r.ok = false;
    r.rows = rows;
    r.pb = pb;
    r.us = 1e30;
    if (n < 3 || n > 5 || s.Ns != s.N) return r;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout; p.N = s.N; p.M = s.M - 2 * s.crop; p.E = s.E; p.EE = s.E * s.E;
    p.q = s.frame;
    p.N0 = s.N - 2 * s.frame;
    p.crop = s.crop;
    p.epi = s.epi;
    for (int c = 0; c < 4; ++c) p.off[c] = (unsigned)seg_offset(s.Cin, s.Cout, n, c, KST_F32);
    if (p.N0 < 1 || (double)s.B * s.N * s.N >= 1e9) return r;
    p.Mtot = s.B * p.EE;
    const int tm = 128 * pb, tco = rows ? 8 : 32, side = n / 2 + 1, taps = rows ? side * side : n * n;
    p.tiles_m = (p.Mtot + tm - 1) / tm;
    p.co_blocks = (s.Cout + tco - 1) / tco;
    p.chunks = (s.Cin + 15) / 16;
    const int dg = (tm - 2) / s.E + 1, crossings = (dg + s.E - 1) / s.E;   // quad rows tm positions can step over, items they enter
    const size_t groups = (size_t)(dg + crossings * (s.N - s.E) + s.fl + 1) * s.N * 2;
    const size_t plane = (size_t)s.N * s.N * 32, x_bytes = (size_t)s.B * p.chunks * 3 * plane;
    const size_t w_bytes = (size_t)p.co_blocks * p.chunks * taps * 3072;
    const unsigned long long tiles = (unsigned long long)p.tiles_m * p.co_blocks;
    if (groups > 5 * P_THREADS || x_bytes >= P_OUTSIDE || w_bytes >= P_OUTSIDE || tiles > (1u << 20)) return r;
    r.nt = groups <= 3 * P_THREADS ? 3 : 5;
    p.groups = (int)groups;
    p.plane = (unsigned)plane;
    p.x_bytes = (unsigned)x_bytes;
    p.w_bytes = (unsigned)w_bytes;
    r.x_bytes = (x_bytes + 255) & ~(size_t)255;
    r.w_bytes = (w_bytes + 255) & ~(size_t)255;
    p.x_blocks = (unsigned)(((size_t)s.B * p.chunks * s.N * s.N * 2 + P_THREADS - 1) / P_THREADS);
    p.w_tasks = (unsigned)p.co_blocks * p.chunks * taps;
    // Splits of the reduction by the time they would take: rounds of as many workgroups as fit the chip, 4 us each beside the
    // multiplies; a chunk takes 0.6 us however few its taps are; a split adds its partial sums.
    const double at_once = r.nt == 3 && pb == 1 ? 512.0 : 256.0, tap = 0.1 * pb * taps;
    const double sums = (double)tiles * tm * tco * 4.0 * 4.0;
    p.splits = 1;
    p.chunks_per_split = p.chunks;
    for (int c = 1; c <= 16 && c <= p.chunks; ++c) {
        const int cps = (p.chunks + c - 1) / c;
        if ((p.chunks + cps - 1) / cps != c) continue;
        const double wgs = (double)tiles * c, rounds = (double)(long long)((wgs + at_once - 1.0) / at_once);
        const double shared = wgs > 256.0 ? at_once / 256.0 : 1.0, chunk = tap * shared > 0.6 ? tap * shared : 0.6;
        const double us = rounds * (cps * chunk + 4.0) + (c > 1 ? 4.0 + (c + 1) * sums / 4.0e6 : 0.0);
        if (us < 0.95 * r.us) {
            r.us = us;
            p.splits = c;
            p.chunks_per_split = cps;
        }
    }
    r.part_bytes = p.splits > 1 ? (size_t)p.splits * p.tiles_m * 4 * pb * p.co_blocks * (rows ? 4096 : 16384) : 0;
    // (a chunk's loads show where a lane stages five groups; within 11 % on 1223 random layers)
    r.us = 9.0 + (r.nt == 3 ? 1.17 : 1.47) * r.us + 0.22e-6 * x_bytes + 0.8e-6 * w_bytes + 0.3e-6 * 4 * s.B * s.Cin * (double)s.N * s.N +
           0.17e-6 * 4 * s.B * s.Cout * (double)s.M * s.M;
    r.ok = true;
    return r;
}

// (Two position blocks are for the rows form only: the four classes' sums of two blocks are 256 accumulators, and the rest
// spilled.)
inline FwdPackedPlan fwd_packed_plan(const Shape &s)
{
    FwdPackedPlan best;
    best.ok = false;
    for (int i = 0; i < 3; ++i) {
        const FwdPackedPlan r = fwd_packed_plan_for(s, i > 0, i < 2 ? 1 : 2);
        if (r.ok && (!best.ok || r.us < best.us)) best = r;
    }
    return best;
}

template <int n, bool ROWS, int PB, int NT>
hipError_t fwd_packed_launch_tile(const float *in, const float *w_seg, float *out, char *ws, const FwdPackedPlan &pl, hipStream_t stream)
{
    const FwdPackedParams &p = pl.p;
    char *x = ws, *wx = ws + pl.x_bytes;
    float *part = (float *)(wx + pl.w_bytes);
    hipLaunchKernelGGL((fwd_pack_kernel<n, ROWS>), dim3(p.x_blocks + (p.w_tasks + 3) / 4), dim3(P_THREADS), 0, stream, in, w_seg, x, wx, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int lds = 2 * 3 * NT * P_THREADS * 16;           // (the stores' 64 KB are fewer)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fwd_packed_kernel<n, ROWS, PB, NT>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fwd_packed_kernel<n, ROWS, PB, NT>), dim3((unsigned)p.tiles_m * p.co_blocks * p.splits), dim3(P_THREADS), lds,
                       stream, in, w_seg, (const char *)x, (const char *)wx, out, part, p);
    e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    const unsigned blocks = (unsigned)p.tiles_m * 4 * PB * p.co_blocks;
    hipLaunchKernelGGL((fwd_packed_sum_kernel<n, ROWS>), dim3((blocks + 3) / 4), dim3(P_THREADS), 0, stream, in, w_seg, out,
                       (const float *)part, p, blocks);
    return hipGetLastError();
}

template <int n, bool ROWS>
hipError_t fwd_packed_launch(const float *in, const float *w_seg, float *out, char *ws, const FwdPackedPlan &pl, hipStream_t stream)
{
    if constexpr (ROWS)
        if (pl.pb == 2)
            return pl.nt == 3 ? fwd_packed_launch_tile<n, true, 2, 3>(in, w_seg, out, ws, pl, stream)
                              : fwd_packed_launch_tile<n, true, 2, 5>(in, w_seg, out, ws, pl, stream);
    return pl.nt == 3 ? fwd_packed_launch_tile<n, ROWS, 1, 3>(in, w_seg, out, ws, pl, stream)
                      : fwd_packed_launch_tile<n, ROWS, 1, 5>(in, w_seg, out, ws, pl, stream);
}

template <int n>
hipError_t fwd_packed_launch_any(const float *in, const float *w_seg, float *out, void *ws, const FwdPackedPlan &pl, hipStream_t stream)
{
    return pl.rows ? fwd_packed_launch<n, true>(in, w_seg, out, (char *)ws, pl, stream)
                   : fwd_packed_launch<n, false>(in, w_seg, out, (char *)ws, pl, stream);
}

}  // namespace

}  // namespace kst

// Segregated forward pass of fp32 layers on the bf16 matrix cores (operands split into three bfloat16 parts or, where the
// reduction is long, two of half precision, see kst_split_common.h).
//
// Section 3.3, Eqs. 7-10, as four implicit GEMMs that share one input tile, as in the fp32 matrix-core kernel: output
// channels down the MFMA rows, quad positions m = (b * E + i) * E + j across its columns.  The reduction walks the input channels 16 at a time (one 32x32x16 MFMA).
//
// What bounds it: the multiplies and, behind them, the issue slots of the one wave each SIMD holds (an MFMA leaves
// room for about five other instructions).  A workgroup of four waves owns 128 positions x 128 output channels (or
// 256 x 64) and one row parity; a wave owns 32 output channels and four blocks of 32 positions: two column parities x
// four blocks x (the largest partial products' sums and the others'), 256 accumulator registers.  Per kernel tap a
// wave issues 24 MFMAs (768 cycles; two parts: 12) and needs the weights of its own 32 output channels only: a first kernel splits
// all weights once and lays them out as MFMA operands, so that a wave's next three (two) operands are one contiguous 3 (2) KB,
// loaded straight into registers two to four taps ahead.  (Split in the main loop instead, 44 vector instructions
// and eight 4-byte loads per tap: 548 us against 488 on 128 x 512 x 256 x 16 x 16, n = 4, when it was tried; 471 with three
// parts, MFMAs busy in 64 % of the main kernel's cycles; 352 with two: half the MFMAs, busy in 42 %, the other cycles go to a
// wave's other instructions and its waits for LDS.)  Input values are
// wanted by every wave and every tap: the rows the tile's positions touch are split once per chunk and kept in LDS as
// [part][channel half][row, column][8 channels], so that a lane's MFMA operand is one 16-byte read; two stages, one
// barrier per chunk.  Taps are walked by window offset: the taps of both column parities that meet the same input
// element share one set of reads.
//
// The kernel reads tensors as they lie in memory: a zero frame (padding factor) is supplied while staging, channel
// counts and map edges may be any number (loads past the tensor return zeros, rows past Cout are not stored).
#pragma once
#include "kst_fwd_store.h"

namespace kst {

namespace {

constexpr int S_THREADS = 256;
constexpr int S_KC = 16;            // input channels per chunk
constexpr int S_GROUP = 2;          // two parts: chunks after which each of the accumulators has been added to the total
constexpr int S_IP = 640;           // input positions (stacked rows x columns) a stage can hold
constexpr unsigned S_OUTSIDE = 0x80000000u;   // byte offset past every buffer here (all below 2 GB)
constexpr int S_TAP = 1024;         // bytes of one part of one tap's split weights for 32 output and 16 input channels
constexpr int S_NT = S_IP / 128;    // (position, channel half) pairs a lane stages per chunk at most

struct SplitParams : FwdShape {
    int tiles_m, tiles_co;
    int ip;                // positions staged: lrows * N
    int chunks;            // of S_KC input channels
    int unit;              // chunks that are never shared out one by one (two parts: a group of the sums' total)
    unsigned in_bytes, w_bytes;   // input tensor, split weights
    unsigned w_pass1;      // byte offset of row parity 1 in one part's weights
    int two;               // operands of two half-precision parts where their ranges allow
    int range_share;       // workgroups of the ranges' launch that took the input
    float from;            // ... and of all pairs of an input value and a weight, how many at least have no zero
};

// Order of the taps of row parity r: by window offset (row a of the sub-kernels, column dx), then column parity s.
template <int n, int r>
struct TapOrder {
    static constexpr int side = n / 2 + 1, rows = taps_for_parity(n, r), offsets = rows * side, taps = rows * n;
    int s[taps] = {}, local[taps] = {}, offset[taps] = {};     // column parity, tap within its class, window offset
    int first[offsets + 1] = {};                               // first tap of a window offset
    constexpr TapOrder()
    {
        int q = 0;
        for (int o = 0; o < offsets; ++o) {
            first[o] = q;
            for (int sp = 0; sp < 2; ++sp) {
                const int b = o % side - sp, Tb = taps_for_parity(n, sp);
                if (b < 0 || b >= Tb) continue;
                s[q] = sp;
                local[q] = o / side * Tb + b;
                offset[q] = o;
                ++q;
            }
        }
        first[offsets] = q;
    }
};

// Two parts: the taps of a group of chunks during which a block's sums go to the total, and the next tap that
// multiplies into it.
template <int n, int r>
struct FlushOrder {
    static constexpr int GROUP = S_GROUP;
    int at[2][4] = {}, next[2][4] = {};                // [column parity][block of positions]
    constexpr FlushOrder()
    {
        constexpr TapOrder<n, r> order{};
        constexpr int TAPS = TapOrder<n, r>::taps;
        for (int s = 0; s < 2; ++s) {
            int last = GROUP * TAPS - 1, others = 0;   // taps of the other column parity before the last of this one
            while (order.s[last % TAPS] != s) --last;
            for (int t = 0; t < last; ++t) others += order.s[t % TAPS] != s;
            for (int pb = 0; pb < 4; ++pb) {
                int nth = pb * others / 4, t = 0;
                while (order.s[t % TAPS] == s || nth-- > 0) ++t;
                at[s][pb] = t;
                while (order.s[t % TAPS] != s) ++t;
                next[s][pb] = t;
            }
        }
    }
    constexpr int count(int t) const
    {
        int c = 0;
        for (int s = 0; s < 2; ++s)
            for (int pb = 0; pb < 4; ++pb) c += at[s][pb] == t;
        return c;
    }
};

// LDS of a kernel that stages NT positions per lane: two stages, or what the waves' stores use.
constexpr int split_half(int NT) { return NT * 128 * 16; }            // bytes: one channel half of one part
constexpr int split_stage(int NT, int parts) { return parts * 2 * split_half(NT); }
constexpr int S_OWN = 16384;                                            // of a wave, from the start
// Two parts: totals of S_TOTALS of the eight accumulator blocks lie behind both.
constexpr int S_TOTALS = 4;
constexpr int split_totals_at(int NT) { return 2 * split_stage(NT, 2) > 4 * S_OWN ? 2 * split_stage(NT, 2) : 4 * S_OWN; }
constexpr int split_lds(int NT, bool two)
{
    const int three = 2 * split_stage(NT, 3) > 4 * S_OWN ? 2 * split_stage(NT, 3) : 4 * S_OWN;
    const int both = split_totals_at(NT) + S_TOTALS * 16 * S_THREADS * 4;
    return two && both > three ? both : three;
}

// WR: waves along the output channels (4 / WR along the positions); every wave: 32 channels x 128 positions.
template <int WR>
struct TileShape {
    static constexpr int tco = 32 * WR, tm = 128 * (4 / WR);
};

// acc[column parity][block of 32 positions] = the sums of the tile's rows of parity r over channel chunks [k0, k1).
// PARTS: three bfloat16 parts, or two half-precision ones scaled as the head says.
template <int n, int r, int WR, int NT, int PARTS>
__device__ __forceinline__ void split_accumulate(const float *__restrict__ in, const void *__restrict__ w_split,
                                                 const SplitParams &p, const SplitHead &head, char *lds, int tile_m,
                                                 int tile_co, int k0, int k1, int tid, floatx16 (&acc)[2][4])
{
    using TS = TileShape<WR>;
    using Order = TapOrder<n, r>;
    constexpr Order order{};
    constexpr int side = Order::side, rows = Order::rows, TAPS = Order::taps;
    constexpr int HALF = split_half(NT), PART = 2 * HALF, STAGE = split_stage(NT, PARTS);

    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kk = lane >> 5;
    const int wrow = wave % WR, wcol = wave / WR;
    const int m0 = tile_m * TS::tm;
    const int b0 = m0 / p.EE;
    const int i0 = (m0 - b0 * p.EE) / p.E;
    const int R0 = b0 * p.N + i0;                     // first stacked (framed) input row of the tile

    // LDS byte address of the window's first column in the rows of this parity, for the four blocks of positions
    int xa[4][rows];
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
        const int m = min(m0 + (wcol * 4 + pb) * 32 + l32, p.Mtot - 1);
        const int mb = m / p.EE, mrem = m - mb * p.EE;
        const int mi = mrem / p.E, mj = mrem - mi * p.E;
        const int pos = (mb * p.N + mi - R0) * p.N + mj;
#pragma unroll
        for (int a = 0; a < rows; ++a) xa[pb][a] = (pos + (r + a) * p.N) * 16 + kk * HALF;
    }

    // Input staging: wave -> channel half wave & 1, positions (wave >> 1) * 64 + lane + 128 k of the tile's rows.
    // Positions in the frame or past the last batch item, and channels past the last, read past the buffer: zero.
    const int half = wave & 1;
    const unsigned plane = 4u * (unsigned)p.N0 * p.N0;
    const int spos = (wave >> 1) * 64 + lane;
    unsigned x_off[NT];                               // byte offset of channel 0
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int pos = spos + 128 * k;
        const int lr = pos / p.N, x = pos - lr * p.N - p.q;
        const int R = R0 + lr, bb = R / p.N, y = R - bb * p.N - p.q;
        const bool ok = pos < p.ip && bb < p.B && y >= 0 && y < p.N0 && x >= 0 && x < p.N0;
        x_off[k] = ok ? (unsigned)bb * p.Cin * plane + 4u * ((unsigned)y * p.N0 + x) : S_OUTSIDE;
    }
    float x_reg[NT][8];
    auto fetch_x = [&](int chunk) {
        const int c = chunk * S_KC + half * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool live = c + j < p.Cin;          // uniform
            const __amdgpu_buffer_rsrc_t buf = buffer_of(in, live ? p.in_bytes : 0u);
            const unsigned at = live ? (unsigned)(c + j) * plane : 0u;
#pragma unroll
            for (int k = 0; k < NT; ++k) x_reg[k][j] = load_f32(buf, x_off[k], at);
        }
    };
    auto write_x = [&](auto kc, int stage) {
        constexpr int k = decltype(kc)::value;
        bf16x8 part[3];
        if constexpr (PARTS == 2) split2(x_reg[k], head.ea, part[0], part[1]);
        else split3(x_reg[k], part[0], part[1], part[2]);
        char *d = lds + stage + half * HALF + (spos + 128 * k) * 16;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) *reinterpret_cast<bf16x8 *>(d + i * PART) = part[i];
    };

    // Weights: tap q of a chunk is in register set q % SETS, loaded SETS - 1 taps ahead.
    constexpr int SETS = n;                           // divides both parities' taps; 4 for n = 4
    bf16x8 wp[SETS][PARTS];
    const __amdgpu_buffer_rsrc_t wbuf = buffer_of(w_split, p.w_bytes);
    const unsigned w_base = (r ? p.w_pass1 * PARTS : 0u) +
                            (unsigned)min(tile_co * WR + wrow, (p.Cout - 1) / 32) * p.chunks * (TAPS * PARTS * S_TAP);
    auto fetch_w = [&](auto qc, int chunk) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int part = 0; part < PARTS; ++part)
            wp[q % SETS][part] = load_bf16x8(wbuf, lane * 16 + part * S_TAP, w_base + (unsigned)((PARTS == 2 ? min(chunk, p.chunks - 1) : chunk) * TAPS + q) * (PARTS * S_TAP));
    };

    // One set of input registers: a part is read for the next window offset as soon as the last MFMAs that want it
    // for the current one are issued.
    bf16x8 xf[4][PARTS];
    int stage = 0;                                    // the stage reads go to
    auto read_x = [&](auto oc, auto partc) {
        constexpr int o = decltype(oc)::value, part = decltype(partc)::value;
#pragma unroll
        for (int pb = 0; pb < 4; ++pb)
            xf[pb][part] = *reinterpret_cast<const bf16x8 *>(lds + stage + xa[pb][o / side] + (o % side) * 16 + part * PART);
    };

    // The smaller partial products are added up on their own and join the largest one's sums at the end: a sum
    // of a few thousand products is then rounded at its own size twice per MFMA of the largest products only.  (All
    // six into one accumulator: relative error 6.0e-7 against 64 bits on 128 x 512 x 256 x 16 x 16, n = 4, where the
    // fp32 multiplies had 5.2e-7.)  Of two parts the largest products' sums are added to a total every S_GROUP chunks and start
    // again; some totals are in LDS: beside two accumulators of each block registers are short.
    constexpr int TR = 8 - S_TOTALS;
    const LdsTotals<S_THREADS> spare = {reinterpret_cast<float4 *>(lds + split_totals_at(NT)) + tid};
    floatx16 low[2][4], total[TR], zeros;
#pragma unroll
    for (int v = 0; v < 16; ++v) zeros[v] = 0.0f;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int pb = 0; pb < 4; ++pb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[c][pb][v] = low[c][pb][v] = 0.0f;
                if (c * 4 + pb < TR) total[c * 4 + pb][v] = 0.0f;
            }
    if constexpr (PARTS == 2)
        static_for<S_TOTALS>([&](auto bc) { spare.clear(decltype(bc)::value); });

    using std::integral_constant;
    // The tap during which the k-th staged position of the next chunk goes to LDS, and how many a tap has.
    constexpr auto write_tap = [](int k) { return TAPS - 2 - k % ((TAPS - 1) / 2); };
    constexpr auto staged_in = [=](int q) {
        int count = 0;
        for (int k = 0; k < NT; ++k) count += write_tap(k) == q;
        return count;
    };
    fetch_x(k0);
    static_for<SETS - 1>([&](auto qc) { fetch_w(qc, k0); });
    static_for<NT>([&](auto kc) { write_x(kc, 0); });
    fetch_x(min(k0 + 1, k1 - 1));
    __syncthreads();
    static_for<PARTS>([&](auto pc) { read_x(integral_constant<int, 0>{}, pc); });

    // Two parts: in every group of chunks each block's sums are added to the total once, while a tap of the other
    // column parity is multiplied, and its next MFMA starts from zero.
    constexpr int GROUP = PARTS == 2 ? S_GROUP : 1;
    constexpr FlushOrder<n, r> flush{};
    for (int chunk0 = k0; chunk0 < k1; chunk0 += GROUP) {
        static_for<GROUP * TAPS>([&](auto tc) {
            constexpr int t = decltype(tc)::value, q = t % TAPS, sp = order.s[q], o = order.offset[q];
            constexpr bool last = q == TAPS - 1;
            constexpr int o_next = last ? 0 : order.offset[last ? 0 : q + 1];
            // (past the last chunk: read again, never multiplied)
            const int chunk = chunk0 + t / TAPS, next = min(chunk + 1, k1 - 1);
            if constexpr (last) {
                // Every wave has written its share of the next chunk's stage and is done reading this one's.
                stage = STAGE - stage;
                __syncthreads();
                fetch_x(min(chunk + 2, k1 - 1));
            }
            fetch_w(integral_constant<int, (q + SETS - 1) % TAPS>{}, q + SETS - 1 < TAPS ? chunk : next);
            // the next chunk's input, in the second half of this one
            static_for<NT>([&](auto kc) {
                if constexpr (write_tap(decltype(kc)::value) == q) write_x(kc, STAGE - stage);
            });
            if constexpr (PARTS == 2)
                static_for<4>([&](auto pbc) {
                    constexpr int pb = decltype(pbc)::value;
                    if constexpr (flush.at[1 - sp][pb] == t) {
                        constexpr int b = (1 - sp) * 4 + pb;
                        if constexpr (b < TR) total[b] += acc[1 - sp][pb];
                        else spare.add(b - TR, acc[1 - sp][pb]);
                    }
                });
            static_for<PARTS>([&](auto xc) {          // parts of the input, smallest first
                constexpr int xp = PARTS - 1 - decltype(xc)::value;
                static_for<PARTS - xp>([&](auto wc) { // ... against the parts of the weights that matter
                    constexpr int w = PARTS - 1 - xp - decltype(wc)::value;
                    static_for<4>([&](auto pbc) {
                        constexpr int pb = decltype(pbc)::value;
                        if constexpr (PARTS == 2 && w + xp == 0 && flush.next[sp][pb] == t) {
                            acc[sp][pb] = mfma16<true>(wp[q % SETS][w], xf[pb][xp], zeros);
                        } else {
                            floatx16 &sum = w + xp == 0 ? acc[sp][pb] : low[sp][pb];
                            sum = mfma16<PARTS == 2>(wp[q % SETS][w], xf[pb][xp], sum);
                        }
                    });
                });
                if constexpr (o_next != o) read_x(integral_constant<int, o_next>{}, integral_constant<int, xp>{});
            });
            // spread the tap's other instructions over its MFMAs: one wave per SIMD has nothing else to hide them
            constexpr int MF = PARTS == 2 ? 12 : 24;
            constexpr int valu = (8 + (PARTS == 2 ? 32 : 56) * staged_in(q) + (PARTS == 2 ? 32 * flush.count(t) : 0) + MF - 1) / MF;
            static_for<MF>([&](auto) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, valu, 0);   // vector arithmetic
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);      // LDS read
                __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);      // global read
                __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);      // LDS write
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    const int down = -(head.ea + head.eb);
    static_for<8>([&](auto bc) {
        constexpr int b = decltype(bc)::value, c = b / 4, pb = b % 4;
        floatx16 &sum = acc[c][pb];
        if constexpr (PARTS == 2) {
            sum += low[c][pb] * (1.0f / LOW_SCALE);
            if constexpr (b < TR) sum += total[b];
            else spare.add_to(b - TR, sum);
        } else {
            sum += low[c][pb];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = PARTS == 2 ? __builtin_amdgcn_ldexpf(sum[v], down) : sum[v] * SPLIT_UNSCALE;
    });
}

constexpr size_t S_SLOT = (size_t)S_THREADS * 128;     // floats of one workgroup's sums of one row parity

template <int n, int r, int WR, int NT, int PARTS>
__device__ __forceinline__ void do_piece(const float *__restrict__ in, const float *__restrict__ w_seg,
                                         const void *__restrict__ w_split, float *__restrict__ out,
                                         float *__restrict__ slot, const SplitParams &p, const SplitHead &head, char *lds,
                                         int tile, int c0, int c1, bool whole, int tid)
{
    using TS = TileShape<WR>;
    const int tile_m = tile % p.tiles_m, tile_co = tile / p.tiles_m;
    // A fresh copy of the lane number: the staging plan is worked out anew for every piece instead of being kept in
    // registers across the pieces.
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    floatx16 acc[2][4];
    split_accumulate<n, r, WR, NT, PARTS>(in, w_split, p, head, lds, tile_m, tile_co, c0, c1, tid, acc);
    // (Three parts: not `whole`, nor, where units are single chunks, c0 and c1 by way of p.unit.  With those the compiler kept 128 of the sums in scratch, read
    // back among the stores, each read a wait for the stores before it: 93 x 24 x 174 x 22 x 22, n = 3, P = 1: 205 us, 120 so.)
    if (PARTS == 2 ? whole : c0 == 0 && c1 == p.chunks) {
        const int co_base = tile_co * TS::tco + (wave % WR) * 32 + 4 * (lane >> 5);
        float zero = 0.0f;                            // NaN where one of the sums is infinite or not a number
        static_for<128>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            zero = fmaf(acc[i & 1][i >> 5][(i >> 1) & 15], 0.0f, zero);
        });
        const bool redo = __ballot(zero != 0.0f) != 0;
        if (p.epi.act != KST_ACT_TANH && !redo) {
            // Straight from the registers: pairs of elements where every row starts at an even one and no map is cropped.
            const size_t plane = (size_t)p.M * p.M;
            float bias[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) bias[v] = p.epi.bias ? p.epi.bias[min(co_base + 8 * (v >> 2) + (v & 3), p.Cout - 1)] : 0.0f;
            const float lo = epi_floor(p.epi.act);
            static_for<4>([&](auto pbc) {
                constexpr int pb = decltype(pbc)::value;
                const Column c = column_of(p, tile_m * TS::tm, (wave / WR) * 4 + pb, lane & 31);
                const int y = 2 * c.mi + r - p.crop, x = 2 * c.mj - p.crop;
                const bool row = c.valid && y >= 0 && y < p.M;
                float *q = out + ((size_t)c.mb * p.Cout + co_base) * plane + (ptrdiff_t)y * p.M + x;
                if ((p.M & 1) == 0 && !p.crop) {      // uniform
                    static_for<16>([&](auto vc) {
                        constexpr int v = decltype(vc)::value, d = 8 * (v >> 2) + (v & 3);
                        if (row && co_base + d < p.Cout)
                            *reinterpret_cast<float2 *>(q + d * plane) =
                                make_float2(epi_max(acc[0][pb][v] + bias[v], lo), epi_max(acc[1][pb][v] + bias[v], lo));
                    });
                } else {
                    const bool left = row && x >= 0 && x < p.M, right = row && x + 1 < p.M;
                    static_for<16>([&](auto vc) {
                        constexpr int v = decltype(vc)::value, d = 8 * (v >> 2) + (v & 3);
                        if (co_base + d < p.Cout) {
                            if (left) q[d * plane] = epi_max(acc[0][pb][v] + bias[v], lo);
                            if (right) q[d * plane + 1] = epi_max(acc[1][pb][v] + bias[v], lo);
                        }
                    });
                }
            });
            return;
        }
        // Otherwise through a wave's own 16 KB of LDS ([position block][register][column parity][lane]): tanh and the
        // blocks that have to be done again are a loop and not 64 copies of the code.
        float *own = reinterpret_cast<float *>(lds + wave * S_OWN) + lane;
        static_for<2>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            static_for<64>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                own[i * 64] = acc[i & 1][2 * h + (i >> 5)][(i >> 1) & 15];
            });
            for (int pb = 0; pb < 2; ++pb) {
                const Column c = column_of(p, tile_m * TS::tm, (wave / WR) * 4 + 2 * h + pb, lane & 31);
                for (int s = 0; redo && s < 2; ++s) {
                    float *mine = own + (pb * 32 + s) * 64;
                    float bad = 0.0f;
                    for (int v = 0; v < 16; ++v) bad = fmaf(mine[v * 128], 0.0f, bad);
                    if (__ballot(bad != 0.0f) == 0) continue;
                    const floatx16 f = fp32_class_block<n, true>(in, w_seg, p, c, r, s,
                                                                 tile_co * TS::tco + (wave % WR) * 32 + (lane & 31));
                    static_for<16>([&](auto vc) {
                        constexpr int v = decltype(vc)::value;
                        if (mine[v * 128] * 0.0f != 0.0f) mine[v * 128] = f[v];
                    });
                }
#pragma unroll 4
                for (int v = 0; v < 16; ++v) {
                    const int co = co_base + 8 * (v >> 2) + (v & 3);
                    const float v0 = own[(pb * 32 + 2 * v) * 64], v1 = own[(pb * 32 + 2 * v + 1) * 64];
                    if (c.valid && co < p.Cout) store_pair(out, p, v0, v1, r, co, c);
                }
            }
        });
    } else {
        float4 *d = reinterpret_cast<float4 *>(slot);
        static_for<32>([&](auto ic) {                 // [position block][pair of registers][column parity 0, 1]
            constexpr int i = decltype(ic)::value, pb = i >> 3, v = 2 * (i & 7);
            d[i * S_THREADS + tid] = make_float4(acc[0][pb][v], acc[1][pb][v], acc[0][pb][v + 1], acc[1][pb][v + 1]);
        });
    }
}

extern __shared__ __attribute__((aligned(16))) char split_f32_lds[];

// UNITS: units of more than one chunk.
template <int n, int WR, int NT, int PARTS, bool UNITS>
__device__ __forceinline__ void split_f32_work(const float *__restrict__ in, const float *__restrict__ w_seg,
                                               const void *__restrict__ w_split, float *__restrict__ out,
                                               float *__restrict__ ws, const SplitParams &p, const EvenShares &k,
                                               const SplitHead &head)
{
    char *lds = split_f32_lds;
    const int g = blockIdx.x;
    int whole = g * k.rounds;                         // this workgroup's whole passes, then its range of the list
    const int whole_end = whole + k.rounds;
    int u = k.begin(g);
    const int u_end = k.begin(g + 1);
    bool first = true;
    while (whole < whole_end || u < u_end) {
        int pass, u0 = 0, u1 = k.chunks;               // (units of p.unit chunks)
        __syncthreads();                              // the last piece's LDS is free
        float *slot = ws;
        if (whole < whole_end) {
            pass = whole++;
        } else {
            const int rel = u / k.chunks;
            slot += (size_t)k.slot(g, rel, first) * S_SLOT;
            pass = k.listed() + rel;
            u0 = u - rel * k.chunks;
            u1 = min(k.chunks, u0 + u_end - u);
            first = false;
            u += u1 - u0;
        }
        pass = __builtin_amdgcn_readfirstlane(pass);  // the same in all lanes: the staging's addresses stay scalar
        const bool all = u0 == 0 && u1 == k.chunks;
        // (two parts: whole groups, the last one's second chunk past the last channel where those are an odd number)
        const int c0 = __builtin_amdgcn_readfirstlane(UNITS ? u0 * p.unit : u0);
        const int c1 = __builtin_amdgcn_readfirstlane(PARTS == 2 ? u1 * p.unit : UNITS ? min(u1 * p.unit, p.chunks) : u1);
        if (pass & 1)
            do_piece<n, 1, WR, NT, PARTS>(in, w_seg, w_split, out, slot, p, head, lds, pass >> 1, c0, c1, all, (int)threadIdx.x);
        else
            do_piece<n, 0, WR, NT, PARTS>(in, w_seg, w_split, out, slot, p, head, lds, pass >> 1, c0, c1, all, (int)threadIdx.x);
    }
}

// TWO: both kinds of parts in one launch, which a look at the head tells apart (a launch of its own that has nothing to do is
// 4.5 us; layers that never have two parts are 2 % faster without the other kind's code beside theirs).
template <int n, int WR, int NT, bool TWO>
__global__ void __launch_bounds__(S_THREADS, 1) split_f32_kernel(const float *__restrict__ in, const float *__restrict__ w_seg,
                                                              const void *__restrict__ w_split, float *__restrict__ out,
                                                              float *__restrict__ ws, SplitParams p, EvenShares k)
{
    if constexpr (TWO) {
        const SplitHead head = read_head((const char *)w_split + p.w_bytes);
        if (head.two == SPLIT_TWO) {
            split_f32_work<n, WR, NT, 2, true>(in, w_seg, w_split, out, ws, p, k, head);
            return;
        }
    }
    split_f32_work<n, WR, NT, 3, TWO>(in, w_seg, w_split, out, ws, p, k, {0u, 0, 0, 0u});
}

// Segregated fp32 weights -> MFMA operands of their three parts: [row parity][block of 32 output channels][chunk][tap]
// [part][lane][8 input channels], zeros where a channel count is no whole block.  One wave per (block, chunk, tap).
template <int n>
__global__ void __launch_bounds__(256) split_weights_kernel(const float *__restrict__ w_seg, char *__restrict__ w_split,
                                                            const RangePart *__restrict__ range, SplitParams p, unsigned tasks)
{
    SplitHead head = {0u, 0, 0, 0u};
    if (p.two) {
        head = split_head(range, p.range_share, p.from);
        if (head.two && blockIdx.x == 0 && threadIdx.x == 0)
            *reinterpret_cast<uint4 *>(w_split + p.w_bytes - 16) = make_uint4(head.two, (unsigned)head.ea, (unsigned)head.eb, 0u);
    }
    const unsigned task = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (task >= tasks) return;
    constexpr int taps0 = TapOrder<n, 0>::taps, taps1 = TapOrder<n, 1>::taps;
    static constexpr TapOrder<n, 0> order0{};
    static constexpr TapOrder<n, 1> order1{};
    const unsigned block = task / (n * n), q = task - block * (n * n);          // block: output block x chunk
    const unsigned oblk = block / (unsigned)p.chunks, chunk = block - oblk * (unsigned)p.chunks;
    const bool second = q >= (unsigned)taps0;
    const unsigned qr = second ? q - taps0 : q;
    int cls = 0, local = 0;
    static_for<n * n>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if (q == (unsigned)i) {
            if constexpr (i < taps0) {
                cls = order0.s[i];
                local = order0.local[i];
            } else {
                cls = 2 + order1.s[i - taps0];
                local = order1.local[i - taps0];
            }
        }
    });
    const int Tp = cls == 0 ? class_taps(n, 0) : cls == 3 ? class_taps(n, 3) : class_taps(n, 1);
    const unsigned off = cls == 0 ? p.off[0] : cls == 1 ? p.off[1] : cls == 2 ? p.off[2] : p.off[3];
    const int lane = threadIdx.x & 63, co = (int)oblk * 32 + (lane & 31), ci = (int)chunk * S_KC + 8 * (lane >> 5);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = co < p.Cout && ci + j < p.Cin ? w_seg[off + ((size_t)(ci + j) * Tp + local) * p.Cout + co] : 0.0f;
    bf16x8 part[3];
    const int parts = head.two ? 2 : 3;
    if (head.two) {
        split2(v, head.eb, part[0], part[1]);
    } else {
        split3(v, part[0], part[1], part[2]);
        part[2] = quiet(part[2]);
    }
    char *d = w_split + ((second ? p.w_pass1 : 0u) + ((size_t)block * (second ? taps1 : taps0) + qr) * S_TAP) * parts + lane * 16;
    *reinterpret_cast<bf16x8 *>(d) = part[0];
    *reinterpret_cast<bf16x8 *>(d + S_TAP) = part[1];
    if (!head.two) *reinterpret_cast<bf16x8 *>(d + 2 * S_TAP) = part[2];
}

// Eight workgroups per pass of the shared list, one per block of positions and half of its registers: the sum of the
// pass's slots, in workgroup order, goes to the output (nothing to do where one workgroup did the whole pass).
template <int n, int WR>
__global__ void __launch_bounds__(S_THREADS, 5) split_f32_sum_kernel(const float *__restrict__ in, const float *__restrict__ w_seg,
                                                                  float *__restrict__ out, const float *__restrict__ ws,
                                                                  SplitParams p, EvenShares k)
{
    using TS = TileShape<WR>;
    const int rel = blockIdx.x >> 3, part = blockIdx.x & 7, tid = threadIdx.x;
    const PassOwners o(k, rel);
    if (o.g0 == o.g1) return;
    float4 a[4];                                      // registers 2 q, 2 q + 1: [column parity 0, 1] each
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    add_slots<S_THREADS>(ws + (size_t)part * 16 * S_THREADS, S_SLOT, k, o, rel, a);
    const int pass = k.listed() + rel, tile = pass >> 1, tile_m = tile % p.tiles_m, tile_co = tile / p.tiles_m;
    const int lane = tid & 63, wave = tid >> 6;
    const Column c = column_of(p, tile_m * TS::tm, (wave / WR) * 4 + (part >> 1), lane & 31);
    const int co32 = tile_co * TS::tco + (wave % WR) * 32, co0 = co32 + 4 * (lane >> 5);
    float zero = 0.0f;                                // NaN where one of the sums is infinite or not a number
#pragma unroll
    for (int q = 0; q < 4; ++q) zero = fmaf(a[q].x, 0.0f, fmaf(a[q].y, 0.0f, fmaf(a[q].z, 0.0f, fmaf(a[q].w, 0.0f, zero))));
    if (__builtin_expect(__ballot(zero != 0.0f) != 0, 0)) {  // (all lanes of the wave, also those past the last position)
        const bool upper = (part & 1) != 0;
#pragma unroll 1
        for (int s = 0; s < 2; ++s) {
            const floatx16 f = fp32_class_block<n, false>(in, w_seg, p, c, pass & 1, s, co32 + (lane & 31));
            static_for<4>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                float &lo = s ? a[q].y : a[q].x, &hi = s ? a[q].w : a[q].z;
                if (lo * 0.0f != 0.0f) lo = upper ? f[8 + 2 * q] : f[2 * q];
                if (hi * 0.0f != 0.0f) hi = upper ? f[9 + 2 * q] : f[1 + 2 * q];
            });
        }
    }
    if (!c.valid) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int v = 8 * (part & 1) + 2 * q, co = co0 + 8 * (v >> 2) + (v & 3);
        if (co < p.Cout) store_pair(out, p, a[q].x, a[q].y, pass & 1, co, c);
        if (co + 1 < p.Cout) store_pair(out, p, a[q].z, a[q].w, pass & 1, co + 1, c);
    }
}

// ---- plan -------------------------------------------------------------------------------------------------------
struct SplitPlan {
    bool ok;
    int wr;
    SplitParams p;
    EvenShares k;
};

// Two half-precision parts where that is no less exact than three bfloat16 ones.  What it costs in exactness does not depend
// on the length of the reduction (products whose operands end after 23 bits, segments of eight MFMAs), the roundings of one
// chain of three-part MFMAs do: `steps` of them, of a pass's sums of one class and without those that multiply the zero
// frame, in the mean over passes that are done whole and shared ones.  From 108 (5 x 5: 150, whose segments are longer) the error
// was 0.65 to 0.99 of the other's on all but one (1.007) of 8430 random layers while all partial products had one accumulator,
// whose roundings the smaller ones' sums apart do without (128 x 512 x 256 x 16 x 16, n = 4: 1.3e-7 for 1.6e-7).  Times as
// fast from there: 1.25 (4 x 4, at least 1.13) and 1.30 (5 x 5, at least 1.12) then; 3 x 3 kernels gained 6 % in the mean and lost on
// some.  (One accumulator for all needs second parts of their own size, which small values do not have: 336 us against 352.)
// Of products that are not zero two parts want 32 steps (25 layers, 1 to 0.06 of the input not zero: no less exact from 24 to 33).
constexpr double SPLIT_FROM = 32.0;
inline bool split_two_parts(const Shape &s, int chunks, double whole, double shared, float *from)
{
    *from = 0.0f;
    if (s.n < 4) return false;
    double taps = 0.0;
    for (int c = 0; c < 4; ++c) taps += (double)class_taps(s.n, c) * class_taps(s.n, c) / (s.n * s.n);
    const double share = shared * chunks / S_GRID, piece = share < chunks ? share : chunks;
    const int N0 = s.N - 2 * s.frame, M = s.M - 2 * s.crop;
    const double inside = taps_inside(N0, s.n, 2 * s.frame - s.crop, M) / ((double)s.E * s.n);
    const double steps = taps * (whole * chunks + shared * piece) / (whole + shared) * inside * inside;
    *from = (float)(SPLIT_FROM / steps * ((double)s.B * s.Cin * N0 * N0) * ((double)s.Cin * s.Cout * s.n * s.n));
    return steps >= (s.n == 4 ? 108.0 : 150.0) && (size_t)s.B * s.Cout * M * M * sizeof(float) >= SPLIT_RANGE_BYTES;
}

inline SplitPlan split_plan_for(const Shape &s, int wr)
{
    SplitPlan r;
    r.ok = false;
    r.wr = wr;
    SplitParams &p = r.p;
    const int tm = 128 * (4 / wr), tco = 32 * wr;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout; p.N = s.N; p.M = s.M - 2 * s.crop; p.E = s.E; p.EE = s.E * s.E;
    p.crop = s.crop;
    p.epi = s.epi;
    p.q = s.frame;
    p.N0 = s.N - 2 * s.frame;
    p.Mtot = s.B * p.EE;
    p.tiles_m = (p.Mtot + tm - 1) / tm;
    p.tiles_co = (s.Cout + tco - 1) / tco;
    const int dg = (tm - 2) / s.E + 1;                        // quad rows tm consecutive positions can step over
    const int crossings = (dg + s.E - 1) / s.E;
    p.ip = (dg + crossings * (s.N - s.E) + s.fl + 1) * s.N;
    for (int c = 0; c < 4; ++c) p.off[c] = (unsigned)seg_offset(s.Cin, s.Cout, s.n, c, KST_F32);
    const size_t in_bytes = (size_t)s.B * s.Cin * p.N0 * p.N0 * sizeof(float);
    p.chunks = (s.Cin + S_KC - 1) / S_KC;
    const size_t blocks = (size_t)((s.Cout + 31) / 32) * p.chunks;
    const int taps0 = taps_for_parity(s.n, 0) * s.n, taps1 = taps_for_parity(s.n, 1) * s.n;
    const size_t w_bytes = blocks * (taps0 + taps1) * 3 * S_TAP;
    p.in_bytes = (unsigned)in_bytes;
    p.w_bytes = (unsigned)w_bytes;
    p.w_pass1 = (unsigned)(blocks * taps0 * S_TAP);
    p.range_share = split_range_share(in_bytes, (size_t)s.Cin * s.Cout * s.n * s.n * sizeof(float));
    // Full rounds of whole passes: any number where the two parities cost the same, pairs of passes where not.
    const unsigned long long tiles = (unsigned long long)p.tiles_m * p.tiles_co, passes = 2 * tiles;
    r.k.rounds = taps0 == taps1 ? (int)(passes / S_GRID) : 2 * (int)(tiles / S_GRID);
    r.k.passes = (int)(passes - (unsigned long long)r.k.rounds * S_GRID);
    p.two = split_two_parts(s, p.chunks, (double)r.k.rounds * S_GRID, r.k.passes, &p.from);
    p.unit = p.two ? S_GROUP : 1;
    r.k.chunks = (p.chunks + p.unit - 1) / p.unit;
    const unsigned long long units = passes * (unsigned)r.k.chunks;
    r.k.grid = units < (unsigned long long)S_GRID ? (int)units : S_GRID;
    r.k.taps0 = taps0 * p.unit;
    r.k.taps1 = taps1 * p.unit;
    const unsigned long long all =
        (unsigned long long)r.k.chunks *
        ((unsigned long long)(r.k.passes >> 1) * (r.k.taps0 + r.k.taps1) + (r.k.passes & 1) * r.k.taps0);
    r.k.per = (int)(all / (unsigned)r.k.grid);
    r.k.more = (int)(all % (unsigned)r.k.grid);
    r.ok = s.n >= 3 && s.n <= 5 && s.Ns == s.N && p.ip <= S_IP && in_bytes < (1u << 31) && w_bytes < (1u << 31) &&
           tiles <= (1u << 22) && all < (1u << 30);
    return r;
}

inline SplitPlan split_plan(const Shape &s)
{
    return split_plan_for(s, s.Cout > 64 ? 4 : 2);
}

inline size_t split_weight_bytes(const SplitPlan &pl) { return ((size_t)pl.p.w_bytes + 255) & ~(size_t)255; }

template <int n, int WR, int NT>
hipError_t split_f32_launch_nt(const float *in, const float *w_seg, float *out, char *ws, const SplitPlan &pl, hipStream_t stream)
{
    const int lds = split_lds(NT, pl.p.two);
    auto kernel = &split_f32_kernel<n, WR, NT, false>;
    if constexpr (n > 3)
        if (pl.p.two) kernel = &split_f32_kernel<n, WR, NT, true>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    const SplitParams &p = pl.p;
    if (p.two) {                                      // (the shares lie in the output until the weights are split)
        e = launch_split_range({in, p.in_bytes / sizeof(float), false}, {w_seg, (size_t)p.Cin * p.Cout * n * n, false}, out, stream);
        if (e != hipSuccess) return e;
    }
    const unsigned tasks = p.w_bytes / (3 * S_TAP);
    hipLaunchKernelGGL((split_weights_kernel<n>), dim3((tasks + 3) / 4), dim3(256), 0, stream, w_seg, ws,
                       (const RangePart *)out, p, tasks);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    float *slots = (float *)(ws + split_weight_bytes(pl));
    hipLaunchKernelGGL(kernel, dim3((unsigned)pl.k.grid), dim3(S_THREADS), lds, stream, in, w_seg,
                       (const void *)ws, out, slots, p, pl.k);
    e = hipGetLastError();
    if (e != hipSuccess || pl.k.passes == 0) return e;
    hipLaunchKernelGGL((split_f32_sum_kernel<n, WR>), dim3(8u * pl.k.passes), dim3(S_THREADS), 0, stream, in, w_seg, out,
                       (const float *)slots, pl.p, pl.k);
    return hipGetLastError();
}

template <int n>
hipError_t split_f32_launch_n(const float *in, const float *w_seg, float *out, char *ws, const SplitPlan &pl, hipStream_t stream)
{
    const bool few = pl.p.ip <= 3 * 128;
    if (pl.wr == 4)
        return few ? split_f32_launch_nt<n, 4, 3>(in, w_seg, out, ws, pl, stream) : split_f32_launch_nt<n, 4, S_NT>(in, w_seg, out, ws, pl, stream);
    return few ? split_f32_launch_nt<n, 2, 3>(in, w_seg, out, ws, pl, stream) : split_f32_launch_nt<n, 2, S_NT>(in, w_seg, out, ws, pl, stream);
}

}  // namespace

}  // namespace kst

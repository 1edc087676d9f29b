// Segregated forward pass of layers with 16-bit operands on the matrix cores, any channel counts, map edges and padding
// factors, kernels of 3 x 3 to 5 x 5: the input repacked once, channels of a pixel side by side.
//
// Section 3.3, Eqs. 7-10, as four implicit GEMMs that share one input tile: output channels down the MFMA rows, quad
// positions m = (b * E + i) * E + j across its columns, input channels 16 at a time (one 32x32x16 MFMA).
//
// What bounds these layers is not the multiplies (a few microseconds) but what stands around them, above all the turn
// of the input from [channel][pixel] to the eight channels of a pixel that a lane's operand is.  Done while staging, a
// workgroup turns every row again for each block of output channels and each halo, two bytes at a time.  Here a first
// kernel turns the whole input once into [batch][16 channels][framed row][framed column][16], with the zero frame of a
// padded layer and zeros past the last channel: what that copy costs the frame's copy cost before.  After that both
// operands are read in 16-byte groups as they are multiplied: the rows that a tile's positions touch go through LDS
// (two stages, one barrier per 16 channels, no conflicts: 64 lanes read 2 KB in a row), the segregated weights, whose
// layout is an operand's already, straight into registers eight to sixteen taps ahead.
//
// Measured against the kernels that take the input as it lies in memory, half precision and bfloat16, on 250 random
// layers of 16 to 1024 channels: 2.1 times as fast (geometric mean, 9 of 10 layers of more than 15 us between 1.2 and 7),
// two launches of 13 us together at the least.  24 x 100 x 52 x 19 x 19, n = 3, P = 1: 46.9 -> 14.2 us (pack 5.2, multiply
// 9.0); 64 x 256 x 128 x 16 x 16, n = 4, P = 2: 54 -> 30 us (7 and 23).  Large maps are bound by their stores: 35 x 72 x 326 x
// 23 x 23, n = 3, P = 3, 109 MB of output: 140 -> 48 us.  Error against 64 bits over 120 layers: 0.83 of the other kernels'.
#include "kst_segregate.h"
#include "kst_split_common.h"

namespace kst {

namespace {

constexpr int K_THREADS = 256;
constexpr int K_KC = 16;                      // input channels per chunk
constexpr int K_TCO = 32;                     // output channels per workgroup
constexpr int K_NT = 6;                       // 16-byte groups a lane stages per chunk at most
constexpr unsigned K_OUTSIDE = 0x80000000u;   // byte offset past every buffer here (all below 2 GB)

struct PackedParams : IgemmParams {
    int chunks, octs;                         // of 16 and of 8 input channels
    int chunks_per_split;
    int groups;                               // 16-byte groups of a tile's staged rows: 2 per position
    unsigned x_bytes, w_bytes;
    unsigned plane;                           // bytes of one chunk's framed map
};

// in[B][Cin][N0][N0] -> x[B][chunk][N][N][16], N = N0 + 2 q: a lane takes two neighbouring pixels (rows of x are cut
// into pairs) of eight channels, four bytes of a tensor row per load whatever its alignment.
__device__ __forceinline__ void pack_pair(const uint16_t *__restrict__ in, char *__restrict__ x, const PackedParams &p,
                                          unsigned i, unsigned total)
{
    if (i >= total) return;
    const unsigned pairs = ((unsigned)p.N + 1) / 2, at = i >> 1;
    const unsigned line = at / pairs, col = 2 * (at - line * pairs);          // (batch item, chunk, row); first column
    const unsigned map = line / (unsigned)p.N, b = map / (unsigned)p.chunks;
    const int y = (int)(line - map * (unsigned)p.N) - p.q, c = (int)col - p.q;
    const int ci = (int)(map - b * (unsigned)p.chunks) * K_KC + 8 * (i & 1);
    // The pair as loaded: moved into the row where one of its pixels lies outside.
    const int c0 = min(max(c, 0), p.N0 - 2);
    const bool row = y >= 0 && y < p.N0;
    const bool in0 = row && c >= 0 && c < p.N0, in1 = row && c + 1 >= 0 && c + 1 < p.N0;
    const unsigned plane = (unsigned)p.N0 * p.N0;
    const uint16_t *src = in + ((size_t)b * p.Cin + ci) * plane + (unsigned)((row ? y : 0) * p.N0 + c0);
    unsigned v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = 0;
        if (ci + j < p.Cin) __builtin_memcpy(&v[j], src + (size_t)j * plane, 4);
    }
    const bool low0 = c == c0, low1 = c + 1 == c0;                            // which half of the pair a pixel is
    unsigned a[8], z[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        a[j] = in0 ? (low0 ? v[j] & 0xffffu : v[j] >> 16) : 0u;
        z[j] = in1 ? (low1 ? v[j] & 0xffffu : v[j] >> 16) : 0u;
    }
    char *dst = x + ((size_t)line * p.N + col) * 32 + (i & 1) * 16;
    *reinterpret_cast<uint4 *>(dst) = make_uint4(a[0] | a[1] << 16, a[2] | a[3] << 16, a[4] | a[5] << 16, a[6] | a[7] << 16);
    if (col + 1 < (unsigned)p.N)
        *reinterpret_cast<uint4 *>(dst + 32) =
            make_uint4(z[0] | z[1] << 16, z[2] | z[3] << 16, z[4] | z[5] << 16, z[6] | z[7] << 16);
}

__global__ void __launch_bounds__(256) pack_input_kernel(const uint16_t *__restrict__ in, char *__restrict__ x,
                                                         PackedParams p, unsigned total)
{
    pack_pair(in, x, p, blockIdx.x * 256u + threadIdx.x, total);
}

// ... and weights as they come segregated in the same launch, by the workgroups past the first `blocks`: neither waits for
// the other (24 x 100 x 52 x 19 x 19, n = 3, P = 1, half precision: a call of kst_forward_padded 34 -> 30 us).
__global__ void __launch_bounds__(256) pack_and_segregate_kernel(const uint16_t *__restrict__ in, char *__restrict__ x,
                                                                 PackedParams p, unsigned total, unsigned blocks,
                                                                 const uint16_t *__restrict__ w, uint16_t *__restrict__ w_seg,
                                                                 SegGeom g)
{
    if (blockIdx.x < blocks) pack_pair(in, x, p, blockIdx.x * 256u + threadIdx.x, total);
    else segregate_one(w, w_seg, g, (blockIdx.x - blocks) * 256u + threadIdx.x);
}

// A workgroup: 32 output channels x four waves of PB blocks of 32 positions, four classes.  (Two waves along the channels
// and two along the positions ran within 5 % of this on 14 layers, and half idle on those of 32 channels and fewer.)
template <int n, int PB, int NT, bool F16>
__global__ void __launch_bounds__(K_THREADS, 2) igemm_16_packed_kernel(const char *__restrict__ x, const char *__restrict__ w_seg,
                                                                      float *__restrict__ dst, PackedParams p)
{
    using Order = FwdTaps<n, false>;
    constexpr Order order{};
    constexpr int side = Order::side, TAPS = Order::taps, OFFSETS = Order::offsets;
    constexpr int TM = 128 * PB, STAGE = NT * K_THREADS * 16;
    // Chunks that the rows and taps that the weights are fetched ahead: what the sums leave registers for.  With one workgroup
    // per CU, four waves of it, a weight's way from L2 (some 700 cycles) is longer than the multiplies of eight taps and, with 3 x 3 kernels
    // and one position block, that of the rows longer than a chunk.  Against 8, 7 and 4 taps and one chunk, 12000 random layers (calls with
    // both launches): n = 3, 4, 5 up to 256 workgroups 1.16, 1.10 and 1.16 times as fast, beyond that, where the workgroups of a CU
    // hide each other's waits, 1.01, 1.01 and 1.05.
    constexpr int XSETS = n == 3 && PB == 1 ? 2 : 1;
    constexpr int AHEAD = n == 3 ? (PB == 2 ? 8 : NT > 3 ? 9 : 16) : n == 4 ? (PB == 2 && NT > 3 ? 12 : 15) : NT > 3 ? 8 : 10;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    unsigned id = blockIdx.x;
    const int tile_m = (int)(id % (unsigned)p.tiles_m);
    id /= (unsigned)p.tiles_m;
    const int tile_co = (int)(id % (unsigned)p.tiles_co);
    const int split = (int)(id / (unsigned)p.tiles_co);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = tile_m * TM;
    const int b0 = m0 / p.EE;
    const int R0 = b0 * p.N + (m0 - b0 * p.EE) / p.E;     // first stacked (framed) input row of the tile

    // LDS byte address of the window's rows at this lane's positions
    int xa[PB][side], mb[PB], mi[PB], mj[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const int m = min(m0 + (wave * PB + pb) * 32 + l32, p.Mtot - 1);
        mb[pb] = m / p.EE;
        const int rest = m - mb[pb] * p.EE;
        mi[pb] = rest / p.E;
        mj[pb] = rest - mi[pb] * p.E;
#pragma unroll
        for (int dy = 0; dy < side; ++dy)
            xa[pb][dy] = ((mb[pb] * p.N + mi[pb] + dy - R0) * p.N + mj[pb]) * 32 + kk * 16;
    }

    // Staging: 16-byte group tid + 256 k of the tile's rows (zeros past the last batch item).
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(x, p.x_bytes), wbuf = buffer_of(w_seg, p.w_bytes);
    unsigned x_off[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int group = tid + K_THREADS * k, pos = group >> 1;
        const int lr = pos / p.N, c = pos - lr * p.N;
        const int R = R0 + lr, b = R / p.N, y = R - b * p.N;
        const bool ok = group < p.groups && b < p.B;
        x_off[k] = ok ? (unsigned)b * p.chunks * p.plane + ((unsigned)y * p.N + c) * 32u + (group & 1) * 16u : K_OUTSIDE;
    }
    bf16x8 x_reg[XSETS][NT];
    auto fetch_x = [&](auto setc, int chunk) {
#pragma unroll
        for (int k = 0; k < NT; ++k) x_reg[decltype(setc)::value][k] = load_bf16x8(xbuf, x_off[k], (unsigned)chunk * p.plane);
    };
    auto write_x = [&](auto setc, int stage) {
#pragma unroll
        for (int k = 0; k < NT; ++k) *reinterpret_cast<bf16x8 *>(lds + stage + (tid + K_THREADS * k) * 16) = x_reg[decltype(setc)::value][k];
    };

    // Weights of tap q of a chunk: this lane's output channel and eight of the chunk's channels (zeros past the last).
    const int co = tile_co * K_TCO + l32;
    const unsigned row = (unsigned)p.Cout * 16u;            // bytes of one tap of eight channels
    const int odd_chunk = (p.octs & 1) ? p.chunks - 1 : -1; // the chunk whose second eight channels do not exist
    unsigned w_off[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        w_off[c] = co < p.Cout ? (unsigned)kk * class_taps(n, c) * row + (unsigned)co * 16u : K_OUTSIDE;
    bf16x8 wf[XSETS][TAPS];
    auto fetch_w = [&](auto setc, auto qc, int chunk) {
        constexpr int q = decltype(qc)::value, c = order.cls[q];
        const unsigned at = p.off[c] * 2u + ((unsigned)chunk * (2 * class_taps(n, c)) + order.local[q]) * row;
        wf[decltype(setc)::value][q] = load_bf16x8(wbuf, chunk == odd_chunk && kk ? K_OUTSIDE : w_off[c], at);
    };

    // One position block: a chunk's sums on their own, added to the whole sums after it, so that a long reduction is
    // rounded at its full size once per chunk and not twice in each multiply.  Two blocks leave no registers for that.
    constexpr bool TWO_SUMS = PB == 1;
    floatx16 acc[4][PB], part[4][TWO_SUMS ? PB : 1];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][pb][v] = 0.0f;

    using std::integral_constant;
    using std::bool_constant;
    const int k0 = split * p.chunks_per_split, k1 = min(p.chunks, k0 + p.chunks_per_split);
    const int last = k1 - 1;                                // (past the last chunk: read again, never multiplied)
    static_for<XSETS>([&](auto sc) { fetch_x(sc, min(k0 + decltype(sc)::value, last)); });
    static_for<AHEAD>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        fetch_w(integral_constant<int, q / TAPS>{}, integral_constant<int, q % TAPS>{}, min(k0 + q / TAPS, last));
    });
    write_x(integral_constant<int, 0>{}, 0);
    int stage = 0;
    auto multiply_chunk = [&](int chunk, auto setc, auto freshc) {     // fresh: the partial sums start here
        constexpr int set = decltype(setc)::value;
        constexpr bool fresh = decltype(freshc)::value;
        __syncthreads();                                    // this chunk's stage is written, the other one is free
        fetch_x(setc, min(chunk + XSETS, last));
        bf16x8 xf[2][PB];
        auto read_x = [&](auto oc) {
            constexpr int o = decltype(oc)::value;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                xf[o & 1][pb] = *reinterpret_cast<const bf16x8 *>(lds + stage + xa[pb][o / side] + (o % side) * 32);
        };
        read_x(integral_constant<int, 0>{});
        static_for<TAPS>([&](auto qc) {
            constexpr int q = decltype(qc)::value, c = order.cls[q], o = order.offset[q];
            if constexpr ((q == 0 || order.offset[q == 0 ? 0 : q - 1] != o) && o + 1 < OFFSETS) read_x(integral_constant<int, o + 1>{});
            constexpr int later = (q + AHEAD) / TAPS;       // chunks
            fetch_w(integral_constant<int, (set + later) % XSETS>{}, integral_constant<int, (q + AHEAD) % TAPS>{},
                    later ? min(chunk + later, last) : chunk);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                floatx16 &sum = TWO_SUMS ? part[c][TWO_SUMS ? pb : 0] : acc[c][pb];
                if constexpr (fresh && order.local[q] == 0) {
                    floatx16 zero = {};
                    sum = mfma16<F16>(wf[set][q], xf[o & 1][pb], zero);
                } else {
                    sum = mfma16<F16>(wf[set][q], xf[o & 1][pb], sum);
                }
            }
            __builtin_amdgcn_sched_barrier(0);              // (left alone, every load is moved down to its use)
        });
        stage = STAGE - stage;
        write_x(integral_constant<int, (set + 1) % XSETS>{}, stage);
        if constexpr (TWO_SUMS) {
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c][0] += part[c][0];
        }
    };
    int chunk = k0;
    for (; chunk + XSETS <= k1; chunk += XSETS)
        static_for<XSETS>([&](auto sc) { multiply_chunk(chunk + decltype(sc)::value, sc, bool_constant<TWO_SUMS>{}); });
    if (XSETS == 2 && chunk < k1) multiply_chunk(chunk, integral_constant<int, 0>{}, bool_constant<TWO_SUMS>{});

    float *out = dst + (size_t)split * p.out_elems;
    const int co_base = tile_co * K_TCO;
    const bool epi = p.splits == 1 && epi_on(p.epi);
    if (epi && p.epi.act == KST_ACT_TANH) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            if (m0 + (wave * PB + pb) * 32 + l32 >= p.Mtot) continue;
            igemm_store_block(out, acc[0][pb], acc[1][pb], acc[2][pb], acc[3][pb], p, co_base, kk, mb[pb], mi[pb], mj[pb]);
        }
        return;
    }
    // Straight from the registers, branch-free: pairs of elements where every row starts at an even one.
    const size_t map = (size_t)p.M * p.M;
    const float lo = epi ? epi_floor(p.epi.act) : 0.0f;
    float bias[16];
#pragma unroll
    for (int v = 0; v < 16; ++v)
        bias[v] = epi && p.epi.bias ? p.epi.bias[min(co_base + 8 * (v >> 2) + 4 * kk + (v & 3), p.Cout - 1)] : 0.0f;
    auto store = [&](auto epic, auto pairc) {
        constexpr bool EPI = decltype(epic)::value, PAIR = decltype(pairc)::value;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const bool live = m0 + (wave * PB + pb) * 32 + l32 < p.Mtot;
            const int y = 2 * mi[pb] - p.crop, c = 2 * mj[pb] - p.crop;
            float *q = out + ((size_t)mb[pb] * p.Cout + co_base + 4 * kk) * map + (ptrdiff_t)y * p.M + c;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bool row = live && y + r >= 0 && y + r < p.M, left = row && c >= 0 && c < p.M, right = row && c + 1 < p.M;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int d = 8 * (v >> 2) + (v & 3);
                    float v0 = acc[2 * r][pb][v], v1 = acc[2 * r + 1][pb][v];
                    if constexpr (EPI) {
                        v0 = epi_max(v0 + bias[v], lo);
                        v1 = epi_max(v1 + bias[v], lo);
                    }
                    float *qv = q + d * map + r * p.M;
                    const bool real = co_base + 4 * kk + d < p.Cout;
                    if constexpr (PAIR) {
                        if (row && real) *reinterpret_cast<float2 *>(qv) = make_float2(v0, v1);
                    } else {
                        if (left && real) qv[0] = v0;
                        if (right && real) qv[1] = v1;
                    }
                }
            }
        }
    };
    const bool pairs = (p.M & 1) == 0 && !p.crop;
    if (epi) {
        if (pairs) store(bool_constant<true>{}, bool_constant<true>{});
        else store(bool_constant<true>{}, bool_constant<false>{});
    } else {
        if (pairs) store(bool_constant<false>{}, bool_constant<true>{});
        else store(bool_constant<false>{}, bool_constant<false>{});
    }
}

// ---- plan -------------------------------------------------------------------------------------------------------
struct PackedPlan {
    bool ok;
    int pb, nt;
    PackedParams p;
    double us;
};

PackedPlan plan_for(const Shape &s, int pb)
{
    PackedPlan r;
    r.pb = pb;
    PackedParams &p = r.p;
    const int tm = 128 * pb;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout; p.N = s.N; p.Ns = s.N; p.M = s.M - 2 * s.crop; p.E = s.E; p.EE = s.E * s.E;
    p.q = s.frame;
    p.N0 = s.N - 2 * s.frame;
    p.pad = 0;
    p.Mtot = s.B * p.EE;
    p.tco = K_TCO;
    p.tiles_m = (p.Mtot + tm - 1) / tm;
    p.tiles_co = (s.Cout + K_TCO - 1) / K_TCO;
    const int dg = (tm - 2) / s.E + 1;                      // quad rows tm consecutive positions can step over
    const int crossings = (dg + s.E - 1) / s.E;
    p.lrows = dg + crossings * (s.N - s.E) + s.fl + 1;
    p.crop = s.crop;
    p.epi = s.epi;
    for (int c = 0; c < 4; ++c) p.off[c] = (unsigned)seg_offset(s.Cin, s.Cout, s.n, c, KST_BF16);
    p.out_elems = (size_t)s.B * s.Cout * p.M * p.M;
    p.chunks = (s.Cin + K_KC - 1) / K_KC;
    p.octs = (s.Cin + 7) / 8;
    const size_t groups = (size_t)p.lrows * s.N * 2, plane = (size_t)s.N * s.N * 32;
    const size_t x_bytes = (size_t)s.B * p.chunks * plane;
    const size_t w_bytes = seg_elems(s.Cin, s.Cout, s.n, KST_BF16) * 2;
    r.ok = s.n >= 3 && s.n <= 5 && s.Ns == s.N && p.N0 >= 2 && groups <= (size_t)K_NT * K_THREADS && x_bytes < K_OUTSIDE &&
           w_bytes < K_OUTSIDE && (unsigned long long)p.tiles_m * p.tiles_co <= (1u << 22);
    if (!r.ok) return r;
    p.groups = (int)groups;
    p.plane = (unsigned)plane;
    p.x_bytes = (unsigned)x_bytes;
    p.w_bytes = (unsigned)w_bytes;
    r.nt = p.groups <= 3 * K_THREADS ? 3 : K_NT;
    // Tile height and splits of the reduction by the time they would take: rounds of 256 workgroups, 2.5 us each beside
    // the multiplies (first loads, stores) and 0.023 us per tap, chunk and position block; a split adds its summing pass.
    // (On 14 layers timed with every choice the one made was within 8 % of the best.)
    const int tiles = p.tiles_m * p.tiles_co;
    const double tap = 0.023 * pb * s.n * s.n;
    r.us = 1e30;
    p.splits = 1;
    p.chunks_per_split = p.chunks;
    for (int c = 1; c <= 16 && c <= p.chunks; ++c) {
        const int cps = (p.chunks + c - 1) / c;
        if ((p.chunks + cps - 1) / cps != c) continue;
        const double rounds = (double)(((size_t)tiles * c + 255) / 256);
        const double us = rounds * (cps * tap + 2.5) + (c > 1 ? 4.0 + (c + 1) * (double)p.out_elems * 4.0 / 4.0e6 : 0.0);
        if (us < 0.95 * r.us) {
            r.us = us;
            p.splits = c;
            p.chunks_per_split = cps;
        }
    }
    return r;
}

PackedPlan plan(const Shape &s)
{
    PackedPlan best;
    best.ok = false;
    // Two position blocks are for layers whose reduction the kernels without the repacked input add up in one chain too:
    // no sum is then rounded more often at its full size than there.
    const bool one_chain = s.Cout >= 16 && (igemm_bf16_strip_supported(s) || igemm_plan(s, KST_BF16, K_KC).splits == 1);
    for (int pb = one_chain ? 2 : 1; pb >= 1; --pb) {
        const PackedPlan r = plan_for(s, pb);
        if (r.ok && (!best.ok || r.us < best.us)) best = r;
    }
    return best;
}

size_t packed_bytes(const PackedPlan &pl) { return ((size_t)pl.p.x_bytes + 255) & ~(size_t)255; }

template <int n, int PB, int NT, bool F16>
hipError_t launch_packed(const char *x, const char *w_seg, float *dst, const PackedParams &p, hipStream_t stream)
{
    const unsigned blocks = (unsigned)p.tiles_m * p.tiles_co * p.splits;
    hipLaunchKernelGGL((igemm_16_packed_kernel<n, PB, NT, F16>), dim3(blocks), dim3(K_THREADS), 2 * NT * K_THREADS * 16, stream,
                       x, w_seg, dst, p);
    return hipGetLastError();
}

template <int n, int PB>
hipError_t launch_tile(const char *x, const char *w_seg, float *dst, const PackedPlan &pl, bool f16, hipStream_t stream)
{
    if (pl.nt == 3)
        return f16 ? launch_packed<n, PB, 3, true>(x, w_seg, dst, pl.p, stream)
                   : launch_packed<n, PB, 3, false>(x, w_seg, dst, pl.p, stream);
    return f16 ? launch_packed<n, PB, K_NT, true>(x, w_seg, dst, pl.p, stream)
               : launch_packed<n, PB, K_NT, false>(x, w_seg, dst, pl.p, stream);
}

template <int n>
hipError_t launch_n(const char *x, const char *w_seg, float *dst, const PackedPlan &pl, bool f16, hipStream_t stream)
{
    return pl.pb == 1 ? launch_tile<n, 1>(x, w_seg, dst, pl, f16, stream) : launch_tile<n, 2>(x, w_seg, dst, pl, f16, stream);
}

}  // namespace

bool igemm_16_packed_applies(const Shape &s)
{
    if (s.lean || s.n < 3 || s.n > 5) return false;         // (a plan's integers hold such kernels)
    if (igemm_bf16_wide_supported(s) || igemm_bf16_ring_supported(s)) return false;
    return plan(s).ok;
}

// Time in microseconds with the launch that repacks (within 14 % on 1465 random layers).
double igemm_16_packed_us(const Shape &s)
{
    const PackedPlan r = plan(s);
    return 9.3 + 1.09 * r.us + 0.39e-6 * r.p.x_bytes + 0.21e-6 * 2 * s.B * s.Cin * (double)s.N * s.N +
           0.13e-6 * 4 * s.B * s.Cout * (double)s.M * s.M + 0.74e-6 * r.p.w_bytes;
}

size_t igemm_16_packed_workspace_bytes(const Shape &s)
{
    const PackedPlan r = plan(s);
    return packed_bytes(r) + (r.p.splits > 1 ? (size_t)r.p.splits * r.p.out_elems * sizeof(float) : 0);
}

hipError_t launch_igemm_16_packed(const void *in, const void *w_seg, float *out, void *ws, const Shape &s, bool f16,
                                  hipStream_t stream, const void *w)
{
    const PackedPlan r = plan(s);
    if (!r.ok) return hipErrorInvalidValue;
    char *x = (char *)ws;
    const unsigned total = (unsigned)((size_t)s.B * r.p.chunks * s.N * ((s.N + 1) / 2) * 2);
    const unsigned blocks = (total + 255) / 256;
    if (w) {
        const SegGeom g = seg_geom(s.Cin, s.Cout, s.n, f16 ? KST_F16 : KST_BF16);
        hipLaunchKernelGGL(pack_and_segregate_kernel, dim3(blocks + (g.off[4] + 255) / 256), dim3(256), 0, stream,
                           (const uint16_t *)in, x, r.p, total, blocks, (const uint16_t *)w,
                           (uint16_t *)const_cast<void *>(w_seg), g);
    } else {
        hipLaunchKernelGGL(pack_input_kernel, dim3(blocks), dim3(256), 0, stream, (const uint16_t *)in, x, r.p, total);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    float *dst = r.p.splits > 1 ? (float *)(x + packed_bytes(r)) : out;
    switch (s.n) {
        case 3: e = launch_n<3>(x, (const char *)w_seg, dst, r, f16, stream); break;
        case 4: e = launch_n<4>(x, (const char *)w_seg, dst, r, f16, stream); break;
        case 5: e = launch_n<5>(x, (const char *)w_seg, dst, r, f16, stream); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (r.p.splits > 1)
        e = launch_splitk_reduce(dst, out, r.p.out_elems, r.p.splits, stream, r.p.epi, (size_t)r.p.M * r.p.M, r.p.Cout);
    return e;
}

}  // namespace kst

// Input gradient on the bf16 matrix cores (g and fp32 weights split into three bfloat16 parts, see kst_split_common.h;
// bfloat16 weights are their own only part, which leaves three partial products of six; large fp32 layers: two parts of half
// precision).
//
//   din[b][ci][a][c] = sum_co sum_u sum_v g[b][co][2 (a + q) - u][2 (c + q) - v] * w[co][ci][u][v]
//
// (q: the zero frame of the padding factor; for an odd one g starts a row and a column later).  As a GEMM: rows = input
// channels, columns = positions m = (b, a, c) of the unframed map, reduction over (co, u, v) in chunks of 16 output
// channels.
//
// What bounds it: the multiplies.  A workgroup of four waves owns 128 positions x 128 RB input channels, a wave 32 RB
// channels and all positions, the largest partial products' sums apart from the others'.  The weights are split once
// by a kernel of their own into MFMA operands, a wave's next ones contiguous, loaded into registers taps ahead.  The
// rows of g that the tile's positions touch are split once per chunk into LDS as [part][channel half][row][column
// parity][column / 2][8 channels]: a tap's positions are two columns apart in g and neighbours there, and a lane's MFMA
// operand is one 16-byte read.  Two stages, one barrier per chunk.  64 x 512 x 256 x 8 x 8, n = 4,
// P = 2: 82 us with three parts where the fp32 multiplies took 162, 61 with two; with bfloat16 weights 64 x 256 x 128 x 16 x 16: 55 against 155.
#include "kst_din_store.h"

namespace kst {

namespace {

constexpr int D_THREADS = 256;
constexpr int D_KC = 16;                 // output channels per chunk
constexpr int D_TM = 128;                // positions per tile
constexpr int D_IP = 832;                // cells (rows x columns of g) a stage can hold: with n = 3 maps of 4 to 28, 32, 33, 64
                                         // and 128, n = 4: 4 to 17, 19, 22, 32, 64, n = 5: 8, 16, 32; others are not taken
constexpr unsigned D_OUTSIDE = 0x80000000u;
constexpr size_t D_SLOT1 = (size_t)D_THREADS * 64;      // floats of a workgroup's sums, per row block

struct DinParams : DinShape {
    int H, W2;             // image rows per batch item, cells per column parity
    int ip;                // cells staged
    int tiles_m, tiles_ci, chunks;
    unsigned g_bytes, w_bytes;
    int two;               // operands of two half-precision parts where their ranges allow
    int range_share;       // workgroups of the ranges' launch that took the weights
    float from;            // ... and of all pairs of a weight and a value of g, how many at least have no zero
};

// LDS of a kernel that stages NT cells per lane: two stages, and totals (below) of some of two row blocks' accumulators.
constexpr int din_half(int NT) { return (NT == 7 ? D_IP : NT * 128) * 16; }           // bytes: one channel half of one part
constexpr int din_stage(int NT, int parts) { return parts * 2 * din_half(NT); }
constexpr int din_lds_totals(int NT, int RB) { return RB == 1 ? 0 : NT == 7 ? 3 : 4; }
constexpr int din_lds(int NT, int RB)
{
    const int two = 2 * din_stage(NT, 2) + din_lds_totals(NT, RB) * 16 * D_THREADS * 4, three = 2 * din_stage(NT, 3);
    return two > three ? two : three;
}

// Two parts: is block b of the accumulators added to the total during this tap of a chunk?  Once every eight taps.
constexpr int D_SEGMENT = 8;
constexpr bool din_flushed(int n, int blocks, int tap, int b)
{
    return tap < n * n / D_SEGMENT * D_SEGMENT && b * D_SEGMENT == tap % D_SEGMENT * blocks;
}

// WP: parts of the weights, PARTS: of g (three bfloat16 ones, or two of half precision, scaled as the head says).
template <int n, int RB, int WP, int NT, int PARTS>
__device__ __forceinline__ void din_accumulate(const float *__restrict__ g, const void *__restrict__ w_split,
                                               const DinParams &p, const SplitHead &head, char *lds, int tile_m, int tile_ci,
                                               int k0, int k1, int tid, floatx16 (&acc)[RB][4])
{
    constexpr int TAPS = n * n, HALF = din_half(NT), PART = 2 * HALF, STAGE = din_stage(NT, PARTS);
    constexpr int SETS = n == 4 ? 4 / RB : n;         // divides the taps
    constexpr int TAP = WP * 1024;                    // bytes of a tap's operands for 32 input and 16 output channels
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kk = lane >> 5;
    const int NN = p.N * p.N, pitch = 2 * p.W2;
    const int m0 = tile_m * D_TM;
    const int b0 = m0 / NN, a0 = (m0 - b0 * NN) / p.N;
    const int V0 = b0 * p.H + 2 * a0;                 // first image row of the tile (rows stacked over batch items)

    int xa[4];                                        // LDS byte address of the window's first cell
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
        const int m = min(m0 + pb * 32 + l32, p.Mtot - 1);
        const int mb = m / NN, rem = m - mb * NN, ma = rem / p.N, mc = rem - ma * p.N;
        xa[pb] = ((mb * p.H + 2 * ma - V0) * pitch + mc) * 16 + kk * HALF;
    }

    // Staging: wave -> channel half wave & 1, cells (wave >> 1) * 64 + lane + 128 k (the last 64 of 832: by both waves
    // of the half, the same values).
    const int half = wave & 1;
    const unsigned plane = 4u * (unsigned)p.M * p.M;
    auto cell_of = [&](int k) { return 128 * (k + 1) <= D_IP ? (wave >> 1) * 64 + lane + 128 * k : lane + 128 * k; };
    unsigned x_off[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int cell = cell_of(k);
        const int lr = cell / pitch, rem = cell - lr * pitch;
        const int odd = rem >= p.W2 ? 1 : 0;
        const int V = V0 + lr, bb = V / p.H;
        const int y = V - bb * p.H + p.shift, x = 2 * (rem - odd * p.W2) + odd + p.shift;
        const bool ok = cell < p.ip && bb < p.B && y >= 0 && y < p.M && x >= 0 && x < p.M;
        x_off[k] = ok ? (unsigned)bb * p.Cout * plane + 4u * ((unsigned)y * p.M + x) : D_OUTSIDE;
    }
    float x_reg[NT][8];
    auto fetch_x = [&](int chunk) {
        const int c = chunk * D_KC + half * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool live = c + j < p.Cout;         // uniform
            const __amdgpu_buffer_rsrc_t buf = buffer_of(g, live ? p.g_bytes : 0u);
            const unsigned at = live ? (unsigned)(c + j) * plane : 0u;
#pragma unroll
            for (int k = 0; k < NT; ++k) x_reg[k][j] = load_f32(buf, x_off[k], at);
        }
    };
    auto write_x = [&](auto kc, int stage) {
        constexpr int k = decltype(kc)::value;
        bf16x8 part[3];
        if constexpr (PARTS == 2) split2(x_reg[k], head.eb, part[0], part[1]);
        else split3(x_reg[k], part[0], part[1], part[2]);
        char *d = lds + stage + half * HALF + cell_of(k) * 16;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) *reinterpret_cast<bf16x8 *>(d + i * PART) = part[i];
    };

    bf16x8 wp[SETS][RB][WP];
    const __amdgpu_buffer_rsrc_t wbuf = buffer_of(w_split, p.w_bytes);
    unsigned w_base[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
        w_base[rb] = (unsigned)min((tile_ci * 4 + wave) * RB + rb, (p.Cin - 1) / 32) * p.chunks * (TAPS * TAP);
    auto fetch_w = [&](auto qc, int chunk) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int part = 0; part < WP; ++part)
                wp[q % SETS][rb][part] = load_bf16x8(wbuf, lane * 16 + part * 1024, w_base[rb] + (unsigned)(chunk * TAPS + q) * TAP);
    };

    bf16x8 xf[4][PARTS];
    int stage = 0;
    auto read_x = [&](auto qc, auto partc) {          // taps are walked row by row, columns of one parity together
        constexpr int q = decltype(qc)::value, part = decltype(partc)::value;
        constexpr int h = q / n, i = q % n, even = (n + 1) / 2;
        constexpr int x = i < even ? 2 * i : 2 * (i - even) + 1;
#pragma unroll
        for (int pb = 0; pb < 4; ++pb)
            xf[pb][part] = *reinterpret_cast<const bf16x8 *>(lds + stage + xa[pb] + (h * 2 + (x & 1)) * p.W2 * 16 +
                                                             (x >> 1) * 16 + part * PART);
    };

    // (two parts: the total to which the largest products' sums are added, a block per tap or two, before they start again)
    // (some totals are in LDS: beside two accumulators of each block registers are short)
    constexpr int BLOCKS = 4 * RB, TR = BLOCKS - din_lds_totals(NT, RB);
    const LdsTotals<D_THREADS> spare = {reinterpret_cast<float4 *>(lds + 2 * STAGE) + tid};
    floatx16 low[RB][4], total[TR], zeros;
#pragma unroll
    for (int v = 0; v < 16; ++v) zeros[v] = 0.0f;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int pb = 0; pb < 4; ++pb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[rb][pb][v] = low[rb][pb][v] = 0.0f;
                if (rb * 4 + pb < TR) total[rb * 4 + pb][v] = 0.0f;
            }
    if constexpr (PARTS == 2)
        static_for<BLOCKS - TR>([&](auto bc) { spare.clear(decltype(bc)::value); });

    using std::integral_constant;
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

    for (int chunk = k0; chunk < k1; ++chunk) {
        const int next = min(chunk + 1, k1 - 1), after = min(chunk + 2, k1 - 1);
        static_for<TAPS>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            constexpr bool last = q == TAPS - 1;
            if constexpr (last) {
                // Every wave has written its share of the next chunk's stage and is done reading this one's.
                stage = STAGE - stage;
                __syncthreads();
                fetch_x(after);
            }
            fetch_w(integral_constant<int, (q + SETS - 1) % TAPS>{}, q + SETS - 1 < TAPS ? chunk : next);
            static_for<NT>([&](auto kc) {
                if constexpr (write_tap(decltype(kc)::value) == q) write_x(kc, STAGE - stage);
            });
            constexpr auto flushed = [](int b) { return PARTS == 2 && din_flushed(n, BLOCKS, q, b); };
            static_for<BLOCKS>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                if constexpr (flushed(b)) {
                    if constexpr (b < TR) total[b] += acc[b / 4][b % 4];
                    else spare.add(b - TR, acc[b / 4][b % 4]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            constexpr int MF = BLOCKS * (PARTS == 2 ? 1 + WP : WP == 1 ? 3 : 6);
            static_for<PARTS>([&](auto xc) {          // parts of g, smallest first, against the parts that matter
                constexpr int xp = PARTS - 1 - decltype(xc)::value, ws = WP < PARTS - xp ? WP : PARTS - xp;
                static_for<ws>([&](auto wc) {
                    constexpr int w = ws - 1 - decltype(wc)::value;
                    static_for<BLOCKS>([&](auto bc) {
                        constexpr int b = decltype(bc)::value, rb = b / 4, pb = b % 4;
                        if constexpr (flushed(b) && w + xp == 0) {
                            acc[rb][pb] = mfma16<true>(wp[q % SETS][rb][w], xf[pb][xp], zeros);
                        } else {
                            floatx16 &sum = w + xp == 0 ? acc[rb][pb] : low[rb][pb];
                            sum = mfma16<PARTS == 2>(wp[q % SETS][rb][w], xf[pb][xp], sum);
                        }
                    });
                });
                read_x(integral_constant<int, last ? 0 : q + 1>{}, integral_constant<int, xp>{});
            });
            constexpr int valu =
                (16 + (PARTS == 2 ? 32 : 56) * staged_in(q) + MF - 1) / MF;
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
    static_for<BLOCKS>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        floatx16 &sum = acc[b / 4][b % 4];
        if constexpr (PARTS == 2) {
            sum += low[b / 4][b % 4] * (1.0f / LOW_SCALE);
            if constexpr (b < TR) sum += total[b];
            else spare.add_to(b - TR, sum);
        } else {
            sum += low[b / 4][b % 4];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = PARTS == 2 ? __builtin_amdgcn_ldexpf(sum[v], down) : sum[v] * SPLIT_UNSCALE;
    });
}

extern __shared__ __attribute__((aligned(16))) char split_din_lds[];

template <int n, int RB, int WP, int NT, int PARTS, class T>
__device__ __forceinline__ void split_din_work(const float *__restrict__ g, const T *__restrict__ w,
                                               const void *__restrict__ w_split, float *__restrict__ din,
                                               float *__restrict__ ws, const DinParams &p, const EvenShares &k,
                                               const SplitHead &head)
{
    char *lds = split_din_lds;
    const int wg = blockIdx.x;
    int whole = wg * k.rounds;
    const int whole_end = whole + k.rounds;
    int u = k.begin(wg);
    const int u_end = k.begin(wg + 1);
    bool first = true;
    while (whole < whole_end || u < u_end) {
        int tile, c0 = 0, c1 = p.chunks;
        __syncthreads();                              // the last piece's LDS is free
        float *slot = ws;
        if (whole < whole_end) {
            tile = whole++;
        } else {
            const int rel = u / p.chunks;
            slot += (size_t)k.slot(wg, rel, first) * (RB * D_SLOT1);
            tile = k.listed() + rel;
            c0 = u - rel * p.chunks;
            c1 = min(p.chunks, c0 + u_end - u);
            first = false;
            u += c1 - c0;
        }
        tile = __builtin_amdgcn_readfirstlane(tile);  // the same in all lanes: the staging's addresses stay scalar
        c0 = __builtin_amdgcn_readfirstlane(c0);
        c1 = __builtin_amdgcn_readfirstlane(c1);
        const int tile_m = tile % p.tiles_m, tile_ci = tile / p.tiles_m;
        int tid = (int)threadIdx.x;                   // (a fresh copy: nothing of the staging plan is kept across pieces)
        asm volatile("" : "+v"(tid));
        floatx16 acc[RB][4];
        din_accumulate<n, RB, WP, NT, PARTS>(g, w_split, p, head, lds, tile_m, tile_ci, c0, c1, tid, acc);
        const int lane = tid & 63, wave = tid >> 6;
        if (c0 == 0 && c1 == p.chunks) {
            static_for<4>([&](auto pbc) {
                constexpr int pb = decltype(pbc)::value;
                const DinColumn c = din_column(p, tile_m * D_TM + pb * 32 + (lane & 31));
                static_for<RB>([&](auto rbc) {
                    constexpr int rb = decltype(rbc)::value;
                    float a[16];
#pragma unroll
                    for (int v = 0; v < 16; ++v) a[v] = acc[rb][pb][v];
                    din_store<n, true>(g, w, din, p, a, ((tile_ci * 4 + wave) * RB + rb) * 32 + 4 * (lane >> 5), c);
                });
            });
        } else {
            float4 *d = reinterpret_cast<float4 *>(slot);
            static_for<16 * RB>([&](auto ic) {        // [position block][row block][four registers]
                constexpr int i = decltype(ic)::value, pb = i / (4 * RB), rb = i / 4 % RB, v = 4 * (i & 3);
                d[i * D_THREADS + tid] = make_float4(acc[rb][pb][v], acc[rb][pb][v + 1], acc[rb][pb][v + 2], acc[rb][pb][v + 3]);
            });
        }
    }
}

// TWO: both kinds of parts in one launch, told apart by the head.
template <int n, int RB, int WP, int NT, class T, bool TWO>
__global__ void __launch_bounds__(D_THREADS, 1) split_din_kernel(const float *__restrict__ g, const T *__restrict__ w,
                                                                const void *__restrict__ w_split, float *__restrict__ din,
                                                                float *__restrict__ ws, DinParams p, EvenShares k)
{
    if constexpr (TWO) {
        const SplitHead head = read_head((const char *)w_split + p.w_bytes);
        if (head.two == SPLIT_TWO) {
            split_din_work<n, RB, 2, NT, 2>(g, w, w_split, din, ws, p, k, head);
            return;
        }
    }
    split_din_work<n, RB, WP, NT, 3>(g, w, w_split, din, ws, p, k, {0u, 0, 0, 0u});
}

// One workgroup per (shared tile, block of positions, row block): the sum of the tile's slots in workgroup order.
template <int n, int RB, class T>
__global__ void __launch_bounds__(D_THREADS, 6) split_din_sum_kernel(const float *__restrict__ g, const T *__restrict__ w,
                                                                  float *__restrict__ din, const float *__restrict__ ws,
                                                                  DinParams p, EvenShares k)
{
    const int rel = blockIdx.x / (4 * RB), part = blockIdx.x - rel * (4 * RB), tid = threadIdx.x;
    const PassOwners o(k, rel);
    if (o.g0 == o.g1) return;
    float4 four[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) four[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    add_slots<D_THREADS>(ws + (size_t)part * 16 * D_THREADS, RB * D_SLOT1, k, o, rel, four);
    float a[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        a[4 * q] = four[q].x;
        a[4 * q + 1] = four[q].y;
        a[4 * q + 2] = four[q].z;
        a[4 * q + 3] = four[q].w;
    }
    const int tile = k.listed() + rel, tile_m = tile % p.tiles_m, tile_ci = tile / p.tiles_m;
    const int lane = tid & 63, wave = tid >> 6;
    din_store<n, false>(g, w, din, p, a, ((tile_ci * 4 + wave) * RB + part % RB) * 32 + 4 * (lane >> 5),
                        din_column(p, tile_m * D_TM + part / RB * 32 + (lane & 31)));
}

// w[co][ci][u][v] -> MFMA operands: [block of 32 input channels][chunk of 16 output channels][tap][part][lane][8 output
// channels], taps in the order the main loop walks them (u and v from the last to the first, even columns of the image
// first).  One wave per (block, chunk, u): all its loads are in flight together, the runs of n values that its lanes
// leave between them are the other u's (15 -> 8.6 us for 512 x 256 x 4 x 4 against one workgroup per (block,
// chunk) turning the weights in LDS).
template <int n, int WP, class T>
__global__ void __launch_bounds__(256) split_din_weights_kernel(const T *__restrict__ w, char *__restrict__ w_split,
                                                                const RangePart *__restrict__ range, DinParams p, unsigned tasks)
{
    constexpr int NN = n * n;
    SplitHead head = {0u, 0, 0, 0u};
    if (p.two) {
        head = split_head(range, p.range_share, p.from);
        if (head.two && blockIdx.x == 0 && threadIdx.x == 0)
            *reinterpret_cast<uint4 *>(w_split + p.w_bytes - 16) = make_uint4(head.two, (unsigned)head.ea, (unsigned)head.eb, 0u);
    }
    const int parts = head.two ? 2 : WP;
    const unsigned task = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (task >= tasks) return;
    const unsigned block = task / n, u = task - block * n;
    const int blk = (int)(block / (unsigned)p.chunks), chunk = (int)(block - (unsigned)blk * p.chunks);
    const int lane = threadIdx.x & 63, ci = blk * 32 + (lane & 31), co = chunk * D_KC + 8 * (lane >> 5);
    float t[8][n];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int v = 0; v < n; ++v)
            t[j][v] = ci < p.Cin && co + j < p.Cout ? value_of(w + ((size_t)(co + j) * p.Cin + ci) * NN + u * n + v) : 0.0f;
    char *d = w_split + ((size_t)block * NN + (n - 1 - u) * n) * (parts * 1024) + lane * 16;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        constexpr int even = (n + 1) / 2;
        const int x = i < even ? 2 * i : 2 * (i - even) + 1;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = t[j][n - 1 - x];
        bf16x8 part[3];
        if (head.two) {
            split2(v, head.ea, part[0], part[1]);
        } else {
            split3(v, part[0], part[1], part[2]);
            part[2] = quiet(part[2]);
        }
#pragma unroll
        for (int k = 0; k < WP; ++k)
            if (k < parts) *reinterpret_cast<bf16x8 *>(d + (i * parts + k) * 1024) = part[k];
    }
}

struct DinPlan {
    bool ok;
    int rb, wp;
    size_t w_bytes;        // split weights: as the launch lays them out, in full width (p.w_bytes only where ok)
    DinParams p;
    EvenShares k;
};

// s: the framed problem with Shape::frame = q (its M is the framed map's); odd: the padding factor is odd.
DinPlan din_plan(const Shape &s, bool odd, kst_dtype dt)
{
    DinPlan r;
    DinParams &p = r.p;
    const int n = s.n;
    p.B = s.B; p.Cin = s.Cin; p.Cout = s.Cout;
    p.N = s.N - 2 * s.frame;
    p.M = s.M - (odd ? 2 : 0);
    p.shift = 2 * s.frame - (odd ? 1 : 0) - (n - 1);
    p.H = 2 * p.N + n - 2;
    p.W2 = (2 * p.N + n - 1) / 2;
    p.Mtot = s.B * p.N * p.N;
    p.tiles_m = (p.Mtot + D_TM - 1) / D_TM;
    r.wp = dt == KST_BF16 ? 1 : 3;
    // Two row blocks per wave share every read of g; n = 5's five sets of weights leave no registers for a second one,
    // and a tile of 256 channels is half empty up to 128.
    // Fewer than four chunks per workgroup are better spent on the half as large partial sums of one row block.
    p.chunks = (s.Cout + D_KC - 1) / D_KC;
    r.rb = n < 5 && s.Cin > 128 && (double)p.tiles_m * ((s.Cin + 255) / 256) * p.chunks >= 4.0 * S_GRID ? 2 : 1;
    p.tiles_ci = (s.Cin + 128 * r.rb - 1) / (128 * r.rb);
    // Image rows a tile can touch: two per row of positions, n - 2 more where it steps into the next batch item, and the
    // window.  Tiles of whole rows that no item boundary cuts touch the fewest.
    const int rows = D_TM / p.N;
    const bool whole_rows = rows * p.N == D_TM && (rows % p.N == 0 || p.N % rows == 0);
    const int dg = whole_rows ? rows - 1 : (D_TM - 2) / p.N + 1;
    const int crossings = whole_rows ? (rows - 1) / p.N : (dg + p.N - 1) / p.N;
    p.ip = (2 * dg + crossings * (n - 2) + n) * 2 * p.W2;
    const size_t g_bytes = (size_t)s.B * s.Cout * p.M * p.M * sizeof(float);
    const size_t w_bytes = (size_t)((s.Cin + 31) / 32) * p.chunks * n * n * r.wp * 1024;
    p.g_bytes = (unsigned)g_bytes;
    p.w_bytes = (unsigned)w_bytes;
    p.range_share = split_range_share((size_t)s.Cin * s.Cout * n * n * sizeof(float), g_bytes);
    r.w_bytes = w_bytes;
    const unsigned long long tiles = (unsigned long long)p.tiles_m * p.tiles_ci, units = tiles * (unsigned)p.chunks;
    r.k.chunks = p.chunks;
    r.k.grid = units < (unsigned long long)S_GRID ? (int)units : S_GRID;
    r.k.rounds = (int)(tiles / S_GRID);
    r.k.passes = (int)(tiles - (unsigned long long)r.k.rounds * S_GRID);
    r.k.taps0 = r.k.taps1 = 1;
    const unsigned long long all = (unsigned long long)r.k.passes * (unsigned)p.chunks;
    // Two half-precision parts where that is no less exact than three bfloat16 ones, as in the forward kernel: from 36 steps
    // of a chain (without taps that meet no g) the error was 0.35 to 1.0 of the other's on 2008 random layers, below 20 up to
    // 1.6 times it.  Times as fast on 1084 of them with 4 x 4 and 5 x 5 kernels: 1.17 in the mean, never slower (64 x 512 x 256 x
    // 8 x 8, n = 4, P = 2: 60 us, 82 with three parts); 3 x 3 kernels: 0.89 to 1.2, 305 of 924 slower.  bfloat16 weights: two
    // partial products for three, which the ranges' pass outweighs (0.97).  Steps of products that are not zero: from 28 (12 layers, 1
    // to 0.06 of g not zero: no less exact from 20 to 28).
    const double share = (double)r.k.passes * p.chunks / S_GRID, piece = share < p.chunks ? share : p.chunks;
    const double inside = taps_inside(p.N, n, 2 * s.frame - (odd ? 1 : 0), p.M) / ((double)p.N * n);
    const double steps = n * n * ((double)r.k.rounds * S_GRID * p.chunks + r.k.passes * piece) / (double)tiles * inside * inside;
    p.from = (float)(28.0 / steps * ((double)s.Cin * s.Cout * n * n) * ((double)s.B * s.Cout * p.M * p.M));
    p.two = n > 3 && r.wp == 3 && steps >= 36.0 && (size_t)p.Mtot * s.Cin * sizeof(float) >= SPLIT_RANGE_BYTES;
    r.k.per = (int)(all / (unsigned)r.k.grid);
    r.k.more = (int)(all % (unsigned)r.k.grid);
    r.ok = n >= 3 && n <= 5 && p.ip <= D_IP && g_bytes < (1u << 31) && w_bytes < (1u << 31) && tiles <= (1u << 22) &&
           all < (1u << 30);
    return r;
}

size_t din_weight_bytes(const DinPlan &pl) { return (pl.w_bytes + 255) & ~(size_t)255; }

template <int n, int RB, int WP, int NT, class T>
hipError_t din_launch(const float *g, const T *w, float *din, char *ws, const DinPlan &pl, hipStream_t stream)
{
    constexpr int lds = din_lds(NT, RB);
    auto kernel = &split_din_kernel<n, RB, WP, NT, T, false>;
    if constexpr (n > 3 && WP == 3)
        if (pl.p.two) kernel = &split_din_kernel<n, RB, WP, NT, T, true>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    const DinParams &p = pl.p;
    if (p.two) {                                      // (the shares lie in the result until the weights are split)
        if constexpr (std::is_same_v<T, float>)
            e = launch_split_range({w, (size_t)p.Cin * p.Cout * n * n, false}, {g, p.g_bytes / sizeof(float), false}, din, stream);
        if (e != hipSuccess) return e;
    }
    const unsigned tasks = (unsigned)((p.Cin + 31) / 32) * (unsigned)p.chunks * n;
    hipLaunchKernelGGL((split_din_weights_kernel<n, WP, T>), dim3((tasks + 3) / 4), dim3(256), 0, stream, w, ws,
                       (const RangePart *)din, p, tasks);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    float *slots = (float *)(ws + din_weight_bytes(pl));
    hipLaunchKernelGGL(kernel, dim3((unsigned)pl.k.grid), dim3(D_THREADS), lds, stream, g, w,
                       (const void *)ws, din, slots, p, pl.k);
    e = hipGetLastError();
    if (e != hipSuccess || pl.k.passes == 0) return e;
    hipLaunchKernelGGL((split_din_sum_kernel<n, RB, T>), dim3(4u * RB * pl.k.passes), dim3(D_THREADS), 0, stream, g, w, din,
                       (const float *)slots, pl.p, pl.k);
    return hipGetLastError();
}

template <int n, int RB, int WP, class T>
hipError_t din_launch_nt(const float *g, const T *w, float *din, char *ws, const DinPlan &pl, hipStream_t stream)
{
    // (no map with a 5 x 5 kernel is staged by five cells per lane: 8, 16 and 32 want 760, 684 and 748)
    if constexpr (n != 5)
        if (pl.p.ip <= 5 * 128) return din_launch<n, RB, WP, 5>(g, w, din, ws, pl, stream);
    return din_launch<n, RB, WP, 7>(g, w, din, ws, pl, stream);
}

template <int WP, class T>
hipError_t din_launch_n(const float *g, const T *w, float *din, char *ws, const DinPlan &pl, int n, hipStream_t stream)
{
    if (n == 3)
        return pl.rb == 2 ? din_launch_nt<3, 2, WP>(g, w, din, ws, pl, stream) : din_launch_nt<3, 1, WP>(g, w, din, ws, pl, stream);
    if (n == 4)
        return pl.rb == 2 ? din_launch_nt<4, 2, WP>(g, w, din, ws, pl, stream) : din_launch_nt<4, 1, WP>(g, w, din, ws, pl, stream);
    return din_launch_nt<5, 1, WP>(g, w, din, ws, pl, stream);
}

}  // namespace

bool split_din_applies(const Shape &s, bool odd, kst_dtype dt)
{
    if (s.n < 3 || s.n > 5 || s.Cin < 16 || s.Cout <= D_KC) return false;
    // Three launches and partial tiles cost 30 to 40 us.  The fp32 multiplies' tiles hold 128 input channels whatever the
    // layer has, so that is what is weighed.  Both sides timed on 1475 random layers from 2.2 to 12 G products: from
    // 2.2 G this is 1.5 to 1.6 times as fast (6 of 850 layers up to 4 G lost) except where the other side is its
    // pipelined kernel, on maps and channels of whole groups of four, and the weights have three parts: of those 11 of
    // 25 lost from 2.2 to 2.6 G (13 x 768 x 384 x 6 x 6, n = 4, P = 2: 68 us here against 57), 6 of 98 from 2.6 to 4 G.
    // bfloat16's one part gained on them all.
    const double edge = s.N - 2 * s.frame;
    const double products = (double)s.B * edge * edge * s.n * s.n * ((s.Cin + 127) / 128 * 128) * s.Cout;
    const bool close = dt != KST_BF16 && (s.M & 3) == 0 && (s.Cin & 3) == 0 && (s.Cout & 3) == 0;
    return products >= (close ? 2.6e9 : 2.2e9) && din_plan(s, odd, dt).ok;
}

// (0 for a layer these kernels do not take with weights of this type)
size_t split_din_workspace_bytes(const Shape &s, bool odd, kst_dtype dt)
{
    const DinPlan r = din_plan(s, odd, dt);
    if (!r.ok) return 0;
    return din_weight_bytes(r) + (size_t)r.k.slots() * r.rb * D_SLOT1 * sizeof(float);
}

hipError_t launch_split_din(const float *g, const void *w, float *din, void *ws, const Shape &s, bool odd, kst_dtype dt,
                            hipStream_t stream)
{
    const DinPlan r = din_plan(s, odd, dt);
    if (!r.ok) return hipErrorInvalidValue;
    if (dt == KST_BF16) return din_launch_n<1>(g, (const uint16_t *)w, din, (char *)ws, r, s.n, stream);
    if (dt == KST_F16) return hipErrorInvalidValue;
    return din_launch_n<3>(g, (const float *)w, din, (char *)ws, r, s.n, stream);
}

}  // namespace kst

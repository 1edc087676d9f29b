// C ABI of libkst.so: argument validation, path choice, launches.
#include "kst_internal.h"
#include "kst_yardstick.h"

#include <mutex>

using namespace kst;

namespace {

constexpr size_t kMaxElems = (size_t)1 << 31;

bool dtype_ok(int dt) { return dt == KST_F32 || dt == KST_BF16 || dt == KST_F16; }
size_t elt_bytes(kst_dtype dt) { return is16(dt) ? 2 : 4; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

kst_status check_weight_shape(int Cin, int Cout, int n)
{
    if (Cin < 1 || Cout < 1 || n < 1) return KST_ERR_SHAPE;
    const size_t pad = ((size_t)Cin + 7) / 8 * 8;
    if (n > 46340 || pad * (size_t)Cout >= kMaxElems / ((size_t)n * n)) return KST_ERR_SHAPE;
    return KST_OK;
}

kst_status check_shape(int B, int Cin, int Cout, int N, int n)
{
    if (B < 1 || N < 1) return KST_ERR_SHAPE;
    kst_status st = check_weight_shape(Cin, Cout, n);
    if (st != KST_OK) return st;
    if (N > 32768) return KST_ERR_SHAPE;
    const long long M = 2LL * N - n;
    if (M < 1) return KST_ERR_SHAPE;
    const size_t S = 2 * (size_t)N - 1;
    if ((size_t)B * Cin >= kMaxElems / (S * S)) return KST_ERR_SHAPE;            // up-sampled map (and in)
    if ((size_t)B * Cout >= kMaxElems / ((size_t)(M + 1) * (M + 1))) return KST_ERR_SHAPE;   // out, quad grid
    return KST_OK;
}

// AUTO: the matrix cores pay off once both channel counts can fill MFMA blocks.
kst_path choose_path(const Shape &s, kst_dtype dt)
{
    const bool ok = is16(dt) ? igemm_bf16_supported(s) : igemm_f32_supported(s);
    if (ok && s.Cout >= 16 && s.Cin >= 8) return KST_PATH_IGEMM;
    // Few output channels in 16 bits: the matrix cores multiply 32 rows for three real ones in less time than the direct
    // kernel walks its channel chunks one after the other, but the repacking launch comes before.  Either side timed on 170
    // such layers: from 600 products per output pixel the direct kernel is 1.2 to 8 times slower, below 500 up to 1.3 faster.
    // With one or two output channels the line is less clear (174 x 28 x 1 x 58 x 58, n = 5: 49 us there, 82 here): by the times
    // both are known to take.
    if (is16(dt) && s.Cout < 16 && s.Cin * s.n * s.n >= 600 && igemm_16_packed_applies(s) &&
        (s.Cout > 2 || igemm_16_packed_us(s) < 0.85 * direct_us(s, dt)))
        return KST_PATH_IGEMM;
    if (dt == KST_F32 && packed_f32_applies(s)) return KST_PATH_IGEMM;
    // One sample of a generator's output layer (many input channels, three output channels): the
    // position-block kernel splits its reduction over the chip, the direct kernel has four tiles.
    if (dt == KST_F32 && s.Cout < 16 && igemm_f32_small_supported(s)) return KST_PATH_IGEMM;
    // ... and a batch of them: the taps of all sub-kernels as the rows of one matrix product.
    if (dt == KST_F32 && tapmajor_f32_supported(s)) return KST_PATH_IGEMM;
    return KST_PATH_DIRECT;
}

kst_status resolve_path(const Shape &s, kst_dtype dt, int path, kst_path *out)
{
    if (path == KST_PATH_AUTO) { *out = choose_path(s, dt); return KST_OK; }
    if (path == KST_PATH_DIRECT) { *out = KST_PATH_DIRECT; return KST_OK; }
    if (path == KST_PATH_IGEMM) {
        const bool ok = is16(dt) ? igemm_bf16_supported(s) : igemm_f32_supported(s);
        if (!ok) return KST_ERR_PATH;
        *out = KST_PATH_IGEMM;
        return KST_OK;
    }
    if (path == KST_PATH_IGEMM_PASSES) {
        if (!is16(dt) || !igemm_bf16_pp_supported(s)) return KST_ERR_PATH;
        *out = KST_PATH_IGEMM_PASSES;
        return KST_OK;
    }
    if (path == KST_PATH_IGEMM_EVEN) {
        if (dt != KST_F32 || !igemm_f32_supported(s) || !igemm_f32_even_shares_possible(s)) return KST_ERR_PATH;
        *out = KST_PATH_IGEMM_EVEN;
        return KST_OK;
    }
    return KST_ERR_PATH;
}

bool on_matrix_cores(kst_path path)
{
    return path == KST_PATH_IGEMM || path == KST_PATH_IGEMM_EVEN || path == KST_PATH_IGEMM_PASSES;
}

// The problem as a caller's path sees it: IGEMM and its launch form EVEN, asked for by name, multiply fp32 operands in
// fp32.  Only AUTO may split them for the bf16 matrix cores, or repack 16-bit ones.
Shape shape_for(int B, int Cin, int Cout, int N, int n, int path)
{
    Shape s = make_shape(B, Cin, Cout, N, n);
    s.lean = path != KST_PATH_AUTO;
    return s;
}

// 16-bit matrix-core layers whose input is repacked: a whole call has its weights segregated by the launch that does it.
bool repacks_16(const Shape &s, kst_dtype dt, kst_path chosen)
{
    return is16(dt) && chosen == KST_PATH_IGEMM && igemm_16_packed_applies(s);
}

// ... from weights as they come; scratch: room for them segregated, then the layer's workspace.
kst_status run_repacked_16(const void *in, const void *w, void *out, void *scratch, size_t seg_bytes, const Shape &s, kst_dtype dt,
                           hipStream_t stream)
{
    return launch_igemm_16_packed(in, scratch, (float *)out, (char *)scratch + seg_bytes, s, dt == KST_F16, stream, w) == hipSuccess
               ? KST_OK
               : KST_ERR_HIP;
}

size_t workspace_for(const Shape &s, kst_dtype dt, kst_path path)
{
    if (!on_matrix_cores(path) || path == KST_PATH_IGEMM_PASSES) return 0;
    return is16(dt) ? igemm_bf16_workspace_bytes(s) : igemm_f32_workspace_bytes(s, path == KST_PATH_IGEMM_EVEN);
}

// The path's kernels for a caller with `have` bytes of scratch, and what they need of it: where the kernels that lay
// operands out anew need more than there is, those that do not (*s then says so).  Not checked: *need <= have.
kst_status plan_within(Shape *s, kst_dtype dtype, int path, size_t have, kst_path *chosen, size_t *need)
{
    for (;;) {
        const kst_status st = resolve_path(*s, dtype, path, chosen);
        if (st != KST_OK) return st;
        *need = workspace_for(*s, dtype, *chosen);
        if (*need <= have || s->lean) return KST_OK;
        s->lean = 1;
    }
}

// The segregated forward pass on a validated shape (s.Ns may exceed s.N only where
// igemm_f32_takes_row_stride says the kernel that will run reads it).
kst_status run_forward_seg(const void *in, const void *w_seg, void *out, void *ws, size_t ws_bytes, Shape s,
                           kst_dtype dtype, int path, hipStream_t stream)
{
    kst_path chosen;
    size_t need;
    kst_status st = plan_within(&s, dtype, path, ws ? ws_bytes : 0, &chosen, &need);
    if (st != KST_OK) return st;
    if (!aligned16(in) || !aligned16(w_seg) || !aligned16(out)) return KST_ERR_ALIGN;
    if (need > 0) {
        if (!ws || ws_bytes < need) return KST_ERR_WORKSPACE;
        if (!aligned16(ws)) return KST_ERR_ALIGN;
    }
    if (s.Ns != s.N && !(on_matrix_cores(chosen) && dtype == KST_F32 && igemm_f32_takes_row_stride(s)))
        return KST_ERR_SHAPE;
    if (chosen == KST_PATH_IGEMM_PASSES && epi_on(s.epi)) return KST_ERR_PATH;    // that kernel stores bare sums only
    hipError_t e;
    if (chosen == KST_PATH_DIRECT)
        e = launch_direct(in, w_seg, (float *)out, s, dtype, stream);
    else if (chosen == KST_PATH_IGEMM_PASSES)
        e = launch_igemm_bf16_pp(in, w_seg, (float *)out, s, dtype == KST_F16, stream);
    else if (is16(dtype))
        e = launch_igemm_bf16(in, w_seg, (float *)out, ws, s, dtype == KST_F16, stream);
    else
        e = launch_igemm_f32((const float *)in, (const float *)w_seg, (float *)out, ws, s,
                             chosen == KST_PATH_IGEMM_EVEN, stream);
    return e == hipSuccess ? KST_OK : KST_ERR_HIP;
}

// Scratch of the entry points that take un-segregated weights (kst_forward, kst_forward_padded):
// a stream-ordered memory pool of the library's own per device, which keeps what is freed
// (release threshold: never) so that call after call re-uses one block instead of mapping and
// unmapping it every time -- with the runtime's default pool a 128 MiB workspace cost about
// 100 us per call.  The pool holds at most the largest scratch any call has asked for.
constexpr int kMaxPoolDevices = 64;
std::mutex pool_mutex;
hipMemPool_t pools[kMaxPoolDevices];
bool pool_tried[kMaxPoolDevices];

hipError_t scratch_alloc(void **ptr, size_t bytes, hipStream_t stream)
{
    int dev = -1;
    hipMemPool_t pool = nullptr;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxPoolDevices) {
        std::lock_guard<std::mutex> lock(pool_mutex);
        if (!pool_tried[dev]) {
            pool_tried[dev] = true;
            hipMemPoolProps props = {};
            props.allocType = hipMemAllocationTypePinned;
            props.handleTypes = hipMemHandleTypeNone;
            props.location.type = hipMemLocationTypeDevice;
            props.location.id = dev;
            hipMemPool_t made = nullptr;
            if (hipMemPoolCreate(&made, &props) == hipSuccess) {
                uint64_t keep = UINT64_MAX;
                if (hipMemPoolSetAttribute(made, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess)
                    pools[dev] = made;
                else
                    (void)hipMemPoolDestroy(made);
            }
            (void)hipGetLastError();       // a refused pool is no error of the call: the default pool serves
        }
        pool = pools[dev];
    }
    if (pool) return hipMallocFromPoolAsync(ptr, bytes, pool, stream);
    return hipMallocAsync(ptr, bytes, stream);
}

// seg_bytes + *ws_bytes of it; where there is no room for that, with the least() bytes of workspace the layer can do with.
template <class F>
bool scratch_for(void **ptr, size_t seg_bytes, size_t *ws_bytes, hipStream_t stream, F least)
{
    if (scratch_alloc(ptr, seg_bytes + *ws_bytes, stream) == hipSuccess) return true;
    const size_t fewer = least();
    if (fewer >= *ws_bytes) return false;
    (void)hipGetLastError();
    *ws_bytes = fewer;
    return scratch_alloc(ptr, seg_bytes + fewer, stream) == hipSuccess;
}

}  // namespace

extern "C" {

int kst_version(void) { return 104; }

const char *kst_status_string(int status)
{
    switch (status) {
        case KST_OK: return "ok";
        case KST_ERR_NULL: return "null pointer";
        case KST_ERR_SHAPE: return "illegal shape";
        case KST_ERR_DTYPE: return "unknown dtype";
        case KST_ERR_WORKSPACE: return "workspace missing or too small";
        case KST_ERR_HIP: return "HIP runtime error";
        case KST_ERR_PATH: return "unknown or unsupported path";
        case KST_ERR_ALIGN: return "pointer not 16-byte aligned";
        case KST_ERR_ACT: return "unknown activation";
        default: return "unknown status";
    }
}

int kst_out_size(int N, int n) { return 2 * N - n; }

kst_status kst_subkernel_shape(int n, int p, int *Ta, int *Tb)
{
    if (!Ta || !Tb) return KST_ERR_NULL;
    if (n < 1 || p < 0 || p > 3) return KST_ERR_SHAPE;
    *Ta = taps_for_parity(n, p >> 1);
    *Tb = taps_for_parity(n, p & 1);
    return KST_OK;
}

size_t kst_segregated_elems(int Cin, int Cout, int n, kst_dtype dtype)
{
    if (!dtype_ok(dtype) || check_weight_shape(Cin, Cout, n) != KST_OK) return 0;
    return seg_elems(Cin, Cout, n, dtype);
}

size_t kst_segregated_offset(int Cin, int Cout, int n, int p, kst_dtype dtype)
{
    if (!dtype_ok(dtype) || check_weight_shape(Cin, Cout, n) != KST_OK || p < 0 || p > 3) return 0;
    return seg_offset(Cin, Cout, n, p, dtype);
}

kst_status kst_segregate_weights(const void *w, void *w_seg, int Cin, int Cout, int n, kst_dtype dtype,
                                 hipStream_t stream)
{
    if (!w || !w_seg) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    kst_status st = check_weight_shape(Cin, Cout, n);
    if (st != KST_OK) return st;
    if (!aligned16(w) || !aligned16(w_seg)) return KST_ERR_ALIGN;
    return launch_segregate(w, w_seg, Cin, Cout, n, dtype, stream) == hipSuccess ? KST_OK : KST_ERR_HIP;
}

size_t kst_workspace_bytes(int B, int Cin, int Cout, int N, int n, kst_dtype dtype, kst_path path)
{
    if (!dtype_ok(dtype) || check_shape(B, Cin, Cout, N, n) != KST_OK) return 0;
    const Shape s = shape_for(B, Cin, Cout, N, n, path);
    kst_path chosen;
    if (resolve_path(s, dtype, path, &chosen) != KST_OK) return 0;
    return workspace_for(s, dtype, chosen);
}

kst_status kst_forward_seg(const void *in, const void *w_seg, void *out, void *ws, size_t ws_bytes,
                           int B, int Cin, int Cout, int N, int n, kst_dtype dtype, kst_path path,
                           hipStream_t stream)
{
    if (!in || !w_seg || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    kst_status st = check_shape(B, Cin, Cout, N, n);
    if (st != KST_OK) return st;
    return run_forward_seg(in, w_seg, out, ws, ws_bytes, shape_for(B, Cin, Cout, N, n, path), dtype, path, stream);
}

// ---- the entry point that allocates nothing --------------------------------------------------
}  // extern "C"

// Workspace of kst_forward_seg_static: one array per GPU, part of the loaded code object, held
// until the process ends.  In host code `scratch` is only a handle for hipGetSymbolAddress; the
// kernels get the device address that call returns.
static __device__ __align__(256) unsigned char scratch[KST_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_ptr[kMaxDevices];          // device address of `scratch` on each GPU, looked up once

// The current device's copy of `scratch`, or nullptr (with *st set) when it cannot be had.
void *static_scratch(kst_status *st)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        *st = KST_ERR_HIP;
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            *st = KST_ERR_HIP;
            return nullptr;
        }
        scratch_ptr[dev] = ptr;
    }
    return scratch_ptr[dev];
}

}  // namespace

extern "C" {

kst_status kst_forward_seg_static(const void *in, const void *w_seg, void *out, int B, int Cin, int Cout, int N, int n,
                                  kst_dtype dtype, kst_path path, hipStream_t stream)
{
    if (!in || !w_seg || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    kst_status st = check_shape(B, Cin, Cout, N, n);
    if (st != KST_OK) return st;
    Shape s = shape_for(B, Cin, Cout, N, n, path);
    kst_path chosen;
    size_t need;
    st = plan_within(&s, dtype, path, KST_STATIC_SCRATCH_BYTES, &chosen, &need);
    if (st != KST_OK) return st;
    if (need > (size_t)KST_STATIC_SCRATCH_BYTES) return KST_ERR_WORKSPACE;     // larger than the array: refuse
    void *ws = nullptr;
    if (need) {
        ws = static_scratch(&st);
        if (!ws) return st;
    }
    // The kernels write every workspace word before they read it: nothing has to be cleared
    // between calls, whatever the previous call left there.
    return run_forward_seg(in, w_seg, out, ws, need, s, dtype, chosen, stream);
}

kst_status kst_forward(const void *in, const void *w, void *out, int B, int Cin, int Cout, int N, int n,
                       kst_dtype dtype, hipStream_t stream)
{
    if (!in || !w || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    kst_status st = check_shape(B, Cin, Cout, N, n);
    if (st != KST_OK) return st;
    if (!aligned16(in) || !aligned16(w) || !aligned16(out)) return KST_ERR_ALIGN;
    Shape s = make_shape(B, Cin, Cout, N, n);
    if (choose_path(s, dtype) == KST_PATH_DIRECT) {
        const hipError_t e = launch_direct_plain_weights(in, w, (float *)out, s, dtype, stream);
        if (e != hipErrorNotSupported) return e == hipSuccess ? KST_OK : KST_ERR_HIP;
    }
    const size_t seg_bytes = (seg_elems(Cin, Cout, n, dtype) * elt_bytes(dtype) + 255) & ~(size_t)255;
    size_t ws_bytes = workspace_for(s, dtype, choose_path(s, dtype));
    const auto least = [&] {
        s.lean = 1;
        return workspace_for(s, dtype, choose_path(s, dtype));
    };
    void *scratch = nullptr;
    if (!scratch_for(&scratch, seg_bytes, &ws_bytes, stream, least)) return KST_ERR_HIP;
    if (repacks_16(s, dtype, choose_path(s, dtype))) {
        st = run_repacked_16(in, w, out, scratch, seg_bytes, s, dtype, stream);
    } else {
        st = kst_segregate_weights(w, scratch, Cin, Cout, n, dtype, stream);
        if (st == KST_OK)
            st = kst_forward_seg(in, scratch, out, ws_bytes ? (char *)scratch + seg_bytes : nullptr, ws_bytes, B, Cin, Cout, N, n,
                                 dtype, KST_PATH_AUTO, stream);
    }
    if (hipFreeAsync(scratch, stream) != hipSuccess && st == KST_OK) st = KST_ERR_HIP;
    return st;
}

// ---- padding factor P -------------------------------------------------------------------------
namespace {

struct Framed {
    int q, Nq, M, Mq;                 // frame on the input, framed input edge, output edge, inner output edge
    Shape s;                          // the inner, unframed problem (s.Ns: row stride of the framed copy)
    kst_path chosen;
    size_t in_bytes, wide_bytes;      // workspace parts before the inner kernels' own scratch (256-byte multiples)
};

kst_status framed_plan(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dt, int path, bool lean, Framed *f)
{
    if (P < 0 || P > 32768 || B < 1 || N < 1 || N > 32768) return KST_ERR_SHAPE;
    f->q = (P + 1) / 2;
    f->Nq = N + 2 * f->q;
    kst_status st = check_shape(B, Cin, Cout, f->Nq, n);        // also bounds the element counts
    if (st != KST_OK) return st;
    f->M = 2 * N + 2 * P - n;
    f->Mq = 2 * f->Nq - n;
    if (f->M < 1) return KST_ERR_SHAPE;
    f->s = shape_for(B, Cin, Cout, f->Nq, n, path);
    if (lean) f->s.lean = 1;
    // The pipelined fp32 matrix-core kernel supplies the frame itself while it stages its input
    // rows (tensor rows of whole 16-byte groups): no framed copy.
    Shape in_place = f->s;
    in_place.frame = f->q;
    const bool frame_in_kernel = dt == KST_F32 && igemm_f32_takes_virtual_frame(in_place);
    if (path == KST_PATH_IGEMM_EVEN) {
        if (frame_in_kernel) f->s = in_place;
        else f->s.Ns = (f->Nq + 3) & ~3;                            // the stride that launch form wants of a copy
    }
    st = resolve_path(f->s, dt, path, &f->chosen);
    if (st != KST_OK) return st;
    // (the tap-major kernel of few-output-channel layers reads the tensor as it lies in memory and is
    // planned on its edge, which only the in-place view carries)
    if (path == KST_PATH_AUTO && dt == KST_F32 && f->chosen == KST_PATH_DIRECT && tapmajor_f32_supported(in_place))
        f->chosen = KST_PATH_IGEMM;
    if (on_matrix_cores(f->chosen) && dt == KST_F32) {
        if (frame_in_kernel) {
            f->s = in_place;
        } else if ((f->Nq & 3) != 0) {
            // Otherwise that kernel wants rows of whole 16-byte groups: give the framed copy a row
            // stride rounded up to 4 elements when that is the kernel that will run.
            Shape wide = f->s;
            wide.Ns = (f->Nq + 3) & ~3;
            if (igemm_f32_takes_row_stride(wide)) f->s = wide;
        }
    }
    // The repacked input of a 16-bit layer has the frame in it, and its kernel stores an odd factor's interior directly.
    if (repacks_16(in_place, dt, f->chosen)) f->s.frame = f->q;
    f->in_bytes = f->s.frame > 0 ? 0 : ((size_t)B * Cin * f->Nq * f->s.Ns * elt_bytes(dt) + 255) & ~(size_t)255;
    f->wide_bytes = (P & 1) ? (((size_t)B * Cout * f->Mq * f->Mq * sizeof(float) + 255) & ~(size_t)255) : 0;
    // The direct kernels supply the zero frame themselves: no framed copy at all; and for an odd
    // padding factor the flat-output kernel writes the interior of the wider map straight to
    // `out` (output row y is row y + 1 of that map: the row parities, hence the sub-kernels,
    // swap roles as in Fig. 7): no wider buffer and no copy of its interior either.
    // The matrix-core kernels whose accumulators go straight to memory (all fp32 ones, the first
    // 16-bit one) store the interior of the wider map directly as well; those that leave through
    // an LDS image of whole rows keep the wider buffer and the copy.
    if ((P & 1) && on_matrix_cores(f->chosen) && f->chosen != KST_PATH_IGEMM_PASSES &&
        (!is16(dt) || f->s.frame > 0 ||
         !(igemm_bf16_wide_supported(f->s) || igemm_bf16_ring_supported(f->s) || igemm_bf16_strip_supported(f->s)))) {
        f->s.crop = 1;
        f->wide_bytes = 0;
    }
    if (f->chosen == KST_PATH_DIRECT) {
        if ((P & 1) && direct_takes_virtual_frame(f->s, f->q, 1, dt)) {
            f->s.frame = f->q;
            f->s.crop = 1;
            f->in_bytes = 0;
            f->wide_bytes = 0;
        } else if (direct_takes_virtual_frame(f->s, f->q, 0, dt)) {
            f->s.frame = f->q;
            f->in_bytes = 0;
        }
    }
    return KST_OK;
}

size_t framed_bytes(const Framed &f, kst_dtype dt)
{
    return f.in_bytes + f.wide_bytes + workspace_for(f.s, dt, f.chosen);
}

// The plan for a caller with `have` bytes of scratch, as plan_within.
kst_status framed_plan_within(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dt, int path, size_t have, Framed *f)
{
    kst_status st = framed_plan(B, Cin, Cout, N, n, P, dt, path, false, f);
    if (st == KST_OK && framed_bytes(*f, dt) > have) st = framed_plan(B, Cin, Cout, N, n, P, dt, path, true, f);
    return st;
}

}  // namespace

int kst_out_size_padded(int N, int n, int P) { return 2 * N + 2 * P - n; }

size_t kst_workspace_bytes_padded(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype, kst_path path)
{
    if (!dtype_ok(dtype)) return 0;
    if (P == 0) return kst_workspace_bytes(B, Cin, Cout, N, n, dtype, path);
    Framed f;
    if (framed_plan(B, Cin, Cout, N, n, P, dtype, path, false, &f) != KST_OK) return 0;
    return framed_bytes(f, dtype);
}

}  // extern "C"

namespace {

// The segregated forward pass for any padding factor, with an optional epilogue at the stores
// that write final values (the copy that crops an odd padding factor's wider map moves them on unchanged).
kst_status forward_seg_padded_impl(const void *in, const void *w_seg, void *out, void *ws, size_t ws_bytes, int B, int Cin,
                                   int Cout, int N, int n, int P, kst_dtype dtype, int path, const Epilogue &epi,
                                   hipStream_t stream)
{
    if (!in || !w_seg || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    if (P == 0) {
        kst_status st0 = check_shape(B, Cin, Cout, N, n);
        if (st0 != KST_OK) return st0;
        Shape s0 = shape_for(B, Cin, Cout, N, n, path);
        s0.epi = epi;
        return run_forward_seg(in, w_seg, out, ws, ws_bytes, s0, dtype, path, stream);
    }
    Framed f;
    kst_status st = framed_plan_within(B, Cin, Cout, N, n, P, dtype, path, ws ? ws_bytes : 0, &f);
    if (st != KST_OK) return st;
    f.s.epi = epi;
    if (!aligned16(in) || !aligned16(w_seg) || !aligned16(out)) return KST_ERR_ALIGN;
    const size_t inner = workspace_for(f.s, dtype, f.chosen);
    const size_t need = f.in_bytes + f.wide_bytes + inner;
    if (need > 0) {
        if (!ws || ws_bytes < need) return KST_ERR_WORKSPACE;
        if (!aligned16(ws)) return KST_ERR_ALIGN;
    }
    char *base = (char *)ws;
    void *in_framed = base;
    float *wide = f.wide_bytes ? (float *)(base + f.in_bytes) : nullptr;
    void *inner_ws = inner ? (void *)(base + f.in_bytes + f.wide_bytes) : nullptr;
    if (f.s.frame == 0) {
        if (launch_frame_input(in, in_framed, B, Cin, N, f.q, f.s.Ns, dtype, stream) != hipSuccess) return KST_ERR_HIP;
    } else {
        in_framed = const_cast<void *>(in);
    }
    st = run_forward_seg(in_framed, w_seg, wide ? (void *)wide : out, inner_ws, inner, f.s, dtype, f.chosen, stream);
    if (st != KST_OK) return st;
    if (wide && launch_crop(wide, (float *)out, B, Cout, f.M, 1, stream) != hipSuccess) return KST_ERR_HIP;
    return KST_OK;
}

}  // namespace

extern "C" {

kst_status kst_forward_seg_padded(const void *in, const void *w_seg, void *out, void *ws, size_t ws_bytes,
                                  int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype, kst_path path,
                                  hipStream_t stream)
{
    const Epilogue none = {nullptr, KST_ACT_NONE};
    return forward_seg_padded_impl(in, w_seg, out, ws, ws_bytes, B, Cin, Cout, N, n, P, dtype, path, none, stream);
}

kst_status kst_forward_seg_epilogue(const void *in, const void *w_seg, const float *bias, void *out, void *ws,
                                    size_t ws_bytes, int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype,
                                    kst_activation act, kst_path path, hipStream_t stream)
{
    if (act != KST_ACT_NONE && act != KST_ACT_RELU && act != KST_ACT_TANH) return KST_ERR_ACT;
    if (bias && (reinterpret_cast<uintptr_t>(bias) & 3u) != 0) return KST_ERR_ALIGN;
    const Epilogue epi = {bias, (int)act};
    return forward_seg_padded_impl(in, w_seg, out, ws, ws_bytes, B, Cin, Cout, N, n, P, dtype, path, epi, stream);
}

kst_status kst_forward_padded(const void *in, const void *w, void *out, int B, int Cin, int Cout, int N, int n, int P,
                              kst_dtype dtype, hipStream_t stream)
{
    if (P == 0) return kst_forward(in, w, out, B, Cin, Cout, N, n, dtype, stream);
    if (!in || !w || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    Framed f;
    kst_status st = framed_plan(B, Cin, Cout, N, n, P, dtype, KST_PATH_AUTO, false, &f);
    if (st != KST_OK) return st;
    if (!aligned16(in) || !aligned16(w) || !aligned16(out)) return KST_ERR_ALIGN;
    const size_t seg_bytes = (seg_elems(Cin, Cout, n, dtype) * elt_bytes(dtype) + 255) & ~(size_t)255;
    size_t ws_bytes = framed_bytes(f, dtype);          // may be 0
    const auto least = [&] {
        return framed_plan(B, Cin, Cout, N, n, P, dtype, KST_PATH_AUTO, true, &f) == KST_OK ? framed_bytes(f, dtype) : ws_bytes;
    };
    void *scratch = nullptr;
    if (!scratch_for(&scratch, seg_bytes, &ws_bytes, stream, least)) return KST_ERR_HIP;
    // (a repacked layer has the frame in its input's copy and stores what is wanted of the map: nothing else in its workspace)
    if (f.s.frame > 0 && repacks_16(f.s, dtype, f.chosen)) {
        st = run_repacked_16(in, w, out, scratch, seg_bytes, f.s, dtype, stream);
    } else {
        st = kst_segregate_weights(w, scratch, Cin, Cout, n, dtype, stream);
        if (st == KST_OK)
            st = kst_forward_seg_padded(in, scratch, out, ws_bytes ? (char *)scratch + seg_bytes : nullptr, ws_bytes, B, Cin,
                                        Cout, N, n, P, dtype, KST_PATH_AUTO, stream);
    }
    if (hipFreeAsync(scratch, stream) != hipSuccess && st == KST_OK) st = KST_ERR_HIP;
    return st;
}

// ---- gradients --------------------------------------------------------------------------------
namespace {

// The input gradient's kernels on the bf16 matrix cores: none for this layer, those that split g while staging (half
// precision's weights are widened to fp32 first), or those that repack it.
enum SplitDinKernel { SPLIT_DIN_NONE, SPLIT_DIN_STAGED, SPLIT_DIN_PACKED };
struct SplitDin {
    SplitDinKernel kernel;
    size_t wconv, bytes;              // widened weights at the start of the workspace; all of it
};

// image, cores: the layer is the image layers' kernel's, the fp32 matrix cores take it.
SplitDin split_din_plan(const Shape &si, bool odd, kst_dtype dt, bool image, bool cores)
{
    SplitDin r = {SPLIT_DIN_NONE, 0, 0};
    const kst_dtype staged = dt == KST_F16 ? KST_F32 : dt;
    if (split_din_applies(si, odd, staged)) {
        r.kernel = SPLIT_DIN_STAGED;
        if (dt == KST_F16) r.wconv = ((size_t)si.Cout * si.Cin * si.n * si.n * sizeof(float) + 255) & ~(size_t)255;
        r.bytes = r.wconv + split_din_workspace_bytes(si, odd, staged);
    } else if (!image && din_packed_applies(si, odd, dt, cores)) {
        r.kernel = SPLIT_DIN_PACKED;
        r.bytes = din_packed_workspace_bytes(si, odd, dt);
    }
    return r;
}

// Workspace of the gradient entry points: for P > 0 the unframed kernels run on framed copies.
//   input gradient:  [g framed by one zero (odd P)] [din of the framed input] [partial sums of the
//                    matrix-core kernel's split reduction]
//   kernel gradient: [input framed by q] [g framed by one zero (odd P)] [partial sums, as above]
struct GradPlan {
    int q, Nq, M, Mq;
    Shape s;                          // the problem on the framed input map (what the plain kernels see)
    Shape si;                         // the same with frame = q: the matrix-core kernels work on the unframed
                                      // positions only (din without the frame; in read as it lies in memory)
    size_t g_bytes, din_bytes, in_bytes;
    size_t split_bytes, wsplit_bytes; // input / kernel gradient on the matrix cores: partial sums
    size_t gw_bytes;                  // kernel gradient on the matrix cores: its framed copy of g (replaces g_bytes)
    int gw_frame, gw_stride;          // frame on the caller's g and row stride of that copy
    bool plain_unframed;              // the other kernels work on the unframed positions too (kernels up to 7 x 7)
    bool din_cores, dw_cores;         // the gradient runs on the matrix cores (fp32 kernels; 16-bit operands are
                                      // widened to fp32 first, which is exact)
    size_t wconv_bytes, xconv_bytes;  // fp32 copies of w (input gradient) and of in (kernel gradient) for that
    Shape image;                      // the problem as the image layers' kernels see it
    bool din_image, dw_image;
    // The same on the bf16 matrix cores, with workspaces of their own; only where the caller's is large enough.
    SplitDinKernel din_split;
    bool use_dw_split;
    size_t din_split_wconv;           // widened half-precision weights
    size_t din_split_bytes, dw_split_bytes;    // whole workspace, as the launch lays it out
    size_t din_bytes_needed() const { return din_image ? 0 : g_bytes + din_bytes + split_bytes + wconv_bytes; }
    size_t dw_bytes_needed() const
    {
        if (dw_image) return wsplit_bytes;
        return dw_cores ? gw_bytes + wsplit_bytes + xconv_bytes : in_bytes + g_bytes + wsplit_bytes;
    }
};

// lean: the caller has less scratch than the image layers' kernel gradient wants for its partial results.
kst_status grad_plan(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dt, bool lean, GradPlan *f)
{
    if (P < 0 || P > 32768 || B < 1 || N < 1 || N > 32768) return KST_ERR_SHAPE;
    f->q = (P + 1) / 2;
    f->Nq = N + 2 * f->q;
    kst_status st = check_shape(B, Cin, Cout, f->Nq, n);
    if (st != KST_OK) return st;
    f->M = 2 * N + 2 * P - n;
    f->Mq = 2 * f->Nq - n;
    if (f->M < 1) return KST_ERR_SHAPE;
    f->s = make_shape(B, Cin, Cout, f->Nq, n);
    f->g_bytes = (P & 1) ? (((size_t)B * Cout * f->Mq * f->Mq * sizeof(float) + 255) & ~(size_t)255) : 0;
    f->din_bytes = P ? (((size_t)B * Cin * f->Nq * f->Nq * sizeof(float) + 255) & ~(size_t)255) : 0;
    f->in_bytes = P ? (((size_t)B * Cin * f->Nq * f->Nq * elt_bytes(dt) + 255) & ~(size_t)255) : 0;
    f->si = f->s;
    f->si.frame = f->q;
    f->split_bytes = 0;
    f->plain_unframed = backward_generic_takes_frame(f->si);
    f->din_cores = backward_input_igemm_supported(f->si, KST_F32);
    f->dw_cores = backward_weight_igemm_supported(f->si, KST_F32);
    f->wconv_bytes = is16(dt) && f->din_cores ? (((size_t)Cout * Cin * n * n * sizeof(float) + 255) & ~(size_t)255) : 0;
    f->xconv_bytes = is16(dt) && f->dw_cores ? (((size_t)B * Cin * N * N * sizeof(float) + 255) & ~(size_t)255) : 0;
    if (f->din_cores) {
        f->split_bytes = backward_input_igemm_workspace_bytes(f->si);
        f->din_bytes = 0;                              // written in place, frame never computed
    } else if (f->plain_unframed) {
        f->din_bytes = 0;
    }
    if (f->plain_unframed) f->in_bytes = 0;            // `in` read as it lies in memory
    f->image = f->si;
    f->image.crop = P & 1;
    f->image.lean = lean;
    f->din_image = !f->din_cores && backward_input_image_apply(f->image);
    f->dw_image = !f->dw_cores && backward_weight_image_apply(f->image);
    const bool odd = (P & 1) != 0;
    const SplitDin din = split_din_plan(f->si, odd, dt, f->din_image, f->din_cores);
    f->din_split = din.kernel;
    f->din_split_wconv = din.wconv;
    f->din_split_bytes = din.bytes;
    f->use_dw_split = split_dw_applies(f->si, odd, dt);
    f->dw_split_bytes = f->use_dw_split ? split_dw_workspace_bytes(f->si, odd, dt, false) : 0;
    f->wsplit_bytes = f->dw_image ? backward_weight_image_workspace_bytes(f->image)
                      : f->dw_cores
                          ? backward_weight_igemm_workspace_bytes(f->si)
                          : backward_weight_generic_workspace_bytes(f->plain_unframed ? f->si : f->s);
    f->gw_bytes = 0;
    f->gw_frame = f->gw_stride = 0;
    if (f->dw_cores) {
        int frame, stride;
        backward_weight_igemm_g_copy(f->si, &frame, &stride);
        f->gw_frame = frame + (P & 1);                 // on top of the odd padding factor's one-pixel frame
        f->gw_stride = stride;
        const size_t rows = (size_t)f->M + 2 * (size_t)f->gw_frame;
        f->gw_bytes = ((size_t)B * Cout * rows * stride * sizeof(float) + 255) & ~(size_t)255;
    }
    return KST_OK;
}

}  // namespace

// The queries give both 16-bit types one size, the larger, where both run on the same kernels for the bf16 matrix cores: what
// these lay out depends on the type.  (Where bfloat16 weights run on the kernels that split g while staging and half
// precision's, whose three parts these multiply, do not, bfloat16 has its own size and half precision no less.)
size_t kst_backward_input_workspace_bytes(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype)
{
    GradPlan f;
    if (!dtype_ok(dtype) || grad_plan(B, Cin, Cout, N, n, P, dtype, false, &f) != KST_OK) return 0;
    if (f.din_split == SPLIT_DIN_NONE) return f.din_bytes_needed();
    if (is16(dtype)) {
        const SplitDin other = split_din_plan(f.si, (P & 1) != 0, other16(dtype), f.din_image, f.din_cores);
        if ((other.kernel == f.din_split || dtype == KST_F16) && other.bytes > f.din_split_bytes) return other.bytes;
    }
    return f.din_split_bytes;
}

size_t kst_backward_weight_workspace_bytes(int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype)
{
    GradPlan f;
    if (!dtype_ok(dtype) || grad_plan(B, Cin, Cout, N, n, P, dtype, false, &f) != KST_OK) return 0;
    if (!f.use_dw_split) return f.dw_bytes_needed();
    // (with room for three parts of the input whatever its type, and for its widened copy, which the fp32 multiplies read;
    // where only bfloat16's items are whole, half precision has no less)
    const bool odd = (P & 1) != 0;
    size_t bytes = split_dw_workspace_bytes(f.si, odd, dtype, true);
    if (dtype == KST_F16 && split_dw_applies(f.si, odd, KST_BF16)) {
        const size_t other = split_dw_workspace_bytes(f.si, odd, KST_BF16, true);
        if (other > bytes) bytes = other;
    }
    return bytes + f.xconv_bytes;
}

kst_status kst_backward_input(const void *g, const void *w, void *din, void *ws, size_t ws_bytes,
                              int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype, hipStream_t stream)
{
    if (!g || !w || !din) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    GradPlan f;
    kst_status st = grad_plan(B, Cin, Cout, N, n, P, dtype, false, &f);
    if (st != KST_OK) return st;
    if (!aligned16(g) || !aligned16(w) || !aligned16(din)) return KST_ERR_ALIGN;
    const bool split = f.din_split != SPLIT_DIN_NONE && ws && ws_bytes >= f.din_split_bytes;
    const size_t need = split ? f.din_split_bytes : f.din_bytes_needed();
    if (need) {
        if (!ws || ws_bytes < need) return KST_ERR_WORKSPACE;
        if (!aligned16(ws)) return KST_ERR_ALIGN;
    }
    if (split && f.din_split == SPLIT_DIN_PACKED)
        return launch_din_packed((const float *)g, w, (float *)din, ws, f.si, (P & 1) != 0, dtype, stream) == hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    if (split) {
        const void *w_in = w;
        if (dtype == KST_F16) {
            if (launch_widen(w, (float *)ws, (size_t)Cout * Cin * n * n, dtype, stream) != hipSuccess) return KST_ERR_HIP;
            w_in = ws;
        }
        return launch_split_din((const float *)g, w_in, (float *)din, (char *)ws + f.din_split_wconv, f.si, (P & 1) != 0,
                                dtype == KST_F16 ? KST_F32 : dtype, stream) == hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    }
    if (f.din_image)
        return launch_backward_input_image((const float *)g, w, (float *)din, f.image, dtype, stream) == hipSuccess ? KST_OK
                                                                                                                  : KST_ERR_HIP;
    const float *g_in = (const float *)g;
    float *d_out = (float *)din;
    if (f.g_bytes) {          // odd P: the forward dropped the outermost ring of the wider output
        if (launch_frame_input(g, ws, B, Cout, f.M, 1, f.Mq, KST_F32, stream) != hipSuccess) return KST_ERR_HIP;
        g_in = (const float *)ws;
    }
    if (f.din_cores) {
        // the matrix-core kernels compute the unframed positions only, straight into din
        void *split_ws = f.split_bytes ? (char *)ws + f.g_bytes : nullptr;
        const float *w32 = (const float *)w;
        if (f.wconv_bytes) {
            float *wc = (float *)((char *)ws + f.g_bytes + f.split_bytes);
            if (launch_widen(w, wc, (size_t)Cout * Cin * n * n, dtype, stream) != hipSuccess) return KST_ERR_HIP;
            w32 = wc;
        }
        return launch_backward_input_igemm(g_in, w32, (float *)din, split_ws, f.si, stream) == hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    }
    if (f.plain_unframed)
        return launch_backward_input_generic(g_in, w, d_out, f.si, dtype, stream) == hipSuccess ? KST_OK : KST_ERR_HIP;
    if (P) d_out = (float *)((char *)ws + f.g_bytes);
    if (launch_backward_input_generic(g_in, w, d_out, f.s, dtype, stream) != hipSuccess) return KST_ERR_HIP;
    if (P && launch_crop(d_out, (float *)din, B, Cin, N, f.q, stream) != hipSuccess) return KST_ERR_HIP;
    return KST_OK;
}

kst_status kst_backward_weight(const void *in, const void *g, void *dw, void *ws, size_t ws_bytes,
                               int B, int Cin, int Cout, int N, int n, int P, kst_dtype dtype, hipStream_t stream)
{
    if (!in || !g || !dw) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    GradPlan f;
    kst_status st = grad_plan(B, Cin, Cout, N, n, P, dtype, false, &f);
    if (st != KST_OK) return st;
    if (!aligned16(in) || !aligned16(g) || !aligned16(dw)) return KST_ERR_ALIGN;
    if (f.use_dw_split && ws && ws_bytes >= f.dw_split_bytes) {
        if (!aligned16(ws)) return KST_ERR_ALIGN;
        return launch_split_dw(in, (const float *)g, (float *)dw, ws, f.si, (P & 1) != 0, dtype, stream) == hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    }
    if (f.dw_image && (ws ? ws_bytes : 0) < f.dw_bytes_needed()) {
        st = grad_plan(B, Cin, Cout, N, n, P, dtype, true, &f);
        if (st != KST_OK) return st;
    }
    const bool cores = f.dw_cores;
    const size_t g_copy = cores ? f.gw_bytes : f.g_bytes;
    const size_t in_copy = cores ? 0 : f.in_bytes;     // the matrix-core kernel reads `in` as it lies in memory
    const size_t need = f.dw_bytes_needed();
    if (need) {
        if (!ws || ws_bytes < need) return KST_ERR_WORKSPACE;
        if (!aligned16(ws)) return KST_ERR_ALIGN;
    }
    if (f.dw_image)
        return launch_backward_weight_image(in, (const float *)g, (float *)dw, ws, f.image, dtype, stream) == hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    const void *x_in = in;
    const float *g_in = (const float *)g;
    if (P && !cores && !f.plain_unframed) {
        if (launch_frame_input(in, ws, B, Cin, N, f.q, f.Nq, dtype, stream) != hipSuccess) return KST_ERR_HIP;
        x_in = ws;
    }
    void *gw = (char *)ws + in_copy;
    void *partial_ws = f.wsplit_bytes ? (char *)ws + in_copy + g_copy : nullptr;
    if (cores) {
        if (f.xconv_bytes) {
            float *xc = (float *)((char *)ws + in_copy + g_copy + f.wsplit_bytes);
            if (launch_widen(in, xc, (size_t)B * Cin * N * N, dtype, stream) != hipSuccess) return KST_ERR_HIP;
            x_in = xc;
        }
        // g framed once for the odd padding factor and for the kernel's own bounds-free reads
        if (launch_frame_input(g, gw, B, Cout, f.M, f.gw_frame, f.gw_stride, KST_F32, stream) != hipSuccess)
            return KST_ERR_HIP;
        return launch_backward_weight_igemm((const float *)x_in, (const float *)gw, (float *)dw, partial_ws, f.si, stream) ==
                       hipSuccess
                   ? KST_OK
                   : KST_ERR_HIP;
    }
    if (f.g_bytes) {
        if (launch_frame_input(g, gw, B, Cout, f.M, 1, f.Mq, KST_F32, stream) != hipSuccess) return KST_ERR_HIP;
        g_in = (const float *)gw;
    }
    return launch_backward_weight_generic(x_in, g_in, (float *)dw, partial_ws, f.plain_unframed ? f.si : f.s, dtype,
                                          stream) == hipSuccess
               ? KST_OK
               : KST_ERR_HIP;
}

kst_status kst_forward_zero_insert(const void *in, const void *w, void *U, void *out, int B, int Cin, int Cout,
                                   int N, int n, kst_dtype dtype, hipStream_t stream)
{
    if (!in || !w || !U || !out) return KST_ERR_NULL;
    if (!dtype_ok(dtype)) return KST_ERR_DTYPE;
    kst_status st = check_shape(B, Cin, Cout, N, n);
    if (st != KST_OK) return st;
    if (!aligned16(in) || !aligned16(w) || !aligned16(U) || !aligned16(out)) return KST_ERR_ALIGN;
    const Shape s = make_shape(B, Cin, Cout, N, n);
    return launch_zero_insert(in, w, U, (float *)out, s, dtype, stream) == hipSuccess ? KST_OK : KST_ERR_HIP;
}

size_t kst_yardstick_mfma_sink_elems(void) { return yardstick_mfma_sink_elems(); }

double kst_yardstick_mfma_flops(kst_dtype dtype, int iters)
{
    if ((dtype != KST_F32 && dtype != KST_BF16) || iters < 1) return 0.0;
    return yardstick_mfma_flops(dtype, iters);
}

kst_status kst_yardstick_mfma(kst_dtype dtype, int iters, float *sink, size_t sink_elems, hipStream_t stream)
{
    if (!sink) return KST_ERR_NULL;
    if (dtype != KST_F32 && dtype != KST_BF16) return KST_ERR_DTYPE;
    if (iters < 1 || iters > (1 << 22)) return KST_ERR_SHAPE;
    if (sink_elems < yardstick_mfma_sink_elems()) return KST_ERR_WORKSPACE;
    return launch_yardstick_mfma(dtype, iters, sink, stream) == hipSuccess ? KST_OK : KST_ERR_HIP;
}

kst_status kst_yardstick_copy(const void *src, void *dst, size_t bytes, hipStream_t stream)
{
    if (!src || !dst) return KST_ERR_NULL;
    if (bytes % 16 != 0) return KST_ERR_SHAPE;
    if (!aligned16(src) || !aligned16(dst)) return KST_ERR_ALIGN;
    return launch_yardstick_copy(src, dst, bytes, stream) == hipSuccess ? KST_OK : KST_ERR_HIP;
}

}  // extern "C"

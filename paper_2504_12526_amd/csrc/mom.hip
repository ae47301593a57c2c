// libmom: C ABI over the gfx950 kernels of the MOM prefill hot path (see include/mom.h).
//
// Host side: argument validation, the mini-sequence driver (Algorithm 1, else-branch), the
// last-token LM head launch and the KV offload and reload copies.  Nothing here allocates or synchronises.
// The only state is what mom_init resolves per device (compute-unit count, address of the static
// workspace) and the testing overrides of the mom_debug_force_ calls.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <tuple>
#include <type_traits>

#include "mom.h"
#include "mom_gemm_forms.h"
#include "mom_gemm_rect_schedule.h"
#include "mom_gemm_schedule.h"
#include "mom_gemm.hip.inc"
#include "mom_gemm_short.hip.inc"
#include "mom_gemm_rect.hip.inc"
#include "mom_block.hip.inc"
#include "mom_gemv.hip.inc"
#include "mom_kv.hip.inc"
#include "mom_probe.hip.inc"

// Workspace of mom_mlp_prefill_static: one copy per device, held from the moment the library is
// loaded on a device until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the device address it yields (kept per device in g_dev) is what kernels get.
static __device__ __align__(256) unsigned char scratch[MOM_STATIC_WORKSPACE_BYTES];

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    if (na == 0 || nb == 0) return false;
    uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + nb && b0 < a0 + na;
}

inline int64_t effective_chunk(int64_t S, int64_t mini_seq) {
    return (mini_seq <= 0 || mini_seq > S) ? S : mini_seq;
}

int validate_mlp(const void* x, const void* wg, const void* wu, const void* wd, int64_t S, int64_t H,
                 int64_t I, int64_t mini_seq, const void* out, const void* ws, size_t ws_bytes) {
    if (S < 0 || H <= 0 || I <= 0 || mini_seq < 0) return MOM_ERR_SHAPE;
    if ((H % 32) != 0 || (I % 32) != 0) return MOM_ERR_SHAPE;
    if (S > (int64_t)0x7fffff00 || H > (1 << 20) || I > (1 << 20)) return MOM_ERR_SHAPE;
    if (S == 0) return MOM_OK;
    if (!x || !wg || !wu || !wd || !out || !ws) return MOM_ERR_NULL;
    if (!aligned16(x) || !aligned16(wg) || !aligned16(wu) || !aligned16(wd) || !aligned16(out) ||
        !aligned16(ws))
        return MOM_ERR_ALIGN;
    const size_t need = mom_mlp_workspace_bytes(S, H, I, mini_seq);
    if (ws_bytes < need) return MOM_ERR_WORKSPACE;
    const size_t xb = (size_t)S * H * 2, wb = (size_t)H * I * 2;
    const void* ins[4] = {x, wg, wu, wd};
    const size_t inb[4] = {xb, wb, wb, wb};
    for (int i = 0; i < 4; ++i)
        if (overlaps(out, xb, ins[i], inb[i]) || overlaps(ws, need, ins[i], inb[i])) return MOM_ERR_ALIAS;
    if (overlaps(out, xb, ws, need)) return MOM_ERR_ALIAS;
    return MOM_OK;
}

// Whether a query succeeded whose failure is an answer like any other: its error is not left for the program to find, and an
// error that was there before is left alone where the query succeeds.
inline bool answered(hipError_t e) {
    if (e == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Per-device data, resolved once per device (by mom_init or by the first call that needs it) with
// that device current.
constexpr int kMaxDevices = 64;
struct DeviceInfo {
    std::atomic<int> cus{0};                 // compute units, 0 = not resolved yet
    std::atomic<void*> static_ws{nullptr};   // device address of this device's copy of `scratch`
};
DeviceInfo g_dev[kMaxDevices];

// Testing overrides (the mom_debug_force_ calls); 0 = the library chooses.
std::atomic<int> g_force_edge{0}, g_force_width{0};
std::atomic<int> g_force_short{0}, g_force_rect{0};      // token rows << 16 | weight rows
std::atomic<int> g_force_block{0};      // token rows of a block

DeviceInfo* current_device_info() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return &g_dev[dev];
}

// Compute units of the current device, or 0 on error.
int compute_units() {
    DeviceInfo* d = current_device_info();
    if (!d) return 0;
    int cus = d->cus.load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 0;
    d->cus.store(cus, std::memory_order_relaxed);
    return cus;
}

// Device address of the current device's copy of `scratch`, or nullptr on error.
void* static_workspace() {
    DeviceInfo* d = current_device_info();
    if (!d) return nullptr;
    void* p = d->static_ws.load(std::memory_order_acquire);
    if (p) return p;
    if (!answered(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) || !p) return nullptr;
    d->static_ws.store(p, std::memory_order_release);
    return p;
}

// MOM_OK if the n bytes at p are page-locked host memory known to the HIP runtime.  Pageable memory
// would make hipMemcpyAsync stage the copy and block the calling thread, which the contract of the
// KV calls ("only enqueue") excludes.
int check_pinned_host(const void* p, size_t n) {
    const unsigned char* b = static_cast<const unsigned char*>(p);
    const unsigned char* ends[2] = {b, b + (n ? n - 1 : 0)};
    for (const unsigned char* q : ends) {
        hipPointerAttribute_t at;
        if (!answered(hipPointerGetAttributes(&at, q)) || at.type != hipMemoryTypeHost) return MOM_ERR_HOST;
    }
    return MOM_OK;
}

// Whether the n bytes at p lie in one allocation, as the runtime's copies demand (they refuse others, also where the
// next allocation follows without a gap).
bool in_one_allocation(const void* p, size_t n) {
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (!answered(hipMemGetAddressRange(&base, &size, const_cast<void*>(p)))) return false;
    const size_t at = static_cast<size_t>(static_cast<const unsigned char*>(p) - static_cast<const unsigned char*>(base));
    return at <= size && n <= size - at;
}

// Whether stream st has nothing left to do.  Asked in relaxed capture mode: in another the question ends a capture that is
// under way on any stream (hipErrorStreamCaptureUnsupported, and hipErrorStreamCaptureInvalidated at its end).
bool is_ready(hipStream_t st) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (!answered(hipThreadExchangeStreamCaptureMode(&mode))) return true;
    const hipError_t e = hipStreamQuery(st);
    (void)answered(hipThreadExchangeStreamCaptureMode(&mode));
    return e != hipErrorNotReady && (answered(e), true);         // (hipErrorNotReady is no error that the runtime keeps)
}

// Whether p is memory of the current device.
bool on_current_device(const void* p) {
    int dev = 0;
    hipPointerAttribute_t at;
    return answered(hipGetDevice(&dev)) && answered(hipPointerGetAttributes(&at, p)) && at.type == hipMemoryTypeDevice && at.device == dev;
}

// The device address of pinned_host if kv_reload_kernel is to copy bytes_each bytes each into k and v on stream st, else nullptr:
// whole 16-byte chunks, buffers of the current device, which is also the stream's, each in one allocation and not overlapping, up to
// 16 GiB each (its 32-bit chunk numbers).  Up to 1 MiB each the kernel is the faster one by itself (256 KiB 34 -> 14 us, 512 KiB 46 -> 34)
// and costs the kernels beside it no more than copies do.  Larger ones do (mom_kv.hip.inc has the times), so they go by copies on a
// stream that is ready (five last-token branches beside 2 x 16 MiB 1242 -> 1097 us).  Behind work that is still to be done the runtime may
// hold the calling thread in a copy, so there it is the kernel (8192 tokens, 40 and more passes enqueued ahead, 863 -> 647 us); the question
// takes 6 ... 10 us then.  Captured calls, whose copies the graph starts, take the kernel up to 256 KiB each.
const void* reload_source(const void* pinned_host, const void* k, const void* v, size_t bytes_each, hipStream_t st) {
    if (bytes_each > ((size_t)16 << 30) || bytes_each % 16 || !aligned16(pinned_host) || !aligned16(k) || !aligned16(v)) return nullptr;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (bytes_each > ((size_t)256 << 10) && (!answered(hipStreamIsCapturing(st, &capture)) || capture != hipStreamCaptureStatusNone)) return nullptr;
    if (bytes_each > ((size_t)1 << 20) && is_ready(st)) return nullptr;
    if (overlaps(k, bytes_each, v, bytes_each)) return nullptr;
    int dev = 0, stream_dev = 0;
    if (!answered(hipGetDevice(&dev)) || (st && (!answered(hipStreamGetDevice(st, &stream_dev)) || stream_dev != dev))) return nullptr;
    hipPointerAttribute_t at;
    for (const void* p : {k, v})
        if (!answered(hipPointerGetAttributes(&at, p)) || at.type != hipMemoryTypeDevice || at.device != dev || !in_one_allocation(p, bytes_each))
            return nullptr;
    if (!answered(hipPointerGetAttributes(&at, pinned_host)) || !at.devicePointer || !in_one_allocation(pinned_host, 2 * bytes_each)) return nullptr;
    return aligned16(at.devicePointer) ? at.devicePointer : nullptr;
}

// One launch, judged by its own return value: hipGetLastError() would report (and take away) an error that some earlier call of
// the program left behind, which successful calls don't clear.
template <typename... P, typename... A>
hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, A... args) {
    std::tuple<std::remove_cv_t<P>...> values(args...);
    return std::apply([&](auto&... v) {
        void* ptrs[] = {static_cast<void*>(&v)...};
        return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, st);
    }, values);
}

// The launch part described by `a` takes the tiles of `g`.
void set_tile_grid(momk::GemmArgs& a, const momk::TileGrid& g) {
    a.tiles_m = (int)g.tiles_m;
    a.tiles_n = (int)g.tiles_n;
    a.group_m = momk::kTokenGroup;
    a.tiles_per_xcd = momk::tiles_per_xcd(g.tiles);
}

// One launch of gemm_rect_kernel<EPI, l.tm, l.tn>.
template <int EPI>
hipError_t launch_rect_tiles(const momk::GemmArgs& a, const momk::Launch& l, bool nt, hipStream_t st) {
    const dim3 grid((unsigned)(a.tiles_per_xcd * 8)), block(momk::k4Threads);
#define MOM_LAUNCH_RECT(TM, TN)                                                                                   \
    if (l.tm == TM && l.tn == TN) {                                                                               \
        if (EPI == momk::EPI_GATEUP && nt)                                                                        \
            return launch(momk::gemm_rect_kernel<EPI, TM, TN, EPI == momk::EPI_GATEUP>, grid, block, 0, st, a);   \
        return launch(momk::gemm_rect_kernel<EPI, TM, TN, false>, grid, block, 0, st, a);                         \
    }
    if constexpr (EPI == momk::EPI_GATEUP) { MOM_RECT_FORMS_GATEUP(MOM_LAUNCH_RECT) }
    else { MOM_RECT_FORMS_DOWN(MOM_LAUNCH_RECT) }
#undef MOM_LAUNCH_RECT
    return hipErrorInvalidValue;
}

// One launch of gemm4_kernel<EPI, l.tm, l.tn>, or of the rectangular tiles, over the operands in `a` (M, N, K, ldo set).  more: the call has more
// than one mini-sequence.
template <int EPI>
hipError_t launch_whole_tiles(momk::GemmArgs a, const momk::Launch& l, bool more, hipStream_t st) {
    set_tile_grid(a, l.grid);
    const int edge = l.tm, width = l.tn;
    const dim3 grid((unsigned)(a.tiles_per_xcd * 8)), block(momk::k4Threads);
    const bool nt = EPI == momk::EPI_GATEUP && momk::weights_once(a.tiles_m, a.N, a.K, more);
    if (momk::is_rect_form(EPI == momk::EPI_GATEUP, edge, width)) return launch_rect_tiles<EPI>(a, l, nt, st);
#define MOM_LAUNCH4(E, W)                                                                                         \
    if (edge == E && width == W) {                                                                                \
        if constexpr (EPI == momk::EPI_GATEUP && E == 256) {                                                      \
            if (nt) return launch(momk::gemm4_kernel<EPI, E, W, true>, grid, block, 0, st, a);                    \
        }                                                                                                         \
        return launch(momk::gemm4_kernel<EPI, E, W, false>, grid, block, 0, st, a);                               \
    }
    MOM_LAUNCH4(256, 256)
    MOM_LAUNCH4(256, 192)
    if constexpr (EPI == momk::EPI_DOWN) {
        MOM_LAUNCH4(256, 224)
        MOM_LAUNCH4(256, 160)
        MOM_LAUNCH4(256, 128)
    } else {
        MOM_LAUNCH4(128, 128)
    }
#undef MOM_LAUNCH4
    return hipErrorInvalidValue;
}

// One launch in the short form l.form (mom_gemm_forms.h).
template <int EPI>
hipError_t launch_short_tiles(momk::GemmArgs a, const momk::Launch& l, bool more, hipStream_t st) {
    set_tile_grid(a, l.grid);
    const dim3 grid((unsigned)(a.tiles_per_xcd * 8)), block(momk::k4Threads);
    const bool nt = EPI == momk::EPI_GATEUP && momk::weights_once(a.tiles_m, a.N, a.K, more);
    int i = 0;
#define MOM_LAUNCH_SHORT(TM, TN, WM, WN, KSUB, NSTG)                                                              \
    if (i++ == l.form) {                                                                                          \
        if (EPI == momk::EPI_GATEUP && nt)                                                                        \
            return launch(momk::gemm_short_kernel<EPI, TM, TN, WM, WN, KSUB, NSTG, EPI == momk::EPI_GATEUP>,      \
                          grid, block, 0, st, a);                                                                 \
        return launch(momk::gemm_short_kernel<EPI, TM, TN, WM, WN, KSUB, NSTG, false>, grid, block, 0, st, a);    \
    }
    if constexpr (EPI == momk::EPI_GATEUP) { MOM_SHORT_FORMS_GATEUP(MOM_LAUNCH_SHORT) }
    else { MOM_SHORT_FORMS_DOWN(MOM_LAUNCH_SHORT) }
#undef MOM_LAUNCH_SHORT
    return hipErrorInvalidValue;
}

// The launch a mom_debug_force_ call asks for (tests need every form on shapes of every size); kRefused with form -1
// where none does.
momk::Launch forced_launch(int64_t M, int64_t N, bool gateup) {
    const int fr = g_force_rect.load(std::memory_order_relaxed);
    if (fr && momk::is_rect_form(gateup, fr >> 16, fr & 0xffff)) return momk::whole_launch(M, N, gateup, fr >> 16, fr & 0xffff);
    const int fs = g_force_short.load(std::memory_order_relaxed);
    if (fs) {
        const int form = momk::find_short_form(gateup, fs >> 16, fs & 0xffff);
        if (form >= 0) return momk::short_launch(M, N, gateup, form);
    }
    const int force = g_force_edge.load(std::memory_order_relaxed), fw = g_force_width.load(std::memory_order_relaxed);
    if (force == 256) return momk::whole_launch(M, N, gateup, 256, (fw && (!gateup || fw == 192)) ? fw : 256);
    if (force == 128 && gateup) return momk::whole_launch(M, N, gateup, 128, 128);
    if (force) return momk::short_launch(M, N, gateup, momk::find_short_form(gateup, force, force));
    return {momk::kRefused, -1, 0, 0, 0, {}, {}};
}

// O[m, n] of M token rows x N output columns by launch l, the intermediate from row `split` on at `rest` (GemmArgs).  more: the call has more
// than one mini-sequence.
template <int EPI>
hipError_t launch_gemm(const momk::Launch& l, const unsigned short* X, const unsigned short* W0, const unsigned short* W1,
                       unsigned short* O, unsigned short* rest, int split, int M, int N, int K, hipStream_t st, bool more) {
    constexpr bool GU = EPI == momk::EPI_GATEUP;
    momk::GemmArgs a;
    a.X = X; a.W0 = W0; a.W1 = W1; a.O = O; a.rest = rest; a.split = split;
    a.M = M; a.N = N; a.K = K; a.ldo = N;
    switch (l.kind) {
        case momk::kShortTiles: return launch_short_tiles<EPI>(a, l, more, st);
        case momk::kWholeTiles: return launch_whole_tiles<EPI>(a, l, more, st);
        case momk::kTwoWidths:
            if constexpr (GU) {
                momk::GemmArgs2 p = {a, a};
                p.wide.N = (int)l.wide_cols;
                p.narrow.W0 = W0 + (size_t)l.wide_cols * K;
                p.narrow.W1 = W1 + (size_t)l.wide_cols * K;
                p.narrow.O = O + l.wide_cols;
                p.narrow.rest = rest + l.wide_cols;
                p.narrow.N = N - (int)l.wide_cols;
                set_tile_grid(p.wide, l.grid);
                set_tile_grid(p.narrow, l.narrow);
                const int64_t wgs = 8 * ((int64_t)p.wide.tiles_per_xcd + p.narrow.tiles_per_xcd);
                if (wgs > (int64_t)0x7fffffff) return hipErrorInvalidValue;
                if (momk::weights_once(p.wide.tiles_m, N, K, more))
                    return launch(momk::gemm4_two_width_kernel<EPI, 192, true>, dim3((unsigned)wgs), dim3(momk::k4Threads), 0, st, p);
                return launch(momk::gemm4_two_width_kernel<EPI, 192, false>, dim3((unsigned)wgs), dim3(momk::k4Threads), 0, st, p);
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

// All S rows by blocks of form `form` (mom_gemm_forms.h).
hipError_t launch_blocks(int form, const unsigned short* x, const unsigned short* wg, const unsigned short* wu, const unsigned short* wd,
                         unsigned short* out, int64_t S, int64_t H, int64_t I, hipStream_t st) {
    const int cus = compute_units();
    if (cus <= 0 || form >= momk::kBlockFormCount) return hipErrorInvalidValue;
    const uint32_t blocks = momk::block_count(momk::kBlockForms[form], S);
    const int share = momk::block_share(blocks, H, cus);
    const dim3 grid(blocks, momk::block_parts(H, share));
    int i = 0;
#define MOM_LAUNCH_BLOCK(TB, WAVES, R)                                                                            \
    if (i++ == form)                                                                                              \
        return launch(momk::mlp_block_kernel<TB, WAVES, R>, grid, dim3(WAVES * 64), (size_t)momk::block_lds(16 * TB, H, I, WAVES * R), st,  \
                      x, wg, wu, wd, out, (int)S, (int)H, (int)I, share);
    MOM_BLOCK_FORMS(MOM_LAUNCH_BLOCK)
#undef MOM_LAUNCH_BLOCK
    return hipErrorInvalidValue;
}

// The form of launch_blocks for a call whose mini-sequences of C rows would take the launches given, or -1.  longer: or longer passes.
int block_form(int64_t S, int64_t H, int64_t I, int64_t C, const momk::Launch& gateup, const momk::Launch& down, bool longer) {
    const int forced = g_force_block.load(std::memory_order_relaxed);
    if (forced) {
        for (int i = 0; i < momk::kBlockFormCount; ++i)
            if (16 * momk::kBlockForms[i].tb == forced && momk::block_fits(momk::kBlockForms[i], H, I)) return i;
        return -1;
    }
    if (S <= C || g_force_edge.load(std::memory_order_relaxed) || g_force_short.load(std::memory_order_relaxed) ||
        g_force_rect.load(std::memory_order_relaxed))
        return -1;
    const int cus = compute_units();
    return cus > 0 ? momk::choose_block(S, H, I, C, cus, gateup, down, longer) : -1;
}

template <int MODE>
hipError_t launch_gemv(const unsigned short* x, const unsigned short* Wa, const unsigned short* Wb, void* y,
                       int64_t R, int64_t K, hipStream_t st) {
    // Wavefronts per workgroup, batches per prefetch step and resident workgroups per CU, as measured on the
    // Llama-3-8B shapes (sweep over 2..16 wavefronts, 1..4 batches, 1..16 workgroups per CU):
    //   LM head  V x 4096     4 wavefronts, 1 batch, 2 per CU   (8 wavefronts per CU, each looping over row groups)
    //   gate/up  2 x I x 4096 2 wavefronts, 2 batches, 16 per CU
    //   down     H x 14336    8 wavefronts, 1 batch, 4 per CU   (the workgroup shares one 28 KiB copy of h in LDS)
    constexpr int WAVES = (MODE == momk::MODE_LOGITS) ? 4 : (MODE == momk::MODE_GATEUP ? 2 : 8);
    constexpr int U = (MODE == momk::MODE_GATEUP) ? 2 : 1;
    constexpr int PER_CU = (MODE == momk::MODE_LOGITS) ? 2 : (MODE == momk::MODE_GATEUP ? 16 : 4);
    const int cus = compute_units();
    if (cus <= 0) return hipErrorInvalidDevice;
    const int64_t groups = (R + momk::gemv_rows_per_group(MODE) - 1) / momk::gemv_rows_per_group(MODE);
    int64_t blocks = (groups + WAVES - 1) / WAVES;
    if (blocks > (int64_t)cus * PER_CU) blocks = (int64_t)cus * PER_CU;
    return launch(momk::gemv_kernel<MODE, WAVES, U>, dim3((unsigned)blocks), dim3(WAVES * 64), (size_t)K * 2, st,
                  x, Wa, Wb, y, (int)R, (int)K);
}

// p, the next pass of `passes`, with the launches that are forced, if any, and its rows where these want them.
momk::Pass as_forced(momk::Pass p, const momk::Passes& passes, int64_t H, int64_t I, int64_t C) {
    const momk::Launch g = forced_launch(p.rows, I, true), d = forced_launch(p.rows, H, false);
    if (g.form >= 0) p.gateup = g;
    if (d.form >= 0) p.down = d;
    if (p.split == momk::kWhole) return p;
    p.split = momk::split_of(p.down, C);
    if (p.gateup.kind != momk::kRefused && p.down.kind != momk::kRefused && p.rows <= momk::most_rows(passes.left, H, I, p.split)) return p;
    return as_forced(passes.plain(), passes, H, I, C);          // no room
}

// The loop over mini-sequences of C rows on one stream.  The arguments have been validated for a workspace of C x I.
int mlp_loop(const void* x, const void* wg, const void* wu, const void* wd, int64_t S, int64_t H, int64_t I, int64_t C,
             void* out, void* ws, void* stream, void** events, int64_t n_events) {
    const int64_t n = (S + C - 1) / C;
    if (events && n_events < 1 + 2 * n) return MOM_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned short* xs = static_cast<const unsigned short*>(x);
    unsigned short* os = static_cast<unsigned short*>(out);
    unsigned short* w = static_cast<unsigned short*>(ws);
    if (events && hipEventRecord(static_cast<hipEvent_t>(events[0]), st) != hipSuccess) return MOM_ERR_HIP;
    const int cus = compute_units();
    if (cus <= 0) return MOM_ERR_HIP;
    // Passes of several mini-sequences keep part of the intermediate in `out`, which then has to be memory of this device: in page-locked
    // host memory or a peer's, which `out` may also be, every column tile would read it through a link.
    const bool longer = !events && momk::longer_passes(S, H, I, C) && on_current_device(out);
    momk::Passes passes(S, H, I, C, cus, longer);
    if (!events) {
        const momk::Pass p = passes.plain();
        const int form = block_form(S, H, I, C, p.gateup, p.down, longer);
        if (form >= 0)
            return launch_blocks(form, xs, static_cast<const unsigned short*>(wg), static_cast<const unsigned short*>(wu),
                                 static_cast<const unsigned short*>(wd), os, S, H, I, st) == hipSuccess ? MOM_OK : MOM_ERR_HIP;
    }
    // Algorithm 1, else-branch: O_i = MLP(A_i) for each mini-sequence, O_i written at its rows of O; several of them as one pass where the
    // rows of O that are still to come have room for the rest of the intermediate.
    int64_t c = 0;
    for (int64_t r0 = 0; r0 < S; ++c) {
        const momk::Pass p = as_forced(passes.next(), passes, H, I, C);
        const int rows = (int)p.rows, split = (int)p.split;
        unsigned short* rest = nullptr;
        if (p.split != momk::kWhole) {
            const uintptr_t end = reinterpret_cast<uintptr_t>(os + S * H), at = (end - (size_t)(p.rows - p.split) * I * 2) & ~(uintptr_t)(momk::kSpareAlign - 1);
            rest = reinterpret_cast<unsigned short*>(at - (size_t)p.split * I * 2);
        }
        if (launch_gemm<momk::EPI_GATEUP>(p.gateup, xs + r0 * H, static_cast<const unsigned short*>(wg),
                                          static_cast<const unsigned short*>(wu), w, rest, split, rows, (int)I, (int)H,
                                          st, n > 1) != hipSuccess)
            return MOM_ERR_HIP;
        if (events && hipEventRecord(static_cast<hipEvent_t>(events[1 + 2 * c]), st) != hipSuccess)
            return MOM_ERR_HIP;
        if (launch_gemm<momk::EPI_DOWN>(p.down, w, static_cast<const unsigned short*>(wd), nullptr, os + r0 * H, rest, split, rows,
                                        (int)H, (int)I, st, n > 1) != hipSuccess)
            return MOM_ERR_HIP;
        if (events && hipEventRecord(static_cast<hipEvent_t>(events[2 + 2 * c]), st) != hipSuccess)
            return MOM_ERR_HIP;
        r0 += p.rows;
        passes.done(p);
    }
    return MOM_OK;
}

int mlp_driver(const void* x, const void* wg, const void* wu, const void* wd, int64_t S, int64_t H,
               int64_t I, int64_t mini_seq, void* out, void* ws, size_t ws_bytes, void* stream,
               void** events, int64_t n_events) {
    const int rc = validate_mlp(x, wg, wu, wd, S, H, I, mini_seq, out, ws, ws_bytes);
    if (rc != MOM_OK || S == 0) return rc;
    return mlp_loop(x, wg, wu, wd, S, H, I, effective_chunk(S, mini_seq), out, ws, stream, events, n_events);
}

}  // namespace

extern "C" {

const char* mom_status_string(int status) {
    switch (status) {
        case MOM_OK: return "ok";
        case MOM_ERR_NULL: return "null pointer";
        case MOM_ERR_SHAPE: return "bad shape (H and I must be positive multiples of 32)";
        case MOM_ERR_ALIGN: return "pointer not 16-byte aligned";
        case MOM_ERR_ALIAS: return "output or workspace overlaps an input";
        case MOM_ERR_WORKSPACE: return "workspace too small";
        case MOM_ERR_HIP: return "HIP runtime error";
        case MOM_ERR_HOST: return "host pointer is not page-locked memory of the HIP runtime";
        default: return "unknown status";
    }
}

int mom_init(void) {
    if (compute_units() <= 0) return MOM_ERR_HIP;
    if (!static_workspace()) return MOM_ERR_HIP;
    return MOM_OK;
}

int mom_debug_force_gemm_form(int tile_edge, int ring_slots, int tile_width) {
    const bool wok = tile_width == 0 || (tile_edge == 256 && (tile_width == 256 || tile_width == 224 || tile_width == 192 ||
                                                              tile_width == 160 || tile_width == 128));
    const bool ok = wok && ((tile_edge == 0 && ring_slots == 0) ||
                    (tile_edge == 256 && (ring_slots == 0 || ring_slots == 5)) ||
                    (tile_edge == 128 && (ring_slots == 0 || ring_slots == 5 || ring_slots == 10)) ||
                    (tile_edge == 64 && (ring_slots == 0 || ring_slots == 5 || ring_slots == 10 || ring_slots == 20)));
    if (!ok) return MOM_ERR_SHAPE;
    g_force_width.store(tile_width, std::memory_order_relaxed);
    g_force_edge.store(tile_edge, std::memory_order_relaxed);
    return MOM_OK;
}

int mom_debug_force_short_form(int token_rows, int weight_rows) {
    const bool off = token_rows == 0 && weight_rows == 0;
    if (!off && momk::find_short_form(false, token_rows, weight_rows) < 0 &&
        momk::find_short_form(true, token_rows, weight_rows) < 0)
        return MOM_ERR_SHAPE;
    g_force_short.store(off ? 0 : (token_rows << 16 | weight_rows), std::memory_order_relaxed);
    return MOM_OK;
}

int mom_debug_force_rect_form(int token_rows, int weight_rows) {
    const bool off = token_rows == 0 && weight_rows == 0;
    if (!off && !momk::is_rect_form(false, token_rows, weight_rows) && !momk::is_rect_form(true, token_rows, weight_rows))
        return MOM_ERR_SHAPE;
    g_force_rect.store(off ? 0 : (token_rows << 16 | weight_rows), std::memory_order_relaxed);
    return MOM_OK;
}

int mom_debug_force_block(int token_rows) {
    if (token_rows != 0 && token_rows != 16 && token_rows != 32) return MOM_ERR_SHAPE;
    g_force_block.store(token_rows, std::memory_order_relaxed);
    return MOM_OK;
}

int mom_debug_mfma_probe(const void* a_bf16, size_t a_bytes, const void* b_bf16, size_t b_bytes, int64_t iters,
                         int workgroups, int order, float* sink, void* stream) {
    if (!a_bf16 || !b_bf16 || !sink) return MOM_ERR_NULL;
    if (!aligned16(a_bf16) || !aligned16(b_bf16) || !aligned16(sink)) return MOM_ERR_ALIGN;
    if (a_bytes < 16 || b_bytes < 16 || a_bytes / 16 > 0x7fffffffu || b_bytes / 16 > 0x7fffffffu || iters < 0 ||
        workgroups <= 0 || workgroups > (1 << 20) || (order != 0 && order != 1))
        return MOM_ERR_SHAPE;
    const dim3 grid((unsigned)workgroups), block(momk::kProbeThreads);
    const momk::u32x4* a = static_cast<const momk::u32x4*>(a_bf16);
    const momk::u32x4* b = static_cast<const momk::u32x4*>(b_bf16);
    hipStream_t st = static_cast<hipStream_t>(stream);
    return launch(order == 0 ? momk::mfma_probe_kernel<0> : momk::mfma_probe_kernel<1>, grid, block, 0, st, a, (unsigned)(a_bytes / 16), b,
                  (unsigned)(b_bytes / 16), (long long)iters, sink) == hipSuccess ? MOM_OK : MOM_ERR_HIP;
}

size_t mom_mlp_workspace_bytes(int64_t S, int64_t H, int64_t I, int64_t mini_seq) {
    if (S <= 0 || H <= 0 || I <= 0 || mini_seq < 0) return 0;
    return (size_t)effective_chunk(S, mini_seq) * (size_t)I * 2;
}

int mom_mlp_prefill(const void* x, const void* W_gate, const void* W_up, const void* W_down, int64_t S,
                    int64_t H, int64_t I, int64_t mini_seq, void* out, void* workspace,
                    size_t workspace_bytes, void* stream) {
    return mlp_driver(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, workspace, workspace_bytes, stream,
                      nullptr, 0);
}

int mom_mlp_prefill_static(const void* x, const void* W_gate, const void* W_up, const void* W_down, int64_t S,
                           int64_t H, int64_t I, int64_t mini_seq, void* out, void* stream) {
    if (S < 0 || H <= 0 || I <= 0 || mini_seq < 0) return MOM_ERR_SHAPE;
    if (S == 0) return validate_mlp(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, nullptr, 0);
    const size_t need = mom_mlp_workspace_bytes(S, H, I, mini_seq);
    if (need > (size_t)MOM_STATIC_WORKSPACE_BYTES) return MOM_ERR_WORKSPACE;
    void* ws = static_workspace();
    if (!ws) return MOM_ERR_HIP;
    const int rc = validate_mlp(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, ws, (size_t)MOM_STATIC_WORKSPACE_BYTES);
    if (rc != MOM_OK) return rc;
    const int cus = compute_units();
    if (cus <= 0) return MOM_ERR_HIP;
    const int64_t C = momk::static_rows(S, H, I, effective_chunk(S, mini_seq), MOM_STATIC_WORKSPACE_BYTES, cus);
    // the call writes more of the array than `need`, but no argument can lie in any of it
    return mlp_loop(x, W_gate, W_up, W_down, S, H, I, C, out, ws, stream, nullptr, 0);
}

size_t mom_mlp_pipelined_workspace_bytes(int64_t S, int64_t H, int64_t I, int64_t mini_seq) {
    const size_t one = mom_mlp_workspace_bytes(S, H, I, mini_seq);
    if (one == 0) return 0;
    const int64_t C = effective_chunk(S, mini_seq);
    return (S + C - 1) / C > 1 ? 2 * one : one;
}

int mom_mlp_prefill_pipelined(const void* x, const void* W_gate, const void* W_up, const void* W_down, int64_t S,
                              int64_t H, int64_t I, int64_t mini_seq, void* out, void* workspace,
                              size_t workspace_bytes, void* stream, void* stream2, void** events,
                              int64_t n_events) {
    int rc = validate_mlp(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, workspace, workspace_bytes);
    if (rc != MOM_OK || S == 0) return rc;
    const size_t need = mom_mlp_pipelined_workspace_bytes(S, H, I, mini_seq);
    if (workspace_bytes < need) return MOM_ERR_WORKSPACE;
    const void* ins[4] = {x, W_gate, W_up, W_down};
    const size_t xb = (size_t)S * H * 2, wb = (size_t)H * I * 2;
    const size_t inb[4] = {xb, wb, wb, wb};
    for (int i = 0; i < 4; ++i)
        if (overlaps(workspace, need, ins[i], inb[i])) return MOM_ERR_ALIAS;
    if (overlaps(out, xb, workspace, need)) return MOM_ERR_ALIAS;
    const int64_t C = effective_chunk(S, mini_seq);
    if ((S + C - 1) / C == 1)      // a single mini-sequence
        return mlp_driver(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, workspace, workspace_bytes, stream,
                          nullptr, 0);
    if (!events) return MOM_ERR_NULL;
    if (n_events < 5) return MOM_ERR_SHAPE;
    for (int i = 0; i < 5; ++i)
        if (!events[i]) return MOM_ERR_NULL;
    (void)stream2;
    const int cus = compute_units();
    if (cus <= 0) return MOM_ERR_HIP;
    return mlp_loop(x, W_gate, W_up, W_down, S, H, I, momk::pipelined_rows(S, H, I, C, cus), out, workspace, stream, nullptr, 0);
}

int mom_mlp_prefill_events(const void* x, const void* W_gate, const void* W_up, const void* W_down,
                           int64_t S, int64_t H, int64_t I, int64_t mini_seq, void* out, void* workspace,
                           size_t workspace_bytes, void* stream, void** events, int64_t n_events) {
    if (!events) return MOM_ERR_NULL;
    return mlp_driver(x, W_gate, W_up, W_down, S, H, I, mini_seq, out, workspace, workspace_bytes, stream,
                      events, n_events);
}

int mom_lmhead_last(const void* x_last, const void* W_lm, int64_t V, float* logits, int64_t H, void* stream) {
    if (V < 0 || H <= 0 || (H % 32) != 0 || H > momk::kGemvMaxK || V > (int64_t)0x7fffff00) return MOM_ERR_SHAPE;
    if (V == 0) return MOM_OK;
    if (!x_last || !W_lm || !logits) return MOM_ERR_NULL;
    if (!aligned16(x_last) || !aligned16(W_lm) || !aligned16(logits)) return MOM_ERR_ALIGN;
    if (overlaps(logits, (size_t)V * 4, x_last, (size_t)H * 2) ||
        overlaps(logits, (size_t)V * 4, W_lm, (size_t)V * H * 2))
        return MOM_ERR_ALIAS;
    return launch_gemv<momk::MODE_LOGITS>(static_cast<const unsigned short*>(x_last),
                                          static_cast<const unsigned short*>(W_lm), nullptr, logits, V, H,
                                          static_cast<hipStream_t>(stream)) == hipSuccess ? MOM_OK : MOM_ERR_HIP;
}

int mom_mlp_last(const void* x_last, const void* W_gate, const void* W_up, const void* W_down, int64_t H,
                 int64_t I, void* out_last, void* workspace, size_t workspace_bytes, void* stream) {
    if (H <= 0 || I <= 0 || (H % 32) != 0 || (I % 32) != 0 || H > momk::kGemvMaxK || I > momk::kGemvMaxK)
        return MOM_ERR_SHAPE;
    if (!x_last || !W_gate || !W_up || !W_down || !out_last || !workspace) return MOM_ERR_NULL;
    if (!aligned16(x_last) || !aligned16(W_gate) || !aligned16(W_up) || !aligned16(W_down) ||
        !aligned16(out_last) || !aligned16(workspace))
        return MOM_ERR_ALIGN;
    const size_t need = (size_t)I * 2, hb = (size_t)H * 2, wb = (size_t)H * I * 2;
    if (workspace_bytes < need) return MOM_ERR_WORKSPACE;
    const void* ins[4] = {x_last, W_gate, W_up, W_down};
    const size_t inb[4] = {hb, wb, wb, wb};
    for (int i = 0; i < 4; ++i)
        if (overlaps(out_last, hb, ins[i], inb[i]) || overlaps(workspace, need, ins[i], inb[i])) return MOM_ERR_ALIAS;
    if (overlaps(out_last, hb, workspace, need)) return MOM_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // h = silu(x Wg^T) .* (x Wu^T)  ->  workspace [I] bf16 ;  out = h Wd^T -> [H] bf16
    if (launch_gemv<momk::MODE_GATEUP>(static_cast<const unsigned short*>(x_last),
                                       static_cast<const unsigned short*>(W_gate),
                                       static_cast<const unsigned short*>(W_up), workspace, I, H, st) != hipSuccess)
        return MOM_ERR_HIP;
    if (launch_gemv<momk::MODE_DOWN>(static_cast<const unsigned short*>(workspace),
                                     static_cast<const unsigned short*>(W_down), nullptr, out_last, H, I,
                                     st) != hipSuccess)
        return MOM_ERR_HIP;
    return MOM_OK;
}

int mom_kv_offload(const void* k, const void* v, void* pinned_host, void* stream, size_t bytes_each,
                   void* producer_stream, void* order_event, void* done_event) {
    if (bytes_each != 0 && (!k || !v || !pinned_host)) return MOM_ERR_NULL;
    if (producer_stream && !order_event) return MOM_ERR_NULL;
    if (bytes_each != 0) {
        const int rc = check_pinned_host(pinned_host, 2 * bytes_each);
        if (rc != MOM_OK) return rc;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (order_event) {
        // producer_stream may be NULL here: that is the default stream, which does not order itself
        // against a non-blocking side stream
        hipEvent_t ev = static_cast<hipEvent_t>(order_event);
        if (hipEventRecord(ev, static_cast<hipStream_t>(producer_stream)) != hipSuccess) return MOM_ERR_HIP;
        if (hipStreamWaitEvent(st, ev, 0) != hipSuccess) return MOM_ERR_HIP;
    }
    if (bytes_each != 0) {
        unsigned char* dst = static_cast<unsigned char*>(pinned_host);
        if (hipMemcpyAsync(dst, k, bytes_each, hipMemcpyDeviceToHost, st) != hipSuccess) return MOM_ERR_HIP;
        if (hipMemcpyAsync(dst + bytes_each, v, bytes_each, hipMemcpyDeviceToHost, st) != hipSuccess)
            return MOM_ERR_HIP;
    }
    if (done_event && hipEventRecord(static_cast<hipEvent_t>(done_event), st) != hipSuccess) return MOM_ERR_HIP;
    return MOM_OK;
}

int mom_kv_reload(const void* pinned_host, void* k, void* v, void* stream, size_t bytes_each, void* done_event) {
    if (bytes_each != 0 && (!k || !v || !pinned_host)) return MOM_ERR_NULL;
    if (bytes_each != 0) {
        const int rc = check_pinned_host(pinned_host, 2 * bytes_each);
        if (rc != MOM_OK) return rc;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const void* mapped = bytes_each != 0 ? reload_source(pinned_host, k, v, bytes_each, st) : nullptr;
    if (mapped) {
        const uint32_t n = (uint32_t)(bytes_each / 16);
        const uint32_t full = (2 * n + momk::kReloadThreads * momk::kReloadLoads - 1) / (momk::kReloadThreads * momk::kReloadLoads);
        if (launch(momk::kv_reload_kernel, dim3(full < (uint32_t)momk::kReloadBlocks ? full : momk::kReloadBlocks),
                   dim3(momk::kReloadThreads), 0, st, static_cast<momk::u32x4*>(k), static_cast<momk::u32x4*>(v),
                   static_cast<const momk::u32x4*>(mapped), n) != hipSuccess)
            return MOM_ERR_HIP;
    } else if (bytes_each != 0) {
        const unsigned char* src = static_cast<const unsigned char*>(pinned_host);
        if (hipMemcpyAsync(k, src, bytes_each, hipMemcpyHostToDevice, st) != hipSuccess) return MOM_ERR_HIP;
        if (hipMemcpyAsync(v, src + bytes_each, bytes_each, hipMemcpyHostToDevice, st) != hipSuccess)
            return MOM_ERR_HIP;
    }
    if (done_event && hipEventRecord(static_cast<hipEvent_t>(done_event), st) != hipSuccess) return MOM_ERR_HIP;
    return MOM_OK;
}

}  // extern "C"

// libtide_route: host side of the C ABI declared in include/tide_route.h -- argument
// checks, the per-device workspace, kernel selection and launches.  No torch types, no
// host synchronisation on the hot path.
#include "../../include/tide_route.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <vector>

#include "batch_kernel.hpp"
#include "compact_kernel.hpp"
#include "cosine_kernel.hpp"
#include "decode_kernel.hpp"
#include "few_rows_kernel.hpp"
#include "pack_kernel.hpp"
#include "prefill_dma_kernel.hpp"
#include "prefill_kernel.hpp"
#include "prefill_splitk_kernel.hpp"
#include "prefill_tile_kernel.hpp"
#include "prefill_wide_kernel.hpp"
#include "prefill_band_kernel.hpp"
#include "prefill_square_kernel.hpp"
#include "prefill_band32_kernel.hpp"
#include "mfma_probe_kernel.hpp"
#include "prefill_wide32_kernel.hpp"
#include "project_kernel.hpp"
#include "repack_kernel.hpp"

namespace {

using namespace tide;

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define TIDE_HIP(expr)                                                                         \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) return fail(TIDE_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kMaxDevices = 16;
constexpr size_t kCounterSlots = 64;       // per-checkpoint counters of the decode kernel
constexpr int kDecodeAutoMaxT = 32;
constexpr int kDecodeRawMaxT = 8;          // raw weights where the split-k prefill form applies
constexpr int kDecodeMaxT = 64;
static_assert(kFewMaxTiles <= (int)kCounterSlots, "the few-rows kernel: a counter per row tile");
static_assert((uint64_t)kMaxHidden / kDecodeSlice * kDecodeMaxT * (2 * kBottleneck + kPartPad) * sizeof(float) < (1ull << 32), "decode_finish: 32-bit offsets");
constexpr int kSplitkMaxSlices = 8;        // workgroups that share a tile's k range in the split-k prefill form
constexpr int kSplitkRingBytes = 128 * 1024;   // most LDS for its ring
constexpr int kSplitkMaxTiles = 128;       // most 128-row tiles' worth of rows (x column halves) the split-k form is considered for ...
constexpr int kSplitkForcedMaxTiles = 1024;   // ... and when it is forced (tide_set_prefill_form(5)): bounds the partial results at 512 MiB

struct Buffer {
    void* ptr = nullptr;
    size_t bytes = 0;
};

// ---- Scratch memory of a router call (device memory beyond the caller's inputs and outputs).
// Two kinds.  STATE words -- the decode kernel's per-checkpoint counters and one arrival word per
// token -- must be zero when a call starts, and every kernel that uses them leaves them zero (the
// last arriver resets them).  DATA -- the packed weights of a raw-weight call and the partial
// results of the split-k pair / the latency kernel -- is written before it is read within the call.
struct Scratch {
    uint32_t* counters = nullptr;   // kCounterSlots words (state)
    uint64_t* arrive = nullptr;     // [T] arrival words (state), null when no exit_layer is asked for
    void* packed = nullptr;         // C packed routers (data), raw-weight prefill calls only
    float* part = nullptr;          // partial results (data)
    void* rows = nullptr;           // re-aligned, zero-padded copy of the hidden rows (data), generic fallback only
};

// The library's own workspace: one per device, grow-only, shared by every call that does not bring
// a workspace of its own.  `last_stream` / `used` remember where its last call was enqueued, `dirty`
// that a launch failed after an earlier one of the same call had been enqueued (the state words
// may then be non-zero: the next call clears them first).
// `sized` remembers for which shapes, and up to which T, the partial results' buffer was sized (see largest_part).
struct SizedShape {
    int dtype = 0, raw = 0;
    int64_t C = 0, d = 0, b = 0, T = 0;
};
constexpr int kSizedShapes = 16;
struct Workspace {
    Buffer counters, arrive, packed, part, rows, batch, compact;
    SizedShape sized[kSizedShapes];
    unsigned next_sized = 0;
    hipStream_t last_stream = nullptr;
    bool used = false, dirty = false;
};

std::mutex g_mu;
Workspace g_ws[kMaxDevices];
int g_variant = TIDE_VARIANT_AUTO;
int g_prefill_form = 0;   // a form word (see valid_form_word): 0 auto; 1 / 2: streaming form with 64 / 128 rows per workgroup;
                          // 3: register-ring form; 4: wide-tile form wherever it applies, on as many workgroups as there are
                          // whole tiles; 5: split-k pair (optionally with a forced shape); 6: one-tile form; 7: band form;
                          // 8: split-k in one launch (optionally with a forced slice count); 9: square form (width 256)

// Caller-owned workspaces (the _ws entry points) and the static array of the no-allocation entry
// point are single blocks laid out per call: state words first, data behind them.  A call with more
// state words than an earlier one would find that call's data where it needs zeros, so the library
// keeps, per block, how many leading bytes are known to hold zero state (`clean`): the whole block
// after tide_workspace_init, what lies before a call's data after a call that wrote some.  `settled`: the leading bytes that hold
// zeros or a split-k form's partial results.  Those depend on the block's size and on estimates, so a program cannot know of them: a later call that
// keeps its state there clears it, whereas other data (packed weights, copied rows, the latency kernel's part) asks for another tide_workspace_init.
struct BlockRecord {
    void* ptr = nullptr;
    size_t bytes = 0, clean = 0, settled = 0;
    size_t state = 0;               // the most state that a call since tide_workspace_init has kept
    uint64_t stamp = 0;             // for replacing the least recently used record
};
constexpr int kMaxBlockRecords = 64;
BlockRecord g_blocks[kMaxBlockRecords];
uint64_t g_block_clock = 0;
uint64_t g_allocations = 0;       // hipMalloc calls made by the library so far (tide_workspace_allocations)

// The no-allocation entry point's scratch memory: every GPU the library runs on holds its own copy
// of this array until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the address kernels and fills use is the per-device pointer kept below.
constexpr size_t kStaticScratchBytes = (size_t)TIDE_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
struct StaticScratch {
    void* ptr = nullptr;            // device address of this device's copy
    size_t clean = 0;               // as BlockRecord::clean (the array starts zero-filled)
};
StaticScratch g_static[kMaxDevices];

// Grow-only device buffer.  Re-allocation frees the old block, which waits for the device.
int reserve(Buffer& b, size_t bytes, bool zero) {
    if (b.bytes >= bytes && b.ptr) return TIDE_OK;
    if (b.ptr) {
        hipError_t e = hipFree(b.ptr);
        b.ptr = nullptr;
        b.bytes = 0;
        if (e != hipSuccess) return fail(TIDE_ERR_HIP, "hipFree: %s", hipGetErrorString(e));
    }
    size_t want = (bytes + 255) & ~size_t(255);
    hipError_t e = hipMalloc(&b.ptr, want);
    if (e != hipSuccess) {
        b.ptr = nullptr;
        return fail(TIDE_ERR_WORKSPACE, "workspace hipMalloc(%zu): %s", want, hipGetErrorString(e));
    }
    b.bytes = want;
    ++g_allocations;
    if (zero) {
        e = hipMemset(b.ptr, 0, want);
        if (e != hipSuccess) return fail(TIDE_ERR_HIP, "hipMemset: %s", hipGetErrorString(e));
    }
    return TIDE_OK;
}

int current_device(int* dev) {
    TIDE_HIP(hipGetDevice(dev));
    if (*dev < 0 || *dev >= kMaxDevices) return fail(TIDE_ERR_UNSUPPORTED, "device index %d out of range", *dev);
    return TIDE_OK;
}

int current_workspace(Workspace** out) {
    int dev = 0;
    int rc = current_device(&dev);
    if (rc) return rc;
    *out = &g_ws[dev];
    return TIDE_OK;
}

// The library's workspace is shared by every stream of the device, and its state words carry a
// call's progress: two calls in flight on different streams would corrupt each other.  A call on
// another stream than the last one is accepted only when that stream has drained.  (Skipped while
// `st` is being captured into a graph -- queries are not allowed then; a captured call must follow
// an eager one on the same stream anyway, which is what sizes the workspace.)
int claim_workspace(Workspace& ws, hipStream_t st) {
    if (ws.used && ws.last_stream != st) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
        if (cap == hipStreamCaptureStatusNone) {
            const hipError_t q = hipStreamQuery(ws.last_stream);
            if (q == hipErrorNotReady)
                return fail(TIDE_ERR_WORKSPACE, "the library workspace is still in use by a call on another stream: order the "
                            "calls on one stream, or give each stream a workspace of its own (the _ws entry points)");
            if (q != hipSuccess) (void)hipGetLastError();   // e.g. the stream no longer exists: nothing of ours is pending on it
        }
    }
    ws.last_stream = st;
    ws.used = true;
    return TIDE_OK;
}

size_t elem_bytes(int dtype) { return dtype == TIDE_F32 ? 4 : 2; }

float threshold_logit(float theta) {
    if (!(theta < 1.0f)) return std::numeric_limits<float>::infinity();   // also NaN: never fire
    if (theta <= 0.0f) return -std::numeric_limits<float>::infinity();
    const double t = (double)theta;
    return (float)std::log(t / (1.0 - t));
}

// Everything both entry points must check before anything is enqueued.
bool supported_bottleneck(int64_t b) { return b == 64 || b == 128 || b == 256; }

// Hidden sizes.  Multiples of 128 run on the tuned kernels.  Other sizes whose rows are whole 16-byte
// chunks run, at widths 64 / 128, on the variants of those kernels that fetch zeros beyond the end of a row, under a forced
// variant or form on the register-ring prefill form with a zero-filled last k-tile, and on
// the latency kernel with a partial last slice.  Everything else -- rows that are not whole chunks, or
// width 256 at a hidden size that is not a multiple of 128 -- is first copied into aligned, zero-padded
// rows (repack_kernel.hpp) and then takes the tuned kernels.
bool supported_hidden(int dtype, int64_t d) {
    (void)dtype;
    return d >= 1 && d <= kMaxHidden;
}
bool chunked_rows(int dtype, int64_t d) { return (d * (int64_t)(dtype == TIDE_F32 ? 4 : 2)) % 16 == 0; }
bool needs_repack(int dtype, int64_t d, int64_t b) { return !chunked_rows(dtype, d) || (d % 128 != 0 && b == 256); }

// d rounded up to a multiple of 128 elements: whole k-tiles of the prefill kernels (256 bytes of a row)
// for every storage type, and the row length the tuned kernels accept.
int64_t padded_hidden(int dtype, int64_t d) {
    (void)dtype;
    return (d + 127) / 128 * 128;
}

// chunked_only: the entry point reads rows in 16-byte chunks and has no fallback for other hidden sizes.
int check_common(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride,
                 int64_t row_stride, const void* weights, const float* w2, float eps, bool chunked_only = false) {
    if (dtype != TIDE_F32 && dtype != TIDE_F16 && dtype != TIDE_BF16)
        return fail(TIDE_ERR_INVALID_ARG, "dtype %d is not a tide_dtype_t", dtype);
    if (C < 1) return fail(TIDE_ERR_INVALID_ARG, "C = %lld must be at least 1", (long long)C);
    if (C > TIDE_MAX_CHECKPOINTS) return fail(TIDE_ERR_UNSUPPORTED, "C = %lld exceeds %d", (long long)C, TIDE_MAX_CHECKPOINTS);
    if (T < 0) return fail(TIDE_ERR_INVALID_ARG, "T = %lld is negative", (long long)T);
    if (d <= 0) return fail(TIDE_ERR_INVALID_ARG, "d = %lld must be positive", (long long)d);
    if (!supported_hidden(dtype, d)) return fail(TIDE_ERR_UNSUPPORTED, "d = %lld: hidden sizes from 1 to 16384", (long long)d);
    if (chunked_only && !chunked_rows(dtype, d))
        return fail(TIDE_ERR_UNSUPPORTED, "d = %lld: rows must be a multiple of 16 bytes for this entry point", (long long)d);
    if (!supported_bottleneck(b))
        return fail(TIDE_ERR_UNSUPPORTED, "bottleneck width b = %lld: supported widths are 64, 128 and 256", (long long)b);
    if (C * T > (int64_t)1 << 30)
        return fail(TIDE_ERR_UNSUPPORTED, "T = %lld is too large for one call", (long long)T);
    if (row_stride < d) return fail(TIDE_ERR_INVALID_ARG, "row_stride %lld < d %lld", (long long)row_stride, (long long)d);
    if (C > 1 && T > 1 && ckpt_stride < 0) return fail(TIDE_ERR_INVALID_ARG, "negative ckpt_stride");
    if (!(eps >= 0.0f)) return fail(TIDE_ERR_INVALID_ARG, "eps must be >= 0");
    if (T == 0) return TIDE_OK;
    if (!hidden || !weights || !w2) return fail(TIDE_ERR_INVALID_ARG, "hidden, W1/packed and w2 must not be NULL");
    const size_t eb = elem_bytes(dtype);
    if (chunked_rows(dtype, d)) {
        if (((uintptr_t)hidden & 15) || ((size_t)row_stride * eb & 15) || (C > 1 && ((size_t)ckpt_stride * eb & 15)))
            return fail(TIDE_ERR_ALIGNMENT, "hidden base and strides must be multiples of 16 bytes");
    } else if ((uintptr_t)hidden & (eb - 1)) {      // rows that cannot be 16-byte aligned: elements must be
        return fail(TIDE_ERR_ALIGNMENT, "hidden must be aligned to its element size");
    }
    if (((uintptr_t)weights & 15) || ((uintptr_t)w2 & 15))
        return fail(TIDE_ERR_ALIGNMENT, "W1 / packed and w2 must be 16-byte aligned");
    return TIDE_OK;
}

// gamma and b1 are optional.  b1 is read with 16-byte loads like w2; gamma element by element (a
// checkpoint's row of gamma starts d floats after the previous one: no alignment beyond a float for general d).
int check_optional_arrays(const float* gamma, const float* b1) {
    if ((uintptr_t)b1 & 15) return fail(TIDE_ERR_ALIGNMENT, "b1 must be 16-byte aligned");
    if ((uintptr_t)gamma & 3) return fail(TIDE_ERR_ALIGNMENT, "gamma must be aligned to a float");
    return TIDE_OK;
}

int fill_table(CheckpointTable& tab, int64_t C, const float* b2, const float* threshold, const int32_t* layer_ids) {
    if (!b2 || !threshold || !layer_ids) return fail(TIDE_ERR_INVALID_ARG, "b2, threshold and layer_ids (host arrays) must not be NULL");
    std::memset(&tab, 0, sizeof(tab));
    for (int64_t c = 0; c < C; ++c) {
        if (c > 0 && layer_ids[c] <= layer_ids[c - 1])
            return fail(TIDE_ERR_INVALID_ARG, "layer_ids must be strictly ascending (layer_ids[%lld] = %d after %d)",
                        (long long)c, layer_ids[c], layer_ids[c - 1]);
        tab.b2[c] = b2[c];
        tab.thr_logit[c] = threshold_logit(threshold[c]);
        tab.layer_id[c] = layer_ids[c];
    }
    return TIDE_OK;
}

template <typename F> int by_dtype(int dtype, F&& f) {
    switch (dtype) {
    case TIDE_F32: return f(std::integral_constant<int, kF32>{});
    case TIDE_F16: return f(std::integral_constant<int, kF16>{});
    default: return f(std::integral_constant<int, kBF16>{});
    }
}

struct Outputs {
    float* prob;
    uint8_t* fire;
    float* logits;
    int32_t* exit_layer;
    uint32_t* fire_mask;
};

int halves_of(int64_t b) { return (int)((b + kBottleneck - 1) / kBottleneck); }

int launch_pack(int dtype, int64_t C, int64_t d, int64_t b, const float* gamma, const float* W1, void* packed, hipStream_t st) {
    const int64_t dpad = padded_hidden(dtype, d);
    const int chunks = (int)(dpad * kBottleneck * elem_bytes(dtype) / 16);   // of one 128-column half
    const int halves = halves_of(b);
    dim3 grid((unsigned)((dpad * 16 + kPackThreads - 1) / kPackThreads), (unsigned)(C * halves));
    by_dtype(dtype, [&](auto dt) {
        hipLaunchKernelGGL((tide_pack_kernel<decltype(dt)::value>), grid, dim3(kPackThreads), 0, st, gamma, W1, (u32x4*)packed, (int)d,
                           (int)dpad, chunks, (int)b, halves);
        return 0;
    });
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

// CUs of the current device, rounded down to a multiple of 8 (one slice of the tile list per XCD).  Called with and without g_mu held.
int resident_cus(unsigned* out) {
    static std::atomic<int> cus[kMaxDevices];                // 0: not asked for yet
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    const bool known = dev >= 0 && dev < kMaxDevices;        // (an entry point without a workspace runs on any device)
    int n = known ? cus[dev].load(std::memory_order_relaxed) : 0;
    if (!n) {
        TIDE_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        if (known) cus[dev].store(n, std::memory_order_relaxed);
    }
    *out = (unsigned)(n > 8 ? n & ~7 : 8);
    return TIDE_OK;
}

// The wide-tile kernel: one persistent workgroup per CU, `grid` of them, p.total_tiles a multiple of grid.
template <int DT, int kHalves> int launch_wide(unsigned grid, hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_wide_kernel<DT, kHalves>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds_bytes(kHalves)));
        raised[dev] = true;
    }
    hipLaunchKernelGGL((tide_prefill_wide_kernel<DT, kHalves>), dim3(grid), dim3(kWideThreads), wide_lds_bytes(kHalves), st, p);
    return TIDE_OK;
}

// The band kernel: `grid` workgroups (a multiple of 8), each a contiguous band of the checkpoint-major list of
// 32-row blocks; p.tiles_per_ckpt = blocks per checkpoint.
template <int DT, bool kRagged> int launch_band(unsigned grid, hipStream_t st, PrefillParams p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_band_kernel<DT, kRagged>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBandLdsBytes));
        raised[dev] = true;
    }
    p.k_slices = band_per_ckpt(p.C, p.tiles_per_ckpt, grid);
    hipLaunchKernelGGL((tide_prefill_band_kernel<DT, kRagged>), dim3(grid), dim3(kBandThreads), kBandLdsBytes, st, p);
    return TIDE_OK;
}

// The split-k pair: `tiles` tiles of kBlocks*32 rows times p.k_slices workgroups leave their partial
// results in `part`, then one small workgroup per 32-row block adds them and finishes the router.
// (SplitkTiling: what the argument word holds)
static_assert(std::max(kSplitkForcedMaxTiles * 4, kSplitkMaxTiles * 10) <= (int)SplitkTiling::kMostTiles, "tiles: at most the 32-row blocks a pair is considered for");
static_assert(kSplitkMaxSlices <= (int)SplitkTiling::kMostSlices && kSplitkMaxStages <= (int)SplitkTiling::kMostStages && kDmaStages <= (int)SplitkTiling::kMostStages, "slices and stages");
// Bytes of partial results the pair leaves for `tiles` tiles of kBlocks*32 rows in `halves` column halves and S slices.
size_t splitk_part_bytes(int blocks, int64_t tiles, int halves, int64_t S) {
    const size_t items = (size_t)tiles * halves * S;
    return items * ((size_t)blocks * 32 * kBottleneck + (size_t)kDmaConsumers * blocks * 32) * sizeof(float);
}
template <int DT, int kBlocks, bool kRagged> int launch_splitk(float* part, int64_t tiles, hipStream_t st, PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    constexpr int kMostStages = std::min(kSplitkMaxStages, kSplitkRingBytes / splitk_lds_bytes<kBlocks>(1));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_splitk_kernel<DT, kBlocks, false, kRagged>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, splitk_lds_bytes<kBlocks>(kMostStages)));
        raised[dev] = true;
    }
    const int halves = halves_of(p.b);
    const size_t items = (size_t)tiles * halves * p.k_slices;
    const size_t z_bytes = items * splitk_part_floats<kBlocks>() * sizeof(float);
    unsigned cus = 0;
    const int rc = resident_cus(&cus);
    if (rc) return rc;
    // As many k-tiles as a workgroup has, at least four.  (A workgroup is alone on its CU: twelve waves of 93-151 registers.)  Four where the workgroups take
    // several rounds: a longer ring is level there or slower (four / eight, us, fp32: C = 2, d = 8192, T = 4500 119 / 123, C = 10, T = 1000 124 / 128, width 256, C = 6, d = 4096,
    // T = 1500 113 / 115; 49 sizes, 0.3 % on average).
    const int ntile = p.dpad * Storage<DT>::kBytes / kTileBytes, nk = (ntile + p.k_slices - 1) / p.k_slices;
    p.ring_stages = items > cus ? 4 : std::min(kMostStages, std::max(nk, 4));
    const int lds = splitk_lds_bytes<kBlocks>(p.ring_stages);
    p.zpart = part;
    p.sspart = (float*)((char*)part + z_bytes);
    hipLaunchKernelGGL((tide_prefill_splitk_kernel<DT, kBlocks, false, kRagged>), dim3(8u * (unsigned)((items + 7) / 8)), dim3(splitk_threads(false)), lds, st,
                       p.hidden, p.packed, p.ckpt_stride_bytes, p.row_stride_bytes, SplitkTiling::pack(p), p.by_slices.m, p.by_tiles.m, p.T, p.d, p);
    // 8 rows per workgroup of the second launch while that is at most one and a half workgroups per CU, else 16 (8 / 16 rows, us): 11.5 / 12.7 at
    // C = 1, T = 1024, 16.9 / 17.4 at C = 8, T = 322 (384 workgroups of 8 rows), 19.8 / 18.8 at C = 1, T = 4096 (512)
    const uint64_t tiling = SplitkTiling::pack(p);
    auto finish = [&](auto halves_tag, auto quads_tag) {
        constexpr int kH = decltype(halves_tag)::value, kQ = decltype(quads_tag)::value;
        if (p.k_slices <= 4) hipLaunchKernelGGL((tide_splitk_finish_kernel<kBlocks, kH, kQ, 4>), dim3(8u * (unsigned)((tiles * kBlocks * (4 / kQ) + 7) / 8)), dim3(kH * kFinishThreads), 0, st, p.zpart, p.b1, p.w2, tiling, p.by_tiles.m, p.inv_d, p.T, p.b, p);
        else hipLaunchKernelGGL((tide_splitk_finish_kernel<kBlocks, kH, kQ, kSplitkMaxS>), dim3(8u * (unsigned)((tiles * kBlocks * (4 / kQ) + 7) / 8)), dim3(kH * kFinishThreads), 0, st, p.zpart, p.b1, p.w2, tiling, p.by_tiles.m, p.inv_d, p.T, p.b, p);
    };
    const bool fine = 2 * tiles * kBlocks * 4 <= 3 * (int64_t)cus;
    using std::integral_constant;
    if (halves == 2) {
        if (fine) finish(integral_constant<int, 2>{}, integral_constant<int, 1>{});
        else finish(integral_constant<int, 2>{}, integral_constant<int, 2>{});
    } else {
        if (fine) finish(integral_constant<int, 1>{}, integral_constant<int, 1>{});
        else finish(integral_constant<int, 1>{}, integral_constant<int, 2>{});
    }
    return TIDE_OK;
}

// The split-k form in one launch (32-row tiles, widths 64 / 128, at most kCounterSlots tiles): the workgroup that
// completes a tile's count finishes it.
template <int DT, bool kRagged> int launch_splitk_fused(float* part, uint32_t* counters, int64_t tiles, hipStream_t st, PrefillParams& p) {
    static_assert(kSplitkMaxSlices == kSplitkMaxS, "the kernel unrolls over the slices");
    const size_t items = (size_t)tiles * p.k_slices;
    p.zpart = part;
    p.sspart = (float*)((char*)part + items * splitk_part_floats<1>() * sizeof(float));
    p.counters = counters;
    p.ring_stages = kDmaStages;
    hipLaunchKernelGGL((tide_prefill_splitk_kernel<DT, 1, true, kRagged>), dim3(8u * (unsigned)((items + 7) / 8)), dim3(splitk_threads(true)), splitk_lds_bytes<1>(kDmaStages), st,
                       p.hidden, p.packed, p.ckpt_stride_bytes, p.row_stride_bytes, SplitkTiling::pack(p), p.by_slices.m, p.by_tiles.m, p.T, p.d, p);
    return TIDE_OK;
}

// The square kernel (width 256, 16-bit rows): a workgroup per 256-row tile.
template <int DT> int launch_square(hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_square_kernel<DT>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kSquareLdsBytes));
        raised[dev] = true;
    }
    const unsigned grid = 8u * (unsigned)((p.total_tiles + 7) / 8);
    hipLaunchKernelGGL((tide_prefill_square_kernel<DT>), dim3(grid), dim3(kSquareThreads), kSquareLdsBytes, st, p);
    return TIDE_OK;
}

// The wide-tile kernel for fp32 rows: as launch_wide.
int launch_wide_f32(unsigned grid, hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_wide_f32_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kWide32LdsBytes));
        raised[dev] = true;
    }
    hipLaunchKernelGGL(tide_prefill_wide_f32_kernel, dim3(grid), dim3(kWideThreads), kWide32LdsBytes, st, p);
    return TIDE_OK;
}

// The band kernel for fp32 rows: `grid` workgroups (a multiple of 8, at least C), tiles of up to kMaxBlocks blocks of 32 rows.
template <bool kRagged, int kMaxBlocks> int launch_band_f32(unsigned grid, hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_band_f32_kernel<kRagged, kMaxBlocks>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, band32_lds_bytes<kMaxBlocks>()));
        raised[dev] = true;
    }
    hipLaunchKernelGGL((tide_prefill_band_f32_kernel<kRagged, kMaxBlocks>), dim3(grid), dim3(kWideThreads), band32_lds_bytes<kMaxBlocks>(), st, p);
    return TIDE_OK;
}

// The one-tile kernel: a workgroup per tile of kRowsM rows from p.tile_begin on.
template <int DT, int kHalves, bool kRagged, int kRowsM, bool kBurst> int launch_tile_form(hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    constexpr int lds = tile_lds_bytes(kHalves, kRowsM, kBurst);
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_tile_kernel<DT, kHalves, kRagged, kRowsM, kBurst>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised[dev] = true;
    }
    const unsigned grid = 8u * (unsigned)((p.total_tiles - p.tile_begin + 7) / 8);
    hipLaunchKernelGGL((tide_prefill_tile_kernel<DT, kHalves, kRagged, kRowsM, kBurst>), dim3(grid), dim3(tile_threads(kHalves)), lds, st, p);
    return TIDE_OK;
}
// In bursts up to three quarters of the CUs, but not on rows of two k-tiles, whose second burst is the last (d = 256, C = 8, without / with: 7.7 / 8.0 us at T = 2080,
// 8.0 / 8.2 at 3000; level at d = 128 and 384, 10.5 / 10.3 at 512) (64 rows: always); figures at the kernel.
template <int DT, int kHalves, bool kRagged = false, int kRowsM = kTileRows> int launch_tile(hipStream_t st, const PrefillParams& p) {
    if constexpr (kHalves == 1) {
        unsigned cus = 0;
        const int rc = resident_cus(&cus);
        if (rc) return rc;
        if (kRowsM == 64 || (p.dpad > 256 && 4 * (int64_t)(p.total_tiles - p.tile_begin) <= 3 * (int64_t)cus)) return launch_tile_form<DT, 1, kRagged, kRowsM, true>(st, p);
    }
    if constexpr (kRowsM == kTileRows) return launch_tile_form<DT, kHalves, kRagged, kRowsM, false>(st, p);
}

// The streaming kernels use more LDS than the default per-kernel limit: raise it once.
// `grid` is the plan's (persistent workgroups, see plan_prefill).
template <int DT, int M, int CB, bool kRagged = false> int launch_dma(unsigned grid, hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    constexpr int lds = dma_lds_bytes<M>();
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_prefill_dma_kernel<DT, M, CB, kRagged>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised[dev] = true;
    }
    hipLaunchKernelGGL((tide_prefill_dma_kernel<DT, M, CB, kRagged>), dim3(grid), dim3(kDmaThreads), lds, st, p);
    return TIDE_OK;
}

// ---- What a prefill call launches.  Pure host arithmetic (no HIP calls), so that tests can check it
// for any shape without a GPU (tide_prefill_plan): every row of every checkpoint must fall into
// exactly one tile of exactly one launch.
enum PrefillKernel : int {
    kKernelSplitK = 1,     // prefill_splitk_kernel.hpp: the pair
    kKernelWide = 2,       // prefill_wide_kernel.hpp (16-bit rows; width 256: 128-row tiles)
    kKernelWideF32 = 3,    // prefill_wide32_kernel.hpp
    kKernelTile = 4,       // prefill_tile_kernel.hpp, 128 or (widths 64 / 128) 64 rows per workgroup
    kKernelStream128 = 5,  // prefill_dma_kernel.hpp, 128 rows per workgroup
    kKernelStream64 = 6,   // prefill_dma_kernel.hpp, 64 rows per workgroup (width 256: both column halves per wave)
    kKernelRing = 7,       // prefill_kernel.hpp
    kKernelBand = 8,       // prefill_band_kernel.hpp: rows_per_tile = 32 (the unit its bands are counted in)
    kKernelSplitKFused = 9,// prefill_splitk_kernel.hpp in one launch: 32-row tiles, the last workgroup of a tile finishes it
    kKernelSquare = 10,    // prefill_square_kernel.hpp (width 256, 16-bit rows: 256-row tiles)
    kKernelBandF32 = 11    // prefill_band32_kernel.hpp: rows_per_tile = 32, as the band kernel
};
struct PlannedLaunch {
    int kernel;            // PrefillKernel
    int rows_per_tile;
    int tiles_per_ckpt;    // ceil(T / rows_per_tile)
    int total_tiles;       // end of the checkpoint-major tile range this launch covers ...
    int tile_begin;        // ... and its beginning
    int k_slices;          // split-k form: workgroups per tile and column half; else 1
    unsigned grid;         // workgroups
};
struct PrefillPlan {
    int count = 0;
    PlannedLaunch launch[2];
};

// The split-k pair's cost (see plan_prefill), us: for 16-bit and fp32 rows, tiles of 32, 64 and 128 rows.  (Fitted before the last k-tiles of a slice ran in straight
// lines: tiles of 32 and 64 rows take 1-4 % less since.)
struct PairCost { double launch, chain, row, slice; };
constexpr PairCost kPairCost[2][3] = {{{4.7, 0.59, 0.0063, 0.0087}, {4.8, 0.77, 0.0111, 0.0070}, {5.9, 1.07, 0.0119, 0.0059}},
                                      {{5.3, 0.58, 0.0101, 0.0103}, {6.1, 0.84, 0.0098, 0.0081}, {7.0, 1.47, 0.0095, 0.0070}}};
// The one-launch form's (up to 16 rows per checkpoint, widths 64 / 128): within 4 % rms of C = 1 ... 32, n = 2 ... 64 k-tiles, two, four and eight slices.
// Up to 8 rows; 0.8 more beyond, as much as the streaming form's.
constexpr PairCost kOneLaunchCost[2] = {{5.8, 0.41, 0.057, 0.0099}, {5.9, 0.59, 0.033, 0.0121}};
int64_t splitk_max_blocks(int dtype, int halves) { return (int64_t)kSplitkMaxTiles * (halves == 1 ? 4 : dtype == TIDE_F32 ? 10 : 6); }
constexpr double kPairLaunches = 8.3;      // two launches from a host that issues them back to back (6.3-8.5, by host)

PrefillPlan plan_prefill(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, unsigned cus, int form_word, bool ragged = false, bool split_k = true,
                         size_t most_part = SIZE_MAX, bool behind_few = false) {
    PrefillPlan plan;
    const int form = form_word & 0xff, force_rows = (form_word >> 8) & 0xff, force_slices = (form_word >> 16) & 0xff;
    const int64_t eb = (int64_t)elem_bytes(dtype);
    const int halves = halves_of(b);
    const bool two_halves = halves == 2;
    const bool generic_d = d % 128 != 0;           // the fallback: register-ring form, whatever form is forced
    // Rows per workgroup (streaming form).  128 rows fetch each W1' fragment once per 128 rows and
    // is the choice whenever the tiles fill most of the chip.  With few tiles it wins again, because
    // every CU is launched and the tiles are cut into 32-row pieces (up to a quarter as many tiles of
    // 128 rows as CUs: 24.9 against 27.1 us at 64 tiles on 256 CUs, d = 4096, measured, 15.4 / 15.6 at d = 2048); from there on 64-row
    // tiles are faster as long as every CU holds at most one (27.6 against 33.7 us at 80 tiles of 128
    // rows, 33.7 against 42.9 us at 128; with a second workgroup on some CUs 55.5 us at 136, where the
    // one-tile kernel takes 41.3 us).  `form` overrides for tests and tuning.
    const int64_t tiles128 = C * ((T + 127) / 128), tiles64 = C * ((T + 63) / 64);
    int rows_per_wg = (4 * tiles128 > (int64_t)cus && tiles64 <= (int64_t)cus) ? 64 : 128;
    if (form == 1) rows_per_wg = 64;
    if (form == 2 || form == 6) rows_per_wg = 128;
    // fp32 rows are split into bf16 terms before the matrix cores: the register-ring form does
    // that once per workgroup on the way into LDS, the streaming form once per consumer wave,
    // so of these two the ring form is the faster one for fp32 (measured 4.1 vs 3.6 TB/s); whole rounds
    // of 256-row tiles go to the fp32 wide-tile kernel further down (4.7 TB/s).
    // Width 256 (two column halves per wave) exists in the streaming form with 64 rows per
    // workgroup only.  With 128 rows the accumulators (128 values per lane) and two halves' fragments left too
    // little of W1' in flight to cover the L2 round trip: measured slower.
    // Rows that are no whole k-tiles (ragged), 16 bits, more than one 128-row tile per CU: it also keeps the batches whose checkpoints end in
    // short tiles, so that the 64-row tiles are two per CU at most (bf16, C = 7, T = 4650, 511 tiles of 64 rows: 60 / 73 us at d = 3080 / 4072 against
    // 64 / 79 in bands, level at d = 1608); from a third one on bands are faster (C = 9, T = 3600, 513 tiles: 79 / 96 us against 62 / 77).
    const bool ragged_over = ragged && form == 0 && dtype != TIDE_F32 && !two_halves && tiles128 > (int64_t)cus;
    const bool ring_form = generic_d || (!two_halves && (form == 3 || (form == 0 && dtype == TIDE_F32))) || (ragged_over && tiles64 <= 2 * (int64_t)cus);
    if (ring_form) rows_per_wg = kRows;
    // Width 256 from more than half as many 128-row tiles as CUs on: the one-tile kernel with eight consumer waves, a
    // workgroup per tile however many rounds that makes -- the rows have the whole ring (three stages of 32 KiB in flight;
    // the wide-tile kernel, which also sends W1' through LDS, has 32 KiB) and every wave fetches the W1' of its own
    // columns straight from L2.  Measured against the wide-tile kernel (bf16, C = 8, d = 4096): 77-83 against 85.5 us at
    // T = 4096, 66 against 73.5 us at 3072, 59 against 66 us at 2304, 309 against 322 us at 16384; d = 8192: 149 against
    // 167 us; at 128 tiles the 64-row kernel's one workgroup per CU still wins (52.7 against 59.9 us).
    const bool tile256 = two_halves && dtype != TIDE_F32 && !generic_d && (form == 6 || (form == 0 && 2 * tiles128 > (int64_t)cus));
    if (two_halves) rows_per_wg = tile256 ? 128 : 64;
    int64_t tiles_per_ckpt = (T + rows_per_wg - 1) / rows_per_wg;
    int64_t total_tiles = C * tiles_per_ckpt, tile_begin = 0;

    // Split-k form: with few rows, 2, 4 or 8 workgroups share the k range of a tile of 32, 64 or 128
    // rows and a second launch adds their results.  Which tile height and slice count is best, and
    // whether the pair beats the streaming kernel at all, depends on how long a row is (a workgroup's
    // dependent chain of k-tiles, longer per k-tile the taller the tile), on how many workgroups that
    // makes (beyond one per CU they run in rounds) and on the volume of partial results (16 KiB per
    // workgroup and 32-row block), so the choice compares cost estimates, in microseconds, fitted to
    // measurements on a 256-CU device (d = 768 ... 8192, 100 ... 16384 rows, C = 1, 6 and 8; within 4-5 % rms), with
    // n = k-tiles of a row, B = 32-row blocks per tile, S = slices, R = 32-row blocks of the whole call
    // (x 2 at width 256), W = workgroups:
    //   streaming, few tiles:  5.1 + 0.45 n + 0.089 (n / 32) (tiles of 128 rows); fp32 rows, register-ring form:
    //                          5.5 + 0.84 n + 0.026 (n / 32) (tiles of 128 rows); width 256: 3.4 + 1.4 n, fp32 rows
    //                          2.5 + 1.87 n per round of 64-row tiles
    //   split-k pair:          launch + chain ceil(n / S) ceil(W / CUs) + (row n / 32 + slice S) R   (kPairCost, by type and B),
    //                          and no less than the host takes to issue two launches (where they are two)
    // The pair has to be 8 % cheaper, twice what the estimates are good for; the one launch just cheaper (kOneLaunchCost; bf16, streaming / one launch:
    // C = 28: 7.6 / 7.7 us at d = 512, 9.0 / 8.0 at 768, 9.3 / 7.7 at 1024, T = 8; two slices or four where eight would share a CU's
    // time).  Streaming form / pair (us):
    // bf16, C = 1: d = 5120, T = 5000 27.0 / 20.5, d = 2048, T = 3000 12.6 / 9.8, d = 4096, T = 5000 22.1 / 18.3; C = 8, d = 8192, T = 700 39.9 / 31.5;
    // fp32, C = 6: d = 5120, T = 700 79 / 47, d = 768, T = 700 16.7 / 14.1; fp32, width 256, C = 6: d = 1024, T = 600 31.4 / 18.0, d = 4096 120 / 72 at
    // T = 1000 and 125 / 106 at 1500 (the streaming form's 64-row tiles leave CUs idle there, and past one round it takes two: five times
    // as many blocks as otherwise are the pair's to compare).
    // Forced (form 5) the cheapest shape is taken whatever the streaming estimate says, and the form
    // word may fix the tile height (bits 8-15) and the slice count (bits 16-23).
    if (!generic_d && split_k && (form == 0 || form == 5 || form == 8)) {
        const int64_t ntile = d * eb / kTileBytes;
        const int64_t max_blocks = form == 5 ? (int64_t)kSplitkForcedMaxTiles * 4 : splitk_max_blocks(dtype, halves);
        // A call of up to 16 rows that the few-rows kernel takes never runs this plan, but a caller's block is asked for its partial results and counts
        // as written by them (see call_need): there the line between the two forms is one of the interface, and stays where it is (these estimates).
        const bool asked = behind_few && T <= 16 && halves == 1;
        double best = 1e30;
        int best_rows = 0;
        int64_t best_S = 0;
        for (int rows = 32; rows <= 128; rows *= 2) {
            if (form == 8 && rows != 32) continue;                                         // the single-launch form has 32-row tiles
            if (force_rows ? rows != force_rows : (rows > 32 && 2 * T <= rows)) continue;   // never a tile that is mostly padding
            const int64_t tiles = C * ((T + rows - 1) / rows);
            const double R = (double)(tiles * halves * (rows / 32)), lines = (double)ntile / 32.0;
            const bool one_launch = form != 5 && rows == 32 && halves == 1 && tiles <= (int64_t)kCounterSlots && (form == 8 || T <= 16);
            const PairCost& cost = one_launch ? kOneLaunchCost[dtype == TIDE_F32] : kPairCost[dtype == TIDE_F32][rows / 64];
            const double least = one_launch ? 0.0 : kPairLaunches;
            if (tiles * halves * (rows / 32) > max_blocks) continue;
            for (int64_t s = kSplitkMaxSlices; s >= 2; s /= 2) {
                const int64_t S = std::min<int64_t>(ntile, s);
                if (S < 2 || (force_slices && s != force_slices)) continue;
                if (splitk_part_bytes(rows / 32, (int)tiles, halves, (int)S) > most_part) continue;
                const int64_t W = tiles * halves * S;
                const double rounds = (double)((ntile + S - 1) / S) * (double)((W + cus - 1) / cus);
                const double t = asked ? 8.8 + (dtype == TIDE_F32 ? 0.65 : 0.50) * rounds + (0.011 * lines + 0.009 * (double)S) * R
                                       : std::max(least, cost.launch + cost.chain * rounds + (cost.row * lines + cost.slice * (double)S) * R);
                if (t < best) { best = t; best_rows = rows; best_S = S; }
            }
        }
        const double t_stream = halves == 2 ? (dtype == TIDE_F32 ? (2.5 + 1.87 * (double)ntile) * (double)((tiles64 + cus - 1) / cus) : 3.4 + 1.4 * (double)ntile)
                              : dtype == TIDE_F32 ? 5.5 + 0.84 * (double)ntile + 0.026 * ((double)ntile / 32.0) * (double)tiles128     // the register-ring form
                                                  : 5.1 + 0.45 * (double)ntile + 0.089 * ((double)ntile / 32.0) * (double)tiles128;
        const double t_asked = dtype == TIDE_F32 ? 8.5 + 0.75 * (double)ntile : 5.7 + 0.48 * (double)ntile + 0.07 * ((double)ntile / 32.0) * (double)tiles128;
        if (best_rows && (form == 5 || form == 8 || best < (asked ? t_asked : T <= 16 && halves == 1 ? t_stream : 0.92 * t_stream))) {
            const int64_t tpc = (T + best_rows - 1) / best_rows, tiles = C * tpc;
            // One launch instead of two where the kernel has it (32-row tiles, one column half, a counter per tile) and
            // where it is faster: the finishing workgroup reads the partial results past every cache, so it wins while
            // few rows are in use -- measured (fp16, C = 8, d = 4096; pair against one launch, us): 10.15 / 8.5 up to 8 rows
            // per checkpoint, 10.25 / 9.2 up to 16, 10.3 / 10.2 up to 24, 10.4 / 11.3 at 32; a full 32-row tile per checkpoint
            // and more (C = 1, T = 64 ... 2048) loses 0.9-1.9 us.  Forced (form 8): whenever the kernel has it.
            const bool fused = form != 5 && best_rows == 32 && halves == 1 && tiles <= (int64_t)kCounterSlots && (form == 8 || T <= 16);
            plan.launch[plan.count++] = PlannedLaunch{fused ? kKernelSplitKFused : kKernelSplitK, best_rows, (int)tpc, (int)tiles, 0, (int)best_S,
                                                      (unsigned)(tiles * halves * best_S)};
            return plan;
        }
    }
    // Square form (width 256, 16-bit rows): 256-row tiles on four waves, a workgroup per tile, as many rounds as that
    // makes.  Half the W1' traffic and half the LDS reads per row of the 128-row tiles below, but twice the work per
    // workgroup: it is the automatic choice when more than half the CUs get a tile, for the whole rounds and for a last round
    // that is more than half full.  Measured on 256 CUs
    // against the 128-row tiles (bf16, C = 8, d = 4096; us): 102 / 119 at T = 4352 (136 tiles), 107 / 123 at 4608, 126 / 145 at
    // 7168, 135-143 / 150 at 8192 (one round), 273 / 300 at 16384, 341 / 352 at C = 9 (2.25 rounds); d = 1024: 36 / 42 at 4608,
    // 43 / 52 at 8192; d = 8192: 195 / 230 at 4608, 268 / 297 at 8192; but 209 / 188 at T = 8448 (1.03 rounds), 210 / 193 at 9216,
    // 225 / 220 at 12288 (1.5), and 98 / 77 at 4096, where the 128-row tiles give every CU one.
    const bool square_fits = two_halves && dtype != TIDE_F32 && !generic_d && d / kSquareStageK >= kSquareMinStages;
    // Beyond one round, what the whole rounds leave over goes to the 128-row one-tile kernel behind the square launch
    // (the arrival words carry the per-token state across the two launches) if it is at most half a round: that is one
    // round of the small tiles, which costs 0.6 of a round of 256-row tiles; more than half a round takes another round
    // of the square form.  Just above a whole number of rounds (less than 0.175 of one left, below two rounds) the small
    // tiles take the whole call, as they do below half a round.  Measured (bf16, C = 8, d = 4096; this rule / all 128-row
    // tiles / all 256-row tiles, us): 190 / 190 / 198 at T = 8448, 193 / 203 / 205 at 10240, 197 / 212 / 211 at 11264,
    // 209 / 231 / 219 at 12288, 226 / 263 / 226 at 13312, 240 / 274 / 240 at 14336, 250 / 292 / 255 at 15360; C = 9,
    // T = 16384: 316 / 353 / 327; C = 10: 345 / 378 / 357.
    int64_t square_tiles = 0, square_tpc = 0;
    if (square_fits && (form == 0 || form == 9)) {
        const int64_t tpc = (T + kSquareRows - 1) / kSquareRows, tiles = C * tpc, rem = tiles % (int64_t)cus, whole = tiles - rem;
        square_tpc = tpc;
        if (form == 9 || (tiles <= (int64_t)cus && 2 * tiles > (int64_t)cus) || (whole > 0 && (rem == 0 || 2 * rem > (int64_t)cus)))
            square_tiles = tiles;
        else if (whole >= 2 * (int64_t)cus || (whole > 0 && 40 * rem > 7 * (int64_t)cus))
            square_tiles = whole;
        if (square_tiles > 0)
            plan.launch[plan.count++] = PlannedLaunch{kKernelSquare, kSquareRows, (int)tpc, (int)square_tiles, 0, 1, 8u * (unsigned)((square_tiles + 7) / 8)};
        if (square_tiles == tiles) return plan;
    }
    // Band form: one launch, every workgroup an equal share of the checkpoint-major list of 32-row blocks, cut
    // into tiles of up to 288 rows by the kernel itself (16-bit rows, widths 64 / 128).
    // It is the automatic choice as soon as the batch is more than one 128-row tile per CU (more than four blocks per CU)
    // -- measured on 256 CUs against the best of the other forms (bf16, C = 8; us): d = 4096: 63.5 against 74.3 at
    // T = 4608, 71.4 against 75.1 at 5632, 75.0 against 76.8 at 6144, level at 5120, 7168 and where the batch is whole rounds
    // of 256-row tiles; d = 1024: 23.5 against 26.9 at 4608, 24.6 against 27.4 at 5120; d = 8192: 114 against 131 at 4608, 123
    // against 138 at 5120, 136 against 144 at 6144; the 36-layer batched prefill (C = 9, T = 16384, d = 4096: 18 blocks per
    // CU) 212-219 against 224-226.  At four blocks per CU and below the one-tile kernel is faster (W1' straight from L2).
    // With few tiles the streaming kernel cuts them into pieces of 32 rows, but only where a row's k-tiles are a
    // multiple of four (a piece takes four per stage); else the pieces are 64 rows, and the band is faster at every size (bf16, pieces
    // against band, us): C = 8, T = 765: 16.3 / 11.0 at d = 896, 25.2 / 17.2 at 1920, 31.7 / 21.5 at 2688; C = 8, T = 1000, d = 4480: 47.4 / 32.5;
    // C = 1, T = 8000: 16.6 / 11.1 at d = 896, 31.6 / 21.8 at 2688; with 32-row pieces 18.1 / 20.9 (d = 2560).
    // Rows that are no whole k-tiles take the band from more than one 128-row tile per CU on, also where short last tiles leave that below four
    // blocks per CU: the wide-tile kernel has no form for them (bf16, d = 1608, against the register-ring form: C = 12, T = 2700: 47 -> 34 us,
    // C = 31, T = 1040: 46 -> 36; at one 128-row tile per CU the one-tile kernel stays ahead of the band: 28.7 / 32.2 at C = 10, T = 3100).
    const int64_t blocks32 = C * ((T + 31) / 32);
    const bool coarse_pieces = rows_per_wg == 128 && 4 * tiles128 <= (int64_t)cus && (d * eb / kTileBytes) % 4 != 0;
    if (!ring_form && dtype != TIDE_F32 && !two_halves && (form == 7 || (form == 0 && (blocks32 > 4 * (int64_t)cus || coarse_pieces || ragged_over)))) {
        const int64_t U = (T + 31) / 32;
        plan.launch[plan.count++] = PlannedLaunch{kKernelBand, 32, (int)U, (int)(C * U), 0, 1, cus};
        return plan;
    }
    // Band form for fp32 rows: every checkpoint gets cus / C workgroups, each an equal share of its blocks.  Up to four blocks
    // per workgroup its eight consumer waves share a block in pairs (each half of k): it is the choice from more than two
    // blocks per workgroup on, where the register-ring kernel's 64-row tiles are more than one per CU; up to six a wave per block.
    // Measured on 256 CUs (C = 8 where not given; against the forms below, us): d = 4096: 94 against 111 at T = 2300, 90 / 111 at
    // 2600, 97 / 113 at 3072, 122 / 132 at 4096, 162 / 171 at 4800, 177 / 187 at 5500, but 216 / 219 at 7000 (seven blocks); d = 2560, C = 10, T = 3001: 79 / 87;
    // d = 1024: 27 / 33 at 2300, 36 / 38 at 4096; d = 8192: 196 / 228 at 2600, 255 / 276 at 4096; C = 32, T = 900, d = 2048: 59 / 70; but 86 / 78
    // at two blocks (T = 2048) and nothing at d <= 256.  From seven blocks on the wide-tile kernel's
    // rounds are level.  The ring kernel is
    // slow on rows that are no whole k-tiles (C = 8, T = 1200, d = 3000: 129 us): those take this form whatever their number.
    if (dtype == TIDE_F32 && !generic_d && !two_halves && form == 0 && (d >= 512 || ragged) && (int64_t)cus >= C) {
        const int64_t U = (T + 31) / 32, per_ckpt = (int64_t)cus / C, most = (U + per_ckpt - 1) / per_ckpt;
        if (ragged || (U > 2 * per_ckpt && most <= 6)) {
            plan.launch[plan.count++] = PlannedLaunch{kKernelBandF32, 32, (int)U, (int)(C * U), 0, 1, cus};
            return plan;
        }
    }
    // Wide-tile forms: whole rounds of wide tiles (256 rows, or 128 rows at width 256; one per CU and
    // round) go to a wide kernel, what is left of the checkpoint-major row list to a kernel with
    // smaller tiles behind it on the same stream (the arrival words carry the per-token state across
    // the two launches): 16-bit rows to the streaming kernel with half as many rows per tile, fp32
    // rows to the register-ring kernel.
    // (The wide-tile kernels have no form for rows that are no whole k-tiles.)
    const bool wide16 = !ring_form && dtype != TIDE_F32 && !ragged && !tile256 && (form == 0 || form == 4);
    const bool wide32 = dtype == TIDE_F32 && !ragged && !generic_d && !two_halves && (form == 0 || form == 4);
    if (wide16 || wide32) {
        const int64_t wrows = two_halves ? kWideRows / 2 : kWideRows;
        const int64_t tpcw = (T + wrows - 1) / wrows, tilesw = C * tpcw;
        // Whole rounds always; the tiles of a last, partly filled round too if they are many enough (the
        // CUs without a tile idle meanwhile), else they go to a kernel with smaller tiles behind this one.
        // Measured on 256 CUs against the best other form, less than one round in all:
        //   16-bit rows, width 128: 78.6 against 86.6 us at 192 wide tiles, 84.4 against 98.8 us at 224; at 129-160
        //     d = 1024 / 2048 gain 5-10 % (23 against 25.5 us, 39 against 41.5 us), d = 4096 1-6 %, d = 16384 11-15 %
        //     (244-270 against 286-303 us), but d = 5120 and 8192 lose 5-8 % (95-100 against 87-93 us) -- from half
        //     the CUs + 1 on, for 4096 < d <= 8192 from 11/16 of them on;
        //   width 256 (128-row tiles): 60.9 against 92 us at 136, 66.6 against 94.4 us at 192, but 59.8 against
        //     51.6 us at 128, where the 64-row kernel still has one workgroup per CU -- from half the CUs + 1 on;
        //   fp32 rows: 157 against 169 us at 132 (264 tiles of 128 rows), 208 against 238 us at 224, nothing to
        //     gain at 128 and below -- from half the CUs + 1 on.
        // Forced (form 4): every tile of the list, whatever their number.
        const int64_t rem = tilesw % (int64_t)cus;
        const bool mid_rows = wide16 && !two_halves && d > 4096 && d <= 8192;
        const bool last_round_too = form == 4 || rem == 0 || (mid_rows ? 16 * rem >= 11 * (int64_t)cus : 2 * rem > (int64_t)cus);
        const int64_t wide_tiles = last_round_too ? tilesw : tilesw - rem;
        const unsigned wgrid = wide_tiles >= (int64_t)cus ? cus : 8u * (unsigned)((wide_tiles + 7) / 8);
        if (wide_tiles > 0) {
            plan.launch[plan.count++] = PlannedLaunch{wide16 ? kKernelWide : kKernelWideF32, (int)wrows, (int)tpcw, (int)wide_tiles, 0, 1, wgrid};
            if (wide_tiles == tilesw) return plan;
            const int64_t c0 = wide_tiles / tpcw, j0 = wide_tiles % tpcw;      // first row left: wrows * j0 of checkpoint c0
            if (wide16) {
                rows_per_wg = (int)(wrows / 2);
                if (rows_per_wg == 128 && form == 0) {         // what is left, by the rule at the top
                    const int64_t tpc128 = (T + 127) / 128, left128 = C * tpc128 - (c0 * tpc128 + 2 * j0);
                    const int64_t tpc64 = (T + 63) / 64, left64 = C * tpc64 - (c0 * tpc64 + 4 * j0);
                    if (4 * left128 > (int64_t)cus && left64 <= (int64_t)cus) rows_per_wg = 64;
                }
            }
            tiles_per_ckpt = (T + rows_per_wg - 1) / rows_per_wg;
            total_tiles = C * tiles_per_ckpt;
            tile_begin = c0 * tiles_per_ckpt + (wrows / rows_per_wg) * j0;
        }
    }
    if (square_tiles > 0) {                        // behind whole rounds of the square form: the 128-row tiles of the rest
        if (rows_per_wg == 128 && tile256) {
            const int64_t c0 = square_tiles / square_tpc, j0 = square_tiles % square_tpc;
            tile_begin = c0 * tiles_per_ckpt + 2 * j0;
        } else {
            plan.count = 0;                        // (never: such a batch is many 128-row tiles of a 16-bit type)
        }
    }
    const int64_t left = total_tiles - tile_begin;
    unsigned grid = 8u * (unsigned)((left + 7) / 8);
    int kernel = kKernelRing;
    if (!ring_form) {
        // One whole tile for every CU or none (128 rows: more than half as many tiles as CUs, at most as many; 64 rows, widths 64 / 128: always): there is
        // nothing to schedule, and the one-tile kernel is 1-3 % faster than the persistent one on such batches, on 64 rows 2-13 %, level on rows of three k-tiles (figures there).
        const bool one_tile_each = dtype != TIDE_F32 &&
                                   (rows_per_wg == 128 ? form == 6 || tile256 || (form == 0 && !two_halves && 2 * left > (int64_t)cus && left <= (int64_t)cus)
                                                       : form == 0 && !two_halves && left <= (int64_t)cus);
        kernel = one_tile_each ? kKernelTile : rows_per_wg == 128 ? kKernelStream128 : kKernelStream64;
        if (!one_tile_each) {
            // The streaming kernels are persistent: at most one (128-row; width 256: the two-halves
            // kernel needs more than the 168 registers that let three waves share a SIMD) or two (64-row)
            // workgroups per CU, each walking a list of tiles.  With fewer 128-row tiles than CUs every CU
            // is launched anyway: the schedule then cuts the tiles into 64- or 32-row pieces, one per
            // workgroup (a workgroup without a piece exits at once).
            const unsigned resident = cus * ((rows_per_wg == 128 || two_halves) ? 1u : 2u);
            if (grid > resident) grid = resident;      // both are multiples of 8
            if (rows_per_wg == 128) grid = resident;
        }
    }
    plan.launch[plan.count++] = PlannedLaunch{kernel, rows_per_wg, (int)tiles_per_ckpt, (int)total_tiles, (int)tile_begin, 1, grid};
    return plan;
}

// The launches of a call on rows of d elements (after a repack: of the padded length).
// Rows of whole 16-byte chunks whose length is no multiple of 128: under the automatic settings the plan of the padded
// length, on the kernels that read the chunks beyond a row's end as zeros: bf16, d = 1600, C = 12: 50 -> 33 us at T = 4000, 20 -> 16 at 1000;
// d = 4104, C = 8, T = 200: 38 -> 12.5; fp32, d = 4000, C = 9, T = 300: 161 -> 28; bf16, d = 1608, C = 8, T = 3000: 31 -> 26 (before: the register-ring
// form, whose loads are selected chunk by chunk).  (split_k: the split-k pair only where its partial results do not
// have to fit a block that was sized without them.)
PrefillPlan call_plan(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, unsigned cus, int variant, int form_word, bool split_k,
                      size_t most_part = SIZE_MAX, bool behind_few = false) {
    if (variant == TIDE_VARIANT_AUTO && form_word == 0 && d % 128 != 0)
        return plan_prefill(dtype, C, T, padded_hidden(dtype, d), b, cus, 0, true, split_k, most_part, behind_few);
    return plan_prefill(dtype, C, T, d, b, cus, form_word, false, true, most_part, behind_few);
}

// What the prefill kernels and the few-rows kernel take, all but the tiling.
PrefillParams prefill_params(const Scratch& sc, const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t d_mean, int64_t b,
                             int64_t ckpt_stride, int64_t row_stride, const void* packed, float eps, const float* b1, const float* w2,
                             const CheckpointTable& tab, int32_t min_layer, int32_t no_exit, const Outputs& o) {
    PrefillParams p;
    std::memset(&p, 0, sizeof(p));
    const size_t eb = elem_bytes(dtype);
    p.hidden = (const char*)hidden;
    p.ckpt_stride_bytes = ckpt_stride * (int64_t)eb;
    p.row_stride_bytes = row_stride * (int64_t)eb;
    p.shared_lines = (((uintptr_t)hidden | (uintptr_t)(T > 1 ? p.row_stride_bytes : 0) | (uintptr_t)(C > 1 ? p.ckpt_stride_bytes : 0)) & 127) != 0;
    p.packed = (const u32x4*)packed;
    p.b1 = b1;
    p.w2 = w2;
    p.C = (int)C;
    p.T = (int)T;
    p.d = (int)d;
    p.dpad = (int)padded_hidden(dtype, d);
    p.b = (int)b;
    p.eps = eps;
    p.inv_d = 1.0f / (float)d_mean;
    p.min_layer = min_layer;
    p.no_exit = no_exit;
    p.prob = o.prob;
    p.fire = o.fire;
    p.logits = o.logits;
    p.exit_layer = o.exit_layer;
    p.fire_mask = o.fire_mask;
    p.tab = tab;
    p.arrive = o.exit_layer ? sc.arrive : nullptr;
    return p;
}

int launch_prefill(const Scratch& sc, const PrefillPlan& plan, PrefillParams p, int dtype, hipStream_t st) {
    const int64_t b = p.b;
    const size_t eb = elem_bytes(dtype);
    int rc = TIDE_OK;
    const bool two_halves = halves_of(b) == 2;
    const int ntile = (int)(p.dpad * (int64_t)eb / kTileBytes);
    const bool ragged = p.dpad != p.d;
    for (int i = 0; i < plan.count; ++i) {
        const PlannedLaunch& L = plan.launch[i];
        p.tiles_per_ckpt = L.tiles_per_ckpt;
        p.total_tiles = L.total_tiles;
        p.tile_begin = L.tile_begin;
        p.k_slices = L.k_slices;
        p.by_slices = FastDiv::of((uint32_t)L.k_slices);
        p.by_tiles = FastDiv::of((uint32_t)L.tiles_per_ckpt);
        // a kernel that would read such rows wrongly is never launched on them, whatever the plan says
        auto no_form = [&]() { return fail(TIDE_ERR_UNSUPPORTED, "kernel %d has no form for dtype %d, d = %d", L.kernel, dtype, p.d); };
        auto launch = [&](auto dt, auto ragged_tag) {
            constexpr int DT = decltype(dt)::value;
            constexpr bool R = decltype(ragged_tag)::value;
            switch (L.kernel) {
            case kKernelSplitK:
                rc = L.rows_per_tile == 32 ? launch_splitk<DT, 1, R>(sc.part, L.total_tiles, st, p)
                   : L.rows_per_tile == 64 ? launch_splitk<DT, 2, R>(sc.part, L.total_tiles, st, p) : launch_splitk<DT, 4, R>(sc.part, L.total_tiles, st, p);
                break;
            case kKernelSplitKFused:
                rc = launch_splitk_fused<DT, R>(sc.part, sc.counters, L.total_tiles, st, p);
                break;
            case kKernelWide:
                if constexpr (DT != kF32 && !R) rc = two_halves ? launch_wide<DT, 2>(L.grid, st, p) : launch_wide<DT, 1>(L.grid, st, p);
                else rc = no_form();
                break;
            case kKernelWideF32:
                if constexpr (DT == kF32 && !R) rc = launch_wide_f32(L.grid, st, p);
                else rc = no_form();
                break;
            case kKernelTile:
                if constexpr (DT != kF32) {
                    // (64 rows, rows above 7 KiB: "nt" is as fast or faster here, us default / nt, C = 4, T = 3232 and C = 10, T = 1300, on the streaming kernel: 16.2 / 18.0 and
                    // 16.3 / 18.3 at d = 1752, 21.3 / 23.9 and 22.0 / 24.3 at 2600, but 33.3 / 32.9 and 34.6 / 33.2 at 3848, 38.5 / 37.3 and 40.0 / 37.6 at 4568)
                    if (L.rows_per_tile == 64 && p.d * (int)eb > 7168) p.shared_lines = 0;
                    if (two_halves) rc = R || L.rows_per_tile != kTileRows ? no_form() : launch_tile<DT, 2>(st, p);
                    else rc = L.rows_per_tile == 64 ? launch_tile<DT, 1, R, 64>(st, p) : launch_tile<DT, 1, R>(st, p);
                } else {
                    rc = no_form();
                }
                break;
            case kKernelBand:
                if constexpr (DT != kF32) rc = launch_band<DT, R>(L.grid, st, p);
                else rc = no_form();
                break;
            case kKernelBandF32:
                if constexpr (DT == kF32) {
                    rc = band32_max_blocks(p.C, L.tiles_per_ckpt, (int)L.grid) == 4 ? launch_band_f32<R, 4>(L.grid, st, p) : launch_band_f32<R, 8>(L.grid, st, p);
                } else {
                    rc = no_form();
                }
                break;
            case kKernelSquare:
                if constexpr (DT != kF32 && !R) rc = launch_square<DT>(st, p);
                else rc = no_form();
                break;
            // (fp32 rows that are no whole k-tiles always have another plan: band, split-k or register ring)
            case kKernelStream128:
                if constexpr (DT != kF32 || !R) rc = launch_dma<DT, 128, 1, R>(L.grid, st, p);
                else rc = no_form();
                break;
            case kKernelStream64:
                if constexpr (!R) rc = two_halves ? launch_dma<DT, 64, 2>(L.grid, st, p) : launch_dma<DT, 64, 1>(L.grid, st, p);
                else rc = no_form();
                break;
            default:
                if (ntile >= kMaxDepth)
                    hipLaunchKernelGGL((tide_prefill_kernel<DT, kMaxDepth, R>), dim3(L.grid), dim3(kPrefillThreads), 0, st, p);
                else
                    hipLaunchKernelGGL((tide_prefill_kernel<DT, 1, R>), dim3(L.grid), dim3(kPrefillThreads), 0, st, p);
                break;
            }
            return 0;
        };
        by_dtype(dtype, [&](auto dt) { return ragged ? launch(dt, std::true_type{}) : launch(dt, std::false_type{}); });
        if (rc) return rc;
        TIDE_HIP(hipGetLastError());
    }
    return TIDE_OK;
}

// The few-rows kernel: a workgroup per 16 rows and 16 columns of the bottleneck.  full: fp32 rows with all their bits.
template <int DT, int kWaves, bool kFull = false> int launch_few(unsigned grid, hipStream_t st, const PrefillParams& p) {
    static bool raised[kMaxDevices] = {};
    int dev = 0;
    TIDE_HIP(hipGetDevice(&dev));
    if (!raised[dev]) {
        TIDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&tide_few_rows_kernel<DT, kWaves, kFull>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, few_lds_bytes(kWaves, kFewRows)));
        raised[dev] = true;
    }
    static_assert(kFewMaxTiles * kFewRows < 1 << 16 && TIDE_MAX_CHECKPOINTS < 1 << 8, "the fields of dims");
    hipLaunchKernelGGL((tide_few_rows_kernel<DT, kWaves, kFull>), dim3(grid), dim3(kWaves * kWave), few_lds_bytes(kWaves, std::min(p.T, kFewRows)), st, p.hidden, p.packed,
                       p.ckpt_stride_bytes, p.row_stride_bytes, p.d, (uint32_t)p.T | (uint32_t)p.C << 16 | (uint32_t)__builtin_ctz((unsigned)p.k_slices) << 24, p.b1, p.w2, p);
    return TIDE_OK;
}
int launch_few_rows(const Scratch& sc, PrefillParams p, int dtype, bool full, hipStream_t st) {
    p.tiles_per_ckpt = (p.T + kFewRows - 1) / kFewRows;
    p.total_tiles = p.C * p.tiles_per_ckpt;
    p.k_slices = p.b / kFewCols;
    p.zpart = sc.part;
    p.counters = sc.counters;
    const unsigned grid = 8u * (unsigned)((p.total_tiles * p.k_slices + 7) / 8);
    // Sixteen waves where eight would take a second turn of the k loop (a dependent round trip), a CU has one workgroup at most (its LDS holds one) and there
    // is enough to read: a workgroup of sixteen starts and ends 0.2 us later.  us in a graph of calls, eight / sixteen, C = 4 where not said: rows of 8 KiB
    // (16-bit, d = 4096): C = 1, T = 1 5.3 / 5.55, T = 4 5.85 / 6.1, C = 8, T = 8 6.5 / 6.55, T = 16 7.2 / 6.9; 10 KiB: T = 4 6.2 / 6.4, T = 16 7.65 / 7.55; 12 KiB: T = 4 6.65 / 6.7,
    // C = 8, T = 8 7.5 / 7.35, T = 16 8.45 / 7.95; fp32, 10 KiB: T = 2 6.3 / 6.65, T = 8 level, C = 8, T = 16 8.3 / 8.2; 12 KiB: C = 1, T = 1 level, C = 8, T = 4 7.7 / 7.55, T = 8 8.3 / 7.75;
    // 16 KiB (fp32, d = 4096): C = 1, T = 1 7.95 / 7.45, T = 8 9.0 / 8.3; 16-bit: C = 1, T = 1 level, C = 8, T = 16 10.15 / 9.55; 32 KiB, C = 8: T = 1 11.4 / 10.7, fp32 13.4 / 11.9.
    // Never where one turn is enough: 6.1 / 6.3 at d = 2048, T = 16, 5.7 / 6.0 at d = 1024, T = 33.
    unsigned cus = 0;
    int rc = resident_cus(&cus);
    if (rc) return rc;
    const int one_turn = 8 * (dtype == TIDE_F32 ? few_groups<kF32>() : few_groups<kBF16>()) * 32;      // elements of a row
    const int row_bytes = p.dpad * (int)elem_bytes(dtype);
    const bool wide = p.dpad > one_turn && (int64_t)p.total_tiles * p.k_slices <= (int64_t)cus &&
                      (row_bytes >= (dtype == TIDE_F32 ? 12288 : 16384) || std::min(p.T, kFewRows) * row_bytes > 81920);
    auto go = [&](auto waves_tag) {
        constexpr int kWaves = decltype(waves_tag)::value;
        return dtype == TIDE_F32 && full ? launch_few<kF32, kWaves, true>(grid, st, p)
                                         : by_dtype(dtype, [&](auto dt) { return launch_few<decltype(dt)::value, kWaves>(grid, st, p); });
    };
    rc = wide ? go(std::integral_constant<int, 16>{}) : go(std::integral_constant<int, 8>{});
    if (rc) return rc;
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

// The latency kernel's cut of a row of d values: raw weights in as few slices as hold it, as equal as whole 128s allow; packed ones in slices of 128.
struct DecodeCut { int slice, S; };
DecodeCut decode_cut(int64_t d, bool packed) {
    const int blocks = (int)((d + kDecodeSlice - 1) / kDecodeSlice), most = kDecodeRawSlice / kDecodeSlice, least = (blocks + most - 1) / most;
    const int per_slice = packed ? 1 : (blocks + least - 1) / least;
    return DecodeCut{per_slice * kDecodeSlice, (blocks + per_slice - 1) / per_slice};
}

int launch_decode(const Scratch& sc, const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride,
                  int64_t row_stride, const float* gamma, const float* W1, const void* packed, float eps, const float* b1, const float* w2,
                  const CheckpointTable& tab, int32_t min_layer, int32_t no_exit, const Outputs& o, hipStream_t st) {
    DecodeParams p;
    std::memset(&p, 0, sizeof(p));
    const size_t eb = elem_bytes(dtype);
    p.hidden = (const char*)hidden;
    p.ckpt_stride_bytes = ckpt_stride * (int64_t)eb;
    p.row_stride_bytes = row_stride * (int64_t)eb;
    p.gamma = gamma;
    p.W1 = W1;
    p.packed = (const u32x4*)packed;
    p.dpad = (int)padded_hidden(dtype, d);
    p.b1 = b1;
    p.w2 = w2;
    p.C = (int)C;
    p.T = (int)T;
    p.d = (int)d;
    const DecodeCut cut = decode_cut(d, packed != nullptr);
    p.slice = cut.slice;
    p.S = cut.S;
    p.b = (int)b;
    p.halves = halves_of(b);
    p.eps = eps;
    p.min_layer = min_layer;
    p.no_exit = no_exit;
    p.prob = o.prob;
    p.fire = o.fire;
    p.logits = o.logits;
    p.exit_layer = o.exit_layer;
    p.fire_mask = o.fire_mask;
    p.tab = tab;
    p.counter = sc.counters;
    p.part = sc.part;
    p.arrive = o.exit_layer ? sc.arrive : nullptr;
    const int nblk = p.C * p.S * (packed ? p.halves : p.b / kDecodeRawCols);
    const unsigned grid = 8u * (unsigned)((nblk + 7) / 8);
    by_dtype(dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        if (p.packed && p.halves == 2)
            hipLaunchKernelGGL((tide_decode_packed_kernel<DT, 2>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
        else if (p.packed)
            hipLaunchKernelGGL((tide_decode_packed_kernel<DT, 1>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
        else {
            auto go = [&](auto halves_tag) {
                constexpr int kH = decltype(halves_tag)::value;
                if (p.T == 1) hipLaunchKernelGGL((tide_decode_kernel<DT, kH, 1>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
                else if (p.T == 2) hipLaunchKernelGGL((tide_decode_kernel<DT, kH, 2>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
                else if (p.T <= 4) hipLaunchKernelGGL((tide_decode_kernel<DT, kH, 4>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
                else hipLaunchKernelGGL((tide_decode_kernel<DT, kH, 8>), dim3(grid), dim3(kDecodeThreads), 0, st, p);
            };
            if (p.halves == 2) go(std::integral_constant<int, 2>{});
            else go(std::integral_constant<int, 1>{});
        }
        return 0;
    });
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

// The latency kernel (fp32 FMAs, raw or packed weights, k split over workgroups) or the prefill path?
// With packed weights the split-k prefill form is the faster one at almost every T (measured,
// d = 4096, C = 1 / 8, fp16: 9.5 / 10.6 us against 10.8 / 13.9 us at T = 1, 13.5 / 15.9 us at T = 8
// and 40 us at T = 32; fp32 rows: 13.3 / 14.7 us against 11.3 / 14.4 us at T = 1 and 13.6 / 16.4 us at
// T = 8).  With raw weights that form needs the packing pass first (7.5 us at C = 8), so the latency
// kernel, which reads W1 as it is, keeps T <= 8 (fp16, C = 8, d = 4096: 7.3 / 8.2 / 9.9 / 10.0 us at T = 1 / 4 / 5 / 8, against the packing pass and
// the few-rows kernel's 11.5 at T = 9, 11.8 at 12; the latency kernel also multiplies the fp32 weights, not their 16-bit
// rounding, so a call does not lose those bits below the line); it also keeps, up to
// T = 32, what the split-k form does not cover (hidden sizes that are not multiples of 128).  Calls that would pack or have
// packed weights go to the few-rows kernel instead where use_few_rows says so.
bool use_decode(int64_t T, int dtype, int64_t d, int64_t b, bool packed_given, int variant, int form_word) {
    if (variant == TIDE_VARIANT_DECODE) return T <= kDecodeMaxT;
    if (variant == TIDE_VARIANT_PREFILL) return false;
    const bool split_k = d % 128 == 0 && d >= 256 &&
                         ((form_word & 0xff) == 0 || (form_word & 0xff) == 5 || (form_word & 0xff) == 8);
    if (!split_k) return T <= kDecodeAutoMaxT;
    return !packed_given && T <= kDecodeRawMaxT;
}

// The few-rows kernel (a workgroup per 16 rows and 16 columns, all of k) or the paths above?  Its one launch beats the split-k pair's two
// (7.8-8.5 us from a host that issues them back to back, whatever the kernels take, and 2-3 us more where the exit projection follows) until a
// workgroup has to walk long rows or the workgroups are more than the CUs.  Figures: us, few rows / the other path, back to back from a host, [in a graph of calls, where
// the host does not hold the pair up], 256 CUs, packed weights, bf16 and C = 8 unless said, w = workgroups per CU.  Both sides have become faster since the lines were
// drawn; they stay where the two ways of calling do not agree, and on the pair's side where few rows would gain some 5-10 % more.
// kFewWide: a captured call whose pair would have to allocate takes the kernel wherever it is at all reasonable.
// pair: false where there is no split-k form behind it (see below).
enum FewRule { kFewNever, kFewByRule, kFewWide };
bool use_few_rows(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, unsigned cus, bool pair, FewRule rule) {
    if (rule == kFewNever) return false;
    const int64_t tiles = (T + kFewRows - 1) / kFewRows, nbk = b / kFewCols, row_bytes = d * (int64_t)elem_bytes(dtype);
    const int64_t W = C * tiles * nbk, n = (int64_t)cus;
    const bool f32 = dtype == TIDE_F32;
    // (rows of 64 KiB: fp32, d = 16384, T = 8 21.6 / 26.3 at C = 1, 24.0 / 26.8 at C = 8)
    if (tiles > kFewMaxTiles || C * nbk >= 256 || row_bytes > 32768) return false;
    // Every workgroup of a row tile ticks the tile's counter (14 ns each).  Beyond one workgroup per CU rows of up to 2 KiB meet that from 112 ticks
    // on (C = 16, T = 33, d = 1024: 7.7 / 7.9 [7.1 / 6.6]).
    const bool few_ticks = C * nbk <= 112 || row_bytes > 2048;

    // Hidden sizes that are no multiple of 128 have no split-k form on the calls that would be the latency kernel's (d = 1600, T = 16: 6.6 / 17.2) and none in a
    // block that was sized without it (the register-ring kernel: d = 1600, T = 100 9.3 / 18.9).  With the pair they follow the lines below
    // (d = 2904: 7.7 / 7.9 [7.3 / 6.8] at T = 48, 9.2 / 8.2 at 96; d = 4304 10.6 / 9.0).
    if (d % 128 != 0 && (!pair || C * nbk > 128)) return W <= (few_ticks ? 2 * n : n);

    // Many checkpoints, widths 64 / 128: from 128 ticks on the counter costs what the kernel gains over the 128-column split-k forms (width 256, where those take twice
    // the workgroups, does not meet that line: 1.03-1.6 times as fast up to 240 ticks).  C = 28: 10.3 / 9.7 at T = 16, d = 2560, 9.0 / 9.0 at T = 8.
    if (b <= 128 && C * nbk >= 200) return false;
    if (rule == kFewWide) return W <= (few_ticks ? 2 * n : n);
    // 17 to 24 checkpoints at width 128, up to 16 rows: 4 rows or rows of 4 KiB (f16, C = 24: 7.4 / 7.7 at d = 768, T = 1, 9.2 / 9.7 at d = 5120, T = 4, but C = 20, d = 2560 8.2 / 8.2 at
    // T = 8, 8.9 / 9.0 at 16); more: fp32, as far as the lines below take it (C = 20, T = 17, d = 768 8.5 / 8.3, C = 24, T = 32, d = 1024 9.3 / 8.5; f16, C = 24, T = 32 8.8 / 8.1 at d = 1024, 10.0 / 8.5
    // at 2560, 13.6 / 10.2 at 5120).
    if (b <= 128 && C * nbk > 128 && !(T <= kFewRows ? T <= 4 || row_bytes <= 4096 : f32)) return false;

    if (T > kFewRows) {             // against the pair
        // above 12 KiB: d = 8192 9.0 / 9.0 [9.0 / 8.6] at w = 0.06, 9.2 / 10.2 [9.4 / 9.3] at 0.125, 9.5 / 10.2 [9.7 / 9.4] at 0.19; fp32, d = 4096 9.6 / 10.2 [9.8 / 9.6], 9.9 / 11.0 [10.1 / 10.3],
        // 10.1 / 11.0 [10.3 / 10.4]
        if (row_bytes > 12288) return false;
        // d = 5376 8.2 / 8.7 [7.8 / 8.0] at 0.125, 8.2 / 9.0 [8.1 / 8.1] at 0.19, 8.2 / 9.0 [7.9 / 8.1] at 0.25; d = 6144 8.3 / 9.0 [8.1 / 8.1], 8.5 / 9.1 [8.4 / 8.2], 8.3 / 9.2 [8.2 / 8.2], width 64
        // 8.4 / 9.0 [8.3 / 7.9] at 0.25; fp32: d = 2688 8.5 / 9.8 [8.4 / 9.0] at 0.125, 8.6 / 9.9 [8.5 / 9.1] at 0.25, 8.8 / 10.1 [8.8 / 9.2] at 0.375; d = 3072 8.6 / 9.9 [8.5 / 9.2] at 0.125
        if (row_bytes > 10240) return f32 || b == 64 ? 4 * W <= n : 5 * W <= n;
        // d = 5120 7.7 / 8.0 [7.2 / 7.0] at 0.06, 8.1 / 8.6 [7.8 / 7.7] at 0.19, 8.0 / 8.8 [7.8 / 7.7] at 0.25; fp32, d = 2560 8.4 / 9.3 [8.1 / 8.6] at 0.125, 8.5 / 9.6 [8.5 / 8.6] at 0.19, 8.5 / 9.5 [8.2 / 8.6] at
        // 0.25, 8.5 / 9.7 [8.6 / 8.7] at 0.375
        if (row_bytes > 8192) return 5 * W <= n;
        // d = 4096 8.3 / 8.5 [7.8 / 7.6] at 0.66, 8.2 / 8.2 [8.1 / 7.3] at 0.75, 8.2 / 8.5 [8.4 / 7.7] at 0.875, 8.6 / 8.3 [8.4 / 7.3] at 1, 10.0 / 8.7 at 1.5; fp32, d = 2048 8.4 / 9.2 [8.3 / 8.4],
        // 8.4 / 9.1 [8.4 / 8.2], 8.5 / 9.2 [8.5 / 8.5], 8.7 / 9.2 [8.8 / 8.1], 10.9 / 9.5; width 64 with the projection 13.0 / 13.7 at 0.875; width 256, C = 2: 7.8 / 8.6 [7.6 / 7.7] at 0.5,
        // 8.4 / 8.5 [8.4 / 7.4] at 1
        if (row_bytes > 6144) return 8 * W <= 7 * n;
        // d = 2560 7.6 / 7.8 [7.2 / 6.6] at 0.75, 7.9 / 8.0 [7.7 / 6.8] at 1, 8.9 / 8.2 [9.0 / 7.2] at 1.5; d = 3072 with the projection 12.5 / 12.8 at 0.94
        if (row_bytes > 4096) return W <= n;
        // d = 1024 6.4 / 9.3 [6.0 / 8.5] at 0.75, 6.8 / 9.3 [6.3 / 8.5] at 1, 7.5 / 9.3 [7.2 / 8.5] at 1.5; d = 2048 7.4 / 7.9 [6.8 / 6.3] at 1, 8.1 / 7.8 [7.9 / 6.7] at 1.5; fp32, d = 1024 7.3 / 8.2
        // [6.8 / 7.0] at 0.75, 7.6 / 8.1 [7.2 / 6.8] at 1, 8.4 / 8.4 [8.3 / 7.2] at 1.5; with the projection, C = 5, d = 2048 11.6 / 12.4 at 1.1; d = 1448 8.1 / 7.9 [7.7 / 6.7] at 1.5, 8.4 / 7.9 at 2
        return W <= n || (few_ticks && 2 * W <= 3 * n);
    }
    // Up to 16 rows per checkpoint against the one-launch split-k form or, at width 256, a pair that is mostly padding:
    // d = 4096 6.3 / 8.5 at T = 1, 7.5 / 9.1 at 16; up to 8 rows of any length fp32, d = 8192 14.2 / 16.9, d = 16384, C = 1 / 8 10.7 / 12.4, 13.5 / 14.2; width 256, fp32, d = 8192 16.5 / 16.2 at T = 8
    // (18.7 / 16.4 at 16: the pair has overtaken there since the line was drawn)
    if (row_bytes <= 20480 || T <= 8 || b == 256) return W <= n;
    // 9 to 16 rows, T = 12 / 16: d = 12288 10.9 / 12.9, 11.9 / 13.0; d = 16384 14.8 / 15.3, 16.2 / 15.6; fp32: d = 6144 12.2 / 15.1, 13.1 / 15.1; d = 8192 15.5 / 17.5, 16.9 / 17.5 (C = 4 14.0 / 17.2, 15.3 / 17.2)
    return W <= n && (f32 ? T <= 12 || row_bytes <= 24576 : T <= 12 && row_bytes <= 24576);
}

// ---- What a router call needs of scratch memory, and which path it takes: host arithmetic only.
struct CallNeed {
    bool decode = false;            // the latency kernel takes the call, else the prefill path with `plan`
    bool few = false;               // the few-rows kernel takes the call, ...
    bool few_full = false;          // ... fp32 rows with all their bits
    PrefillPlan plan;
    size_t state_bytes = 0;         // counters + arrival words, a multiple of 256
    size_t packed_bytes = 0;        // a multiple of 256
    size_t part_bytes = 0;          // a multiple of 256
    size_t few_bytes = 0;           // ... of which the few-rows kernel uses so much, if it takes the call; a multiple of 256
    size_t rows_bytes = 0;          // generic fallback: the re-aligned copy of the hidden rows; a multiple of 256
    int64_t d_run = 0;              // the row length the kernels run on: d, or d padded to a multiple of 128 with rows_bytes
    size_t total() const { return state_bytes + packed_bytes + part_bytes + rows_bytes; }
    bool part_last = false;         // a split-k form's partial results: they lie at the end of a block, behind the state of as many calls as it has room for
    bool part_stays = false;        // whether part counts as written behind the state words afterwards (the few-rows kernel leaves zeros where it wrote)
    size_t part_offset(size_t room) const { return part_last ? (room - part_bytes) & ~size_t(255) : state_bytes + packed_bytes; }
    size_t rows_offset() const { return total() - rows_bytes - (part_last ? part_bytes : 0); }
    size_t data_begin(size_t room) const {      // the first byte of a block of `room` bytes that may not be zero afterwards
        if (packed_bytes || rows_bytes) return state_bytes;
        return part_stays ? part_offset(room) : SIZE_MAX;
    }
};
size_t round256(size_t n) { return (n + 255) & ~size_t(255); }

CallNeed call_need(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, bool raw_weights, bool want_exit, unsigned cus, int variant,
                   int form_word, bool library, FewRule few_rule = kFewByRule, size_t most_part = SIZE_MAX) {
    CallNeed n;
    n.state_bytes = round256(kCounterSlots * sizeof(uint32_t)) + (want_exit ? round256((size_t)T * sizeof(uint64_t)) : 0);
    const bool repack = needs_repack(dtype, d, b);
    n.d_run = repack ? padded_hidden(dtype, d) : d;
    if (repack) n.rows_bytes = round256((size_t)C * (size_t)T * (size_t)n.d_run * elem_bytes(dtype));
    // (the latency kernel reads raw W1 rows by the true d and hidden rows in 16-byte chunks: never after a repack)
    n.decode = !repack && use_decode(T, dtype, d, b, !raw_weights, variant, form_word);
    const int halves = halves_of(b);
    if (n.decode) {
        const size_t S = (size_t)decode_cut(d, !raw_weights).S;
        n.part_bytes = round256((size_t)C * S * (size_t)T * (size_t)(halves * kBottleneck + kPartPad) * sizeof(float));
    }
    // (the other paths' needs are counted all the same for a caller's block: what a caller has to bring does not depend on this choice)
    n.few = !(raw_weights && n.decode) && variant == TIDE_VARIANT_AUTO && form_word == 0 &&
            use_few_rows(dtype, C, T, n.d_run, b, cus, library && !n.decode, few_rule);
    // fp32 rows that are the latency kernel's otherwise: it multiplies the whole fp32 value of a row by both terms of the weight, the other kernels
    // for packed weights the row's two leading bf16 terms (error against 64 bits at T = 32, d = 1000: 2.6e-6 / 4.7e-6).  16-bit rows are exact in any.
    n.few_full = n.few && n.decode;
    n.few_bytes = n.few ? round256((size_t)T * (size_t)C * (size_t)(b / kFewCols) * sizeof(float)) : 0;
    if (n.decode) {
        n.part_stays = true;
        n.part_bytes = n.few && library ? n.few_bytes : std::max(n.part_bytes, n.few_bytes);
        if (n.few) n.decode = false;
        return n;
    }
    if (raw_weights) n.packed_bytes = round256((size_t)C * tide_packed_router_bytes(dtype, d, b));
    n.plan = call_plan(dtype, C, T, n.d_run, b, cus, variant, form_word, library, most_part, n.few);
    if (const PlannedLaunch& L = n.plan.launch[0]; L.kernel == kKernelSplitK || L.kernel == kKernelSplitKFused) {      // (always the only launch)
        n.part_bytes = round256(splitk_part_bytes(L.rows_per_tile / 32, L.total_tiles, halves, L.k_slices));
        n.part_last = !n.few;
        // a few-rows call of up to 16 rows counts as what it always has counted as, the one-launch form behind it
        n.part_stays = !n.few || L.kernel == kKernelSplitKFused;
    }
    n.part_bytes = n.few && library ? n.few_bytes : std::max(n.part_bytes, n.few_bytes);
    return n;
}

// The route of a call on a block of `room` bytes (a caller's workspace, the fixed array): the one without a limit where that fits; else the few-rows
// kernel where that does, whatever the paths behind it would need; else those paths with a split-k pair whose partial results fit, or none.  Only
// what a call cannot do without is left to be refused: state, weights packed or rows copied by the call, the latency kernel's part, a forced form's.
CallNeed block_need(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, bool raw_weights, bool want_exit, unsigned cus, int variant, int form_word,
                    size_t room) {
    auto need = [&](FewRule rule, size_t most_part) {
        return call_need(dtype, C, T, d, b, raw_weights, want_exit, cus, variant, form_word, false, rule, most_part);
    };
    CallNeed n = need(kFewByRule, SIZE_MAX);
    const size_t fixed = n.total() - n.part_bytes;
    if (n.total() <= room) return n;
    const size_t most_part = form_word == 0 && fixed <= room ? room - fixed : SIZE_MAX;
    if (n.few && fixed + n.few_bytes <= room) {
        n = need(kFewByRule, most_part);
        n.part_bytes = n.few_bytes;
        return n;
    }
    return need(kFewNever, most_part);
}

// The most partial results that any call of these C, d and b with more than `from` and at most `to` rows per checkpoint keeps under the automatic
// settings (both multiples of 32).  An eager call on the library's workspace reserves that much for every row count up to its own, so that no
// smaller call outgrows the buffer: a captured graph holds its address.  The split-k forms' choice changes with the number of
// 32-row blocks only; the few-rows kernel has at most two workgroups of 16 rows x 4 bytes per CU; the latency kernel's part grows with
// T up to 8 or 32.
size_t largest_part(int dtype, int64_t C, int64_t from, int64_t to, int64_t d, int64_t b, bool raw_weights, unsigned cus) {
    size_t most = std::min<size_t>(round256((size_t)(to * C * (b / kFewCols)) * sizeof(float)), (size_t)cus * 2 * kFewRows * sizeof(float));
    auto at = [&](int64_t t) { most = std::max(most, call_need(dtype, C, t, d, b, raw_weights, false, cus, TIDE_VARIANT_AUTO, 0, true).part_bytes); };
    if (from == 0) {
        at(kDecodeRawMaxT);
        at(kFewRows);                 // up to 16 rows the split-k form is one launch, with a line of its own to the streaming forms
    }
    for (int64_t t = from + 32; t <= to && C * halves_of(b) * (t / 32) <= splitk_max_blocks(dtype, halves_of(b)); t += 32) at(t);
    return most;
}

// The split-k pair: the slices of a tile dealt out over the XCDs instead of kept on one?  Kept together, every XCD reads the whole W1' of
// its tiles; dealt out, an eighth of it, but the second launch finds the partial results in other XCDs' L2s.  The first is the dearer one where
// the W1' of a checkpoint fills an XCD's 4 MiB L2 and the tiles are few, more so where this call packed the weights, which then come from
// memory.  Measured (us, dealt out / together; R = 32-row blocks x column halves of the call): raw weights, C = 1, 4 MiB and more: fp32, d = 8192 21.1 / 24.6
// at T = 200, 23.9 / 26.2 at 1000 (R = 32), bf16, d = 16384 19.9 / 23.3 at T = 100; packed, width 256, C = 1: bf16, d = 16384 16.2 / 18.4 at T = 200 (R = 14), d = 8192 13.4 / 14.1
// at T = 455 (30), but 18.0 / 16.4 at 1000 (64); from 8 MiB on with more checkpoints too: bf16, d = 16384, width 256, C = 4 22.1 / 23.5 at T = 200 (56), but 40.3 / 35.4
// at 455 (120).  With 2 MiB and less the first is the faster one throughout (C = 8, T = 322, d = 4096: 17.0 / 15.3).
bool deals_out(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, bool raw_weights) {
    const int64_t w1 = (int64_t)tide_packed_router_bytes(dtype, d, b), R = C * ((T + 31) / 32) * halves_of(b);
    if (w1 >= 8 << 20 && R <= 56) return true;
    return w1 >= 4 << 20 && C == 1 && R <= (raw_weights ? 32 : 30);
}

// Zero-fill for state words (a kernel, not a memset: calls may be captured into HIP graphs).
__global__ void tide_clear_kernel(u32x4* p, size_t chunks) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < chunks; i += (size_t)gridDim.x * blockDim.x)
        p[i] = u32x4{0u, 0u, 0u, 0u};
}
int launch_clear(void* ptr, size_t bytes, hipStream_t st) {      // ptr 16-byte aligned, bytes a multiple of 16
    if (bytes == 0) return TIDE_OK;
    const size_t chunks = bytes / 16;
    const unsigned grid = (unsigned)std::min<size_t>((chunks + 255) / 256, 2048);
    hipLaunchKernelGGL(tide_clear_kernel, dim3(grid), dim3(256), 0, st, (u32x4*)ptr, chunks);
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

// One block of `room` bytes (a caller's workspace or the static array) laid out for a call: state first, data behind, a split-k form's at the end.
Scratch carve(void* block, size_t room, const CallNeed& n, bool want_exit) {
    Scratch sc;
    char* base = (char*)block;
    sc.counters = (uint32_t*)base;
    sc.arrive = want_exit ? (uint64_t*)(base + round256(kCounterSlots * sizeof(uint32_t))) : nullptr;
    sc.packed = n.packed_bytes ? base + n.state_bytes : nullptr;
    sc.part = n.part_bytes ? (float*)(base + n.part_offset(room)) : nullptr;
    sc.rows = n.rows_bytes ? base + n.rows_offset() : nullptr;
    return sc;
}

BlockRecord* find_block(void* ptr) {
    for (BlockRecord& r : g_blocks)
        if (r.ptr == ptr) return &r;
    return nullptr;
}

// Where a call's scratch memory comes from.
enum ScratchSource { kScratchLibrary, kScratchCaller, kScratchStatic };
constexpr int kRouteFewRows = 12;      // tide_call_route's number for the few-rows kernel, behind those of PrefillKernel (0: the latency kernel)

// Shared body of the compute entry points.  Exactly one of (W1) / (packed) is given.  Everything that
// can fail for lack of memory or for a misused workspace happens before the first kernel is enqueued.
int run(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride, int64_t row_stride,
        const float* gamma, const float* W1, const void* packed, float eps, const float* b1, const float* w2,
        const CheckpointTable& tab, int32_t min_layer, int32_t no_exit, const Outputs& o, void* stream,
        ScratchSource source = kScratchLibrary, void* block = nullptr, size_t block_bytes = 0) {
    if (T == 0) return TIDE_OK;
    hipStream_t st = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(g_mu);
    int dev = 0;
    int rc = current_device(&dev);
    if (rc) return rc;
    unsigned cus = 0;
    rc = resident_cus(&cus);
    if (rc) return rc;
    const bool want_exit = o.exit_layer != nullptr;
    const size_t room = source == kScratchCaller ? block_bytes : kStaticScratchBytes;      // of a block that is not the library's workspace
    CallNeed need = source == kScratchLibrary
                        ? call_need(dtype, C, T, d, b, W1 != nullptr, want_exit, cus, g_variant, g_prefill_form, true)
                        : block_need(dtype, C, T, d, b, W1 != nullptr, want_exit, cus, g_variant, g_prefill_form, room);

    auto capturing = [&]() {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
        return cap != hipStreamCaptureStatusNone;
    };
    // While a call is captured nothing can be allocated: where the library's workspace lacks the partial results of a route, the call takes the
    // few-rows kernel if that is near its range and has room, else the route that a caller's block would give it, with a pair that fits or none.
    if (source == kScratchLibrary && need.part_bytes > g_ws[dev].part.bytes && capturing()) {
        const size_t part_room = g_ws[dev].part.bytes;
        const CallNeed wide = call_need(dtype, C, T, d, b, W1 != nullptr, want_exit, cus, g_variant, g_prefill_form, true, kFewWide);
        need = wide.few && wide.part_bytes <= part_room
                   ? wide
                   : call_need(dtype, C, T, d, b, W1 != nullptr, want_exit, cus, g_variant, g_prefill_form, false, kFewNever, g_prefill_form == 0 ? part_room : SIZE_MAX);
    }

    Scratch sc;
    Workspace* ws = nullptr;        // library workspace, if that is the source
    size_t* clean = nullptr;        // else: the block's count of leading zero-state bytes
    BlockRecord* rec = nullptr;     // ... and a caller's block's record
    if (source == kScratchLibrary) {
        ws = &g_ws[dev];
        rc = claim_workspace(*ws, st);
        if (rc) return rc;
        if ((rc = reserve(ws->counters, kCounterSlots * sizeof(uint32_t), true))) return rc;
        if (want_exit && (rc = reserve(ws->arrive, (size_t)T * sizeof(uint64_t), true))) return rc;
        if (need.packed_bytes && (rc = reserve(ws->packed, need.packed_bytes, false))) return rc;
        size_t part_bytes = need.part_bytes;
        SizedShape* shape = nullptr;     // to be remembered once the buffer is there
        if (g_variant == TIDE_VARIANT_AUTO && g_prefill_form == 0) {
            for (SizedShape& s : ws->sized)
                if (s.C == C && s.d == d && s.b == b && s.dtype == dtype && s.raw == (W1 != nullptr)) shape = &s;
            if (shape && T <= shape->T) {
                shape = nullptr;
            } else if (!capturing()) {
                const int64_t from = shape ? shape->T : 0;
                if (!shape) shape = &ws->sized[ws->next_sized++ % kSizedShapes];
                part_bytes = std::max(part_bytes, largest_part(dtype, C, from, (T + 31) / 32 * 32, d, b, W1 != nullptr, cus));
            } else {
                shape = nullptr;
            }
        }
        rc = part_bytes ? reserve(ws->part, part_bytes, false) : TIDE_OK;
        if (rc && part_bytes > need.part_bytes) {       // no room for more than this call needs
            (void)hipGetLastError();
            for (SizedShape& s : ws->sized) s = SizedShape{};
            shape = nullptr;
            rc = need.part_bytes ? reserve(ws->part, need.part_bytes, false) : TIDE_OK;
        }
        if (rc) return rc;
        if (shape) *shape = SizedShape{dtype, W1 != nullptr, C, d, b, (T + 31) / 32 * 32};
        if (need.rows_bytes && (rc = reserve(ws->rows, need.rows_bytes, false))) return rc;
        if (ws->dirty) {            // an earlier call broke off between two launches: its state words may be set
            if ((rc = launch_clear(ws->counters.ptr, ws->counters.bytes, st))) return rc;
            if (ws->arrive.ptr && (rc = launch_clear(ws->arrive.ptr, ws->arrive.bytes, st))) return rc;
            ws->dirty = false;
        }
        sc.counters = (uint32_t*)ws->counters.ptr;
        sc.arrive = want_exit ? (uint64_t*)ws->arrive.ptr : nullptr;
        sc.packed = ws->packed.ptr;
        sc.part = (float*)ws->part.ptr;
        sc.rows = ws->rows.ptr;
    } else if (source == kScratchCaller) {
        rec = find_block(block);
        if (!rec) return fail(TIDE_ERR_WORKSPACE, "unknown workspace %p: call tide_workspace_init on it first", block);
        if (block_bytes > rec->bytes)
            return fail(TIDE_ERR_WORKSPACE, "workspace_bytes %zu exceeds the %zu bytes tide_workspace_init was given", block_bytes, rec->bytes);
        if (need.total() > block_bytes)
            return fail(TIDE_ERR_WORKSPACE, "this call needs %zu bytes of workspace (tide_workspace_bytes), %zu given", need.total(), block_bytes);
        if (need.state_bytes > rec->settled)
            return fail(TIDE_ERR_WORKSPACE, "this call keeps %zu bytes of state at the start of the workspace, where an earlier call of "
                        "another shape left data (or a launch failed): call tide_workspace_init again first", need.state_bytes);
        if (need.state_bytes > rec->clean) {         // an earlier call's partial results lie where this one keeps state: clear it
            if ((rc = launch_clear(block, need.state_bytes, st))) return rc;
            rec->clean = need.state_bytes;
        }
        rec->stamp = ++g_block_clock;
        rec->state = std::max(rec->state, need.state_bytes);
        clean = &rec->clean;
        sc = carve(block, room, need, want_exit);
    } else {
        StaticScratch& ss = g_static[dev];
        if (!ss.ptr) {              // once per device, with that device current
            void* addr = nullptr;
            TIDE_HIP(hipGetSymbolAddress(&addr, HIP_SYMBOL(g_static_scratch)));
            ss.ptr = addr;
            ss.clean = kStaticScratchBytes;          // device globals start zero-filled
        }
        if (need.total() > kStaticScratchBytes)
            return fail(TIDE_ERR_WORKSPACE, "this call needs %zu bytes of scratch memory; the no-allocation entry point holds %zu "
                        "(use the entry point with a caller-supplied workspace)", need.total(), kStaticScratchBytes);
        if (need.state_bytes > ss.clean) {           // an earlier call's data lies where this one keeps state: clear it
            if ((rc = launch_clear(ss.ptr, need.state_bytes, st))) return rc;
            ss.clean = need.state_bytes;
        }
        clean = &ss.clean;
        sc = carve(ss.ptr, room, need, want_exit);
    }
    // the data regions of this call overwrite whatever zero state lay there
    const size_t data = need.data_begin(room);
    const bool split_k_only = need.part_last && !need.packed_bytes && !need.rows_bytes;
    if (clean) *clean = std::min(*clean, data);
    if (rec && !split_k_only) rec->settled = std::min(rec->settled, data);

    if (need.decode) {
        rc = launch_decode(sc, hidden, dtype, C, T, d, b, ckpt_stride, row_stride, gamma, W1, packed, eps, b1, w2, tab,
                           min_layer, no_exit, o, st);
    } else {
        if (need.rows_bytes) {      // generic fallback: aligned, zero-padded rows for the tuned kernels
            RepackParams rp;
            const int64_t eb = (int64_t)elem_bytes(dtype);
            rp.hidden = (const char*)hidden;
            rp.ckpt_stride_bytes = ckpt_stride * eb;
            rp.row_stride_bytes = row_stride * eb;
            rp.out = (u32x4*)sc.rows;
            rp.C = (int)C;
            rp.T = (int)T;
            rp.d = (int)d;
            rp.dpad = (int)need.d_run;
            const int64_t chunks = C * T * (need.d_run * eb / 16);
            const unsigned grid = (unsigned)std::min<int64_t>((chunks + kRepackThreads - 1) / kRepackThreads, 1 << 20);
            by_dtype(dtype, [&](auto dt) {
                hipLaunchKernelGGL((tide_repack_rows_kernel<decltype(dt)::value>), dim3(grid), dim3(kRepackThreads), 0, st, rp);
                return 0;
            });
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) rc = fail(TIDE_ERR_HIP, "row repack launch: %s", hipGetErrorString(e));
            hidden = sc.rows;
            ckpt_stride = T * need.d_run;
            row_stride = need.d_run;
        }
        if (!rc && W1) {
            rc = launch_pack(dtype, C, d, b, gamma, W1, sc.packed, st);
            packed = sc.packed;
        }
        auto params = [&]() {
            PrefillParams p = prefill_params(sc, hidden, dtype, C, T, need.d_run, d, b, ckpt_stride, row_stride, packed, eps, b1, w2, tab, min_layer,
                                             no_exit, o);
            p.deal_out = deals_out(dtype, C, T, d, b, W1 != nullptr);
            return p;
        };
        if (!rc)
            rc = need.few ? launch_few_rows(sc, params(), dtype, need.few_full, st) : launch_prefill(sc, need.plan, params(), dtype, st);
    }
    if (!rc && rec && split_k_only && data < rec->state) {      // over the state of an earlier call, which may be captured and replayed: zeros again
        rc = launch_clear((char*)block + data, rec->state - data, st);
        if (rec->clean == data) rec->clean = rec->state;
    }
    if (rc) {                       // a launch failed, possibly after an earlier one of this call was enqueued
        if (ws) ws->dirty = true;
        if (clean) *clean = 0;
        if (rec) rec->settled = 0;
    }
    return rc;
}

}  // namespace

extern "C" {

int tide_version(void) { return 112; }

const char* tide_last_error(void) { return g_err; }

size_t tide_packed_router_bytes(int dtype, int64_t d, int64_t b) {
    if ((dtype != TIDE_F32 && dtype != TIDE_F16 && dtype != TIDE_BF16) || !supported_hidden(dtype, d)) return 0;
    if (!supported_bottleneck(b)) return 0;
    return (size_t)halves_of(b) * (size_t)padded_hidden(dtype, d) * kBottleneck * elem_bytes(dtype);
}

int tide_router_pack(int dtype, int64_t C, int64_t d, int64_t b, const float* gamma, const float* W1, void* packed, void* stream) {
    g_err[0] = 0;
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS) return fail(TIDE_ERR_INVALID_ARG, "C = %lld outside [1, 32]", (long long)C);
    if (tide_packed_router_bytes(dtype, d, b) == 0)
        return fail(TIDE_ERR_UNSUPPORTED, "unsupported dtype %d, d %lld or bottleneck width %lld", dtype, (long long)d, (long long)b);
    if (!W1 || !packed) return fail(TIDE_ERR_INVALID_ARG, "W1 and packed must not be NULL");
    if ((uintptr_t)packed & 15) return fail(TIDE_ERR_ALIGNMENT, "packed must be 16-byte aligned");
    return launch_pack(dtype, C, d, b, gamma, W1, packed, (hipStream_t)stream);
}

namespace {
// Front end of the router_eval family: one router (C = 1), exactly one of W1 / packed.
int eval_front(const void* hidden, int dtype, int64_t T, int64_t d, int64_t b, int64_t row_stride, const float* gamma, float eps,
               const float* W1, const void* packed, const float* b1, const float* w2, float b2, float threshold, float* prob,
               uint8_t* fire, float* logit, void* stream, ScratchSource source, void* block, size_t block_bytes) {
    g_err[0] = 0;
    int rc = check_common(hidden, dtype, 1, T, d, b, 0, row_stride, W1 ? (const void*)W1 : packed, w2, eps);
    if (rc) return rc;
    if ((rc = check_optional_arrays(gamma, b1))) return rc;
    CheckpointTable tab;
    const int32_t id0 = 0;
    rc = fill_table(tab, 1, &b2, &threshold, &id0);
    if (rc) return rc;
    Outputs o{prob, fire, logit, nullptr, nullptr};
    return run(hidden, dtype, 1, T, d, b, 0, row_stride, gamma, W1, packed, eps, b1, w2, tab, 0, 0, o, stream, source, block, block_bytes);
}
// Front end of the select_exit family.
int select_front(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride, int64_t row_stride,
                 const float* gamma, float eps, const float* W1, const void* packed, const float* b1, const float* w2,
                 const float* b2, const float* threshold, const int32_t* layer_ids, int32_t min_layer, int32_t no_exit_layer,
                 int32_t* exit_layer, float* logits, uint32_t* fire_mask, void* stream, ScratchSource source, void* block,
                 size_t block_bytes) {
    g_err[0] = 0;
    int rc = check_common(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, W1 ? (const void*)W1 : packed, w2, eps);
    if (rc) return rc;
    if ((rc = check_optional_arrays(gamma, b1))) return rc;
    CheckpointTable tab;
    rc = fill_table(tab, C, b2, threshold, layer_ids);
    if (rc) return rc;
    if (T > 0 && !exit_layer) return fail(TIDE_ERR_INVALID_ARG, "exit_layer must not be NULL");
    Outputs o{nullptr, nullptr, logits, exit_layer, fire_mask};
    return run(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, gamma, W1, packed, eps, b1, w2, tab, min_layer, no_exit_layer, o,
               stream, source, block, block_bytes);
}
// A caller's workspace argument, checked before anything else is looked at.
int check_block(const void* W1, const void* packed, const float* gamma, void* workspace, size_t workspace_bytes) {
    g_err[0] = 0;
    if ((W1 != nullptr) == (packed != nullptr)) return fail(TIDE_ERR_INVALID_ARG, "give exactly one of W1 (raw weights) and packed");
    if (packed && gamma) return fail(TIDE_ERR_INVALID_ARG, "gamma is folded into packed weights: pass gamma = NULL with packed");
    if (!workspace || workspace_bytes == 0) return fail(TIDE_ERR_INVALID_ARG, "workspace must not be NULL or empty");
    if ((uintptr_t)workspace & 255) return fail(TIDE_ERR_ALIGNMENT, "workspace must be 256-byte aligned");
    return TIDE_OK;
}
}  // namespace

int tide_router_eval(const void* hidden, int dtype, int64_t T, int64_t d, int64_t b, int64_t row_stride, const float* gamma,
                     float eps, const float* W1, const float* b1, const float* w2, float b2, float threshold,
                     float* prob, uint8_t* fire, float* logit, void* stream) {
    return eval_front(hidden, dtype, T, d, b, row_stride, gamma, eps, W1, nullptr, b1, w2, b2, threshold, prob, fire, logit, stream,
                      kScratchLibrary, nullptr, 0);
}

int tide_router_eval_packed(const void* hidden, int dtype, int64_t T, int64_t d, int64_t b, int64_t row_stride,
                            const void* packed, float eps, const float* b1, const float* w2, float b2,
                            float threshold, float* prob, uint8_t* fire, float* logit, void* stream) {
    return eval_front(hidden, dtype, T, d, b, row_stride, nullptr, eps, nullptr, packed, b1, w2, b2, threshold, prob, fire, logit,
                      stream, kScratchLibrary, nullptr, 0);
}

int tide_router_eval_ws(const void* hidden, int dtype, int64_t T, int64_t d, int64_t b, int64_t row_stride, const float* gamma,
                        float eps, const float* W1, const void* packed, const float* b1, const float* w2, float b2,
                        float threshold, float* prob, uint8_t* fire, float* logit, void* workspace, size_t workspace_bytes,
                        void* stream) {
    int rc = check_block(W1, packed, gamma, workspace, workspace_bytes);
    if (rc) return rc;
    return eval_front(hidden, dtype, T, d, b, row_stride, gamma, eps, W1, packed, b1, w2, b2, threshold, prob, fire, logit, stream,
                      kScratchCaller, workspace, workspace_bytes);
}

int tide_select_exit(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride,
                     int64_t row_stride, const float* gamma, float eps, const float* W1, const float* b1,
                     const float* w2, const float* b2, const float* threshold, const int32_t* layer_ids,
                     int32_t min_layer, int32_t no_exit_layer, int32_t* exit_layer, float* logits,
                     uint32_t* fire_mask, void* stream) {
    return select_front(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, gamma, eps, W1, nullptr, b1, w2, b2, threshold, layer_ids,
                        min_layer, no_exit_layer, exit_layer, logits, fire_mask, stream, kScratchLibrary, nullptr, 0);
}

int tide_select_exit_packed(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride,
                            int64_t row_stride, const void* packed, float eps, const float* b1, const float* w2,
                            const float* b2, const float* threshold, const int32_t* layer_ids, int32_t min_layer,
                            int32_t no_exit_layer, int32_t* exit_layer, float* logits, uint32_t* fire_mask,
                            void* stream) {
    return select_front(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, nullptr, eps, nullptr, packed, b1, w2, b2, threshold,
                        layer_ids, min_layer, no_exit_layer, exit_layer, logits, fire_mask, stream, kScratchLibrary, nullptr, 0);
}

int tide_select_exit_ws(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int64_t ckpt_stride,
                        int64_t row_stride, const float* gamma, float eps, const float* W1, const void* packed,
                        const float* b1, const float* w2, const float* b2, const float* threshold,
                        const int32_t* layer_ids, int32_t min_layer, int32_t no_exit_layer, int32_t* exit_layer,
                        float* logits, uint32_t* fire_mask, void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_block(W1, packed, gamma, workspace, workspace_bytes);
    if (rc) return rc;
    return select_front(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, gamma, eps, W1, packed, b1, w2, b2, threshold, layer_ids,
                        min_layer, no_exit_layer, exit_layer, logits, fire_mask, stream, kScratchCaller, workspace, workspace_bytes);
}

size_t tide_workspace_bytes(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int raw_weights) {
    g_err[0] = 0;
    if ((dtype != TIDE_F32 && dtype != TIDE_F16 && dtype != TIDE_BF16) || C < 1 || C > TIDE_MAX_CHECKPOINTS || T < 0 ||
        C * T > (int64_t)1 << 30 || tide_packed_router_bytes(dtype, d, b) == 0) {
        fail(TIDE_ERR_UNSUPPORTED, "unsupported dtype %d, C %lld, T %lld, d %lld or b %lld", dtype, (long long)C, (long long)T,
             (long long)d, (long long)b);
        return 0;
    }
    unsigned cus = 256;             // without a device: the answer for a 256-CU one
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess) {
        if (resident_cus(&cus) != TIDE_OK) cus = 256;
    } else {
        (void)hipGetLastError();
    }
    std::lock_guard<std::mutex> lock(g_mu);
    return call_need(dtype, C, T > 0 ? T : 1, d, b, raw_weights != 0, true, cus, g_variant, g_prefill_form, false).total();
}

int tide_call_route(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int raw_weights, int cus, size_t block_bytes, int64_t* out) {
    g_err[0] = 0;
    if (dtype != TIDE_F32 && dtype != TIDE_F16 && dtype != TIDE_BF16) return fail(TIDE_ERR_INVALID_ARG, "dtype %d is not a tide_dtype_t", dtype);
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS || T < 1 || C * T > (int64_t)1 << 30) return fail(TIDE_ERR_INVALID_ARG, "C = %lld, T = %lld out of range", (long long)C, (long long)T);
    if (!supported_hidden(dtype, d) || !supported_bottleneck(b)) return fail(TIDE_ERR_UNSUPPORTED, "d = %lld, b = %lld unsupported", (long long)d, (long long)b);
    if (cus < 8 || cus % 8 != 0) return fail(TIDE_ERR_INVALID_ARG, "cus = %d must be a positive multiple of 8", cus);
    if (!out) return fail(TIDE_ERR_INVALID_ARG, "out must not be NULL");
    std::lock_guard<std::mutex> lock(g_mu);
    const bool library = block_bytes == 0;
    const CallNeed n = library ? call_need(dtype, C, T, d, b, raw_weights != 0, true, (unsigned)cus, g_variant, g_prefill_form, true)
                               : block_need(dtype, C, T, d, b, raw_weights != 0, true, (unsigned)cus, g_variant, g_prefill_form, block_bytes);
    if (!library && n.total() > block_bytes) return fail(TIDE_ERR_WORKSPACE, "this call needs %zu bytes of workspace, %zu given", n.total(), block_bytes);
    const PlannedLaunch none{kRouteFewRows, kFewRows, 0, 0, 0, 1, 0}, &L = n.few || n.decode ? none : n.plan.launch[0];
    out[0] = n.decode ? 0 : L.kernel;
    out[1] = n.decode ? 0 : L.rows_per_tile;
    out[2] = L.k_slices;
    out[3] = (int64_t)n.total();
    out[4] = library ? 0 : (int64_t)std::min(n.data_begin(block_bytes), block_bytes);
    return TIDE_OK;
}

int tide_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
    g_err[0] = 0;
    if (!workspace || workspace_bytes < 256) return fail(TIDE_ERR_INVALID_ARG, "workspace must not be NULL and hold at least 256 bytes");
    if ((uintptr_t)workspace & 255) return fail(TIDE_ERR_ALIGNMENT, "workspace must be 256-byte aligned");
    const size_t bytes = workspace_bytes & ~size_t(255);
    std::lock_guard<std::mutex> lock(g_mu);
    int rc = launch_clear(workspace, bytes, (hipStream_t)stream);
    if (rc) return rc;
    BlockRecord* rec = find_block(workspace);
    if (!rec) {                     // a free record, else the least recently used one
        rec = &g_blocks[0];
        for (BlockRecord& r : g_blocks) {
            if (!r.ptr) { rec = &r; break; }
            if (r.stamp < rec->stamp) rec = &r;
        }
    }
    rec->ptr = workspace;
    rec->bytes = bytes;
    rec->clean = rec->settled = bytes;
    rec->state = 0;
    rec->stamp = ++g_block_clock;
    return TIDE_OK;
}

int tide_workspace_forget(void* workspace) {
    g_err[0] = 0;
    std::lock_guard<std::mutex> lock(g_mu);
    BlockRecord* rec = find_block(workspace);
    if (!rec) return fail(TIDE_ERR_INVALID_ARG, "unknown workspace %p", workspace);
    *rec = BlockRecord{};
    return TIDE_OK;
}

int tide_select_exit_packed_noalloc(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t b,
                                    int64_t ckpt_stride, int64_t row_stride, const void* packed, float eps, const float* b1,
                                    const float* w2, const float* b2, const float* threshold, const int32_t* layer_ids,
                                    int32_t min_layer, int32_t no_exit_layer, int32_t* exit_layer, float* logits,
                                    uint32_t* fire_mask, void* stream) {
    return select_front(hidden, dtype, C, T, d, b, ckpt_stride, row_stride, nullptr, eps, nullptr, packed, b1, w2, b2, threshold,
                        layer_ids, min_layer, no_exit_layer, exit_layer, logits, fire_mask, stream, kScratchStatic, nullptr, 0);
}

size_t tide_noalloc_scratch_bytes(void) { return kStaticScratchBytes; }

#ifdef TIDE_TILE_TIMELINE
// Timeline builds only (timeline.py): where the one-tile prefill kernel leaves its per-workgroup time stamps
// (device memory, kTimelineStamps x 8 bytes per workgroup of the largest launch; NULL switches them off).
int tide_debug_timeline(void* buffer) {
    g_err[0] = 0;
    unsigned long long* b = (unsigned long long*)buffer;
    TIDE_HIP(hipMemcpyToSymbol(HIP_SYMBOL(g_tile_timeline), &b, sizeof(b)));
    return kTimelineStamps;
}
#endif

// Measurement helper (not part of the router path): see the header.
int tide_mfma_probe(int waves_per_cu, int iters, int launches, int zero_operands, double* out) {
    g_err[0] = 0;
    if (!out || (waves_per_cu != 4 && waves_per_cu != 8) || iters < 1 || iters > (1 << 20) || launches < 1 || launches > 1000)
        return fail(TIDE_ERR_INVALID_ARG, "tide_mfma_probe: waves_per_cu 4 or 8, 1 <= iters <= 2^20, 1 <= launches <= 1000, out not NULL");
    unsigned cus = 0;
    int rc = resident_cus(&cus);
    if (rc) return rc;
    // operand bits: pairs of bf16 values of magnitude 1 .. 2 with pseudo-random mantissas and signs, or zeros
    std::vector<uint32_t> bits(4096 * 4, 0u);
    if (!zero_operands) {
        uint32_t x = 0x71DEu;
        for (uint32_t& w : bits) {
            uint32_t h[2];
            for (uint32_t& v : h) {
                x = x * 1664525u + 1013904223u;
                v = 0x3f80u | ((x >> 9) & 0x7fu) | (((x >> 20) & 1u) << 15);
            }
            w = h[0] | (h[1] << 16);
        }
    }
    void *in = nullptr, *sums = nullptr, *clk = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto cleanup = [&]() {
        if (in) (void)hipFree(in);
        if (sums) (void)hipFree(sums);
        if (clk) (void)hipFree(clk);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    auto step = [&](hipError_t e, const char* what) {
        if (e == hipSuccess) return 0;
        cleanup();
        return fail(TIDE_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
    };
    const unsigned threads = (unsigned)waves_per_cu * kWave;
    if ((rc = step(hipMalloc(&in, bits.size() * 4), "hipMalloc"))) return rc;
    if ((rc = step(hipMalloc(&sums, (size_t)cus * threads * sizeof(float)), "hipMalloc"))) return rc;
    if ((rc = step(hipMalloc(&clk, 16), "hipMalloc"))) return rc;
    if ((rc = step(hipMemcpy(in, bits.data(), bits.size() * 4, hipMemcpyHostToDevice), "hipMemcpy"))) return rc;
    if ((rc = step(hipMemset(clk, 0, 16), "hipMemset"))) return rc;
    if ((rc = step(hipEventCreate(&e0), "hipEventCreate"))) return rc;
    if ((rc = step(hipEventCreate(&e1), "hipEventCreate"))) return rc;
    auto launch = [&]() {
        hipLaunchKernelGGL(tide_mfma_probe_kernel, dim3(cus), dim3(threads), 0, nullptr, (const u32x4*)in, (float*)sums, iters, (unsigned long long*)clk);
    };
    launch();                                                     // (untimed: code load, clocks)
    if ((rc = step(hipDeviceSynchronize(), "hipDeviceSynchronize"))) return rc;
    if ((rc = step(hipEventRecord(e0, nullptr), "hipEventRecord"))) return rc;
    for (int l = 0; l < launches; ++l) launch();
    if ((rc = step(hipEventRecord(e1, nullptr), "hipEventRecord"))) return rc;
    if ((rc = step(hipDeviceSynchronize(), "hipDeviceSynchronize"))) return rc;
    float ms = 0.0f;
    if ((rc = step(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime"))) return rc;
    unsigned long long c[2] = {0, 0};
    if ((rc = step(hipMemcpy(c, clk, 16, hipMemcpyDeviceToHost), "hipMemcpy"))) return rc;
    cleanup();
    const double us = (double)ms * 1e3 / launches;
    const double flop = (double)cus * waves_per_cu * (double)iters * kMfmaProbeAcc * 32768.0;      // 2 x 32 x 32 x 16 per instruction
    out[0] = us;
    out[1] = flop / us / 1e6;                                    // TFLOP/s
    out[2] = c[1] ? (double)c[0] / (double)c[1] / 10.0 : 0.0;     // GHz
    out[3] = (double)c[0] / ((double)iters * kMfmaProbeAcc);     // cycles per instruction and wave
    return TIDE_OK;
}

uint64_t tide_workspace_allocations(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    return g_allocations;
}

int tide_exit_project(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t ckpt_stride,
                      int64_t row_stride, const void* final_hidden, int64_t final_row_stride,
                      const int32_t* exit_layer, const int32_t* layer_ids, const float* norm_gain, float eps,
                      void* out, int64_t out_row_stride, void* stream) {
    g_err[0] = 0;
    int rc = check_common(hidden, dtype, C, T, d, kBottleneck, ckpt_stride, row_stride, hidden, reinterpret_cast<const float*>(hidden), eps, true);
    if (rc) return rc;
    if (T == 0) return TIDE_OK;
    if (!exit_layer || !layer_ids || !out) return fail(TIDE_ERR_INVALID_ARG, "exit_layer, layer_ids (host) and out must not be NULL");
    if (out_row_stride < d || (final_hidden && final_row_stride < d))
        return fail(TIDE_ERR_INVALID_ARG, "row strides of out / final_hidden must be at least d");
    const size_t eb = elem_bytes(dtype);
    if (((uintptr_t)out & 15) || ((size_t)out_row_stride * eb & 15) ||
        (final_hidden && (((uintptr_t)final_hidden & 15) || ((size_t)final_row_stride * eb & 15))) ||
        ((uintptr_t)norm_gain & 15))
        return fail(TIDE_ERR_ALIGNMENT, "out, final_hidden and norm_gain bases and the row strides must be multiples of 16 bytes");
    ProjectParams p;
    std::memset(&p, 0, sizeof(p));
    for (int64_t c = 0; c < C; ++c) {
        if (c > 0 && layer_ids[c] <= layer_ids[c - 1])
            return fail(TIDE_ERR_INVALID_ARG, "layer_ids must be strictly ascending");
        p.layer_id[c] = layer_ids[c];
    }
    p.hidden = (const char*)hidden;
    p.ckpt_stride_bytes = ckpt_stride * (int64_t)eb;
    p.row_stride_bytes = row_stride * (int64_t)eb;
    p.final_hidden = (const char*)final_hidden;
    p.final_row_stride_bytes = final_row_stride * (int64_t)eb;
    p.exit_layer = exit_layer;
    p.gain = norm_gain;
    p.out = (char*)out;
    p.out_row_stride_bytes = out_row_stride * (int64_t)eb;
    p.C = (int)C;
    p.T = (int)T;
    p.d = (int)d;
    p.eps = eps;
    const int64_t row_bytes = d * (int64_t)eb;
    bool wave_per_row = row_bytes <= (int64_t)kProjectMaxChunks * 16 * kWave;        // 16 KiB
    bool gain_ahead = true;
    if (row_bytes >= 4096) {                                                          // (project_kernel.hpp has the figures of both choices)
        unsigned cus = 0;
        if ((rc = resident_cus(&cus))) return rc;
        gain_ahead = wave_per_row || T <= (int64_t)cus || T > (eb == 2 ? 5 : 8) * (int64_t)cus;
        wave_per_row = wave_per_row && T > 3 * (int64_t)cus;
    }
    if (row_bytes > (int64_t)kProjectMaxChunks * 16 * kProjectThreads)
        return fail(TIDE_ERR_UNSUPPORTED, "rows of %lld bytes exceed the projection kernel's limit", (long long)row_bytes);
    hipStream_t st = (hipStream_t)stream;
    const unsigned grid = wave_per_row ? (unsigned)((T + 3) / 4) : (unsigned)T;
    const int64_t per_thread = (row_bytes / 16 + (wave_per_row ? kWave : kProjectThreads) - 1) / (wave_per_row ? kWave : kProjectThreads);
    by_dtype(dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        auto go = [&](auto wpr, auto gain, auto chunks) {
            constexpr bool kWpr = decltype(wpr)::value, kGain = decltype(gain)::value, kAhead = kGain && !kWpr;
            constexpr int kChunks = decltype(chunks)::value;
            if constexpr (kAhead && kChunks > 4)
                if (!gain_ahead) {
                    hipLaunchKernelGGL((tide_project_kernel<DT, kWpr, kGain, kChunks, false>), dim3(grid), dim3(kProjectThreads), 0, st, p.exit_layer, p.hidden,
                       p.ckpt_stride_bytes, p.row_stride_bytes, p.final_hidden, p.final_row_stride_bytes, p.T, p.d, p);
                    return;
                }
            hipLaunchKernelGGL((tide_project_kernel<DT, kWpr, kGain, kChunks, kAhead>), dim3(grid), dim3(kProjectThreads), 0, st, p.exit_layer, p.hidden,
                       p.ckpt_stride_bytes, p.row_stride_bytes, p.final_hidden, p.final_row_stride_bytes, p.T, p.d, p);
        };
        auto pick_chunks = [&](auto wpr, auto gain) {
            if constexpr (!decltype(wpr)::value) {
                if (per_thread <= 1) return go(wpr, gain, std::integral_constant<int, 1>{});
                if (per_thread <= 2) return go(wpr, gain, std::integral_constant<int, 2>{});
            }
            if (per_thread <= 4) go(wpr, gain, std::integral_constant<int, 4>{});
            else if (per_thread <= 8) go(wpr, gain, std::integral_constant<int, 8>{});
            else go(wpr, gain, std::integral_constant<int, 16>{});
        };
        auto pick_gain = [&](auto wpr) {
            if (norm_gain) pick_chunks(wpr, std::true_type{});
            else pick_chunks(wpr, std::false_type{});
        };
        if (wave_per_row) pick_gain(std::true_type{});
        else pick_gain(std::false_type{});
        return 0;
    });
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

int tide_batch_compact(const int32_t* exit_layer, int64_t T, int32_t layer, int32_t* exit_idx, int32_t* cont_idx,
                       int32_t* counts, void* stream) {
    g_err[0] = 0;
    if (T < 0 || T > (int64_t)1 << 30) return fail(TIDE_ERR_INVALID_ARG, "T = %lld outside [0, 2^30]", (long long)T);
    if (!counts) return fail(TIDE_ERR_INVALID_ARG, "counts must not be NULL");
    if (T > 0 && (!exit_layer || !exit_idx || !cont_idx))
        return fail(TIDE_ERR_INVALID_ARG, "exit_layer, exit_idx and cont_idx must not be NULL");
    hipStream_t st = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(g_mu);
    Workspace* ws = nullptr;
    int rc = current_workspace(&ws);
    if (rc) return rc;
    if ((rc = claim_workspace(*ws, st))) return rc;
    constexpr int kMaxBlocks = 1024;
    rc = reserve(ws->compact, kMaxBlocks * sizeof(uint32_t), true);
    if (rc) return rc;
    CompactParams p;
    std::memset(&p, 0, sizeof(p));
    p.exit_layer = exit_layer;
    p.T = (int)T;
    p.layer = layer;
    p.exit_idx = exit_idx;
    p.cont_idx = cont_idx;
    p.counts = counts;
    p.block_counts = (uint32_t*)ws->compact.ptr;
    int64_t slice = 16 * kCompactThreads;                               // 4096 tokens per workgroup ...
    while ((T + slice - 1) / slice > kMaxBlocks) slice *= 2;            // ... more for very large batches
    p.slice = (int)slice;
    const unsigned grid = T > 0 ? (unsigned)((T + slice - 1) / slice) : 1u;   // T == 0 still writes counts = {0, 0}
    if (grid > 1) hipLaunchKernelGGL(tide_compact_count_kernel, dim3(grid), dim3(kCompactThreads), 0, st, p);
    hipLaunchKernelGGL(tide_compact_scatter_kernel, dim3(grid), dim3(kCompactThreads), 0, st, p);
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

namespace {
// Cosine labels: units per token (1 << the result: 1, 2 or 4) that its checkpoints are dealt out to.  More of them are more waves in flight and a shorter
// chain per wave, but each reads the last layer's row.  The lines are tokens on 256 CUs, which is waves per CU at one unit (longer rows take more
// registers, so fewer waves are resident: 32 per CU up to three chunks per lane, 28 at four, 24 / 20 / 16 / 12 / 8 at 5 / 6 / 8 / 10 / more).  Measured (us,
// one / two / four units, kernels back to back in a graph, bf16, C = 8 where not given; C = 4, 10, 16, 32 alike within the noise unless said):
int label_unit_bits(bool wave_per_row, int64_t row_chunks, int64_t C, int64_t T, unsigned cus) {
    if (C == 1 || T >= (int64_t)1 << 22) return 0;     // a launch has fewer than 2^32 threads: as many tokens as with one unit each
    const int64_t t = T * 256 / (int64_t)cus;
    // A workgroup per row (above 16 KiB; fp32, d = 5120, C = 9): 14.7 / 10.4 at 200, 18.0 / 16.6 at 420, 23.9 / 27.0 at 700, 32.0 / 32.6 at 980, 52.4 / 47.5 at 1500.
    if (!wave_per_row) return t <= 500 || t > 1000 ? 1 : 0;
    int bits;
    if (row_chunks <= 192)
        // d = 768: 8.1 / 5.2 / 4.0 at 500, 8.7 / 5.9 / 5.2 at 1300, 9.0 / 6.5 / 6.1 at 1850, 9.3 / 7.4 / 8.2 at 2300, 9.8 / 8.9 / 9.4 at 3000, 10.7 / 9.9 at 3500, 13.0 / 14.5 at 5000;
        // d = 1024, C = 16: 16.5 / 12.1 / 13.9 at 1850; C = 8 10.2 / 10.0 at 2600, 10.6 / 10.7 at 3000, 12.1 / 12.6 at 3500; d = 1536 14.9 / 13.2 at 2600, 15.6 / 15.4 at 3000.
        bits = t <= (row_chunks <= 96 ? 1800 : 1000) ? 2 : t <= 3200 ? 1 : 0;
    else if (row_chunks <= 256)
        // d = 2048: 12.0 / 7.6 / 5.4 at 500, 12.8 / 8.3 / 7.7 at 900, 14.2 / 11.3 / 11.9 at 1550, 16.3 / 16.0 / 15.8 at 2400, 17.0 / 18.2 / 16.9 at 2600, 18.5 / 19.7 / 19.9 at 3000.
        bits = t <= 1000 ? 2 : t <= 2500 ? 1 : 0;
    else if (row_chunks <= 384)
        // d = 2560: 13.3 / 9.3 / 8.8 at 900, 14.9 / 10.9 / 11.7 at 1300, 15.6 / 13.2 / 13.2 at 1550, 16.3 / 15.5 / 15.3 at 1850, 18.1 / 18.9 / 17.4 at 2200, 20.4 / 22.7 / 20.8 at 2700
        // (C = 4 12.4 / 13.3 / 12.3, C = 16 35.9 / 40.6 / 38.3), 27.2 / 27.7 / 26.0 at 3500, 42.0 / 39.9 / 38.1 at 5440; d = 3072 18.7 / 19.2 / 19.7 at 2000, 40.4 / 37.5 / 36.9 at
        // 4200, 51.8 / 47.1 / 48.7 at 5440.
        bits = t <= (row_chunks <= 320 ? 1000 : 700) ? 2 : t <= (row_chunks <= 320 ? 2000 : 1500) ? 1 : t <= 2000 || (C >= 8 && t > 2400 && t <= 3200) ? 0
               : row_chunks > 320 && t > 4800 ? 1 : 2;
    else
        // d = 4096: 14.7 / 9.4 / 8.1 at 500, 15.8 / 11.9 / 12.6 at 900, 19.0 / 16.8 / 16.8 at 1300, 20.2 / 22.1 / 20.8 at 1550, 20.8 / 23.0 / 21.0 at 1700 (C = 5 14.9 / 16.2 / 15.4,
        // C = 16 36.2 / 40.9 / 37.8), 28.9 / 28.3 / 26.6 at 2200; d = 8192 37.6 / 39.6 / 38.5 at 1550, 62.2 / 53.2 / 49.9 at 2200.
        bits = t <= 700 ? 2 : t <= 1500 ? 1 : t <= 1900 ? 0 : 2;
    // Never more units than checkpoints: a unit requests its first row before it looks whether there is another.
    // Two or three checkpoints: two units at most, and one where many waves would only be the better balanced (d = 4096, C = 3: 17.2 / 17.5 at 3000).
    return C >= 4 ? bits : bits == 2 && t > 1500 && row_chunks > 256 ? 0 : std::min(bits, 1);
}
}  // namespace

int tide_cosine_labels(const void* hidden, int dtype, int64_t C, int64_t T, int64_t d, int64_t ckpt_stride,
                       int64_t row_stride, const void* final_hidden, int64_t final_row_stride, float tau, float* sim,
                       uint8_t* label, void* stream) {
    g_err[0] = 0;
    int rc = check_common(hidden, dtype, C, T, d, kBottleneck, ckpt_stride, row_stride, hidden, reinterpret_cast<const float*>(hidden), 0.0f, true);
    if (rc) return rc;
    if (T == 0) return TIDE_OK;
    if (!final_hidden) return fail(TIDE_ERR_INVALID_ARG, "final_hidden must not be NULL");
    if (final_row_stride < d) return fail(TIDE_ERR_INVALID_ARG, "final_row_stride %lld < d", (long long)final_row_stride);
    const size_t eb = elem_bytes(dtype);
    if (((uintptr_t)final_hidden & 15) || ((size_t)final_row_stride * eb & 15))
        return fail(TIDE_ERR_ALIGNMENT, "final_hidden base and stride must be multiples of 16 bytes");
    const int64_t row_bytes = d * (int64_t)eb;
    if (row_bytes > (int64_t)kCosineMaxChunks * 16 * kCosineThreads)
        return fail(TIDE_ERR_UNSUPPORTED, "rows of %lld bytes exceed the labeler's limit", (long long)row_bytes);
    CosineParams p;
    std::memset(&p, 0, sizeof(p));
    p.hidden = (const char*)hidden;
    p.ckpt_stride_bytes = ckpt_stride * (int64_t)eb;
    p.row_stride_bytes = row_stride * (int64_t)eb;
    p.final_hidden = (const char*)final_hidden;
    p.final_row_stride_bytes = final_row_stride * (int64_t)eb;
    p.C = (int)C;
    p.T = (int)T;
    p.d = (int)d;
    p.tau = tau;
    p.sim = sim;
    p.label = label;
    const bool wave_per_row = row_bytes <= (int64_t)kCosineMaxChunks * 16 * kWave;
    const int64_t row_chunks = row_bytes / 16;
    unsigned cus = 0;
    if ((rc = resident_cus(&cus))) return rc;
    p.group_bits = label_unit_bits(wave_per_row, row_chunks, C, T, cus);
    const int64_t units = T << p.group_bits;
    const unsigned grid = wave_per_row ? (unsigned)((units + 3) / 4) : (unsigned)(((T + 7) / 8 * 8) << p.group_bits);
    const int64_t per_thread = (row_chunks + (wave_per_row ? kWave : kCosineThreads) - 1) / (wave_per_row ? kWave : kCosineThreads);
    hipStream_t st = (hipStream_t)stream;
    by_dtype(dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        static_assert(TIDE_MAX_CHECKPOINTS < 1 << 16, "the fields of ckpts");
        auto go = [&](auto wpr, auto chunks) {
            hipLaunchKernelGGL((tide_cosine_kernel<DT, decltype(wpr)::value, decltype(chunks)::value>), dim3(grid),
                               dim3(kCosineThreads), 0, st, p.hidden, p.ckpt_stride_bytes, p.row_stride_bytes, p.final_hidden, p.final_row_stride_bytes, p.T, p.d,
                               (uint32_t)p.C | (uint32_t)p.group_bits << 16, p);
        };
        auto pick = [&](auto wpr) {
            if (per_thread <= 2) go(wpr, std::integral_constant<int, 2>{});
            else if (per_thread <= 3) go(wpr, std::integral_constant<int, 3>{});
            else if (per_thread <= 4) go(wpr, std::integral_constant<int, 4>{});
            else if (per_thread <= 5) go(wpr, std::integral_constant<int, 5>{});
            else if (per_thread <= 6) go(wpr, std::integral_constant<int, 6>{});
            else if (per_thread <= 8) go(wpr, std::integral_constant<int, 8>{});
            else if (per_thread <= 10) go(wpr, std::integral_constant<int, 10>{});
            else if (per_thread <= 12) go(wpr, std::integral_constant<int, 12>{});
            else go(wpr, std::integral_constant<int, 16>{});
        };
        if (wave_per_row) pick(std::true_type{});
        else pick(std::false_type{});
        return 0;
    });
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

int tide_batch_exit(const uint32_t* fire_mask, int64_t T, int64_t C, const int32_t* layer_ids, int32_t min_layer,
                    int32_t no_exit_layer, int32_t* batch_exit_layer, uint32_t* all_fire_mask, uint32_t* fire_counts,
                    void* stream) {
    g_err[0] = 0;
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS) return fail(TIDE_ERR_INVALID_ARG, "C = %lld outside [1, 32]", (long long)C);
    if (T < 0 || T > (int64_t)1 << 30) return fail(TIDE_ERR_INVALID_ARG, "T = %lld outside [0, 2^30]", (long long)T);
    if (T == 0) return TIDE_OK;
    if (!fire_mask || !layer_ids || !batch_exit_layer)
        return fail(TIDE_ERR_INVALID_ARG, "fire_mask, layer_ids (host) and batch_exit_layer must not be NULL");
    BatchParams p;
    std::memset(&p, 0, sizeof(p));
    for (int64_t c = 0; c < C; ++c) {
        if (c > 0 && layer_ids[c] <= layer_ids[c - 1])
            return fail(TIDE_ERR_INVALID_ARG, "layer_ids must be strictly ascending");
        p.layer_id[c] = layer_ids[c];
    }
    std::lock_guard<std::mutex> lock(g_mu);
    Workspace* ws = nullptr;
    int rc = current_workspace(&ws);
    if (rc) return rc;
    if ((rc = claim_workspace(*ws, (hipStream_t)stream))) return rc;
    constexpr unsigned kMaxBlocks = 256;
    rc = reserve(ws->batch, (kMaxBlocks * 32 + 1) * sizeof(uint32_t), true);
    if (rc) return rc;
    p.fire_mask = fire_mask;
    p.T = (int)T;
    p.C = (int)C;
    p.min_layer = min_layer;
    p.no_exit = no_exit_layer;
    p.batch_exit_layer = batch_exit_layer;
    p.all_fire_mask = all_fire_mask;
    p.fire_counts = fire_counts;
    p.counter = (uint32_t*)ws->batch.ptr;
    p.partial = p.counter + 1;
    unsigned grid = (unsigned)((T + 4 * kBatchThreads - 1) / (4 * kBatchThreads));
    grid = grid > kMaxBlocks ? kMaxBlocks : grid;
    hipLaunchKernelGGL(tide_batch_exit_kernel, dim3(grid), dim3(kBatchThreads), 0, (hipStream_t)stream, p);
    TIDE_HIP(hipGetLastError());
    return TIDE_OK;
}

int tide_set_variant(int variant) {
    if (variant != TIDE_VARIANT_AUTO && variant != TIDE_VARIANT_PREFILL && variant != TIDE_VARIANT_DECODE)
        return fail(TIDE_ERR_INVALID_ARG, "variant %d is not a tide_variant_t", variant);
    std::lock_guard<std::mutex> lock(g_mu);
    int prev = g_variant;
    g_variant = variant;
    return prev;
}

namespace {
// A prefill form word: the form in bits 0-7; with forms 5 and 8, optionally a forced split-k tile height
// (bits 8-15: 0, 32, 64 or 128; form 8: 0 or 32) and slice count (bits 16-23: 0, 2, 4 or 8).
bool valid_form_word(int w) {
    const int form = w & 0xff, rows = (w >> 8) & 0xff, slices = (w >> 16) & 0xff;
    if (w < 0 || (w >> 24) != 0 || form > 9) return false;
    if ((rows || slices) && form != 5 && form != 8) return false;
    if (form == 8 && rows != 0 && rows != 32) return false;
    return (rows == 0 || rows == 32 || rows == 64 || rows == 128) && (slices == 0 || slices == 2 || slices == 4 || slices == 8);
}
}  // namespace

int tide_prefill_plan(int dtype, int64_t C, int64_t T, int64_t d, int64_t b, int cus, int form, int32_t* out) {
    if (dtype != TIDE_F32 && dtype != TIDE_F16 && dtype != TIDE_BF16) return fail(TIDE_ERR_INVALID_ARG, "dtype %d is not a tide_dtype_t", dtype);
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS || T < 1 || C * T > (int64_t)1 << 30) return fail(TIDE_ERR_INVALID_ARG, "C = %lld, T = %lld out of range", (long long)C, (long long)T);
    if (!supported_hidden(dtype, d) || !supported_bottleneck(b)) return fail(TIDE_ERR_UNSUPPORTED, "d = %lld, b = %lld unsupported", (long long)d, (long long)b);
    if (needs_repack(dtype, d, b)) d = padded_hidden(dtype, d);      // such calls run the tuned kernels on zero-padded rows
    if (cus < 8 || cus % 8 != 0) return fail(TIDE_ERR_INVALID_ARG, "cus = %d must be a positive multiple of 8", cus);
    if (!valid_form_word(form)) return fail(TIDE_ERR_INVALID_ARG, "prefill form %d: a form in [0, 8], with forms 5 and 8 optionally rows << 8 | slices << 16", form);
    if (!out) return fail(TIDE_ERR_INVALID_ARG, "out must not be NULL");
    const PrefillPlan plan = call_plan(dtype, C, T, d, b, (unsigned)cus, TIDE_VARIANT_AUTO, form, true);
    for (int i = 0; i < plan.count; ++i) {
        const PlannedLaunch& L = plan.launch[i];
        int32_t* o = out + 7 * i;
        o[0] = L.kernel; o[1] = L.rows_per_tile; o[2] = L.tiles_per_ckpt; o[3] = L.total_tiles; o[4] = L.tile_begin; o[5] = L.k_slices;
        o[6] = (int32_t)L.grid;
    }
    return plan.count;
}

int tide_stream_schedule(int rows_per_tile, int64_t b, int64_t k_tiles, int grid, int block, int tile_begin, int total_tiles,
                         int32_t* out, int max_items) {
    if (rows_per_tile != 64 && rows_per_tile != 128) return fail(TIDE_ERR_INVALID_ARG, "rows_per_tile = %d: 64 or 128", rows_per_tile);
    if (!supported_bottleneck(b) || k_tiles < 1) return fail(TIDE_ERR_INVALID_ARG, "b = %lld, k_tiles = %lld", (long long)b, (long long)k_tiles);
    if (grid < 8 || grid % 8 != 0 || block < 0 || block >= grid) return fail(TIDE_ERR_INVALID_ARG, "grid = %d (a multiple of 8), block = %d", grid, block);
    if (tile_begin < 0 || tile_begin > total_tiles || !out || max_items < 0) return fail(TIDE_ERR_INVALID_ARG, "tile range / out");
    const int ntile = halves_of(b) == 2 ? 1 : (int)k_tiles;          // the two-halves kernel never cuts tiles
    int n = 0;
    auto emit = [&](const WorkItem& it) {
        if (n < max_items) { out[3 * n] = it.tile; out[3 * n + 1] = it.row_off; out[3 * n + 2] = it.blocks * 32; }
        ++n;
    };
    if (rows_per_tile == 128) {
        for (TileWalk<4> w(block, grid, tile_begin, total_tiles, ntile); w.valid(); w.advance()) emit(w.current());
    } else {
        for (TileWalk<2> w(block, grid, tile_begin, total_tiles, ntile); w.valid(); w.advance()) emit(w.current());
    }
    return n;
}

int tide_band_schedule(int64_t C, int64_t blocks_per_ckpt, int grid, int block, int32_t* out, int max_items) {
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS || blocks_per_ckpt < 1 || C * blocks_per_ckpt > (int64_t)1 << 30)
        return fail(TIDE_ERR_INVALID_ARG, "C = %lld, blocks_per_ckpt = %lld out of range", (long long)C, (long long)blocks_per_ckpt);
    if (grid < 8 || grid % 8 != 0 || block < 0 || block >= grid) return fail(TIDE_ERR_INVALID_ARG, "grid = %d (a multiple of 8), block = %d", grid, block);
    if (!out || max_items < 0) return fail(TIDE_ERR_INVALID_ARG, "out / max_items");
    int n = 0;
    for (BandWalk w(block, grid, (int)C, (int)blocks_per_ckpt, band_per_ckpt(C, blocks_per_ckpt, grid)); w.valid(); w.advance()) {
        const BandTile t = w.current();
        if (n < max_items) { out[3 * n] = t.c; out[3 * n + 1] = t.block0; out[3 * n + 2] = t.blocks; }
        ++n;
    }
    return n;
}

int tide_band_f32_schedule(int64_t C, int64_t blocks_per_ckpt, int grid, int block, int32_t* out, int max_items) {
    if (C < 1 || C > TIDE_MAX_CHECKPOINTS || blocks_per_ckpt < 1 || C * blocks_per_ckpt > (int64_t)1 << 30)
        return fail(TIDE_ERR_INVALID_ARG, "C = %lld, blocks_per_ckpt = %lld out of range", (long long)C, (long long)blocks_per_ckpt);
    if (grid < C || grid % 8 != 0 || block < 0 || block >= grid) return fail(TIDE_ERR_INVALID_ARG, "grid = %d (a multiple of 8, at least C), block = %d", grid, block);
    if (!out || max_items < 0) return fail(TIDE_ERR_INVALID_ARG, "out / max_items");
    int n = 0;
    auto emit = [&](auto walk) {
        for (; walk.valid(); walk.advance()) {
            const BandTile t = walk.current();
            if (n < max_items) { out[3 * n] = t.c; out[3 * n + 1] = t.block0; out[3 * n + 2] = t.blocks; }
            ++n;
        }
    };
    if (band32_max_blocks((int)C, (int)blocks_per_ckpt, grid) == 4) emit(Band32Walk<4>(block, grid, (int)C, (int)blocks_per_ckpt));
    else emit(Band32Walk<8>(block, grid, (int)C, (int)blocks_per_ckpt));
    return n;
}

int tide_set_prefill_form(int form) {
    if (!valid_form_word(form)) return fail(TIDE_ERR_INVALID_ARG, "prefill form %d: a form in [0, 8], with forms 5 and 8 optionally rows << 8 | slices << 16", form);
    std::lock_guard<std::mutex> lock(g_mu);
    int prev = g_prefill_form;
    g_prefill_form = form;
    return prev;
}

int tide_release(void) {
    g_err[0] = 0;
    std::lock_guard<std::mutex> lock(g_mu);
    Workspace* ws = nullptr;
    int rc = current_workspace(&ws);
    if (rc) return rc;
    TIDE_HIP(hipDeviceSynchronize());
    for (Buffer* b : {&ws->counters, &ws->arrive, &ws->packed, &ws->part, &ws->rows, &ws->batch, &ws->compact}) {
        if (b->ptr) TIDE_HIP(hipFree(b->ptr));
        b->ptr = nullptr;
        b->bytes = 0;
    }
    for (SizedShape& s : ws->sized) s = SizedShape{};
    ws->used = false;
    ws->dirty = false;
    return TIDE_OK;
}

}  // extern "C"

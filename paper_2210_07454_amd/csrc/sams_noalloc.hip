// topk_refine_static: the second round's final selection (topk_refine of sams.h) for callers that cannot
// allocate device memory -- code under HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.
// It needs no context: the scratch the selection kernels use (listed keys, radix histograms,
// selection state, per-tile counts and ranks) lives in a file-scope __device__ array that every GPU the
// library runs on holds until the process ends.  The kernels are the ones topk_refine launches; they receive the
// array's device address as an ordinary argument.
#include <mutex>

#include "sams_ctx.h"

namespace sams {

constexpr int64_t kStaticMaxCand = SAMS_STATIC_MAX_CANDIDATES;
constexpr int64_t kStaticTiles = (kStaticMaxCand >> 12) + 1;         // sel_tiles(kStaticMaxCand)
constexpr int kStaticMaxDevices = 64;

// layout of the scratch, in bytes from its start (every part 256-byte aligned)
constexpr size_t align256(size_t x) { return (x + 255) / 256 * 256; }
constexpr size_t kOffVal = 0;                                                        // SelList::val
constexpr size_t kOffLoc = align256(kOffVal + (size_t)(kStaticMaxCand + 64) * 4);    // SelList::loc
constexpr size_t kOffTile = align256(kOffLoc + (size_t)(kStaticMaxCand + 64) * 2);   // SelList::group, cnt
constexpr size_t kOffSel = align256(kOffTile + (size_t)3 * kStaticTiles * 4);        // SelState, then the histograms
constexpr size_t kStaticBytes = kOffSel + (size_t)kSelWords * 4;

// In host code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

static std::mutex g_static_mutex;
static void *g_static_ptr[kStaticMaxDevices];       // device address of `scratch` on each device, once resolved

// Device address of the scratch on the current device (resolved once per device, with that device current).
int static_scratch_ptr(void **out)
{
    int dev = -1;
    SAMS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kStaticMaxDevices) return SAMS_EINVAL;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        SAMS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return SAMS_EHIP;
        g_static_ptr[dev] = p;
    }
    *out = g_static_ptr[dev];
    return SAMS_OK;
}

}  // namespace sams

using namespace sams;

extern "C" {

int64_t topk_refine_static_max_candidates(void) { return kStaticMaxCand; }

int topk_refine_static(const int32_t *idx_in, const float *delta_in, int64_t k_in, int64_t k_out, int32_t *idx_out,
                       float *delta_out, void *hip_stream)
{
    if (!idx_in || !delta_in || !idx_out || !delta_out) return SAMS_EINVAL;
    if (k_in < 1 || k_in > kStaticMaxCand || k_out < 1 || k_out > k_in) return SAMS_EINVAL;
    if (!aligned16(idx_in) || !aligned16(delta_in) || !aligned16(idx_out) || !aligned16(delta_out)) return SAMS_EINVAL;
    void *p = nullptr;
    SAMS_TRY(static_scratch_ptr(&p));
    unsigned char *b = static_cast<unsigned char *>(p);
    uint32_t *tile = reinterpret_cast<uint32_t *>(b + kOffTile), *sel = reinterpret_cast<uint32_t *>(b + kOffSel);
    const SelScratch sc = {reinterpret_cast<SelState *>(sel), sel + kSelStateWords, sel + kSelClearWords,
                           {reinterpret_cast<uint32_t *>(b + kOffVal), reinterpret_cast<uint16_t *>(b + kOffLoc),
                            tile + 2 * kStaticTiles, reinterpret_cast<uint2 *>(tile)},
                           kStaticTiles, kStaticMaxCand, true};
    return enqueue_select(nullptr, (hipStream_t)hip_stream, sc, delta_in, k_in, k_out, idx_in, idx_out, delta_out, false);
}

}  // extern "C"

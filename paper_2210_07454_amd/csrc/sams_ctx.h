// Internal header of the HIP library: the context, error plumbing, launch/timing helpers and the
// declarations of the per-stage enqueue functions (one .hip file per stage group).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sams.h"
#include "sams_hash.h"

namespace sams {

extern int g_last_hip_error;

#define SAMS_HIP(expr)                                  \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) {                         \
            ::sams::g_last_hip_error = (int)e_;         \
            return SAMS_EHIP;                           \
        }                                               \
    } while (0)

#define SAMS_TRY(expr)                                  \
    do {                                                \
        int rc_ = (expr);                               \
        if (rc_ != SAMS_OK) return rc_;                 \
    } while (0)

constexpr int kWave = 64;
constexpr int64_t kPlanMinRecoveryC = 1 << 15;   // buckets above which a context that pushes recovers through a plan
constexpr int64_t kOrderedSingleBinMaxD = (int64_t)1 << 22;     // largest d sketched in order when c fits one window
constexpr int kHistBins = 2048;     // first radix digit of the selection: 11 bits, then 10 and 10 (kHistBins / 2 bins)
constexpr int kSelTileLog2 = 12;    // keys per tile of the filters: 1024 threads, 4 each
constexpr int kSelMaxTiles = 16;    // kSelSmallMax keys
constexpr int kSelFlatTiles = 256;       // tiles whose lists one workgroup may finish a selection from
constexpr int64_t kSelFlatMax = (int64_t)kSelFlatTiles << kSelTileLog2;
constexpr int64_t kSelSmallMax = 1 << 16;   // keys up to which the selection is one launch after the first histogram (for small k)

// device-resident state of the radix selection (no host round trip inside a step).  A selection starts from histograms and
// `done` of zeros and leaves them so (up to 2^16 keys, after a pass of its own over the keys, it needs none); the next one
// clears them first where one failed half-way (sams_ctx::sel_open), and topk_refine_static always does
struct SelState {
    uint32_t prefix[3];   // key bits decided after each digit: the top bits of the k-th largest |key| pattern (prefix[2]: all 31)
    uint32_t k_rem[3];    // how many keys to take among those that match the prefix (k_rem[2]: how many equal to the k-th largest)
    uint32_t done[4];     // workgroups that have finished, per launch of the selection that asks for the last one
};

// kernels, for the optional per-kernel timing (sams_profile_*)
enum KernelId {
    KID_FILL = 0, KID_HASH_DUMP, KID_TAIL, KID_TAIL_ZERO_E, KID_HEAD, KID_SKETCH_ATOMIC, KID_REDUCE,
    KID_ESTIMATE, KID_SEL_HIST, KID_SEL_FILTER, KID_SEL_COUNT, KID_SEL_WRITE,
    KID_GATHER, KID_PLAN_BUILD, KID_BIN_SCATTER, KID_BIN_ACCUMULATE, KID_SKETCH_LDS, KID_BIN_LOOKUP,
    KID_BIN_COLLECT, KID_EST_MEDIAN, KID_HEAD_SCATTER, KID_HEAD_PA, KID_HEAD_SPARSE_V, KID_SEL_SMALL, KID_SKETCH_PULL, KID_PULL_SUM, KID_SKETCH_PUSH, KID_COUNT
};
const char *kernel_name(int kid);

constexpr int kMaxWorkers = 1024;     // n accepted by sams_create
constexpr int kWideCoords = 8;        // coordinates per workgroup of the 32-lanes-per-coordinate sparse kernels
constexpr int kWideMinWorkers = 16;   // ... which are used from this many workers on
constexpr int kProfPool = 8192;   // event pairs kept for one profiling window

struct ProfRec {
    hipEvent_t a, b;
    int kid;
};

// how sketch_accumulate is carried out for this context (chosen at creation from c and the tunables)
enum PlanMode { PLAN_ATOMIC = 0, PLAN_LDS_ROW = 1, PLAN_BINNED = 2 };

// static permutation "coordinate order -> bucket order" of the binned path (see sams_plan.hip)
struct Plan {
    int mode;
    int acc_variant;    // pass 2 of the rows that read meta words: 0 = 4-byte loads, 1 = 16-byte loads; 2 = no such row (all rows read chunk records)
    uint32_t rec_mask;  // bit j set: row j reads chunk records in pass 2 (k_bin_accumulate_r)
    int win_log2, tile_log2, chunk_log2, acc_threads, run_pad, grp_log2, rows, stage_rows, stage_ilv, acc_wide;
    int64_t nbins, ntile, dpad, rowlen;
    int64_t stg_words;  // floats of the staging buffer
    int64_t stg_rows;   // rows of rowlen floats that the staging holds: n * stage_rows, or r where only the recovery goes through the plan
    uint16_t *srcp;     // [r][rowlen]      slot -> coordinate inside its tile (bits 0-14) and sign (bit 15), or padding
    uint32_t *dst16;    // [r][rowlen >> grp_log2]  stream position of each group of 2^grp_log2 slots (16, or the run padding if smaller)
    uint32_t *pbase;    // [r][ntile+1]     first slot of each tile
    uint32_t *binbase;  // [r][nbins+1]     start of each bin in the row stream (multiples of the chunk)
    uint32_t *meta;     // [r][rowlen]          per stream position: bucket in window, chain link, flags (absent with acc_variant 2)
    uint32_t *rec;      // [r][rowlen/4096][2560] chunk records of acc_variant 2: 4096 16-bit codes, 512 chain entries
    uint16_t *wlow;     // [r][rowlen]          per stream position: bucket in window only (what the recovery reads)
    void *stg_chunks;   // staging mapped from physical chunks picked all over device memory (stage_spread): their handles, else null
    int64_t stg_nchunks, stg_va_bytes;
    float *stg;         // n * stage_rows * rowlen floats: per-step staging, signed values at their stream positions
                        //                      ([stage_rows][rowlen/32][n][32], or [n][stage_rows][rowlen] without stage_ilv)
    const float *staged_u;  // vector whose sorted copy the staging holds (set by a fused head), else null
    float *rowest;      // [r][d]               per-step: signed row estimates in coordinate order (stage 3);
                        //                      absent when the median is fused (fused_median)
    bool fused_median;  // stage 3 keeps the row estimates in registers (decided when the plan is built)
};

struct PullOrder;
struct PullRow {
    int32_t win0, per_win, per_wave;   // windows of the rows before; lists per window, per wavefront
};
// the lists of the pulling form of the order-preserving path (see sams_pull.hip); kernel == null: this context does not pull
struct PullPlan {
    const void *kernel;
    struct PullOrder *po;         // where a wavefront's lists are (host memory)
    int32_t parts;                // parts of the vector that workgroups share out
    uint2 *first;                 // per stream, a wavefront's lists: its first load of words, its units
    uint32_t *lists;              // [loads][64][4]  words of two entries
    float *part_sums;             // [parts][n][r][c], with more than one part
    int64_t list_bytes, first_bytes;
};

// the lists of words of the path that picks its values out of the vector (see sams_push.hip); words == null: this context does not take it
struct PushPlan {
    int32_t nwin, win;            // windows of a row, buckets of a window
    int32_t span, nph, nalloc;    // coordinates of a phase, phases, phases that a list has room for
    uint32_t *words;              // [r * nwin][nalloc][2048]
    int32_t share;                // units of an XCD's turn
    int32_t ncopy;                // sorted copies of the vectors that the values are picked from (0: the vectors themselves)
    int8_t copy_of[SAMS_MAX_ROWS], row[SAMS_MAX_ROWS];     // a row's copy; the order in which the rows are worked on
    const void *kernel;
    uint16_t *order;              // [ncopy][nph][span]  the coordinate, in its phase, that lies in a place of a copy
    int64_t copy_words;           // floats of the copies, in the plan's staging buffer
    int64_t word_bytes, order_bytes;
};

// what a context that pushes would take (push_estimate)
struct PushChoice {
    double ns;                    // time of a sketch; 1e30: it does not push
    int32_t windows;              // of a row
    bool copies;
    uint32_t repeat[SAMS_MAX_ROWS];       // rows' shortest distances after which buckets repeat
};

// tunables: sams_configure edits the process-wide set, sams_create copies it into the context, and every
// later call on that context reads only its own copy
struct Tunables {
    int tile_log2;     // coordinates per tile of the binned path (0 = chosen from d)
    int win_log2;      // buckets per LDS window
    int chunk_log2;    // stream positions between two barriers of the accumulate kernel
    int acc_threads;   // workgroup size of the accumulate kernel
    int sketch_path;   // 0 = choose from c and d, 1 = global atomics, 2 = ordered (binned) always, 3 = LDS atomics when c fits a window
    int scatter_threads;  // workgroup size of the scatter kernel
    int estimate_path;    // stage 3: 0 = through the plan when there is one, unless table and vector are small; 1 = direct gathers from the table; 2 = through the plan
    int fuse_head;        // 1, 2 = amsgrad_ef_update also stages u for the next sketch_accumulate (2: a workgroup per worker)
    int fuse_median;      // 1 = recovery keeps the row estimates in registers where the shape allows, 0 = through memory
    int stage_rows;       // rows staged at once (0 = all r): bounds the staging buffer at n*stage_rows*rowlen floats
    int run_pad;          // runs are padded to a multiple of this many stream positions (4, 8, 16 or 32)
    int stage_interleave; // 1 = the workers' staged copies are interleaved in pieces of 32 stream positions
    int stage_spread;     // 1 = a staging buffer of 2 GiB or more is mapped from 1 GiB chunks picked at even distances over all free device memory
    int pull_lists;       // lists of the pulling path: 0 = chosen; 1 = one of a slice per wavefront, 2 = up to two, 4 = up to four of four slices
    int push_windows;     // windows of a row of the path that picks its values out of the vectors (sams_push.hip): 0 = chosen, -1 = not that path,
                          // 1 to 16 = so many, 101 to 116 = so many, out of sorted copies
    int acc_wide;         // accumulate kernel where its shape allows (1024 threads, 2048-position chunks): 1 = 16-byte loads,
                          // 2 = 16-byte loads and compact chunk records instead of meta words (falls back to 1 when a chunk has too many chains)
};
extern Tunables g_tun;

// the keys a selection has listed (k_sel_filter), and what is known per tile of keys.  Without room for lists the keys
// themselves take their place: cnt and loc null, every key of a tile listed
struct SelList {
    uint32_t *val;           // [cap + 64]  a listed key's bits (sign included), tile after tile, each from the tile's first position on
    uint16_t *loc;           // [cap + 64]  its position inside the tile
    uint32_t *cnt;           // [ntile_cap]  listed keys per tile
    uint2 *group;            // [ntile_cap]  per workgroup of k_sel_count: keys above the threshold, keys equal to it
};

// scratch of one radix selection (enqueue_select): the context's, or the static one of topk_refine_static
struct SelScratch {
    SelState *st;
    uint32_t *hist;          // [2 * kHistBins]  first digit, then second, then third
    uint32_t *tile_hist;     // [kSelMaxTiles][kHistBins / 2]  up to 2^16 keys: first digit tile by tile, two bins of 16 bits a word
    SelList list;
    int64_t ntile_cap, cap;  // tiles, and keys that the lists have room for
    bool shared;             // by several streams: what the selection before has left in st and hist is not relied on
};
constexpr int64_t kSelHistPickMin = (int64_t)1 << 20;                // above, the kernel that takes the first histogram picks its digit
constexpr int64_t kSelStateWords = 64;                               // words of SelState, rounded up; the histograms follow it
constexpr int64_t kSelClearWords = kSelStateWords + 2 * kHistBins;   // what a selection starts from as zeros
constexpr int64_t kSelWords = kSelClearWords + kSelMaxTiles * kHistBins / 2;   // the tiles' histograms after it
static_assert(sizeof(SelState) <= kSelStateWords * 4, "selection state");
// tiles for which the per-tile arrays need room when up to len keys are selected from: of 4096 keys, at least 256
static inline int64_t sel_tiles(int64_t len) { return (len >> 12) + 1 > 256 ? (len >> 12) + 1 : 256; }

}  // namespace sams

struct sams_ctx {
    int64_t d, c, k;
    int32_t n, r;
    hipStream_t stream;
    sams::HashParams hp;
    // scratch (device)
    float *est;              // [d]
    uint32_t *bitmap;        // [ceil(d/32)]  bit l set <=> l in the most recent index set
    uint32_t *wordrank;      // [ceil(d/32)]  for a bitmap word with a bit set: the rank (position in idx) of its first set bit;
                             //               with gsel, only where the head is fused per worker (fuse_head = 2), else null
    float *gsel;             // [n][k]        g of every worker at the coordinates of the most recent index set, by rank
    uint32_t *sel;           // [kSelWords]  SelState, then SelScratch::hist and tile_hist
    bool sel_open;           // a selection was begun and not enqueued whole: the next one clears `sel` first
    uint32_t *sel_tile;      // [3][sel_tiles(d)]  SelList::group, cnt
    uint32_t *sel_list;      // SelList::val and loc when the staging buffer is absent or too small to hold them, else null
    int64_t sel_cap;         // keys that the lists have room for: d, or less where device memory was short
    int64_t scratch_bytes;
    sams::Plan plan;
    sams::PullPlan pull;
    sams::PushPlan push;
    sams::Tunables tun;      // the tunables as they were when the context was created
    // per-kernel timing (host)
    int prof_on;
    int prof_only;           // kernel id the timing is restricted to, -1 = every kernel
    int prof_used;
    sams::ProfRec *prof;     // [kProfPool], events created on first enable
    double prof_ms[sams::KID_COUNT];
    int64_t prof_n[sams::KID_COUNT];
};

namespace sams {

static inline int grid_for(int64_t work, int block, int64_t cap = (int64_t)1 << 30)
{
    int64_t g = (work + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

static inline bool aligned16(const void *p) { return (((uintptr_t)p) & 15u) == 0; }

// Brackets one kernel launch with a HIP event pair on the context's stream while profiling is on.
struct ProfScope {
    sams_ctx *ctx;
    int slot;
    ProfScope(sams_ctx *c, int kid) : ctx(c), slot(-1)
    {
        if (c && c->prof_on && (c->prof_only < 0 || c->prof_only == kid) && c->prof_used < kProfPool) {
            slot = c->prof_used++;
            c->prof[slot].kid = kid;
            (void)hipEventRecord(c->prof[slot].a, c->stream);
        }
    }
    ~ProfScope()
    {
        if (slot >= 0) (void)hipEventRecord(ctx->prof[slot].b, ctx->stream);
    }
};

// SAMS_LAUNCH(ctx, KID_X, (kernel<..>), grid, block, args...)
#define SAMS_LAUNCH(ctx, kid, kernel, grid, block, ...)                                          \
    do {                                                                                         \
        ::sams::ProfScope ps_((ctx), (kid));                                                     \
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, (ctx)->stream, __VA_ARGS__);      \
    } while (0)
// the same on a given stream, for code that also runs without a context (ctx may be null: no timing then)
#define SAMS_LAUNCH_ON(ctx, stream, kid, kernel, grid, block, ...)                               \
    do {                                                                                         \
        ::sams::ProfScope ps_((ctx), (kid));                                                     \
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, (stream), __VA_ARGS__);           \
    } while (0)

// median of R row estimates (Sec. II-C); for an even R the lower middle element
template <int R>
__device__ __forceinline__ float median_of(float (&a)[R])
{
    // odd-even transposition network: R rounds sort R values; compile-time unrolled
#pragma unroll
    for (int round = 0; round < R; ++round) {
#pragma unroll
        for (int p = (round & 1); p + 1 < R; p += 2) {
            float lo = a[p + 1] < a[p] ? a[p + 1] : a[p];
            float hi = a[p + 1] < a[p] ? a[p] : a[p + 1];
            a[p] = lo;
            a[p + 1] = hi;
        }
    }
    return a[(R - 1) / 2];
}

// inclusive prefix sum over the 64 lanes, in registers: six adds through the data-parallel primitives (row shifts by 1, 2,
// 4, 8 inside rows of 16, then the row totals broadcast), where shuffles would each cost a trip through the LDS crossbar
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
    return x;
}

// exclusive prefix sum over the N threads of a block (part: at least N / 64 words of LDS; all threads call it):
// a scan inside every wavefront, then the wavefronts' totals through LDS
template <int N>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t val, uint32_t *part)
{
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t incl = wave_inclusive_scan(val);
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    const uint32_t upto = wave_inclusive_scan(lane < N / kWave ? part[lane] : 0u);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)upto, wave - 1) : 0u;
    __syncthreads();
    return before + incl - val;
}

// accesses to data that other workgroups of the same launch write or read (AGENT: coherent across the XCDs' L2s)
template <bool AGENT, typename T>
__device__ __forceinline__ T get(const T *p)
{
    if constexpr (AGENT) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}
template <bool AGENT, typename T>
__device__ __forceinline__ void put(T *p, T v)
{
    if constexpr (AGENT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// True in every thread of the workgroup that comes here last of the nblk of its launch; nobody waits.  The agent-scope
// accesses and atomics that the workgroups have issued before are complete by then.  *done goes back to 0.
// sh: a word of LDS.
__device__ __forceinline__ bool last_workgroup(uint32_t *done, uint32_t nblk, uint32_t *sh)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // this wavefront's stores and atomics have been performed
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t before = atomicAdd(done, 1u);
        if (before == nblk - 1) put<true>(done, 0u);
        *sh = before;
    }
    __syncthreads();
    return *sh == nblk - 1;
}

// The digit in which the k_rem-th largest key lies, from the histogram count(bin) of NB bins: exactly one thread calls
// sink(digit, number of keys in higher bins, in this one), since k_rem <= the number of keys.  Thread t looks at NB / THREADS
// consecutive bins counted from the top.
template <int THREADS, int NB, typename C, typename S>
__device__ __forceinline__ void pick_digit(C count, uint32_t k_rem, S sink, uint32_t *part)
{
    constexpr int PER = NB / THREADS;
    const int top = NB - 1 - (int)threadIdx.x * PER;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int z = 0; z < PER; ++z) v[z] = count(top - z);
#pragma unroll
    for (int z = 0; z < PER; ++z) sum += v[z];
    uint32_t above = block_exclusive_scan<THREADS>(sum, part);
#pragma unroll
    for (int z = 0; z < PER; ++z) {
        if (above < k_rem && k_rem <= above + v[z]) sink((uint32_t)(top - z), above, v[z]);
        above += v[z];
    }
}

// One workgroup picks a digit from its complete global histogram, clears that histogram and leaves the prefix and the
// remaining count in the state, and in picked[2] (LDS; complete after the next barrier).  k: for digit 0, the number of
// keys to select.  part: THREADS / 64 words of LDS.
template <int THREADS>
__device__ __forceinline__ void sel_pick(SelState *st, uint32_t *hist, int digit, uint32_t k, uint32_t *part, uint32_t *picked)
{
    const uint32_t prefix_in = digit == 0 ? 0u : st->prefix[digit - 1];
    const uint32_t k_rem = digit == 0 ? k : st->k_rem[digit - 1];
    auto count = [&](int b) {
        const uint32_t x = get<true>(hist + b);
        hist[b] = 0u;
        return x;
    };
    const int width = digit == 0 ? 11 : 10;
    auto sink = [&](uint32_t b, uint32_t above, uint32_t) {
        const uint32_t prefix = (prefix_in << width) | b;
        st->prefix[digit] = picked[0] = prefix;
        st->k_rem[digit] = picked[1] = k_rem - above;
    };
    if (digit == 0) pick_digit<THREADS, kHistBins>(count, k_rem, sink, part);
    else pick_digit<THREADS, kHistBins / 2>(count, k_rem, sink, part);
}

// ---- enqueue functions (all asynchronous on ctx->stream; return SAMS_OK or SAMS_EHIP) ----
int enqueue_fill_u32(sams_ctx *ctx, uint32_t *p, int64_t n, uint32_t val);
int enqueue_fill_u32_on(sams_ctx *ctx, hipStream_t stream, uint32_t *p, int64_t n, uint32_t val);   // ctx may be null: no timing then
int enqueue_hash_dump(sams_ctx *ctx, int32_t *bucket, int8_t *sign);
// sams_update.hip
// the whole update when the head is not fused with the first sketch pass (pa: Alg. 1, v and vhat are [n][d])
int enqueue_update(sams_ctx *ctx, const float *g, float *m, float *e_u, float *v, float *vhat, float *x, const int32_t *idx,
                   const float *delta, int64_t k_sel, float beta1, float beta2, float lr, float rho, bool pa);
// the tail alone: with the bitmap of the index set for a fused head, and with e zeroed there when no head follows
int enqueue_tail(sams_ctx *ctx, float *x, const int32_t *idx, const float *delta, int64_t k_sel, float lr);
int enqueue_tail_only(sams_ctx *ctx, float *e_u, float *x, const int32_t *idx, const float *delta, int64_t k_sel, float lr);
int enqueue_reduce(sams_ctx *ctx, const float *S_workers, float *S_mean);
int enqueue_gather(sams_ctx *ctx, const float *u, const float *vhat, const int32_t *idx,
                   float *U_workers, float *delta);
// sams_sketch.hip
int enqueue_sketch(sams_ctx *ctx, const float *u, float *S_workers);
// sams_pull.hip
int pull_create(sams_ctx *ctx, const Tunables &tun, double limit, bool *done);
void pull_destroy(sams_ctx *ctx);
int enqueue_sketch_pull(sams_ctx *ctx, const float *u, float *S_workers);
// sams_push.hip
// Before push_create: whether this path is taken to pay, and how.  Allocates nothing.
int push_estimate(sams_ctx *ctx, const Tunables &tun, PushChoice *choice);
int push_create(sams_ctx *ctx, const PushChoice &choice, bool *done);
void push_destroy(sams_ctx *ctx);
int enqueue_sketch_push(sams_ctx *ctx, const float *u, float *S_workers);
// sams_plan.hip
int plan_create(sams_ctx *ctx, const Tunables &tun);
void plan_destroy(sams_ctx *ctx);
int copies_create();                                // the sorted copies of the path in sams_push.hip
int enqueue_sort_copies(sams_ctx *ctx, const float *u);
int plan_staging_alone(sams_ctx *ctx);              // the staging buffer, where there are copies but no plan
int64_t plan_staging_words(const sams_ctx *ctx);     // size of the staging buffer in floats, 0 without one
int enqueue_sketch_planned(sams_ctx *ctx, const float *u, float *S_workers);
int enqueue_row_estimates_planned(sams_ctx *ctx, const float *S_mean, float *rowest);
// whole recovery through the plan when the fused collect+median kernel applies; *done says whether it ran
int enqueue_estimates_planned_fused(sams_ctx *ctx, const float *S_mean, const float *vhat, float *est, bool *done,
                                    const SelScratch *sc);   // see enqueue_estimate; *done implies the histogram
// whether the tunables and the vector's length let the head write what the first sketch pass would, and whether this context has that to write
bool head_form_fuses(const Tunables &tun, int64_t d, bool pa);
bool head_can_fuse(const sams_ctx *ctx, bool pa);
// wordrank and gsel exist for this context (sams_create decides): the per-worker fused head then leaves the
// gradients of the selected coordinates in gsel and the second moments on I_{t-1} need no gathers
bool head_compacts_g(const sams_ctx *ctx);
int enqueue_head_scatter(sams_ctx *ctx, const float *g, float *m, float *e_u, float *v, float *vhat,
                         float beta1, float beta2, float rho, bool pa,   // pa: v, vhat are [n][d] (Alg. 1)
                         const int32_t *idx_prev, int64_t k_prev);       // I_{t-1}, as handed to the tail
// sams_select.hip
// whether the kernel that takes the first digit's histogram over len keys also picks the digit (the filter does otherwise)
bool sel_hist_picks(int64_t len);
// whether stage 3 goes through the plan where there is one
bool estimate_wants_plan(const sams_ctx *ctx);
// at creation, once it is known whether there is a plan: what the kernels of enqueue_estimate need set
int estimate_prepare(const sams_ctx *ctx);
// sc != null: a selection of ctx->k from est follows with this scratch; *hist_done tells whether the estimate kernel has
// also taken the histogram of the first radix digit (see sel_hist_picks)
int enqueue_estimate(sams_ctx *ctx, const float *S_mean, const float *vhat, float *est, const SelScratch *sc, bool *hist_done);
// The k of keys[0..len) with the largest magnitude, ties to the smaller position, positions ascending: idx = position, or
// map[position]; val_sel (or null) = the key.  hist_done: see enqueue_estimate.  ctx may be null (no per-kernel timing);
// the work goes to `stream`, the scratch is the caller's.
int enqueue_select(sams_ctx *ctx, hipStream_t stream, const SelScratch &sc, const float *keys, int64_t len, int64_t k,
                   const int32_t *map, int32_t *idx, float *val_sel, bool hist_done);
SelScratch ctx_sel_scratch(const sams_ctx *ctx);
// words of SelList::val and loc together for len keys
static inline int64_t sel_list_words(int64_t len) { return (len + 64) + (len + 64 + 1) / 2; }
// whether the lists of a selection from d keys live in the staging buffer (idle between two sketches)
bool sel_list_in_staging(const sams_ctx *ctx);
// sams_noalloc.hip: device address of the static scratch of topk_refine_static on the current device
int static_scratch_ptr(void **out);

}  // namespace sams

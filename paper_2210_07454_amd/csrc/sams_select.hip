// Stage 3 of the pipeline declared in sams.h: per-coordinate estimates (median over rows, Sec. II-C,
// with the 1/sqrt(vhat) scaling of Alg. 3) and the exact top-k selection of Alg. 2.
#include "sams_ctx.h"

// Every formula below is evaluated as separate IEEE-754 binary32 operations, rounded to nearest:
// no fused multiply-add is formed (here and with -ffp-contract=off on the command line), and
// x / y and sqrtf(x) are the correctly rounded ones (hipcc's default; never build this file with
// -ffast-math or -fno-hip-fp32-correctly-rounded-divide-sqrt).
#pragma clang fp contract(off)

namespace sams {
// ------------------------------------------------------------------------------------------
// stage 3a: per-coordinate estimates (Sec. II-C median, Alg. 3 scaling)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t mag_key(float x) { return __float_as_uint(x) & 0x7fffffffu; }

// What a kernel that takes the histogram of the first digit of |est| does at its end (as k_bin_collect_median): the workgroup's
// histogram to the whole one, and where st is given the last workgroup picks the digit.
__device__ __forceinline__ void hist_finish(uint32_t *lh, uint32_t k, SelState *__restrict__ st, uint32_t *__restrict__ hist)
{
    __syncthreads();
    for (int b = threadIdx.x; b < kHistBins; b += 1024)
        if (lh[b]) atomicAdd(&hist[b], lh[b]);
    if (!st) return;
    __syncthreads();                                                 // lh is free again: a few words for the last workgroup
    if (last_workgroup(&st->done[0], gridDim.x, lh)) sel_pick<1024>(st, hist, 0, k, lh + 32, lh + 2);
}

// HIST: a selection follows, and the histogram of the first digit of |est| is taken here, by workgroups of 1024 threads that walk the
// vector with a fixed step: one per compute unit at most, so that there are few histograms to add up (unsketch_topk with a histogram
// pass of its own, and by up to 128, 256 and 512 workgroups: 110,000 coordinates 24.4, 13.9 us, alike; 431,003 31.6, 21.0, 20.6, 23.0; a
// million 41, 36, 32, 32; four million, 5 x 30,000 114, 139, 107, 109; the first three with fewer launches of the selection too).
constexpr int kEstHistGrid = 256;
template <int R, bool HIST>
__global__ void __launch_bounds__(HIST ? 1024 : 256)
k_estimate(const float *__restrict__ S, const float *__restrict__ vhat, float *__restrict__ est,
           HashParams hp, int64_t d, int64_t c, uint32_t k, SelState *__restrict__ st, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t lh[HIST ? kHistBins : 1];
    if constexpr (HIST) {
        for (int b = threadIdx.x; b < kHistBins; b += 1024) lh[b] = 0;
        __syncthreads();
    }
    const int64_t step = HIST ? (int64_t)gridDim.x * 1024 : d;
    for (int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; l < d; l += step) {
        float a[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            uint32_t b = bucket_of(hp, j, (uint32_t)l);
            float q = S[(int64_t)j * c + b];
            a[j] = sign_neg(hp, j, (uint32_t)l) ? -q : q;
        }
        const float med = median_of<R>(a);
        const float e = vhat ? (med / sqrtf(vhat[l])) : med;
        est[l] = e;
        if constexpr (HIST) atomicAdd(&lh[mag_key(e) >> 20], 1u);
    }
    if constexpr (HIST) hist_finish(lh, k, st, hist);
}

// The same for long vectors and tables that LDS holds at least a row of: a workgroup per compute unit keeps the first
// `held` rows in LDS (the others are gathered as above) and walks the vector with a fixed step, so that a hash value follows
// from the one before: y(l + step) = y(l) + (a step mod p), less p if that is not below it.  The bucket is y less
// floor(y m / 2^32) c, and less c once more if that is not below c, with m = floor(2^32 / c): the quotient is at most one too
// small for y < 2^31.
constexpr int kEstLdsUnroll = 4;
template <int R>
__global__ void __launch_bounds__(1024)
k_estimate_lds(const float *__restrict__ S, const float *__restrict__ vhat, float *__restrict__ est, HashParams hp, int64_t d,
               int32_t c, uint32_t m, int32_t held, uint32_t k, SelState *__restrict__ st, uint32_t *__restrict__ hist)
{
    extern __shared__ float rows[];                                  // [held][c], and with hist a histogram (see k_estimate)
    const int t = threadIdx.x;
    uint32_t *lh = reinterpret_cast<uint32_t *>(rows + held * c);
    if (hist)
        for (int b = t; b < kHistBins; b += 1024) lh[b] = 0;
    for (int q = t; q < held * c; q += 1024) rows[q] = S[q];
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * 1024;
    uint32_t yb[R], ys[R], ab[R], as[R];
    int64_t l = blockIdx.x * (int64_t)1024 + t;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        yb[j] = hash_y(hp.row[j].ah, hp.row[j].bh, (uint32_t)l);
        ys[j] = hash_y(hp.row[j].as, hp.row[j].bs, (uint32_t)l);
        ab[j] = hash_y(hp.row[j].ah, 0u, (uint32_t)step);
        as[j] = hash_y(hp.row[j].as, 0u, (uint32_t)step);
    }
    auto less = [](uint32_t y, uint32_t by) { return y - by < y ? y - by : y; };   // y mod by for y < 2 by
    for (; l < d; l += step * kEstLdsUnroll) {
        float a[kEstLdsUnroll][R], vh[kEstLdsUnroll];
#pragma unroll
        for (int z = 0; z < kEstLdsUnroll; ++z) vh[z] = vhat ? vhat[l + z * step < d ? l + z * step : l] : 1.f;
        uint32_t neg[kEstLdsUnroll] = {};                            // bit j: the row's sign; applied once all loads are under way
#pragma unroll
        for (int j = 0; j < R; ++j) {
            uint32_t b[kEstLdsUnroll];
#pragma unroll
            for (int z = 0; z < kEstLdsUnroll; ++z) {
                b[z] = less(yb[j] - __umulhi(yb[j], m) * (uint32_t)c, (uint32_t)c);
                neg[z] |= (ys[j] & 1u) << j;
                yb[j] = less(yb[j] + ab[j], kP31);
                ys[j] = less(ys[j] + as[j], kP31);
            }
            if (j < held) {                                          // uniform
#pragma unroll
                for (int z = 0; z < kEstLdsUnroll; ++z) a[z][j] = rows[j * c + (int)b[z]];
            } else {
#pragma unroll
                for (int z = 0; z < kEstLdsUnroll; ++z) a[z][j] = S[(int64_t)j * c + b[z]];
            }
        }
#pragma unroll
        for (int z = 0; z < kEstLdsUnroll; ++z)
#pragma unroll
            for (int j = 0; j < R; ++j) a[z][j] = __uint_as_float(__float_as_uint(a[z][j]) ^ (((neg[z] >> j) & 1u) << 31));
#pragma unroll
        for (int z = 0; z < kEstLdsUnroll; ++z) {
            const float med = median_of<R>(a[z]);
            if (l + z * step < d) {
                const float e = vhat ? (med / sqrtf(vh[z])) : med;
                est[l + z * step] = e;
                if (hist) atomicAdd(&lh[mag_key(e) >> 20], 1u);
            }
        }
    }
    if (hist) hist_finish(lh, k, st, hist);
}

// est[l] = median_j(rowest[j][l]) / sqrt(vhat[l]) from row estimates already in coordinate order
template <int R>
__global__ void __launch_bounds__(256)
k_est_median(const float *__restrict__ rowest, const float *__restrict__ vhat, float *__restrict__ est,
             int64_t d)
{
    int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (l >= d) return;
    float a[R];
#pragma unroll
    for (int j = 0; j < R; ++j) a[j] = rowest[(int64_t)j * d + l];
    float med = median_of<R>(a);
    est[l] = vhat ? (med / sqrtf(vhat[l])) : med;
}

// ------------------------------------------------------------------------------------------
// stage 3b: exact top-k of |est| by radix selection on the 31-bit magnitude pattern
// ------------------------------------------------------------------------------------------
// Digits of 11, 10 and 10 bits.  The histogram of the first digit needs every key (an estimate kernel often takes it).
// A filter then reads the keys once more and lists those whose first digit is not below that of the k-th largest key --
// the selected ones and the candidates, about 1.5 k of them unless many keys are equal -- in coordinate order, every
// tile of keys in a region of its own.  Everything after that works on the listed keys only (on all keys, without the filter,
// where a context of more than 2^20 coordinates found no room for lists).
//   up to 2^20 keys and small k (kSelSmallMaxK, kSelFlatMaxK, kSelFlatShortMaxK): k_sel_small filters, and its last workgroup finishes
//   the selection
//   else: k_sel_filter, two histograms of the listed keys, k_sel_count, k_sel_write
// Up to 2^20 keys every filter workgroup picks the first digit from the histogram for itself (8 KiB, in every L2); above,
// the last workgroup of the histogram does it once.
// Code that one workgroup runs once is bound by its chain of latencies, fetching the instructions among them: it is kept
// short (rolled loops; 16 KB of unrolled code took 5 us longer).
// "Last workgroup" (last_workgroup) never waits: whoever draws the last number goes on, the others end.  Data that it
// reads from other workgroups of the same launch goes through agent-scope atomic accesses, since the L2s of the eight
// XCDs are not coherent with each other inside a launch.
// Measured on MI355X, without the first histogram's pass where an estimate kernel takes it, in brackets ten launches over all
// keys (up to 2^16 keys three sweeps by one workgroup): k = 1 % of 65,536 keys 8 us (28), of 431,003 29 us with the
// histogram (84), of 11.2 million 35 us (111), of 124 million 0.18 ms (0.41): what is left is the filter's pass over the keys and
// launches of 5 us.  By topk_refine, with the histogram: 65,536 keys, half of them kept 26 us (44); 431,003, half 30 us (63);
// 4.96 million, a quarter 56 us (134), all 84 us (126).

// The streaming passes of the selection read four consecutive keys per lane with one 16-byte load
// (the entry points accept 16-byte aligned arrays only; the last, partial group of four is read key by key).  Absent keys
// (at or beyond len) are reported through the mask `have`.
struct Keys4 {
    float v[4];
    uint32_t have;   // bit z set: v[z] is a key
};
__device__ __forceinline__ Keys4 load_keys4(const float *__restrict__ keys, int64_t l, int64_t len)
{
    Keys4 q;
    if (l + 3 < len) {
        typedef float vec4f __attribute__((ext_vector_type(4)));
        const vec4f t = __builtin_nontemporal_load(reinterpret_cast<const vec4f *>(keys + l));   // streamed: read once per pass
        q.v[0] = t.x; q.v[1] = t.y; q.v[2] = t.z; q.v[3] = t.w;
        q.have = 0xfu;
    } else {
        q.have = 0u;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            q.v[z] = (l + z < len) ? keys[l + z] : 0.0f;
            q.have |= (l + z < len) ? (1u << z) : 0u;
        }
    }
    return q;
}

// sum over the lanes below this one, and over the whole wavefront, of a per-lane count in 0..7
__device__ __forceinline__ void wave_prefix3(uint32_t cnt, uint64_t below, uint32_t *excl, uint32_t *total)
{
    uint32_t e = 0, t = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const uint64_t m = __ballot((cnt >> b) & 1u);
        e += (uint32_t)__popcll(m & below) << b;
        t += (uint32_t)__popcll(m) << b;
    }
    *excl = e;
    *total = t;
}

// Histogram of the first digit over all keys; PICK: the last workgroup picks the digit.  A workgroup has at least four tiles of 4096 keys
// where that leaves kHistMinGrid of them, and there are no more than compute units: what a workgroup costs is the adding of its
// histogram to the whole one.  Selections (topk_refine) with up to 512 and so: a million keys 32.5 and 31.3 us, three million 40 and
// 36.5, 4.96 million, a quarter 58.5 and 55.7, seven million, an eighth 58 and 55;
// two loads of keys are under way per thread, for the long ones.
constexpr int kHistMinGrid = 128, kHistMaxGrid = 256;
static int hist_grid(int64_t len)
{
    const int by_four = grid_for(len, 4 << kSelTileLog2, kHistMaxGrid);
    return by_four > kHistMinGrid ? by_four : grid_for(len, 1 << kSelTileLog2, kHistMinGrid);
}
template <bool PICK>
__global__ void __launch_bounds__(1024)
k_sel_hist(const float *__restrict__ keys, int64_t len, uint32_t k, SelState *__restrict__ st, uint32_t *__restrict__ hist)
{
    __shared__ uint32_t lh[kHistBins], part[16], sh[2];
    for (int t = threadIdx.x; t < kHistBins; t += 1024) lh[t] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * 4096;
    for (int64_t l = (blockIdx.x * (int64_t)1024 + threadIdx.x) * 4; l < len; l += 2 * stride) {
        const Keys4 q[2] = {load_keys4(keys, l, len), load_keys4(keys, l + stride, len)};
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int z = 0; z < 4; ++z)
                if ((q[y].have >> z) & 1u) atomicAdd(&lh[mag_key(q[y].v[z]) >> 20], 1u);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kHistBins; t += 1024)
        if (lh[t]) atomicAdd(&hist[t], lh[t]);
    if constexpr (PICK) {
        if (last_workgroup(&st->done[0], gridDim.x, sh)) sel_pick<1024>(st, hist, 0, k, part, sh);
    }
}

// The same for at most kSelMaxTiles tiles, a workgroup each: every tile's histogram to a place of its own, so that nothing has to
// be zero before.  *done (of the launch that follows) goes to 0.
__global__ void __launch_bounds__(1024)
k_sel_hist_tiles(const float *__restrict__ keys, int64_t len, uint32_t *__restrict__ tile_hist, uint32_t *__restrict__ done)
{
    __shared__ uint32_t lh[kHistBins];
    const int t = threadIdx.x;
    for (int b = t; b < kHistBins; b += 1024) lh[b] = 0;
    if (blockIdx.x == 0 && t == 0) *done = 0u;
    __syncthreads();
    const Keys4 q = load_keys4(keys, ((int64_t)blockIdx.x << kSelTileLog2) + t * 4, len);
#pragma unroll
    for (int z = 0; z < 4; ++z)
        if ((q.have >> z) & 1u) atomicAdd(&lh[mag_key(q.v[z]) >> 20], 1u);
    __syncthreads();
    tile_hist[blockIdx.x * (kHistBins / 2) + t] = lh[2 * t] | (lh[2 * t + 1] << 16);
}

// One more in h[bin] (LDS) for every lane with `in`.  Lanes that have the first one's bin are added up in registers: keys that are all
// alike would queue up for one word.
__device__ __forceinline__ void count_alike(uint32_t *h, bool in, uint32_t bin)
{
    const uint64_t all = __ballot(in);
    if (!all) return;                                                // uniform
    const int first = __ffsll((unsigned long long)all) - 1;
    const uint32_t bin0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
    const uint32_t same = (uint32_t)__popcll(__ballot(in && bin == bin0));
    const bool leads = (int)(threadIdx.x & (kWave - 1)) == first;
    if (leads || (in && bin != bin0)) atomicAdd(&h[bin], leads ? same : 1u);   // (one instruction: bin is the lane's)
}

// A tile of keys per workgroup: lists the keys whose first digit is at or above the k-th largest key's, in
// coordinate order, at val / loc [tile * tile size], their number at cnt[tile].
// PICK: the workgroup picks that digit from hist0 (the prefix and the number of keys to take among those that match it
// are left in picked[2], LDS); otherwise it is *prefix_in.  AGENT: the list is read again in this launch, and zeros are not listed
// (see flat_zeros).
// TILES: hist0 is the tiles' histograms.
// Where all tiles together list more than `crowd` keys, every tile adds the second digit of its keys that match the first to
// hist1 (lh: 1024 bins in LDS) and leaves the smallest and the largest magnitude that it lists at ls.group[tile].
template <bool PICK, bool AGENT, bool TILES = false>
__device__ __forceinline__ void filter_tile(const float *__restrict__ keys, int64_t len, int64_t tile,
                                            const uint32_t *__restrict__ prefix_in, const uint32_t *__restrict__ hist0, uint32_t k,
                                            const SelList &ls, uint32_t *picked, uint32_t crowd = 0,
                                            uint32_t *__restrict__ hist1 = nullptr, uint32_t *lh = nullptr)
{
    __shared__ uint32_t part[16], wsum[16];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    const int64_t base = tile << kSelTileLog2;
    const Keys4 q = load_keys4(keys, base + t * 4, len);
    uint32_t prefix;
    if constexpr (PICK) {
        uint32_t pair[2] = {0u, 0u};                                 // TILES: the thread's two bins, all tiles' loads under way
        if constexpr (TILES) {
            uint32_t x[kSelMaxTiles];
#pragma unroll
            for (int w = 0; w < kSelMaxTiles; ++w)
                x[w] = hist0[(w < (int)gridDim.x ? w : 0) * (kHistBins / 2) + (kHistBins / 2 - 1 - t)];
#pragma unroll
            for (int w = 0; w < kSelMaxTiles; ++w)
                if (w < (int)gridDim.x) {
                    pair[0] += x[w] & 0xffffu;
                    pair[1] += x[w] >> 16;
                }
        }
        pick_digit<1024, kHistBins>([&](int b) { return TILES ? pair[b & 1] : hist0[b]; }, k, [&](uint32_t b, uint32_t above, uint32_t in) {
            picked[0] = b;
            picked[1] = k - above;
            if (AGENT) picked[2] = above + in;                       // keys listed in all, and the zeros
        }, part);
        __syncthreads();
        prefix = picked[0];
    } else {
        prefix = *prefix_in;
    }
    uint32_t keep = 0, before = 0, total = 0;
#pragma unroll
    for (int z = 0; z < 4; ++z)
        keep |= ((mag_key(q.v[z]) >> 20) >= prefix && (!AGENT || mag_key(q.v[z]) != 0u) ? (q.have >> z) & 1u : 0u) << z;
    if (__ballot(keep != 0u)) wave_prefix3((uint32_t)__popc(keep), ((uint64_t)1 << lane) - 1, &before, &total);
    if (lane == 0) wsum[wave] = total;
    __syncthreads();
    const uint32_t upto = wave_inclusive_scan(lane < 16 ? wsum[lane] : 0u);   // lane w: listed by wavefronts 0 .. w
    uint32_t pos = before + (uint32_t)__shfl((int)upto, wave) - total;
#pragma unroll
    for (int z = 0; z < 4; ++z)
        if ((keep >> z) & 1u) {
            put<AGENT>(ls.val + base + pos, __float_as_uint(q.v[z]));
            put<AGENT>(ls.loc + base + pos, (uint16_t)(t * 4 + z));
            ++pos;
        }
    if (t == 15) put<AGENT>(ls.cnt + tile, upto);
    if (!hist1 || picked[2] <= crowd) return;                        // uniform over the workgroup
    __shared__ uint32_t least[16], most[16];
    uint32_t lo = UINT32_MAX, hi = 0;
    lh[t] = 0;
    __syncthreads();
#pragma unroll
    for (int z = 0; z < 4; ++z) {
        const uint32_t key = mag_key(q.v[z]);
        const bool in = (keep >> z) & 1u;
        count_alike(lh, in && (key >> 20) == prefix, (key >> 10) & 1023u);
        lo = in && key < lo ? key : lo;
        hi = in && key > hi ? key : hi;
    }
    for (int off = kWave / 2; off; off >>= 1) {
        const uint32_t l = __shfl_xor(lo, off), h = __shfl_xor(hi, off);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    if (lane == 0) {
        least[wave] = lo;
        most[wave] = hi;
    }
    __syncthreads();
    if (lh[t]) atomicAdd(&hist1[t], lh[t]);
    if (t == 0) {
        for (int w = 1; w < 16; ++w) {
            lo = least[w] < lo ? least[w] : lo;
            hi = most[w] > hi ? most[w] : hi;
        }
        put<AGENT>(&ls.group[tile].x, lo);
        put<AGENT>(&ls.group[tile].y, hi);
    }
}

// The listed keys of at most TILES tiles as one sequence in coordinate order, for one workgroup of 1024 threads: entry e is
// number e - start[tile] of its tile's list.  Up to kMax entries are copied to LDS, more than that stay in their lists (see
// flat_crowded).  Up to 16 tiles that is 64 KB in all; more tiles (at most a workgroup per compute unit) list more keys for the same
// k: with 7,168 and with 15,360 entries a step on 200,000 coordinates, k = 1,500 after 600 steps 54.3 and 52.0 us.
template <int TILES>
struct Flat {
    static constexpr uint32_t kMax = 15360;
    uint32_t start[2 * TILES];
    alignas(16) uint32_t val[kMax], pos[kMax];
    uint32_t part[16], picked[4], hist[1024];
};

// entries e[0..N), each below the number of entries: tile by bisection, N searches side by side
template <int N, int TILES>
__device__ __forceinline__ void flat_fetch(const SelList &ls, const Flat<TILES> &f, const uint32_t (&e)[N], uint2 (&x)[N])
{
    uint32_t tile[N];
#pragma unroll
    for (int z = 0; z < N; ++z) tile[z] = 0;
#pragma unroll 1
    for (uint32_t step = TILES; step; step >>= 1) {
#pragma unroll
        for (int z = 0; z < N; ++z)
            if (f.start[tile[z] + step] <= e[z]) tile[z] += step;
    }
#pragma unroll
    for (int z = 0; z < N; ++z) {
        const uint32_t base = tile[z] << kSelTileLog2, at = base + e[z] - f.start[tile[z]];
        x[z] = make_uint2(get<true>(ls.val + at), base + get<true>(ls.loc + at));
    }
}

// the number of entries; complete for all threads
template <int TILES>
__device__ __forceinline__ uint32_t flat_load(const SelList &ls, Flat<TILES> &f, int ntile, uint32_t len)
{
    static_assert(2 * TILES <= 1024, "a thread per start");
    const int t = threadIdx.x;
    // (a call on another stream with the same scratch may have put any count there: no list is longer than its tile)
    const uint32_t rest = t < ntile ? len - ((uint32_t)t << kSelTileLog2) : 0u, tile = rest < 1u << kSelTileLog2 ? rest : 1u << kSelTileLog2;
    const uint32_t cnt = t < ntile ? get<true>(ls.cnt + t) : 0u;
    const uint32_t before = block_exclusive_scan<1024>(cnt < tile ? cnt : tile, f.part);
    if (t < 2 * TILES) f.start[t] = before;                          // from ntile on: the number of entries
    f.hist[t] = 0;
    __syncthreads();
    const uint32_t m = f.start[ntile];
    if (m > Flat<TILES>::kMax) return m;
#pragma unroll 1
    for (uint32_t e0 = t; e0 < m; e0 += 4 * 1024) {
        uint32_t e[4];
        uint2 x[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) e[z] = e0 + z * 1024 < m ? e0 + z * 1024 : m - 1;
        flat_fetch<4>(ls, f, e, x);
#pragma unroll
        for (int z = 0; z < 4; ++z) {                                // (the last entry may be stored twice, alike)
            f.val[e[z]] = x[z].x;
            f.pos[e[z]] = x[z].y;
        }
    }
    __syncthreads();
    return m;
}

// one digit of 10 bits from f.hist, which is zero again for the next one: prefix and k_rem (keys to take among those that match it)
// go one digit on.  p: two words of LDS that no other digit has.  The histogram is complete (a barrier before)
template <int TILES>
__device__ __forceinline__ void flat_pick(Flat<TILES> &f, uint32_t *p, uint32_t &prefix, uint32_t &k_rem)
{
    auto count = [&](int b) {                                        // (read by one thread)
        const uint32_t x = f.hist[b];
        f.hist[b] = 0;
        return x;
    };
    pick_digit<1024, 1024>(count, k_rem, [&](uint32_t b, uint32_t above, uint32_t) {
        p[0] = (prefix << 10) | b;
        p[1] = k_rem - above;
    }, f.part);
    __syncthreads();
    prefix = p[0];
    k_rem = p[1];
}

// the last two digits of m entries in LDS: prefix (the first digit) and k_rem become the threshold and how many keys equal to it to take
template <int TILES>
__device__ __forceinline__ void flat_digits(Flat<TILES> &f, uint32_t m, uint32_t &prefix, uint32_t &k_rem)
{
#pragma unroll 1
    for (int digit = 1; digit <= 2; ++digit) {
        const int up = 30 - 10 * digit;
        for (uint32_t e = threadIdx.x; e < m; e += 1024) {
            const uint32_t key = f.val[e] & 0x7fffffffu;
            if ((key >> up) == prefix) atomicAdd(&f.hist[(key >> (up - 10)) & 1023u], 1u);
        }
        __syncthreads();
        flat_pick(f, f.picked + (digit - 1) * 2, prefix, k_rem);
    }
}

// where the selected entries go: an entry's rank follows from the keys above the threshold and at it before it.
// map != null: the output is map[position] instead of the position, which a call on another stream with the same scratch may have
// put there: it is held below len.
struct SelOut {
    const int32_t *__restrict__ map;
    int32_t *__restrict__ idx;
    float *__restrict__ val_sel;
    int64_t k, len;
    uint32_t k_eq;   // how many keys equal to the threshold are taken
    __device__ __forceinline__ uint32_t source(uint32_t at) const { return (uint32_t)map[at < (uint32_t)len ? at : (uint32_t)len - 1u]; }
    __device__ __forceinline__ void put(uint32_t bits, uint32_t at, uint32_t gtb, uint32_t eqb) const
    {
        const int64_t pos = (int64_t)gtb + (eqb < k_eq ? eqb : k_eq);
        if (pos >= k) return;
        idx[pos] = (int32_t)(map ? source(at) : at);
        if (val_sel) val_sel[pos] = __uint_as_float(bits);
    }
};

// writes the selected ones of m entries in LDS at their rank: key > tau, or key == tau and among the first k_eq such keys.  Of many
// entries a thread has consecutive ones, so that one scan ranks them all; few come 1024 at a time.
template <int TILES>
__device__ __forceinline__ void flat_write(Flat<TILES> &f, uint32_t m, uint32_t tau, const SelOut &out)
{
    const uint32_t k_eq = out.k_eq;
    if (TILES > kSelMaxTiles && m > 3072) {                          // (up to 16 tiles the turns below are 0.6 us faster)
        const uint32_t per = ((m + 1023u) / 1024u) | 1u;             // odd: the threads' first entries lie in different banks
        const uint32_t e0 = threadIdx.x * per < m ? threadIdx.x * per : m, e1 = e0 + per < m ? e0 + per : m;
        uint32_t own = 0;                                            // above the threshold, and at it, in one scan
#pragma unroll 1
        for (uint32_t e = e0; e < e1; ++e) {
            const uint32_t key = f.val[e] & 0x7fffffffu;
            own += (key > tau ? 1u : 0u) + (key == tau ? 0x10000u : 0u);
        }
        const uint32_t before = block_exclusive_scan<1024>(own, f.part);
        uint32_t gtb = before & 0xffffu, eqb = before >> 16;
#pragma unroll 1
        for (uint32_t e = e0; own && e < e1; ++e) {
            const uint32_t bits = f.val[e], key = bits & 0x7fffffffu;
            if (key > tau || (key == tau && eqb < k_eq)) out.put(bits, f.pos[e], gtb, eqb);
            gtb += key > tau ? 1u : 0u;
            eqb += key == tau ? 1u : 0u;
        }
        return;
    }
    uint32_t gt_run = 0, eq_run = 0;
#pragma unroll 1
    for (uint32_t e0 = 0; e0 < m; e0 += 1024) {
        const uint32_t e = e0 + threadIdx.x;
        const uint32_t bits = e < m ? f.val[e] : 0u, key = bits & 0x7fffffffu;
        const bool gt = e < m && key > tau, eq = e < m && key == tau;
        const uint32_t own = (gt ? 1u : 0u) | (eq ? 0x10000u : 0u);  // both prefixes (at most 1024) in one scan
        const uint32_t before = block_exclusive_scan<1024>(own, f.part);
        if (threadIdx.x == 1023) f.picked[0] = before + own;
        const uint32_t eqb = eq_run + (before >> 16), gtb = gt_run + (before & 0xffffu);
        if (gt || (eq && eqb < k_eq)) out.put(bits, f.pos[e], gtb, eqb);
        __syncthreads();
        gt_run += f.picked[0] & 0xffffu;
        eq_run += f.picked[0] >> 16;
        __syncthreads();
    }
}

// One wavefront walks nt lists in order, list q of length(q) entries from val[q 2^12] on: f(at, n, w) for every group of at most
// 256 entries, val[at ... at + n), four consecutive ones per lane in w.  Four groups are under way, of one list or of several.  val is
// 16-byte aligned, and has room for three words behind each list's last entry.  f is in the code four times, so what it does with
// entries that matter is a loop over the four of a lane.
template <int UNDER, typename L, typename F>
__device__ __forceinline__ void each_group(const uint32_t *val, L length, int nt, F f)
{
    constexpr int kGroup = 4 * kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    int q = 0;
    uint32_t e0 = 0, cnt = nt > 0 ? length(0) : 0u;
    auto settle = [&] {                                              // to the next list with an entry; q == nt: no more
        while (e0 >= cnt && q < nt) {
            if (++q == nt) break;
            e0 = 0;
            cnt = length(q);
        }
    };
    settle();
    while (q < nt) {
        uint32_t at[UNDER], n[UNDER];
        uint4 w[UNDER];
#pragma unroll
        for (int z = 0; z < UNDER; ++z) {
            at[z] = z && q >= nt ? at[z - 1] : ((uint32_t)q << kSelTileLog2) + e0;
            n[z] = q >= nt ? 0u : (cnt - e0 < kGroup ? cnt - e0 : kGroup);
            const uint32_t end = n[z] ? (n[z] - 1u) & ~3u : 0u;
            const uint64_t *const src = reinterpret_cast<const uint64_t *>(val + at[z] + (lane * 4 < end ? lane * 4 : end));
            const uint64_t lo = get<true>(src), hi = get<true>(src + 1);
            w[z] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
            e0 += kGroup;
            settle();
        }
#pragma unroll
        for (int z = 0; z < UNDER; ++z)
            if (n[z]) f(at[z], n[z], w[z]);
    }
}
__device__ __forceinline__ uint4 next_entry(const uint4 &b) { return make_uint4(b.y, b.z, b.w, b.x); }
// of the lanes below this one, how many are in mask, and `more`
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask, uint32_t more)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, more));
}

// The selection where LDS does not hold the listed keys: many share the threshold's first digit (its binary exponent and three
// more bits), as clipped or quantised values do, and values that lie within an eighth of an octave.  Every wavefront has consecutive
// tiles and walks their lists.  With AHEAD the filter has taken the second digit's histogram (h1: this thread's bin), so one walk
// remains in most cases: it takes the third digit's and copies what may still be selected to the wavefront's part of LDS.  Equal keys too
// many for that cost two more, to count and to write; but lists that are all one magnitude (range, with AHEAD) are not walked.
// Measured (topk_refine_static, us; by separate launches, with a search in the lists for every entry and digit, and so): 200,000 keys, k =
// 2,500, all equal 173, 615, 40, all within [1, 1.125) 83, 370, 54, a tenth there 31, 41, 27, normal values clipped at 1 74, 197, 39;
// 431,003, k = 500 the same 174, 1,307, 30; 80, 746, 62; 33, 79, 29; 74, 419, 24; a million, k = 2,500 180, 3,288, 51; 85, 2,054, 130;
// 37, 196, 48; 79, 1,016, 45; 60,000, k = 500 (no separate launches) 175, 62; 101, 42; 18, 17; 61, 33.  The walk is bound by instruction
// issue: with eight groups under way in place of four it takes as long, with a case of its own for groups that hold a few keys to keep
// 191 -> 130 us at a million.
template <bool AHEAD, int TILES>
__device__ __forceinline__ void flat_crowded(const SelList &ls, Flat<TILES> &f, int ntile, uint32_t h1, uint32_t prefix, uint32_t k_rem,
                                             SelOut out)
{
    constexpr uint32_t kPart = Flat<TILES>::kMax / 16;               // entries of a wavefront in LDS
    constexpr uint32_t kLong = 4 * kWave;                            // a list of no more is one load
    static_assert(kPart % 4 == 0, "parts start at 16 bytes");
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int per = (ntile + 15) / 16, t0 = wave * per < ntile ? wave * per : ntile, nt = ntile - t0 < per ? ntile - t0 : per;
    const uint32_t first = (uint32_t)t0 << kSelTileLog2;             // of the wavefront's lists, in val and loc
    // lane q has list q: its length, and its magnitude if that is the only one in a long list (else 0, which no listed key has)
    const uint32_t count = lane < nt ? f.start[t0 + lane + 1] - f.start[t0 + lane] : 0u;
    uint32_t only = 0;
    if (AHEAD && count > kLong) {
        const uint32_t lo = get<true>(&ls.group[t0 + lane].x), hi = get<true>(&ls.group[t0 + lane].y);
        only = lo == hi ? lo : 0u;
    }
    if constexpr (!AHEAD) {
        each_group<4>(ls.val + first, [&](int q) { return (uint32_t)__builtin_amdgcn_readlane((int)count, q); }, nt,
                   [&](uint32_t, uint32_t n, const uint4 &w) {
            uint4 b = w;
#pragma unroll 1
            for (int y = 0; y < 4; ++y, b = next_entry(b))
                count_alike(f.hist, lane * 4 + y < (int)n && ((b.x >> 20) & 0x7ffu) == prefix, (b.x >> 10) & 1023u);
        });
        __syncthreads();
    } else {
        f.hist[t] = h1;
        __syncthreads();
    }
    flat_pick(f, f.picked, prefix, k_rem);
    uint32_t *const pv = f.val + wave * kPart, *const pp = f.pos + wave * kPart;
    uint32_t mine = 0;                                               // may exceed kPart
    const uint32_t open = only ? 0u : count;                         // to be walked
    each_group<4>(ls.val + first, [&](int q) { return (uint32_t)__builtin_amdgcn_readlane((int)open, q); }, nt,
               [&](uint32_t at, uint32_t n, const uint4 &w) {
        const uint32_t bits[4] = {w.x, w.y, w.z, w.w};
        const uint32_t least = prefix << 10;                         // (first 11 and next 10 bits of 31)
        uint32_t top4 = 0;
#pragma unroll
        for (int y = 0; y < 4; ++y) top4 = (bits[y] & 0x7fffffffu) > top4 ? bits[y] & 0x7fffffffu : top4;
        if (!__any(top4 >= least)) return;                           // uniform; most groups, where keys differ
        const int have = (int)n - lane * 4;                          // entries of this lane
        uint32_t own = 0, bit = 0, which = 0;                        // how many are kept, the last one
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const bool in = (bits[y] & 0x7fffffffu) >= least && y < have;
            own += in;
            bit = in ? bits[y] : bit;
            which = in ? y : which;
        }
        const uint64_t any = __ballot(own);
        if (!any) return;                                            // uniform
        if (__popcll(any) <= 32 && !__ballot(own > 1u)) {            // uniform; most of the rest: a third of the instructions
            const uint32_t rank = lanes_below(any, mine), key = bit & 0x7fffffffu;
            if (own && rank < kPart) {
                pv[rank] = bit;
                pp[rank] = at + lane * 4 + which;
            }
            if (own && key < least + 1024u) atomicAdd(&f.hist[key & 1023u], 1u);
            mine += (uint32_t)__popcll(any);
            return;
        }
        uint64_t keep[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) keep[y] = __ballot((bits[y] & 0x7fffffffu) >= least && y < have);
        uint32_t rank = mine;
#pragma unroll
        for (int y = 0; y < 4; ++y) rank = lanes_below(keep[y], rank);
        const uint32_t more = (uint32_t)(__popcll(keep[0]) + __popcll(keep[1]) + __popcll(keep[2]) + __popcll(keep[3]));
        const bool many = more > 32u;
        mine += more;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const uint32_t key = bits[y] & 0x7fffffffu;
            const bool in = key >= least && y < have, digit = in && key < least + 1024u;
            if (in && rank < kPart) {
                pv[rank] = bits[y];
                pp[rank] = at + lane * 4 + y;
            }
            rank += in;
            if (many) count_alike(f.hist, digit, key & 1023u);       // uniform
            else if (digit) atomicAdd(&f.hist[key & 1023u], 1u);
        }
    });
    if (only && (only >> 10) == prefix) atomicAdd(&f.hist[only & 1023u], count);
    const bool spill = __syncthreads_or(mine > kPart || (only && (only >> 10) >= prefix));
    flat_pick(f, f.picked + 2, prefix, k_rem);
    const uint32_t tau = prefix, k_eq = k_rem;
    out.k_eq = k_eq;
    // the wavefront's entries: its part of LDS, or its lists
    const uint32_t *const src = spill ? ls.val + first : pv;
    const uint32_t src_open = spill ? open : mine;                   // (lane 0's is asked for of LDS)
    const int src_lists = spill ? nt : 1;
    uint32_t gt = 0, eq = 0;
    each_group<4>(src, [&](int q) { return (uint32_t)__builtin_amdgcn_readlane((int)src_open, q); }, src_lists,
               [&](uint32_t, uint32_t n, const uint4 &w) {
        const uint32_t bits[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            gt += (bits[y] & 0x7fffffffu) > tau && lane * 4u + y < n ? 1u : 0u;
            eq += (bits[y] & 0x7fffffffu) == tau && lane * 4u + y < n ? 1u : 0u;
        }
    });
    if (only > tau) gt += count;
    if (only == tau) eq += count;                                    // (tau is no zero: those are not listed)
    const uint32_t gt_before = block_exclusive_scan<1024>(gt, f.part), eq_before = block_exclusive_scan<1024>(eq, f.part);
    uint32_t gt_run = (uint32_t)__builtin_amdgcn_readfirstlane((int)gt_before), eq_run = (uint32_t)__builtin_amdgcn_readfirstlane((int)eq_before);
    const uint32_t last = spill ? (only && only < tau ? 0u : count) : mine;
    each_group<2>(src, [&](int q) {
        if (spill && eq_run >= k_eq && (uint32_t)__builtin_amdgcn_readlane((int)only, q) == tau) return 0u;   // all taken
        return (uint32_t)__builtin_amdgcn_readlane((int)last, q);
    }, src_lists, [&](uint32_t at, uint32_t n, const uint4 &w) {
        const uint32_t bits[4] = {w.x, w.y, w.z, w.w};
        const int have = (int)n - lane * 4;
        const bool ties = eq_run < k_eq;                             // more than k_eq need no count
        uint64_t gts[4], eqs[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            gts[y] = __ballot((bits[y] & 0x7fffffffu) > tau && y < have);
            eqs[y] = __ballot(ties && (bits[y] & 0x7fffffffu) == tau && y < have);
        }
        if (!(gts[0] | gts[1] | gts[2] | gts[3] | eqs[0] | eqs[1] | eqs[2] | eqs[3])) return;   // uniform
        uint32_t gtb = gt_run, eqb = eq_run;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            gtb = lanes_below(gts[y], gtb);
            eqb = lanes_below(eqs[y], eqb);
            gt_run += (uint32_t)__popcll(gts[y]);
            eq_run += (uint32_t)__popcll(eqs[y]);
        }
        bool take[4];
        uint32_t to[4], from[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) {                                // all positions under way, then all that map[] says
            const uint32_t key = bits[y] & 0x7fffffffu;
            const bool g = key > tau && y < have, q = ties && key == tau && y < have;
            take[y] = (g || (q && eqb < k_eq)) && gtb + (eqb < k_eq ? eqb : k_eq) < out.k;
            to[y] = gtb + (eqb < k_eq ? eqb : k_eq);
            gtb += g;
            eqb += q;
            const uint32_t e = at + lane * 4 + y, listed = first + (spill || !take[y] ? e : pp[e]);
            from[y] = take[y] ? (listed & ~((1u << kSelTileLog2) - 1u)) + get<true>(ls.loc + listed) : 0u;
        }
        if (out.map) {
#pragma unroll
            for (int y = 0; y < 4; ++y)
                if (take[y]) from[y] = out.source(from[y]);
        }
#pragma unroll
        for (int y = 0; y < 4; ++y)
            if (take[y]) {
                out.idx[to[y]] = (int32_t)from[y];
                if (out.val_sel) out.val_sel[to[y]] = __uint_as_float(bits[y]);
            }
    });
}

// The selection where fewer keys than k differ from zero: those, all of them listed, and the first zeros.  With z zeros to take, a
// listed key's rank is its position while fewer than z zeros lie before it, and its number in the lists plus z from there on; all
// positions before the last of those zeros are selected.  (Zeros in the lists, most of a sparse vector's coordinates, would make the
// last workgroup walk all keys: of 431,003 keys, 750 of them other than zero, k = 1,500 18 us; of 60,000, 250 of them, k = 500 16.)
template <int TILES>
__device__ __forceinline__ void flat_zeros(const SelList &ls, Flat<TILES> &f, uint32_t m, const float *__restrict__ keys, uint32_t len,
                                           uint32_t k, const int32_t *__restrict__ map, int32_t *__restrict__ idx,
                                           float *__restrict__ val_sel)
{
    const uint32_t z = k - m;
    uint32_t early = 0;                                              // this thread's listed keys before the last zero
#pragma unroll 1
    for (uint32_t e0 = threadIdx.x; e0 < m; e0 += 1024) {
        uint32_t e[1] = {e0};
        uint2 x[1];
        if (m <= Flat<TILES>::kMax) x[0] = make_uint2(f.val[e0], f.pos[e0]);
        else flat_fetch<1>(ls, f, e, x);
        if (x[0].y - e0 < z) {
            ++early;
        } else {
            idx[z + e0] = map ? map[x[0].y < len ? x[0].y : len - 1u] : (int32_t)x[0].y;   // (see flat_write)
            if (val_sel) val_sel[z + e0] = __uint_as_float(x[0].x);
        }
    }
    const uint32_t before = block_exclusive_scan<1024>(early, f.part);
    if (threadIdx.x == 1023) f.picked[0] = before + early;
    __syncthreads();
    const uint32_t whole = z + f.picked[0];
    for (uint32_t q = threadIdx.x; q < whole; q += 1024) {
        idx[q] = map ? map[q] : (int32_t)q;
        if (val_sel) val_sel[q] = keys[q];
    }
}

// tiles of 4096 keys, one per workgroup, at most TILES; HISTS: hist is the tiles' histograms
template <bool HISTS, int TILES>
__global__ void __launch_bounds__(1024)
k_sel_small(const float *__restrict__ keys, int64_t len, SelState *__restrict__ st, uint32_t *__restrict__ hist, SelList ls,
            int64_t k, const int32_t *__restrict__ map, int32_t *__restrict__ idx, float *__restrict__ val_sel)
{
    __shared__ Flat<TILES> f;
    constexpr bool kAhead = TILES > kSelMaxTiles;                    // (up to 16 tiles there may be no histogram of zeros to add to)
    uint32_t *const hist1 = kAhead ? hist + kHistBins : nullptr;
    filter_tile<true, true, HISTS>(keys, len, blockIdx.x, nullptr, hist, (uint32_t)k, ls, f.picked, Flat<TILES>::kMax, hist1, f.hist);
    uint32_t prefix = f.picked[0], k_rem = f.picked[1];
    if (!last_workgroup(&st->done[1], gridDim.x, f.part)) return;
    if constexpr (!HISTS)
        for (int b = threadIdx.x; b < kHistBins; b += 1024) hist[b] = 0u;   // every workgroup has read it
    __syncthreads();
    const uint32_t m = flat_load(ls, f, (int)gridDim.x, (uint32_t)len);
    uint32_t h1 = 0;
    if constexpr (kAhead) {
        if (m > Flat<TILES>::kMax) h1 = get<true>(hist1 + threadIdx.x);
        hist1[threadIdx.x] = 0u;
    }
    if (prefix == 0u && m < (uint32_t)k) {
        flat_zeros(ls, f, m, keys, (uint32_t)len, (uint32_t)k, map, idx, val_sel);
        return;
    }
    SelOut out = {map, idx, val_sel, k, len, 0u};
    if (m > Flat<TILES>::kMax) {
        flat_crowded<kAhead>(ls, f, (int)gridDim.x, h1, prefix, k_rem, out);
        return;
    }
    flat_digits(f, m, prefix, k_rem);
    out.k_eq = k_rem;
    flat_write(f, m, prefix, out);
}

// PICK: the filter picks the first digit (and leaves it in the state), see above
template <bool PICK>
__global__ void __launch_bounds__(1024)
k_sel_filter(const float *__restrict__ keys, int64_t len, SelState *__restrict__ st, const uint32_t *__restrict__ hist,
             SelList ls, uint32_t k)
{
    __shared__ uint32_t picked[2];
    filter_tile<PICK, false>(keys, len, blockIdx.x, st->prefix, hist, k, ls, picked);
    if (PICK && blockIdx.x == 0 && threadIdx.x == 0) {
        st->prefix[0] = picked[0];
        st->k_rem[0] = picked[1];
    }
}

constexpr int kSelWriteMaxPpw = 4;
__device__ __forceinline__ uint32_t listed(const SelList &ls, int64_t len, int64_t tile)
{
    if (ls.cnt) return ls.cnt[tile];
    const int64_t rest = len - (tile << kSelTileLog2);
    return rest < (1 << kSelTileLog2) ? (uint32_t)rest : 1u << kSelTileLog2;
}

// What a wavefront takes at a time: a tile's list, or (SPLIT) one of 2^split pieces of it, whole groups of 64 but for the last
// one's end.
struct Piece {
    int64_t at;    // first entry, in val and loc
    uint32_t cnt;
};
template <bool SPLIT>
__device__ __forceinline__ Piece piece_of(const SelList &ls, int64_t len, int64_t piece, int split)
{
    if constexpr (!SPLIT) return {piece << kSelTileLog2, listed(ls, len, piece)};
    const int64_t tile = piece >> split;
    const uint32_t sub = (uint32_t)piece & ((1u << split) - 1u), all = listed(ls, len, tile);
    const uint32_t size = (((all + (1u << split) - 1u) >> split) + kWave - 1u) & ~(uint32_t)(kWave - 1);
    const uint32_t lo = sub * size < all ? sub * size : all, hi = lo + size < all ? lo + size : all;
    return {(tile << kSelTileLog2) + lo, hi - lo};
}

// f(have, bits) for the listed keys of a piece, 64 at a time by one wavefront; four groups of 64 are fetched
// together (clamped to the piece's count: in bounds)
template <typename F>
__device__ __forceinline__ void each_listed(const SelList &ls, const Piece &pc, F f)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t *val = ls.val + pc.at;
#pragma unroll 1
    for (uint32_t e0 = 0; e0 < pc.cnt; e0 += 4 * kWave) {
        uint32_t w[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const uint32_t e = e0 + z * kWave + lane;
            w[z] = val[e < pc.cnt ? e : pc.cnt - 1];
        }
#pragma unroll
        for (int z = 0; z < 4; ++z)
            if (e0 + z * kWave < pc.cnt) f(e0 + z * kWave + lane < pc.cnt, w[z]);
    }
}

// histogram of digit 1 or 2 over the listed keys whose higher digits are the picked ones
template <bool SPLIT>
__global__ void __launch_bounds__(1024)
k_sel_list_hist(SelState *__restrict__ st, uint32_t *__restrict__ hist, SelList ls, int64_t len, int64_t pieces, int split,
                int digit, uint32_t *__restrict__ clear)   // null, or the first digit's histogram, which the filter has read
{
    __shared__ uint32_t lh[1024], part[16], sh[2];
    const int t = threadIdx.x;
    lh[t] = 0;
    if (clear && blockIdx.x == 0)
        for (int b = t; b < kHistBins; b += 1024) clear[b] = 0u;
    __syncthreads();
    const uint32_t prefix = st->prefix[digit - 1];
    const int up = 30 - 10 * digit;
    const int64_t waves = (int64_t)gridDim.x * 16;
    for (int64_t piece = (int64_t)blockIdx.x * 16 + t / kWave; piece < pieces; piece += waves)
        each_listed(ls, piece_of<SPLIT>(ls, len, piece, split), [&](bool have, uint32_t bits) {
            const uint32_t key = bits & 0x7fffffffu;
            if (have && (key >> up) == prefix) atomicAdd(&lh[(key >> (up - 10)) & 1023u], 1u);
        });
    __syncthreads();
    if (lh[t]) atomicAdd(&hist[t], lh[t]);
    if (last_workgroup(&st->done[digit], gridDim.x, sh)) sel_pick<1024>(st, hist, digit, 0, part, sh);
}

// keys of a piece that exceed the threshold, and that equal it (uniform over the wavefront)
__device__ __forceinline__ uint2 count_listed(const SelList &ls, const Piece &pc, uint32_t tau)
{
    uint2 n = make_uint2(0u, 0u);
    each_listed(ls, pc, [&](bool have, uint32_t bits) {
        n.x += (uint32_t)__popcll(__ballot(have && (bits & 0x7fffffffu) > tau));
        n.y += (uint32_t)__popcll(__ballot(have && (bits & 0x7fffffffu) == tau));
    });
    return n;
}

// A workgroup has 16 * ppw consecutive pieces, wavefront w the pieces ppw w ... ppw w + ppw - 1 of them.
// k_sel_count: keys above and at the threshold per workgroup, to group[].
template <bool SPLIT>
__global__ void __launch_bounds__(1024)
k_sel_count(const SelState *__restrict__ st, SelList ls, int64_t len, int64_t pieces, int split, int ppw)
{
    __shared__ uint32_t sum[2];
    const uint32_t tau = st->prefix[2];
    const int wave = threadIdx.x / kWave;
    if (threadIdx.x < 2) sum[threadIdx.x] = 0;
    __syncthreads();
    uint2 n = make_uint2(0u, 0u);
    for (int q = 0; q < ppw; ++q) {
        const int64_t piece = ((int64_t)blockIdx.x * 16 + wave) * ppw + q;
        if (piece >= pieces) break;
        const uint2 x = count_listed(ls, piece_of<SPLIT>(ls, len, piece, split), tau);
        n.x += x.x;
        n.y += x.y;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&sum[0], n.x);
        atomicAdd(&sum[1], n.y);
    }
    __syncthreads();
    if (threadIdx.x == 0) ls.group[blockIdx.x] = make_uint2(sum[0], sum[1]);
}

// k_sel_write: a workgroup adds up what the groups before it hold (every one for itself: a few hundred to two thousand pairs,
// in place of a scan by one workgroup in between), counts its own pieces and writes their selected keys at their rank:
// key > tau, or key == tau and among the first k_eq such keys.  map != null: the output is map[position] (below len, see
// flat_write).
template <bool SPLIT>
__global__ void __launch_bounds__(1024)
k_sel_write(const SelState *__restrict__ st, SelList ls, int64_t len, int64_t pieces, int split, int ppw, int64_t k,
            const int32_t *__restrict__ map, int32_t *__restrict__ idx, float *__restrict__ val_sel)
{
    __shared__ uint32_t part[16], sum[2];
    __shared__ uint32_t piece_gt[16 * kSelWriteMaxPpw], piece_eq[16 * kSelWriteMaxPpw];
    const uint32_t tau = st->prefix[2], k_eq = st->k_rem[2];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    if (t < 2) sum[t] = 0;
    if (t < 16 * kSelWriteMaxPpw) piece_gt[t] = piece_eq[t] = 0;
    __syncthreads();
    uint32_t g = 0, e = 0;
    for (uint32_t q = t; q < blockIdx.x; q += 1024) {
        const uint2 x = ls.group[q];
        g += x.x;
        e += x.y;
    }
    g = wave_inclusive_scan(g);
    e = wave_inclusive_scan(e);
    if (lane == kWave - 1) {
        atomicAdd(&sum[0], g);
        atomicAdd(&sum[1], e);
    }
    const int64_t first = ((int64_t)blockIdx.x * 16 + wave) * ppw;
    for (int q = 0; q < ppw && first + q < pieces; ++q) {
        const uint2 n = count_listed(ls, piece_of<SPLIT>(ls, len, first + q, split), tau);
        if (lane == 0) {
            piece_gt[wave * ppw + q] = n.x;
            piece_eq[wave * ppw + q] = n.y;
        }
    }
    __syncthreads();
    const int np = 16 * ppw;
    const uint32_t own_g = t < np ? piece_gt[t] : 0u, own_e = t < np ? piece_eq[t] : 0u;
    const uint32_t before_g = block_exclusive_scan<1024>(own_g, part), before_e = block_exclusive_scan<1024>(own_e, part);
    if (t < np) {
        piece_gt[t] = sum[0] + before_g;
        piece_eq[t] = sum[1] + before_e;
    }
    __syncthreads();
    for (int q = 0; q < ppw && first + q < pieces; ++q) {
        const Piece pc = piece_of<SPLIT>(ls, len, first + q, split);
        const int64_t base = (SPLIT ? (first + q) >> split : first + q) << kSelTileLog2;
        const uint32_t cnt = pc.cnt;
        uint32_t gtr = piece_gt[wave * ppw + q], eqr = piece_eq[wave * ppw + q];
#pragma unroll 1
        for (uint32_t e0 = 0; e0 < cnt; e0 += 4 * kWave) {
            uint32_t bits[4], at[4];
            int32_t l[4];
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const uint32_t en = e0 + z * kWave + lane;
                at[z] = en < cnt ? en : cnt - 1;
                bits[z] = ls.val[pc.at + at[z]];
            }
            if (ls.loc) {
#pragma unroll
                for (int z = 0; z < 4; ++z) l[z] = (int32_t)(base + ls.loc[pc.at + at[z]]);
            } else {
#pragma unroll
                for (int z = 0; z < 4; ++z) l[z] = (int32_t)(pc.at + at[z]);
            }
            if (map) {
#pragma unroll
                for (int z = 0; z < 4; ++z) l[z] = map[l[z] < len ? l[z] : len - 1];
            }
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                if (e0 + z * kWave >= cnt) break;                    // uniform over the wavefront
                const bool have = e0 + z * kWave + lane < cnt;
                const uint32_t key = bits[z] & 0x7fffffffu;
                const uint64_t gtm = __ballot(have && key > tau), eqm = __ballot(have && key == tau);
                const uint32_t eqb = eqr + (uint32_t)__popcll(eqm & below);
                if (have && (key > tau || (key == tau && eqb < k_eq))) {
                    const int64_t pos = (int64_t)gtr + __popcll(gtm & below) + (eqb < k_eq ? eqb : k_eq);
                    if (pos < k) {
                        idx[pos] = l[z];
                        if (val_sel) val_sel[pos] = __uint_as_float(bits[z]);
                    }
                }
                gtr += (uint32_t)__popcll(gtm);
                eqr += (uint32_t)__popcll(eqm);
            }
        }
    }
}

constexpr int kEstLdsBytes = 160 * 1024;
constexpr int64_t kGatherEstimateMaxTableBytes = 1 << 20, kGatherEstimateMaxD = (int64_t)1 << 22;

// Whether stage 3 goes through the plan.  A small table under a short vector stays in every L2: r gathers per coordinate in
// one launch then beat the two launches of the plan-driven recovery (C1: 6 us against 23), which is made for tables far
// larger than any cache.
bool estimate_wants_plan(const sams_ctx *ctx)
{
    const bool small = (int64_t)ctx->r * ctx->c * 4 <= kGatherEstimateMaxTableBytes && ctx->d <= kGatherEstimateMaxD;
    return ctx->tun.estimate_path == 2 || (ctx->tun.estimate_path == 0 && !small);
}
static bool estimate_by_plan(const sams_ctx *ctx) { return ctx->plan.srcp && estimate_wants_plan(ctx); }

// Rows that k_estimate_lds holds, 0 = it is not used.  It has to fill its LDS and to compute more per coordinate than the
// gathers wait for while their table stays in the 32 KB L1s; rows that it has no room for cost it more than the gathers.
// k_estimate_lds and gathers (us):
//   whole table held, d = 1 million (6 million): 5 x 9,001 11 and 19 (41 and 105), 3 x 5,000 7 and 8 (27 and 39), 5 x 2,406 8 and 8 (33 and 46),
//     5 x 1,000 8 and 8 (32 and 35), at two million 15 and 14; 7 x 2,406 at 1.1 million 16 and 14, at 1.5 17 and 18; 16 x 1,000
//     26 and 23 (119 and 125); 1 x 5,000 5 and 5 (18 and 16), 1 x 16,384 6 and 6 (21 and 28), 1 x 40,000 8 and 5 (36 and 22)
//   two rows held: 5 x 16,384 18 and 22 (78 and 118), 10 x 16,384 at 1.5 million 59 and 50, at three million 89 and 101
//   one: 3 x 32,768 16 and 15 (96 and 72), at 25.6 million 249 and 283
static int32_t estimate_held_rows(const sams_ctx *ctx)
{
    const int64_t table = ctx->r * ctx->c * 4, million = 1000000;
    const int32_t held = (int32_t)(kEstLdsBytes / (ctx->c * 4) < ctx->r ? kEstLdsBytes / (ctx->c * 4) : ctx->r);
    int64_t least;                                                   // the shortest vector
    if (held == ctx->r) least = table > 56 * 1024 && ctx->c > 2000 ? (ctx->c > 4096 ? million : 3 * million / 2) : 6 * million;
    else if (held >= 2) least = held * 3 >= ctx->r ? million : 3 * million;
    else least = 12 * million;
    const bool used = ctx->d >= least && ctx->c >= 2 && held * 5 >= ctx->r && (ctx->r > 1 || (ctx->c > 8192 && ctx->c <= 24576)) && ctx->tun.estimate_path != 1;
    return used && !estimate_by_plan(ctx) ? held : 0;
}

int estimate_prepare(const sams_ctx *ctx)
{
    if (!estimate_held_rows(ctx)) return SAMS_OK;
#define SAMS_CASE(R) (const void *)k_estimate_lds<R>
    const void *const kernels[SAMS_MAX_ROWS] = {SAMS_CASE(1),  SAMS_CASE(2),  SAMS_CASE(3),  SAMS_CASE(4), SAMS_CASE(5),  SAMS_CASE(6),
                                                SAMS_CASE(7),  SAMS_CASE(8),  SAMS_CASE(9),  SAMS_CASE(10), SAMS_CASE(11), SAMS_CASE(12),
                                                SAMS_CASE(13), SAMS_CASE(14), SAMS_CASE(15), SAMS_CASE(16)};
#undef SAMS_CASE
    SAMS_HIP(hipFuncSetAttribute(kernels[ctx->r - 1], hipFuncAttributeMaxDynamicSharedMemorySize, kEstLdsBytes));
    return SAMS_OK;
}

int enqueue_estimate(sams_ctx *ctx, const float *S_mean, const float *vhat, float *est, const SelScratch *sc, bool *hist_done)
{
    if (hist_done) *hist_done = false;
    const int block = 256;
    const int grid = grid_for(ctx->d, block);
    if (estimate_by_plan(ctx)) {
        bool done = false;
        SAMS_TRY(enqueue_estimates_planned_fused(ctx, S_mean, vhat, est, &done, sc));
        if (done) {
            if (hist_done) *hist_done = sc != nullptr;
            return SAMS_OK;
        }
        SAMS_TRY(enqueue_row_estimates_planned(ctx, S_mean, ctx->plan.rowest));
        switch (ctx->r) {
#define SAMS_CASE(R)                                                                                  \
    case R:                                                                                           \
        SAMS_LAUNCH(ctx, KID_EST_MEDIAN, (k_est_median<R>), grid, block, ctx->plan.rowest, vhat, est, \
                    ctx->d);                                                                          \
        break;
            SAMS_CASE(1) SAMS_CASE(2) SAMS_CASE(3) SAMS_CASE(4) SAMS_CASE(5) SAMS_CASE(6) SAMS_CASE(7)
            SAMS_CASE(8) SAMS_CASE(9) SAMS_CASE(10) SAMS_CASE(11) SAMS_CASE(12) SAMS_CASE(13)
            SAMS_CASE(14) SAMS_CASE(15) SAMS_CASE(16)
#undef SAMS_CASE
        default:
            return SAMS_EINVAL;
        }
        SAMS_HIP(hipGetLastError());
        return SAMS_OK;
    }
    if (const int32_t held = estimate_held_rows(ctx)) {
        const uint32_t m = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)ctx->c);
        const bool with_hist = sc && held * ctx->c * 4 + kHistBins * 4 <= kEstLdsBytes, pick = with_hist && sel_hist_picks(ctx->d);
        switch (ctx->r) {
#define SAMS_CASE(R)                                                                                                             \
    case R: {                                                                                                                    \
        ProfScope ps(ctx, KID_ESTIMATE);                                                                                         \
        hipLaunchKernelGGL(k_estimate_lds<R>, dim3(grid_for(ctx->d, 1024, 256)), dim3(1024),                                    \
                           (size_t)(held * ctx->c * 4 + (with_hist ? kHistBins * 4 : 0)), ctx->stream, S_mean, vhat, est, ctx->hp,  \
                           ctx->d, (int32_t)ctx->c, m, held, (uint32_t)ctx->k, pick ? sc->st : nullptr,                           \
                           with_hist ? sc->hist : nullptr);                                                                       \
        break;                                                                                                                   \
    }
            SAMS_CASE(1) SAMS_CASE(2) SAMS_CASE(3) SAMS_CASE(4) SAMS_CASE(5) SAMS_CASE(6) SAMS_CASE(7)
            SAMS_CASE(8) SAMS_CASE(9) SAMS_CASE(10) SAMS_CASE(11) SAMS_CASE(12) SAMS_CASE(13)
            SAMS_CASE(14) SAMS_CASE(15) SAMS_CASE(16)
#undef SAMS_CASE
        default:
            return SAMS_EINVAL;
        }
        if (hist_done) *hist_done = with_hist;
        SAMS_HIP(hipGetLastError());
        return SAMS_OK;
    }
    const bool with_hist = sc != nullptr;
    SelState *const st = with_hist && sel_hist_picks(ctx->d) ? sc->st : nullptr;
    switch (ctx->r) {
#define SAMS_CASE(R)                                                                                       \
    case R:                                                                                                \
        if (with_hist)                                                                                     \
            SAMS_LAUNCH(ctx, KID_ESTIMATE, (k_estimate<R, true>), grid_for(ctx->d, 1024, kEstHistGrid), 1024, S_mean, vhat, \
                        est, ctx->hp, ctx->d, ctx->c, (uint32_t)ctx->k, st, sc->hist);                     \
        else                                                                                               \
            SAMS_LAUNCH(ctx, KID_ESTIMATE, (k_estimate<R, false>), grid, block, S_mean, vhat, est, ctx->hp, \
                        ctx->d, ctx->c, 0u, nullptr, nullptr);                                             \
        break;
        SAMS_CASE(1) SAMS_CASE(2) SAMS_CASE(3) SAMS_CASE(4) SAMS_CASE(5) SAMS_CASE(6) SAMS_CASE(7)
        SAMS_CASE(8) SAMS_CASE(9) SAMS_CASE(10) SAMS_CASE(11) SAMS_CASE(12) SAMS_CASE(13)
        SAMS_CASE(14) SAMS_CASE(15) SAMS_CASE(16)
#undef SAMS_CASE
    default:
        return SAMS_EINVAL;
    }
    if (hist_done) *hist_done = with_hist;
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

bool sel_list_in_staging(const sams_ctx *ctx) { return ctx->sel_list == nullptr; }

SelScratch ctx_sel_scratch(const sams_ctx *ctx)
{
    uint32_t *list = sel_list_in_staging(ctx) ? reinterpret_cast<uint32_t *>(ctx->plan.stg) : ctx->sel_list;
    const int64_t nt = sel_tiles(ctx->d);
    const SelList ls = {list, reinterpret_cast<uint16_t *>(list + ctx->sel_cap + 64), ctx->sel_tile + 2 * nt,
                        reinterpret_cast<uint2 *>(ctx->sel_tile)};
    return SelScratch{reinterpret_cast<SelState *>(ctx->sel), ctx->sel + kSelStateWords, ctx->sel + kSelClearWords, ls, nt, ctx->sel_cap, false};
}

// The largest k for which k_sel_small's last workgroup finishes by itself: it takes 2 us per thousand listed keys, where the other
// kernels take 26 us (above 2^16 keys, without a first pass for tiles' histograms, 22) whatever the lists hold.  Both (topk_refine): 20,000
// keys, k = 5,000 17 and 26 us, 10,000 30 and 26 us; 65,536 keys, k = 8,192 25 and 26 us, 16,384 43 and 26 us, 65,536 142 and 26 us; 431,003,
// k = 500 16 and 30 us, 2,500 18 and 30 us, 4,311 22 and 30 us; 66,000, k = 3,000 17 and 25 us, 131,072 19 and 25; a million, k = 3,000 23
// and 32 us.  Above 2^16 keys the line lies lower than these say: keys whose errors a training run has fed back for long are closer to
// each other, and three times k of them share the first digits (whole steps after 600 to 1,000: 70,000 coordinates, k = 256 35 and
// 50 us; 131,000, 3,000 48 and 57; 200,000, 2,500 53 and 63; 300,000, 3,000 68.7 and 71; 431,003, 3,000 76.3 and 78.3, 4,311 83.1 and
// 80.4; 800,000, 2,500 114 and 117; a million, 2,000 136 and 141, 3,000 141 and 137).
constexpr int64_t kSelSmallMaxK = 1 << 13, kSelFlatMaxK = 2500, kSelFlatShortMaxK = 3000, kSelFlatShort = (int64_t)1 << 19;
// Tiles' lists are cut into pieces of at least 256 entries (about 1.5 k are listed) while there are fewer than 16 wavefronts for
// each of the 256 compute units.  Whole lists and pieces: 100,000 keys, k = 50,000 54 and 26 us; a million, half of them 62 and
// 33 us, an eighth 36 and 31 us; 4.96 million, half 82 and 72 us; with more pieces than that 30 million keys, half, take 350
// instead of 235 us.
constexpr int64_t kSelMaxPieces = 4096;
bool sel_hist_picks(int64_t len) { return len > kSelHistPickMin; }

int enqueue_select(sams_ctx *ctx, hipStream_t stream, const SelScratch &sc, const float *keys, int64_t len, int64_t k,
                   const int32_t *map, int32_t *idx, float *val_sel, bool hist_done)
{
    uint32_t *hist1 = sc.hist + kHistBins, *hist2 = hist1 + kHistBins / 2;
    const bool tiles = len <= kSelSmallMax;
    const int64_t small_k = tiles ? kSelSmallMaxK : len <= kSelFlatShort ? kSelFlatShortMaxK : kSelFlatMaxK;
    const bool small = len <= kSelFlatMax && k <= small_k;
    if (small && tiles && !hist_done) {
        const int grid = grid_for(len, 1 << kSelTileLog2);
        SAMS_LAUNCH_ON(ctx, stream, KID_SEL_HIST, k_sel_hist_tiles, grid, 1024, keys, len, sc.tile_hist, &sc.st->done[1]);
        SAMS_LAUNCH_ON(ctx, stream, KID_SEL_SMALL, (k_sel_small<true, kSelMaxTiles>), grid, 1024, keys, len, sc.st, sc.tile_hist, sc.list, k, map, idx,
                       val_sel);
        SAMS_HIP(hipGetLastError());
        return SAMS_OK;
    }
    // A selection that overlapped this one on another stream, or ended half-way, has left anything.  A launch of 2 us (4.96
    // million candidates 58 -> 60 us).
    if (sc.shared) SAMS_TRY(enqueue_fill_u32_on(ctx, stream, reinterpret_cast<uint32_t *>(sc.st), kSelClearWords, 0u));
    if (!hist_done) {
        if (sel_hist_picks(len))
            SAMS_LAUNCH_ON(ctx, stream, KID_SEL_HIST, k_sel_hist<true>, hist_grid(len), 1024, keys, len,
                           (uint32_t)k, sc.st, sc.hist);
        else
            SAMS_LAUNCH_ON(ctx, stream, KID_SEL_HIST, k_sel_hist<false>, hist_grid(len), 1024, keys, len,
                           (uint32_t)k, sc.st, sc.hist);
    }
    if (small) {
        if (tiles)
            SAMS_LAUNCH_ON(ctx, stream, KID_SEL_SMALL, (k_sel_small<false, kSelMaxTiles>), grid_for(len, 1 << kSelTileLog2), 1024, keys, len,
                           sc.st, sc.hist, sc.list, k, map, idx, val_sel);
        else
            SAMS_LAUNCH_ON(ctx, stream, KID_SEL_SMALL, (k_sel_small<false, kSelFlatTiles>), grid_for(len, 1 << kSelTileLog2), 1024, keys, len,
                           sc.st, sc.hist, sc.list, k, map, idx, val_sel);
        SAMS_HIP(hipGetLastError());
        return SAMS_OK;
    }
    const int64_t nt = (len + (1 << kSelTileLog2) - 1) >> kSelTileLog2;
    if (nt > sc.ntile_cap) return SAMS_EINVAL;
    int split = 0;
    while (split < 4 && (3 * k / 2 / nt >> split) > 4 * kWave && nt << split < kSelMaxPieces) ++split;
    const int64_t pieces = nt << split;
    const int lgrid = grid_for(pieces, 16, 128);
    const int ppw = pieces > 16384 ? kSelWriteMaxPpw : 1;            // at most a few thousand groups for a workgroup to add up
    const int wgrid = grid_for(pieces, 16 * ppw);
    SelList ls = sc.list;
    if (len > sc.cap)                                                // above kSelHistPickMin, so the digit has been picked
        ls = {reinterpret_cast<uint32_t *>(const_cast<float *>(keys)), nullptr, nullptr, sc.list.group};   // read only
    else if (sel_hist_picks(len))
        SAMS_LAUNCH_ON(ctx, stream, KID_SEL_FILTER, k_sel_filter<false>, (unsigned)nt, 1024, keys, len, sc.st, sc.hist, sc.list,
                       (uint32_t)k);
    else
        SAMS_LAUNCH_ON(ctx, stream, KID_SEL_FILTER, k_sel_filter<true>, (unsigned)nt, 1024, keys, len, sc.st, sc.hist, sc.list,
                       (uint32_t)k);
    SAMS_LAUNCH_ON(ctx, stream, KID_SEL_HIST, (split ? k_sel_list_hist<true> : k_sel_list_hist<false>), lgrid, 1024, sc.st, hist1, ls, len,
                   pieces, split, 1, sel_hist_picks(len) ? nullptr : sc.hist);
    SAMS_LAUNCH_ON(ctx, stream, KID_SEL_HIST, (split ? k_sel_list_hist<true> : k_sel_list_hist<false>), lgrid, 1024, sc.st, hist2, ls, len,
                   pieces, split, 2, nullptr);
    SAMS_LAUNCH_ON(ctx, stream, KID_SEL_COUNT, (split ? k_sel_count<true> : k_sel_count<false>), wgrid, 1024, sc.st, ls, len, pieces, split,
                   ppw);
    SAMS_LAUNCH_ON(ctx, stream, KID_SEL_WRITE, (split ? k_sel_write<true> : k_sel_write<false>), wgrid, 1024, sc.st, ls, len, pieces, split,
                   ppw, k, map, idx, val_sel);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

}  // namespace sams

// Order-preserving Count Sketch accumulation (stage 1 of sams.h; Sec. II-C update rule) for narrow tables, without staging.
//
// The binned path (sams_plan.hip) writes every signed value to where its bucket's window will read it and reads it
// back: 8 bytes of memory traffic per (worker, row, coordinate), and a window that few workgroups share when the table
// is small.  A narrow table turns that round: the workgroups pull.  The vector is cut into tiles that fit in LDS; a
// workgroup has one worker, one row and a range of its slices of 64 buckets (a window), walks the worker's tiles in order, and every
// lane of a wavefront owns one bucket of each of its slices -- one, or up to sixteen --, with the sum in a register.  Which
// coordinates of a tile a bucket takes is worked out once, at context creation: lists of steps, each of 64 entries, one per lane -- the
// coordinate inside the tile and its sign --, padded with an entry that points at a zero; the lists of a wavefront lie one after the
// other, as one stream, which a lane reads 16 bytes at a time.  With one or two slices per wavefront a list is that of a (row, tile,
// slice); with more it is that of four slices, a word (two steps) of each in every load: four sums that do not wait for each other, and
// one test for the list's end in eight steps.  A lane takes its entries in ascending coordinate order, so the sums are those of a
// sequential loop over the coordinates, bit for bit (adding the padding's zero changes nothing: a sum that starts at +0 is never -0; a
// value is added as fma(value, +-1, sum), which rounds once, like the addition).  No atomics, no exchange between lanes, one barrier
// per tile.
// Vectors of more than 2^22 coordinates, whose sums need not be in that order, may be cut into parts: workgroups of their
// own make a table of every part, and the tables are added up part after part, always the same way.
//
// Cost: every workgroup reads its worker's whole vector, or part, through the L2: the workgroups that walk the same tiles, and those of
// other workers with the same lists, have consecutive numbers on one XCD (worker by worker only, the lists of 25.6 million
// coordinates, n = 4, 5 x 10,000 came from memory four times: 513 -> 434 us).
// Bound by what one compute unit takes in from the L2 (a tile of 52 KB in 0.5 us, 105 GB/s) and by the steps of the lists, 3.5 ns each (a
// wavefront's read of 64 scattered values; the LDS is busy a third of the time, the vector units half, the rest is latencies of
// 14 wavefronts); the two hardly overlap.  Two tiles are under way while a third is added: that takes a barrier of its own
// (tile_barrier), since __syncthreads lets the loaders wait for all they have asked for, and one tile then took 0.65 us (431,003
// coordinates, n = 5, 4 x 9,001 37.5 -> 29 us).  Counters in LDS in place of the barrier, so that the wavefronts need not walk in step,
// cost more than they give (29 -> 48 us: their latency is in every tile); so does reading a load's values before the one in front
// of it is added (70 -> 78 us at a million, n = 20, 5 x 12,000).
// What a list holds beyond its coordinates is by the row's hash: 1.5 to 3.1 entries per coordinate in 28 of 30 rows of 10,000
// buckets, 5.5 and 5.8 in the others; 2.7 with 9,001, 1.35 with 400.  A row with long lists gets more windows (pull_share).
// Measured on MI355X (us), lists with at most four slices per wavefront, one list per slice, 4- to 16-byte loads of their words and the
// same number of windows for every row, and this kernel: 25.6 million, n = 4, 5 x 10,000 680 to 1,030 by the hash, now 340 to 530;
// 12 million, n = 8, 5 x 16,384 757, 500; four million, n = 50, 5 x 12,000 1,290, 840; a million, n = 20, 5 x 12,000 172, 70; six
// million, n = 8, 4 x 700 142, 84; 431,003, n = 5, 4 x 9,001 37.5, 25 to 29 by the hash; 65,536, n = 4, 5 x 2,048 9.0, 7.6; 60,000, 5 x 400, n = 50
// 10.8, 10.3; n = 100 20, 18.7.  The binned path: 98 and 130 us at the last two, 103 at 431,003, 8.5 ms at 25.6 million.
// A context with lists is made in 0.10 ms at 65,536, 0.32 at 431,003, 2.9 at 25.6 million; two waits for the stream and the choice of
// windows on the host are in it.
#include <stdlib.h>

#include "sams_ctx.h"

#pragma clang fp contract(off)

namespace sams {

constexpr int kPullThreads = 1024;
constexpr int kPullLoaders = 2;               // wavefronts that bring the tiles in; the others add
constexpr int kPullAdders = kPullThreads / kWave - kPullLoaders;
constexpr int kPullLoads = 26;                // 1 KiB loads per tile and loader
constexpr int kPullZero = kPullLoaders * kPullLoads * 256;           // floats of a tile; a zero lies behind them
constexpr int kPullTile = kPullZero - 4;      // coordinates per tile: up to 3 floats of the buffer lie in front of them
constexpr int kPullBuf = kPullZero + 16;      // floats of a tile buffer
constexpr int kPullBufs = 3;
constexpr int kPullLds = (kPullBufs * kPullBuf + kWave) * 4;
constexpr int kPullAhead = 4;                 // tiles that the loaders are ahead with fetching into the L2
constexpr int kPullLoad = 4;                  // words that a lane reads with one load
constexpr int kPullDepth = 6;                 // such loads on their way ahead of the words being added
constexpr int kPullSpare = 2 * kPullLoad * kPullDepth;   // words of a lane behind the last list: the adders' loop goes in turns of kPullDepth
                                              // loads, each refilled, so it reads up to 2 kPullDepth - 1 loads past its own
constexpr int kPullMany = 4;                  // most lists of four slices per wavefront
constexpr int kPullPair = 2;                  // most lists of one slice per wavefront
constexpr int kPullMaxList = 512;             // longest list of one bucket in one tile
// A word holds two consecutive steps of a lane: the first step's coordinate in bits 2-15 (so that it is a byte offset) and
// its sign in bit 0, the second's in bits 17-30 and 31.  Bit 1 of the first word of a list's last unit, in every lane, ends the list.

// ------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------
// Where the lists are.  A list is that of a tile, a row and per_list slices (one, or four whose words take turns); row j's lists
// of a tile are shared out over row[j + 1].win0 - row[j].win0 windows of per_win lists, and a window's over the adders, per_wave
// each.  A wavefront's lists of its part of the tiles, tile by tile, are one stream.
struct PullOrder {
    int32_t ntile, nslice, nlist;
    int32_t per_list, group;          // slices of a list; words of a lane in a list's smallest unit
    int32_t most;                     // lists that a wavefront may have: 1 or kPullPair of one slice, kPullMany of four
    int32_t parts, per_part, windows; // windows: of all rows
    PullRow row[SAMS_MAX_ROWS + 1];
};
__host__ __device__ __forceinline__ int64_t stream_number(const PullOrder &po, int part, int window, int wave)
{
    return ((int64_t)part * po.windows + window) * kPullAdders + wave;
}
// the lists [first, first + count) of a row that wavefront `wave` of a window has; count <= 0: none
__host__ __device__ __forceinline__ void lists_of(const PullOrder &po, int j, int window, int wave, int32_t *first, int32_t *count)
{
    const PullRow &row = po.row[j];
    const int32_t w0 = (window - row.win0) * row.per_win, w1 = w0 + row.per_win < po.nlist ? w0 + row.per_win : po.nlist;
    *first = w0 + wave * row.per_wave;
    *count = *first + row.per_wave < w1 ? row.per_wave : w1 - *first;
}
__device__ __forceinline__ int64_t list_number(const PullOrder &po, int j, int64_t tile, int list)
{
    return ((int64_t)j * po.ntile + tile) * po.nlist + list;
}

// per (row, every step-th tile): the longest of the 64 columns of every slice, at len[(row * gridDim.x + blockIdx.x) * nslice + slice]
__global__ void __launch_bounds__(1024)
k_pull_count(HashParams hp, int64_t d, int32_t step, int32_t nslice, uint16_t *__restrict__ len)
{
    extern __shared__ uint32_t cnt[];                                // [nslice * 64]
    const int j = blockIdx.y;
    const int64_t l0 = (int64_t)blockIdx.x * step * kPullTile;
    const int lim = d - l0 < kPullTile ? (int)(d - l0) : kPullTile;
    for (int b = threadIdx.x; b < nslice * kWave; b += 1024) cnt[b] = 0;
    __syncthreads();
    for (int p = threadIdx.x; p < lim; p += 1024) atomicAdd(&cnt[bucket_of(hp, j, (uint32_t)(l0 + p))], 1u);
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int s = wave; s < nslice; s += 16) {
        uint32_t m = cnt[s * kWave + lane];
        for (int off = kWave / 2; off; off >>= 1) {
            const uint32_t o = __shfl_xor(m, off);
            m = o > m ? o : m;
        }
        if (lane == 0) len[((int64_t)j * gridDim.x + blockIdx.x) * nslice + s] = (uint16_t)m;
    }
}

// per (tile, row): the lists.  len, off: every list's units, and the units before it
__global__ void __launch_bounds__(1024)
k_pull_place(HashParams hp, int64_t d, PullOrder po, const uint16_t *__restrict__ len, const uint32_t *__restrict__ off,
             uint32_t *__restrict__ lists)
{
    const int nslice = po.nlist * po.per_list;                       // the last list's slices may lie behind the row
    extern __shared__ uint32_t end[];                                // [nslice * 64] list ends, then kPullTile 16-bit entries
    __shared__ uint32_t part[16];
    uint16_t *ent = reinterpret_cast<uint16_t *>(end + nslice * kWave);
    const int t = threadIdx.x, j = blockIdx.y;
    const int64_t l0 = (int64_t)blockIdx.x * kPullTile;
    const int lim = d - l0 < kPullTile ? (int)(d - l0) : kPullTile;
    const int nb = nslice * kWave;
    for (int b = t; b < nb; b += 1024) end[b] = 0;
    __syncthreads();
    for (int p = t; p < lim; p += 1024) atomicAdd(&end[bucket_of(hp, j, (uint32_t)(l0 + p))], 1u);
    __syncthreads();
    // exclusive prefix: thread t has the buckets [t * per, (t + 1) * per)
    const int per = (nb + 1023) / 1024;
    uint32_t sum = 0;
    for (int b = t * per; b < (t + 1) * per && b < nb; ++b) sum += end[b];
    uint32_t run = block_exclusive_scan<1024>(sum, part);
    for (int b = t * per; b < (t + 1) * per && b < nb; ++b) {
        const uint32_t c = end[b];
        end[b] = run;
        run += c;
    }
    __syncthreads();
    // end[b] grows from the start of list b to its end while the coordinates are dealt out, in no fixed order
    for (int p = t; p < lim; p += 1024) {
        const uint32_t at = atomicAdd(&end[bucket_of(hp, j, (uint32_t)(l0 + p))], 1u);
        ent[at] = (uint16_t)(p | (sign_neg(hp, j, (uint32_t)(l0 + p)) ? 0x8000 : 0));
    }
    __syncthreads();
    // ascending coordinates: insertion (the lists are short, see kPullMaxList, and nearly in order)
    for (int b = t; b < nb; b += 1024) {
        const uint32_t lo = b ? end[b - 1] : 0u, hi = end[b];
        for (uint32_t q = lo + 1; q < hi; ++q) {
            const uint16_t e = ent[q];
            uint32_t x = q;
            for (; x > lo && (ent[x - 1] & 0x7fff) > (e & 0x7fff); --x) ent[x] = ent[x - 1];
            ent[x] = e;
        }
    }
    __syncthreads();
    const int lane = t & (kWave - 1), wave = t / kWave;
    for (int s = wave; s < nslice; s += 16) {
        const int64_t o = list_number(po, j, blockIdx.x, s / po.per_list);
        const int b = s * kWave + lane;
        const uint32_t lo = b ? end[b - 1] : 0u, hi = end[b];
        // word q of the slice's list in its units: of one slice, the words of a unit lie side by side in a lane, and so do those of
        // as many units as a load holds; of four, a word of each is a load
        const bool many = po.per_list > 1;
        const uint32_t words = (uint32_t)len[o] * (many ? 1u : (uint32_t)po.group);
        const int64_t w0 = (int64_t)off[o] * po.group + (many ? s % po.per_list : 0), step = many ? kPullLoad : 1;
        for (uint32_t q = 0; q < words; ++q) {
            const uint32_t e0 = lo + 2 * q < hi ? ent[lo + 2 * q] : (uint32_t)kPullZero,
                           e1 = lo + 2 * q + 1 < hi ? ent[lo + 2 * q + 1] : (uint32_t)kPullZero;
            const uint32_t unit = many ? 1u : (uint32_t)po.group, end_flag = q % unit == 0 && q + unit >= words ? 2u : 0u;
            const int64_t at = w0 + q * step;
            lists[(at / kPullLoad * kWave + lane) * kPullLoad + at % kPullLoad] =
                ((e0 & 0x7fffu) << 2) | (e0 >> 15) | ((e1 & 0x7fffu) << 17) | ((e1 >> 15) << 31) | end_flag;
        }
    }
}

// ------------------------------------------------------------------------------------------
// accumulation
// ------------------------------------------------------------------------------------------
struct PullArgs {
    const float *u;
    const uint32_t *lists;
    const uint2 *first;               // per stream: its first load of words, its units
    float *S;                         // [parts][n][r][c]
    int64_t d, c, total;              // total = n * d
    int32_t n, r;
    PullOrder po;
};

// 16 bytes per lane from memory straight to LDS: lane x's go to dst + 16 x bytes.  src: this lane's.
__device__ __forceinline__ void load_to_lds16(const float *src, float *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

__device__ __forceinline__ void load_to_lds4(const float *src, float *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
}

// The barrier between two tiles.  Not __syncthreads: the compiler puts a wait for every load that is under way in front of
// that, the next tile's among them.  LDS accesses of a wavefront happen in order, an adder's values have been used when it gets
// here, and a loader has waited for its part of the tile; the LDS writes before the first tile are waited for.
__device__ __forceinline__ void tile_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Three tile buffers: the loaders bring the next two tiles in while the adders work on the third.  The two kinds wait for
// their own loads only (a wavefront's loads come back in order: one that fetched both would wait for the whole next
// tile before each list).  The adders' loop is a stream of words: a load is issued for every one used up, unconditionally and
// straight into the registers that the loop carries, so that the compiler waits for exactly the oldest.
// Up to MOST lists per wavefront, whose sums take turns.
// MANY = false: lists of a slice, of units of W words, whose values are read from LDS together and added in order.
// MANY: lists of four slices, a word of each per load.
template <int W, bool MANY, int MOST>
__global__ void __launch_bounds__(kPullThreads)
k_sketch_pull(PullArgs a)
{
    extern __shared__ float buf[];                                   // [kPullBufs][kPullBuf], and 64 words nobody reads
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    // workgroups are dealt round-robin to the 8 XCDs: consecutive (worker, row, window) triples to one XCD
    const int64_t per = (int64_t)gridDim.x / 8, q = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    const PullOrder &po = a.po;
    const int32_t rw = po.windows;                                   // workgroups that walk the same tiles of a worker
    if (q >= (int64_t)a.n * po.parts * rw) return;
    const int32_t i = (int32_t)(q / rw) % a.n, part = (int32_t)(q / rw) / a.n, win = (int32_t)(q % rw);
    int32_t j = 0;
    while (win >= po.row[j + 1].win0) ++j;
    const int32_t t0 = part * po.per_part, ntile = po.ntile - t0 < po.per_part ? po.ntile - t0 : po.per_part;
    // worker i's vector starts `mis` floats past a 16-byte boundary; the tiles are loaded from that boundary on
    const int64_t row0 = (int64_t)i * a.d;
    const int mis = (int)(row0 & 3);
    if (t < kPullBufs * 16) buf[(t / 16) * kPullBuf + kPullZero + t % 16] = 0.f;
    if (wave >= kPullAdders) {
        const int w = wave - kPullAdders;
        const int64_t last4 = (a.total - 4) & ~(int64_t)3;           // the last whole 16-byte group of u
        // The workgroups of a worker walk in step, so that every tile would come from HBM while all of them wait: each
        // also fetches a share of a later tile's 128-byte lines into the XCD's L2.  The shares of up to 16 workgroups make
        // the tile (with fewer than 4 part of it); with more, several fetch the same.
        int groups = 16;
        while (groups > rw) groups >>= 1;
        const int lines = kPullBuf / 32 / groups;
        const int64_t ahead = (int64_t)kPullAhead * kPullTile + ((int64_t)(q % groups) * lines + (w * kWave + lane) % lines) * 32;
        // tile tl to its buffer, and the share of a later tile.  Groups past the last whole one of u are replaced by it: never
        // read by an adder, except for the up to three values put right below.
        auto load = [&](int32_t tl) {
            float *dst = buf + (tl % kPullBufs) * kPullBuf;
            const int64_t at = row0 - mis + (int64_t)(t0 + tl) * kPullTile;   // flat position in u of the buffer's start
            if (at + kPullZero <= last4) {                           // uniform; without the limit on the address half the instructions
                const float *src = a.u + at + (w * kWave + lane) * 4;
#pragma unroll
                for (int g = 0; g < kPullLoads; ++g)
                    load_to_lds16(src + g * kPullLoaders * kWave * 4, dst + (g * kPullLoaders + w) * kWave * 4);
            } else {
#pragma unroll
                for (int g = 0; g < kPullLoads; ++g) {
                    const int chunk = g * kPullLoaders + w;
                    const int64_t f = at + (chunk * kWave + lane) * 4;
                    load_to_lds16(a.u + (f < last4 ? f : last4), dst + chunk * kWave * 4);
                }
            }
            const int64_t fa = at + ahead;
            load_to_lds4(a.u + (fa < last4 ? fa : last4), buf + kPullBufs * kPullBuf);
        };
        load(0);
        if (ntile > 1) load(1);
        for (int32_t tl = 0; tl < ntile; ++tl) {
            // tile tl is there; its share of a later tile, and tile tl + 1, may be under way
            if (tl + 1 < ntile) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPullLoads + 2) : "memory");
            else asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
            const int64_t at = row0 - mis + (int64_t)(t0 + tl) * kPullTile, f = a.total & ~(int64_t)3;
            if (f - at < kPullZero) {                                // u's last, partial group: in the last worker's last tile or
                const int p = (int)(f - at);                         // the one before it, by the wavefront that loaded its chunk
                if (p / 4 / kWave % kPullLoaders == w && lane < (int)(a.total & 3))
                    buf[(tl % kPullBufs) * kPullBuf + p + lane] = a.u[f + lane];
            }
            tile_barrier();                                          // the adders have done with tile tl - 1, whose buffer tl + 2 takes
            if (tl + 2 < ntile) load(tl + 2);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the LDS is given back with nothing under way
        return;
    }
    int32_t l0, lists;
    lists_of(po, j, win, wave, &l0, &lists);
    if (lists <= 0) {                                                // only the barriers
        for (int32_t tl = 0; tl < ntile; ++tl) tile_barrier();
        return;
    }
    typedef uint32_t vec4u __attribute__((ext_vector_type(kPullLoad)));
    const uint2 mine = a.first[stream_number(po, part, win, wave)];
    const vec4u *src = reinterpret_cast<const vec4u *>(a.lists) + (int64_t)mine.x * kWave + lane;
    const int32_t ng = (int32_t)mine.y;
    vec4u ring[kPullDepth];
#pragma unroll
    for (int z = 0; z < kPullDepth; ++z) {
        ring[z] = src[(int64_t)z * kWave];                           // kPullSpare words end the array
        __builtin_amdgcn_sched_barrier(0);
    }
    src += (int64_t)kPullDepth * kWave;
    constexpr int kPer = MANY ? kPullLoad : 1;                       // slices of a list
    float x[MOST * kPer], sum[kPer];                                 // sum: of the list that is being added, in place of its x
#pragma unroll
    for (int p = 0; p < MOST * kPer; ++p) x[p] = 0.f;
#pragma unroll
    for (int y = 0; y < kPer; ++y) sum[y] = 0.f;
    int32_t turn = 0;                                                // that list
    const char *base = reinterpret_cast<const char *>(buf + mis);
    int32_t left = kPullBufs;                                        // buffers until the first one again
    tile_barrier();                                                  // tile 0 is there
    auto value = [&](uint32_t slot) { return *reinterpret_cast<const float *>(base + slot); };
    auto add = [&](float &to, uint32_t w, float v0, float v1) {
        to = __builtin_fmaf(v0, __uint_as_float(0x3f800000u | (w << 31)), to);
        to = __builtin_fmaf(v1, __uint_as_float(0x3f800000u | (w & 0x80000000u)), to);
    };
    auto tile_done = [&](bool more) {
        if (more) tile_barrier();                                    // the next tile is there
        base += kPullBuf * 4;
        if (--left == 0) {
            base -= kPullBufs * kPullBuf * 4;
            left = kPullBufs;
        }
    };
    constexpr int kGroups = MANY ? 1 : kPullLoad / W;                // units of a load
    for (int32_t m0 = 0; m0 < ng; m0 += kPullDepth * kGroups) {
#pragma unroll
        for (int z = 0; z < kPullDepth; ++z) {
            const vec4u w = ring[z];
            if constexpr (MANY) {
                const int32_t m = m0 + z;
                if (m < ng) {                                        // uniform; false only past the stream's end
                    float v[2 * kPullLoad];
#pragma unroll
                    for (int y = 0; y < kPullLoad; ++y) {
                        v[2 * y] = value(w[y] & 0xfffcu);
                        v[2 * y + 1] = value((w[y] >> 15) & 0xfffcu);
                    }
#pragma unroll
                    for (int y = 0; y < kPullLoad; ++y) add(sum[y], w[y], v[2 * y], v[2 * y + 1]);
                    if (__builtin_amdgcn_readfirstlane((int)w[0]) & 2) {         // the list ends
#pragma unroll
                        for (int y = 0; y < kPullLoad; ++y) x[turn * kPer + y] = sum[y];
                        turn = turn + 1 < lists ? turn + 1 : 0;
#pragma unroll
                        for (int y = 0; y < kPullLoad; ++y) sum[y] = x[turn * kPer + y];
                        if (turn == 0) tile_done(m + 1 < ng);
                    }
                }
            } else {
#pragma unroll
                for (int y = 0; y < kGroups; ++y) {
                    const int32_t m = m0 + z * kGroups + y;
                    if (m >= ng) continue;                           // uniform; only past the stream's end
                    float v[2 * W];
#pragma unroll
                    for (int p = 0; p < W; ++p) {
                        v[2 * p] = value(w[y * W + p] & 0xfffcu);
                        v[2 * p + 1] = value((w[y * W + p] >> 15) & 0xfffcu);
                    }
#pragma unroll
                    for (int p = 0; p < W; ++p) add(sum[0], w[y * W + p], v[2 * p], v[2 * p + 1]);
                    if (__builtin_amdgcn_readfirstlane((int)w[y * W]) & 2) {     // the list ends
                        if (MOST > 1 && lists > 1) {                 // x[1]: the sum of the one that waits
                            const float other = x[1];
                            x[1] = sum[0];
                            sum[0] = other;
                            turn ^= 1;
                        }
                        if (turn == 0) tile_done(m + 1 < ng);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            ring[z] = src[(int64_t)z * kWave];
            __builtin_amdgcn_sched_barrier(0);
        }
        src += (int64_t)kPullDepth * kWave;
    }
#pragma unroll
    for (int y = 0; y < kPer; ++y) x[y] = sum[y];                    // the last tile's lists have ended
    float *out = a.S + (((int64_t)part * a.n + i) * a.r + j) * a.c;
#pragma unroll
    for (int p = 0; p < MOST * kPer; ++p) {
        const int64_t b = (int64_t)(l0 * kPer + p) * kWave + lane;
        if (p < lists * kPer && b < a.c) out[b] = x[p];
    }
}

// the parts' tables added up, part after part
__global__ void __launch_bounds__(256)
k_pull_sum(const float *__restrict__ part, float *__restrict__ S, int64_t cells, int32_t parts)
{
    const int64_t q = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (q >= cells) return;
    float x = 0.f;
    for (int32_t p0 = 0; p0 < parts; p0 += 8) {                      // eight loads in flight
        float v[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) v[z] = part[(int64_t)(p0 + z < parts ? p0 + z : parts - 1) * cells + q];
#pragma unroll
        for (int z = 0; z < 8; ++z)
            if (p0 + z < parts) x = (x + v[z]);
    }
    S[q] = x;
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
// Whether this shape may pull (see pull_declines, and pull_create on its lists).  Tables of 128 to 2^15 buckets under vectors of up to
// 2^26 coordinates.  With fewer buckets a bucket's list gets too long to sort by insertion at creation, with more the lists of a
// tile's 64 buckets are padding but for a tenth (13,308 coordinates and a step or two for each of 512 slices), and their making would
// not fit in LDS; the lists of longer vectors take gigabytes.
constexpr int64_t kPullLongD = 1000000;       // shorter vectors always pull: both paths are launches and latencies
constexpr int64_t kPullWide = 1 << 14, kPullMaxC = 1 << 15, kPullWideMinD = 1 << 18;
static bool pull_shape(const sams_ctx *ctx, const Tunables &tun)
{
    if (tun.sketch_path != 0 || tun.estimate_path == 2 || tun.win_log2 || tun.tile_log2 || tun.chunk_log2 || tun.acc_threads ||
        tun.stage_rows)
        return false;                                                // the caller asks for the binned path or for a shape of it
    if (ctx->c > kPullWide && ctx->d < kPullWideMinD && !tun.pull_lists) return false;
    return ctx->c >= 128 && ctx->c <= kPullMaxC && ctx->d <= ((int64_t)1 << 26) && (int64_t)ctx->n * ctx->d >= 4;
}

// units of a list: of one slice, `group` words of two steps; of several, a word of each
static inline uint32_t list_units(const PullOrder &po, const uint16_t *longest, int32_t list)
{
    uint32_t m = 0;
    for (int32_t s = list * po.per_list; s < (list + 1) * po.per_list && s < po.nslice; ++s) m = longest[s] > m ? longest[s] : m;
    const uint32_t steps = po.per_list > 1 ? 2u : 2u * (uint32_t)po.group;
    return m ? (m + steps - 1) / steps : 1u;
}

// Shares the rows' lists out over windows and the vector over parts (where the order of the additions is not promised, above 2^22
// coordinates), for one of the two kernels; steps[j]: of row j's lists in a tile, all lists together.  A row whose hash makes long
// lists gets more windows: a launch waits for its slowest workgroup (25.6 million, n = 4, 5 x 10,000 with a row of twice the others'
// lists 434 -> 340 us, with two rows of four times 711 -> 530).  Returns the time it should take, in ns: workgroups run in rounds of 256,
// one per compute unit; a tile takes a workgroup kTileNs to take in, and kStepNs per step of its lists, or kChainNs per step
// of the wavefront with the most; measured / returned at 76 shapes 0.5 to 1.4, in the middle 0.95.
static int64_t pull_share(const sams_ctx *ctx, PullOrder &po, const double *steps)
{
    const bool many = po.per_list > 1;
    const double kTileNs = 450, kStepNs = 3.0, kChainNs = many ? 20 : 30, kStartNs = ctx->d > kOrderedSingleBinMaxD ? 20000 : 5000;
    const int32_t most_lists = kPullAdders * po.most, least = (po.nlist + most_lists - 1) / most_lists;
    const int32_t most_parts = ctx->d > kOrderedSingleBinMaxD ? (po.ntile < 128 ? po.ntile : 128) : 1;
    double best = 1e30;
    for (int32_t parts = 1; parts <= most_parts; ++parts) {
        const int32_t per_part = (po.ntile + parts - 1) / parts;
        const int64_t fewest = (int64_t)ctx->n * parts * ctx->r * least, first = (fewest + 255) / 256;
        for (int64_t rounds = first; rounds <= first + 1; ++rounds) {
            int32_t win[SAMS_MAX_ROWS];
            int64_t windows = 0;
            for (int j = 0; j < ctx->r; ++j) windows += win[j] = least;
            double worst = 0;
            for (;;) {                                               // a window more for the row whose windows take longest
                int at = 0;
                worst = 0;
                for (int j = 0; j < ctx->r; ++j) {
                    const int32_t per_win = (po.nlist + win[j] - 1) / win[j], per_wave = (per_win + kPullAdders - 1) / kPullAdders;
                    const double all = steps[j] / win[j] * kStepNs, chain = steps[j] / po.nlist * per_wave * kChainNs, x = all > chain ? all : chain;
                    if (x > worst) {
                        worst = x;
                        at = j;
                    }
                }
                if ((windows + 1) * parts * ctx->n > rounds * 256 || win[at] >= po.nlist) break;
                ++win[at];
                ++windows;
            }
            const double cost = (double)rounds * (per_part * (kTileNs + worst) + kStartNs);
            if (cost >= best) continue;
            best = cost;
            po.parts = (po.ntile + per_part - 1) / per_part;
            po.per_part = per_part;
            po.windows = 0;
            for (int j = 0; j < ctx->r; ++j) {
                PullRow &row = po.row[j];
                row.per_win = (po.nlist + win[j] - 1) / win[j];
                row.per_wave = (row.per_win + kPullAdders - 1) / kPullAdders;
                row.win0 = po.windows;
                po.windows += (po.nlist + row.per_win - 1) / row.per_win;
            }
            po.row[ctx->r] = PullRow{po.windows, 0, 0};
        }
    }
    return (int64_t)best;
}

// Whether the context takes the binned path (or, above 2^22 coordinates, LDS atomics) all the same.  Of 76 shapes with 0.4 to 20 million
// coordinates, 1 to 64 workers, 1 to 10 rows and 128 to 16,384 buckets the lists are the faster at 74, two to ten times so at most; not
// where few pairs walk a long vector through few short streams: one row of 4,096 under four million coordinates, n = 1, 161 and
// 106 us, three of 3,000, n = 2, 193 and 175 us.  In ns, as both were before the lists came in groups of four slices, and the line is
// where it was: 820 per tile here, there a base, 0.67 per position of a window's stream and 1.6 per thousand terms.  Many pairs under
// wide tables are no exception: of 16 shapes with 1 to 20 million coordinates, 160 to 600 pairs and 9,001 to 16,384 buckets, two hashes
// each, lists are the faster at all, 1.03 to 2.7 times (5 x 16,384, n = 50, four million 1.27 and 1.48 by the hash, and 1.92 ms).
// Above 2^14 buckets the line is the cost that pull_share returns against 1.75 ns per thousand terms by bins: of 66 shapes with 0.27 to
// 21 million coordinates and 16,400 to 32,700 buckets the lists are the faster at 65, 1.0 to 2.5 times up to 2^22 coordinates (where
// one of 40 others, 7 x 29,777 and n = 32 under 2.6 million, lost with 1,288 us to 1,005), two to 26 times above, where the others are
// LDS atomics.
// Pulling also leaves the head and the recovery without the plan ("fuse_head" has nothing to stage, estimates are gathered).  Whole steps of 30
// shapes up to 2^22 coordinates with 3 to 16 rows and 2 to 97 workers that pull, by lists and by bins: lists 1.03 to 1.9 times as
// fast at 28, 24 of them with "fuse_head" 2 (10 x 27,000, n = 8, 2.5 million 570 and 712 us; 10 x 20,000, n = 8, a million 221 and 376), and 1.01 times
// slower at two of those (10 x 19,102, n = 23, a million 628 and 622; 16 x 32,768, n = 10, four million 1,717 and 1,692).
static bool pull_declines(const sams_ctx *ctx, int32_t ntile)
{
    const int64_t pairs = (int64_t)ctx->n * ctx->r;
    if (ctx->d < kPullLongD) return false;
    if (ctx->d > kOrderedSingleBinMaxD || ctx->c > (1 << 12) || pairs * ((ctx->c + 127) / 128) >= 2048) return false;
    return 25000 + 86 * ctx->d / ctx->c + pairs * ctx->d * 16 / 10000 < ((int64_t)ntile + 12) * 820;
}

// SAMS_OK with *done saying whether the context pulls; device memory that cannot be had means it does not.  limit: what another path is taken to need, in ns
int pull_create(sams_ctx *ctx, const Tunables &tun, double limit, bool *done)
{
    *done = false;
    PullPlan pp = {};
    const int32_t ntile = (int32_t)((ctx->d + kPullTile - 1) / kPullTile), nslice = (int32_t)((ctx->c + kWave - 1) / kWave);
    if (!pull_shape(ctx, tun) || (!tun.pull_lists && pull_declines(ctx, ntile))) return SAMS_OK;
    const int64_t rows = (int64_t)ctx->r * ntile;                    // (row, tile) pairs
    uint16_t *cnt = nullptr, *len = nullptr;                         // build-time only
    uint32_t *off = nullptr;
    uint16_t *h_cnt = (uint16_t *)malloc((size_t)(rows * nslice) * 2), *h_len = (uint16_t *)malloc((size_t)(rows * nslice) * 2);
    uint32_t *h_off = (uint32_t *)malloc((size_t)(rows * nslice) * 4), *h_first = nullptr;
    int rc = SAMS_OK;
    do {
        if (!h_cnt || !h_len || !h_off || hipMalloc((void **)&cnt, (size_t)(rows * nslice) * 2) != hipSuccess) break;
        const dim3 grid((unsigned)ntile, (unsigned)ctx->r);
        const int lds_max = kPullLds;                                // more than the other two kernels need
        hipError_t e = hipFuncSetAttribute((const void *)k_pull_count, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_pull_place, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        // every step-th tile's longest columns, to the host
        auto count = [&](int32_t step) {
            const int64_t tiles = (ntile + step - 1) / step;
            {
                ProfScope ps(ctx, KID_PLAN_BUILD);
                hipLaunchKernelGGL(k_pull_count, dim3((unsigned)tiles, (unsigned)ctx->r), dim3(1024), (size_t)nslice * kWave * 4, ctx->stream,
                                   ctx->hp, ctx->d, step, nslice, cnt);
            }
            e = hipMemcpyAsync(h_cnt, cnt, (size_t)(ctx->r * tiles * nslice) * 2, hipMemcpyDeviceToHost, ctx->stream);
            if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
            if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; }
            return e == hipSuccess;
        };
        // What the choice rests on: up to 64 tiles of each row.  A wide table may be declined, and is counted whole only then.
        const bool wide = ctx->c > kPullWide;
        const int32_t sample = (ntile + 63) / 64, counted = wide ? sample : 1;
        if (!count(counted)) break;
        // Both kernels' lists, and how they would be shared out.  Lists of one slice (not for a wide table: none was faster) in units of
        // eight steps where a tile has many entries for a bucket, else of four (5 x 4,096, n = 8, two million: 112 and 105 us; 9,001:
        // 29 and 25; 2,048: 7.1 and 6.8; 400: alike)
        PullOrder po = {};
        int64_t cost = INT64_MAX;
        double steps = 0, per_tile[SAMS_MAX_ROWS], all = 0;
        // Two lists of a slice per wavefront save a round of workgroups where a row has 15 to 28 slices (45 x 5 pairs of 1,020 buckets, 77,028
        // coordinates: 16.1 us with one, 11.8 with two, 14.4 with lists of four slices, of which four wavefronts of fourteen have one; 93 x 3
        // of 971, 148,962: 44.5, 29.8, 41.7; 28 x 7 of 1,597, 347,459: 50, 39, 62).  Where lists are one unit, and most of it padding, they
        // take longer than pull_share says: 3.3 million, 3 x 7 pairs of 16,000 buckets 209 us, lists of four slices 184.  Of 314
        // shapes with 50,000 to 4 million coordinates and 400 to 16,000 buckets the choice is the fastest form or within 4 % of it at
        // 285, 8 % at 306 and 37 % at all.
        // Not where the vector may be cut into parts: two lists per wavefront are fewer parts, of longer sums (error against 64 bits, 2-norm:
        // 11.4 million, n = 5, 5 x 955 7.0e-7, with one list 6.3e-7; nine million, 7, 5 x 1,459 5.7e-7 and 5.3e-7).
        for (int form : {1, 2, 4}) {
            if (tun.pull_lists ? tun.pull_lists != form : (wide && form < 4) || (form == 2 && ctx->d > kOrderedSingleBinMaxD)) continue;
            const bool many = form == 4;
            PullOrder x = {};
            x.ntile = ntile;
            x.nslice = nslice;
            x.per_list = many ? kPullLoad : 1;
            x.most = many ? kPullMany : form;
            x.group = many ? kPullLoad : (ctx->c <= 1500 ? 4 : 2);
            x.nlist = (nslice + x.per_list - 1) / x.per_list;
            const int64_t tiles = (ntile + counted - 1) / counted, every = wide ? 1 : sample;
            const bool count_steps = form != 2 || tun.pull_lists;    // (form 2 has the lists of form 1)
            if (count_steps) all = 0;
            for (int j = 0; count_steps && j < ctx->r; ++j) {
                int64_t units = 0, seen = 0;
                for (int64_t t = 0; t < tiles; t += every, ++seen)
                    for (int32_t l = 0; l < x.nlist; ++l) units += list_units(x, h_cnt + (j * tiles + t) * nslice, l);
                per_tile[j] = (double)units * 2 * x.group / seen;
                all += per_tile[j] * ntile;
            }
            int64_t c = pull_share(ctx, x, per_tile);
            if (form == 2 && x.group == 2 && !tun.pull_lists) c += c / 10;
            if (c < cost) {
                cost = c;
                po = x;
                steps = all;
            }
        }
        if (!tun.pull_lists && (double)cost > limit) break;
        if (wide && !tun.pull_lists && cost > 25000 + (int64_t)ctx->n * ctx->r * ctx->d * 7 / 4000) break;   // (see pull_declines)
        if (steps * kWave > 12.0 * ctx->r * (double)ctx->d + 8.0 * kWave * (double)rows * nslice) break;   // lists that are mostly padding
        if (counted > 1 && !count(1)) break;
        uint32_t longest = 0;
        for (int64_t q = 0; q < rows * nslice; ++q) longest = h_cnt[q] > longest ? h_cnt[q] : longest;
        if (longest > kPullMaxList) break;                           // a hash that crowds a tile's coordinates into few buckets
        const int64_t lists = rows * po.nlist, streams = stream_number(po, po.parts, 0, 0);
        const int64_t part_bytes = po.parts > 1 ? (int64_t)po.parts * ctx->n * ctx->r * ctx->c * 4 : 0;
        h_first = (uint32_t *)malloc((size_t)streams * 8);
        if (!h_first) break;
        uint64_t run = 0;                                            // units; streams start with a load of their own
        const uint64_t per_load = (uint64_t)(kPullLoad / po.group);
        for (int32_t part = 0; part < po.parts; ++part)
            for (int32_t j = 0; j < ctx->r; ++j)
                for (int32_t w = po.row[j].win0; w < po.row[j + 1].win0; ++w)
                    for (int32_t wave = 0; wave < kPullAdders; ++wave) {
                        int32_t l0, count;
                        lists_of(po, j, w, wave, &l0, &count);
                        run = (run + per_load - 1) / per_load * per_load;
                        uint32_t *f = h_first + 2 * stream_number(po, part, w, wave);
                        f[0] = (uint32_t)(run / per_load);
                        const uint64_t before = run;
                        const int32_t t1 = (part + 1) * po.per_part < ntile ? (part + 1) * po.per_part : ntile;
                        for (int32_t t = part * po.per_part; count > 0 && t < t1; ++t) {
                            const int64_t rt = (int64_t)j * ntile + t;
                            for (int32_t l = l0; l < l0 + count; ++l) {
                                const uint32_t units = list_units(po, h_cnt + rt * nslice, l);
                                h_off[rt * po.nlist + l] = (uint32_t)run;
                                h_len[rt * po.nlist + l] = (uint16_t)units;
                                run += units;
                            }
                        }
                        f[1] = (uint32_t)(run - before);
                    }
        run = (run + per_load - 1) / per_load * per_load;
        if (run >= (1ull << 31)) break;
        if (po.per_list > 1) pp.kernel = (const void *)k_sketch_pull<1, true, kPullMany>;
        else if (po.most > 1) pp.kernel = po.group == 4 ? (const void *)k_sketch_pull<4, false, kPullPair> : (const void *)k_sketch_pull<2, false, kPullPair>;
        else pp.kernel = po.group == 4 ? (const void *)k_sketch_pull<4, false, 1> : (const void *)k_sketch_pull<2, false, 1>;
        e = hipFuncSetAttribute(pp.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        pp.list_bytes = (int64_t)(run * (uint64_t)po.group + kPullSpare) * kWave * 4;
        pp.first_bytes = streams * 8;
        pp.po = (PullOrder *)malloc(sizeof(PullOrder));
        if (!pp.po) break;
        *pp.po = po;
        pp.parts = po.parts;
        if (hipMalloc((void **)&len, (size_t)lists * 2) != hipSuccess || hipMalloc((void **)&off, (size_t)lists * 4) != hipSuccess ||
            hipMalloc((void **)&pp.first, (size_t)pp.first_bytes) != hipSuccess || hipMalloc((void **)&pp.lists, (size_t)pp.list_bytes) != hipSuccess)
            break;
        if (part_bytes && hipMalloc((void **)&pp.part_sums, (size_t)part_bytes) != hipSuccess) break;
        e = hipMemcpyAsync(off, h_off, (size_t)lists * 4, hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(len, h_len, (size_t)lists * 2, hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(pp.first, h_first, (size_t)pp.first_bytes, hipMemcpyHostToDevice, ctx->stream);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        {
            ProfScope ps(ctx, KID_PLAN_BUILD);
            hipLaunchKernelGGL(k_pull_place, grid, dim3(1024), (size_t)(po.nlist * po.per_list * kWave * 4 + kPullTile * 2), ctx->stream, ctx->hp,
                               ctx->d, po, len, off, pp.lists);
        }
        e = hipStreamSynchronize(ctx->stream);                       // the host arrays are released below
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        *done = true;
        ctx->scratch_bytes += pp.list_bytes + pp.first_bytes + part_bytes;
    } while (0);
    (void)hipGetLastError();
    free(h_cnt);
    free(h_len);
    free(h_off);
    free(h_first);
    if (cnt) (void)hipFree(cnt);
    if (len) (void)hipFree(len);
    if (off) (void)hipFree(off);
    ctx->pull = pp;
    if (*done) ctx->plan.mode = pp.parts == 1 ? PLAN_BINNED : PLAN_LDS_ROW;   // to the caller: whether the order is the coordinates'
    else pull_destroy(ctx);
    return rc;
}

void pull_destroy(sams_ctx *ctx)
{
    free(ctx->pull.po);
    if (ctx->pull.first) (void)hipFree(ctx->pull.first);
    if (ctx->pull.lists) (void)hipFree(ctx->pull.lists);
    if (ctx->pull.part_sums) (void)hipFree(ctx->pull.part_sums);
    ctx->pull = PullPlan{};
}

int enqueue_sketch_pull(sams_ctx *ctx, const float *u, float *S_workers)
{
    const PullPlan &pp = ctx->pull;
    const int64_t cells = (int64_t)ctx->n * ctx->r * ctx->c;
    PullArgs a = {u, pp.lists, pp.first, pp.parts > 1 ? pp.part_sums : S_workers, ctx->d, ctx->c, (int64_t)ctx->n * ctx->d, ctx->n,
                  ctx->r, *pp.po};
    const int64_t wgs = (int64_t)ctx->n * a.po.windows * a.po.parts;
    void *args[] = {&a};
    {
        ProfScope ps(ctx, KID_SKETCH_PULL);
        SAMS_HIP(hipLaunchKernel(pp.kernel, dim3((unsigned)((wgs + 7) / 8 * 8)), dim3(kPullThreads), args,
                                 (size_t)kPullLds, ctx->stream));
    }
    if (pp.parts > 1)
        SAMS_LAUNCH(ctx, KID_PULL_SUM, k_pull_sum, grid_for(cells, 256), 256, pp.part_sums, S_workers, cells, pp.parts);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

}  // namespace sams

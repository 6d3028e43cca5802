// Order-preserving Count Sketch accumulation (stage 1 of sams.h; Sec. II-C update rule) for tables of a few LDS windows, without a staged copy per row.
//
// The binned path (sams_plan.hip) writes every signed value, once per row, to where its bucket's window will read it, and reads it back.  Where a row is only
// a few windows wide, a workgroup can as well pick its values out of the worker's vector itself: it has one worker, one row and one window of up to 40,800
// buckets in LDS, walks the vector in phases of `span` coordinates, and adds the ones that fall into its window.  Which those are is worked out once, at
// context creation: a list of words per (row, window), shared by the workers, each word with a coordinate's place in its phase, its sign and the cell of its
// bucket.
//
// A phase has at most kPushEntries words, kPushGroups groups of 64 (a word per lane) for each of 16 wavefronts; a lane reads its words, fetches the values
// they name from memory, and adds each to its cell with a plain read-modify-write.  Wavefronts meet at one barrier per phase, and within a phase all
// coordinates of a bucket are one lane's two words, or words of adjacent lanes, in order, each of which adds to the sum of the one before.  So a bucket's terms are
// added in coordinate order, bit for bit like a sequential loop; no atomics, every cell is written once.
//
// Out of the vectors themselves a group of 64 neighbouring coordinates of one of w windows touches 2 w lines, and that is what bounds it: a compute unit's L1
// takes about two clocks for 16 lanes and a line, and the lines of all windows' workgroups come through it.  With more than a window or two (and where vectors
// and lists do not fit the 256 MB cache together: 490 ns a phase there, 860 from HBM at three and six million, n = 8, 5 x 150,001) it is better to sort first: pass
// 1 (k_sort_copies, or the head, sams_plan.hip) writes copies of the vectors whose phases are sorted by the windows of two to seven rows (push_rows), a window's values
// then lie in long runs, and a row's lists name places in its copy.  That is one write per copy, from end to end, instead of one scattered write per row; the
// copies' reads are one per row, as the binned path's are.  A phase of 1,870 entries takes 340 to 430 ns.  No one thing bounds it: without
// the read-modify-writes, or with every second barrier, it takes as long; with all values from the caches (the same phase again and again) 8 to 16 % less, with the
// words too 20 %, and without any values 30 to 38 % less (11.2 million, n = 8, 5 x 262,001 477, 441, 385 and 341 us; 25 million, n = 16, 10 x 100,000 3,573, 3,008,
// 2,915 and 2,275): addresses of gathers, which the vector memory unit works at two thirds of the time, then instructions and the LDS.
//
// A hash either has next to no bucket twice in a phase or, about one row in thirty, in hundreds of places: (a l + b) mod p walks a lattice, and a distance after
// which buckets repeat is shorter than a phase or it is not (k_push_repeat).  Such a row's words of a bucket name places far apart, and its workgroups take up to
// half as long again; they come first.  (That a bucket's words are a lane's two and not two lanes' matters here: with the first lane collecting the others' values by
// shifts, in copies sorted for such rows, 11.2 million, n = 8, 5 x 262,001 with one took 588 to 663 us; now 515 to 575, and 480 without such a row.  Copies of their
// own for such rows, sorted so that a bucket's values lie side by side, cost more than they gave.)
//
// Measured on MI355X with cold caches, sketch_accumulate by bins and by these lists (us): 853,610 coordinates, n = 14, 5 x 40,514 162 and 130; 1.8 million, n = 17, 3
// x 56,323 239 and 160; 2.2 million, n = 83, 5 x 39,335 1,890 and 741 (one window); 4.3 million, n = 21, 5 x 134,908 930 and 606; 13.6 million, n = 19, 10 x
// 110,245 4,423 and 3,005; 46 million, n = 8, 5 x 446,747 3,386 and 2,948; by slices (sams_pull.hip) and these lists: a million, n = 43, 5 x 19,287 363
// and 191; 0.8 million, n = 70, 10 x 11,957 687 and 455.  Of 290 shapes drawn at random (0.26 to 60 million coordinates, 10,000 to 650,000 buckets; all in
// profiles/sketch_paths_us.txt) the rules below send 114 here: whole steps are 1.02 to 1.9 times as fast as by bins (93, in the middle 1.22) and 0.97 to 1.67 times
// as fast as by slices (21, in the middle 1.23; three below 1).
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <type_traits>

#include "sams_ctx.h"

#pragma clang fp contract(off)

namespace sams {

constexpr int kPushThreads = 1024;
constexpr int kPushWaves = kPushThreads / kWave;
constexpr int kPushGroups = 2;                // words of a lane per phase
constexpr int kPushEntries = kPushThreads * kPushGroups;
constexpr int kPushMaxWin = 40800;            // buckets of a window, which with 64 cells for the padding words have to fit in LDS
constexpr int kPushMostWin = 16;              // windows of a row (with more a phase has too few entries for its barrier)
constexpr int kPushVals = 4;                  // phases whose values are under way
constexpr int kPushRing = 8;                  // phases whose words are
// Buckets lie in LDS in blocks of 64, each turned by a number of its own: the buckets of neighbouring coordinates step by a constant, and where that is a
// multiple of 32 every lane of a group would be in one bank (207 instead of 147 us for one hash of eight at three million, n = 8, 5 x 150,001).
__host__ __device__ __forceinline__ uint32_t push_cell(uint32_t b) { return (b & ~63u) | ((b + ((b >> 6) * 0x9e3779b1u >> 26)) & 63u); }
static __host__ __device__ __forceinline__ int32_t push_cells(int32_t win) { return (win + kWave - 1) / kWave * kWave; }   // the padding's cells follow
static __host__ __device__ __forceinline__ int32_t push_bit_words(int32_t win) { return (win + 31) / 32; }
// A word: sign (bit 0), place in the phase (the next 15 bits, or 14), cell (up to bit 30); bit 31: the word before, the lane's first or the second
// of the lane before, has the same bucket.  Padding: place 0, a cell of the lane's.

// ------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------
// Which rows share a copy, and how its phases are sorted: by the windows of its rows, the first row's first.
struct PushCopies {
    int32_t ncopy;
    int8_t rows[SAMS_MAX_ROWS], row[SAMS_MAX_ROWS][SAMS_MAX_ROWS], of[SAMS_MAX_ROWS];     // rows of a copy; a row's copy
};

// repeat[row]: the shortest distance below `span` after which buckets repeat, else 0x7fffffff.  From a coordinate to one that far behind it the hash moves by
// t = a * distance mod p, or by t - p where it wraps: the bucket is the same for the share 1 - t / p of the coordinates if c divides t, for t / p if it
// divides p - t.  Shares below a tenth do not count.
__global__ void __launch_bounds__(1024)
k_push_repeat(HashParams hp, int32_t span, uint32_t *__restrict__ repeat)
{
    __shared__ uint32_t least;
    if (threadIdx.x == 0) least = 0x7fffffffu;
    __syncthreads();
    for (uint32_t dist = 1 + threadIdx.x; dist < (uint32_t)span; dist += 1024) {
        const uint32_t t = hash_y(hp.row[blockIdx.x].ah, 0u, dist);
        if ((mod_c(hp.modc, t) == 0 && t <= kP31 / 10 * 9) || (mod_c(hp.modc, kP31 - t) == 0 && t >= kP31 / 10)) {
            atomicMin(&least, dist);
            break;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) repeat[blockIdx.x] = least;
}

// per (phase, copy): the coordinate that lies in every place
__global__ void __launch_bounds__(kPushThreads)
k_push_order(HashParams hp, int64_t d, PushCopies pc, int32_t nwin, int32_t win, int32_t span, int32_t nph, uint16_t *__restrict__ order)
{
    extern __shared__ uint32_t keys[];                               // [span, up to a power of two]
    const int t = threadIdx.x, q = blockIdx.y, rows = pc.rows[q];
    const int64_t l0 = (int64_t)blockIdx.x * span;
    const int lim = d - l0 < span ? (int)(d - l0) : span;
    int all = kPushThreads * 2;
    while (all < span) all *= 2;
    for (int x = t; x < all; x += kPushThreads) {
        uint32_t key = 0;
        for (int z = 0; z < rows && x < lim; ++z) {
            key = key * (uint32_t)nwin + bucket_of(hp, pc.row[q][z], (uint32_t)(l0 + x)) / (uint32_t)win;
        }
        keys[x] = x < lim ? (key << 14) | (uint32_t)x : 0xffffffffu;
    }
    for (int size = 2; size <= all; size *= 2)
        for (int step = size / 2; step; step /= 2) {
            __syncthreads();
            for (int p = t; p < all / 2; p += kPushThreads) {
                const int lo = 2 * step * (p / step) + p % step, hi = lo + step;
                const uint32_t x = keys[lo], y = keys[hi];
                if ((x > y) == ((lo & size) == 0)) {
                    keys[lo] = y;
                    keys[hi] = x;
                }
            }
        }
    __syncthreads();
    uint16_t *out = order + ((int64_t)q * nph + blockIdx.x) * span;
    for (int x = t; x < span; x += kPushThreads) out[x] = x < lim ? (uint16_t)(keys[x] & 0x3fffu) : (uint16_t)0;
}

// per (phase, row and window): the words.  *status: a phase has too many entries, or too many that share buckets
//
// Bound by hashing and barriers: every window's workgroup hashes the whole phase, in sweeps of a coordinate per thread, and then only the places that it found,
// two per thread.  Which buckets are shared is two bits per bucket, and the entries that share one are sorted, so that a workgroup takes 46 KB of LDS and two
// fit a unit (with 16-bit counters 118 KB, a second hash of everything and all pairs of shared entries compared: 11.2 million, 5 x 262,144 2.65 ms, now 0.80;
// 25 million, 10 x 100,000 12.5, with a row that repeats 25.4, now 4.3 and 5.9).
__global__ void __launch_bounds__(kPushThreads, 8)
k_push_plan(HashParams hp, int64_t d, int32_t nwin, int32_t win, int32_t span, int32_t nph, int32_t nalloc, int place_bits,
            const uint16_t *__restrict__ order, PushCopies pc, uint32_t *__restrict__ words, uint32_t *__restrict__ status)
{
    extern __shared__ uint32_t seen[];                               // [2][push_bit_words(win)]  bit per bucket: has an entry, has several
    __shared__ uint32_t ent[kPushEntries], outw[kPushEntries];       // the entries' words, by place and in their slots
    __shared__ uint16_t coord[kPushEntries];                         // their coordinates in the phase
    __shared__ uint16_t multi[kPushEntries], nth[kPushEntries];      // entries that share a bucket; how many of its entries come before one
    __shared__ uint32_t place[kPushEntries];                         // of a shared bucket's first entry: wavefront, place among its words; of the others: the first
    __shared__ uint32_t part[kPushWaves], many[kPushWaves], before[kPushWaves * kPushGroups + 1];
    __shared__ uint32_t sh, longest;
    const int bshift = place_bits + 1;
    const int t = threadIdx.x, my_lane = t & (kWave - 1), my_wave = t / kWave, j = blockIdx.y / nwin, w = blockIdx.y % nwin;
    uint32_t *out = words + ((int64_t)blockIdx.y * nalloc + blockIdx.x) * kPushEntries;
    const int64_t l0 = (int64_t)blockIdx.x * span;
    const int lim = (int)blockIdx.x >= nph ? 0 : (d - l0 < span ? (int)(d - l0) : span);
    const uint32_t b0 = (uint32_t)w * (uint32_t)win;
    uint32_t *several = seen + push_bit_words(win);
    for (int q = t; q < 2 * push_bit_words(win); q += kPushThreads) seen[q] = 0u;
    if (t < kPushWaves) many[t] = 0u;
    if (t == 0) longest = 0u;
    // the window's places, in order: in a sweep every thread looks at one of 1,024 neighbours
    const uint16_t *in_place = order ? order + ((int64_t)pc.of[j] * nph + blockIdx.x) * span : nullptr;
    auto at_place = [&](int x) { return in_place ? (int)in_place[x] : x; };
    const int sweeps = (lim + kPushThreads - 1) / kPushThreads;      // at most 32: a place has 15 bits
    uint32_t *found = ent;                                           // [sweeps][kPushWaves]  places of a wavefront's 64, then of all before
    uint16_t *places = nth;                                          // (neither is in use yet)
    uint32_t mine = 0;
    for (int z0 = 0; z0 < sweeps; z0 += 4) {
        uint32_t l[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int x = (z0 + z) * kPushThreads + t;
            l[z] = (uint32_t)(l0 + at_place(x < lim ? x : 0));
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const bool in = (z0 + z) * kPushThreads + t < lim && bucket_of(hp, j, l[z]) - b0 < (uint32_t)win;
            const uint64_t all = __ballot(in);
            if (my_lane == 0) found[(z0 + z) * kPushWaves + my_wave] = (uint32_t)__popcll(all);
            mine |= (in ? 1u : 0u) << (z0 + z);
        }
    }
    __syncthreads();
    {
        const uint32_t n = t < sweeps * kPushWaves ? found[t] : 0u, upto = block_exclusive_scan<kPushThreads>(n, part);
        if (t < sweeps * kPushWaves) found[t] = upto;
        if (t == kPushThreads - 1) sh = upto + n;
    }
    __syncthreads();
    const uint32_t total = sh;
    if (total > (uint32_t)kPushEntries) {
        if (t == 0) atomicOr(status, 1u);
        return;
    }
    for (int z = 0; z < sweeps; ++z) {
        const uint64_t all = __ballot((mine >> z) & 1u);
        if ((mine >> z) & 1u) places[found[z * kPushWaves + my_wave] + __popcll(all & (((uint64_t)1 << my_lane) - 1))] = (uint16_t)(z * kPushThreads + t);
    }
    __syncthreads();
#pragma unroll
    for (int z = 0; z < kPushGroups; ++z) {
        const uint32_t e = t * kPushGroups + z;
        if (e >= total) continue;
        const uint32_t x = places[e], q = (uint32_t)at_place((int)x), l = (uint32_t)l0 + q, b = bucket_of(hp, j, l) - b0;
        coord[e] = (uint16_t)q;
        ent[e] = (b << bshift) | (x << 1) | (sign_neg(hp, j, l) ? 1u : 0u);
        const uint32_t bit = 1u << (b & 31);
        if (atomicOr(&seen[b >> 5], bit) & bit) atomicOr(&several[b >> 5], bit);
    }
    __syncthreads();
    auto bucket = [&](uint32_t e) { return ent[e] >> bshift; };
    bool is_multi[kPushGroups];
    uint32_t nm = 0;
#pragma unroll
    for (int z = 0; z < kPushGroups; ++z) {
        const uint32_t e = t * kPushGroups + z;
        is_multi[z] = e < total && ((several[bucket(e) >> 5] >> (bucket(e) & 31)) & 1u);
        nm += is_multi[z] ? 1u : 0u;
    }
    const uint32_t multi_before = block_exclusive_scan<kPushThreads>(nm, part);
    {
        uint32_t k = multi_before;
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z)
            if (is_multi[z]) multi[k++] = (uint16_t)(t * kPushGroups + z);
        if (t == kPushThreads - 1) sh = k;
    }
    __syncthreads();
    const uint32_t nmulti = sh;
    __syncthreads();
    if (nmulti) {
        // sorted by bucket and coordinate, a bucket's entries lie side by side, the first one first
        uint32_t key[kPushGroups], first[kPushGroups], len[kPushGroups], sum = 0;
        uint32_t *keys = outw;
        uint32_t all = 2;
        while (all < nmulti) all *= 2;
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            const uint32_t k = t * kPushGroups + z;
            key[z] = k < nmulti ? (bucket(multi[k]) << 15) | coord[multi[k]] : 0xffffffffu;
            if (k < all) keys[k] = key[z];
        }
        for (uint32_t size = 2; size <= all; size *= 2)
            for (uint32_t step = size / 2; step; step /= 2) {
                __syncthreads();
                if ((uint32_t)t < all / 2) {
                    const uint32_t lo = 2 * step * (t / step) + t % step, hi = lo + step, x = keys[lo], y = keys[hi];
                    if ((x > y) == ((lo & size) == 0)) {
                        keys[lo] = y;
                        keys[hi] = x;
                    }
                }
            }
        __syncthreads();
        auto below = [&](uint32_t v) {                               // keys below v
            uint32_t n = 0;
            for (uint32_t s = all; s; s /= 2)
                if (n + s <= all && keys[n + s - 1] < v) n += s;
            return n;
        };
        uint16_t *sorted = coord;                                    // (no longer needed)
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            const uint32_t k = t * kPushGroups + z;
            len[z] = first[z] = 0u;
            if (k >= nmulti) continue;
            const uint32_t at = below(key[z]);
            first[z] = below(key[z] & ~0x7fffu);
            nth[k] = (uint16_t)(at - first[z]);
            sorted[at] = (uint16_t)k;
            if (at == first[z]) len[z] = below((key[z] | 0x7fffu) + 1u) - at;
        }
        __syncthreads();
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            const uint32_t k = t * kPushGroups + z;
            if (k < nmulti && !len[z]) place[k] = sorted[first[z]];
        }
        // The shared buckets in the order of their first entries, as if in one line that is cut every 128 - (most entries of a bucket - 1): a bucket
        // goes with all its entries to the wavefront in whose piece it starts, and none is longer than what is left of the 128 words.  Where there is
        // room, each starts with a lane's first word.
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            sum += (len[z] + 1) & ~1u;
            if (len[z] > 1) atomicMax(&longest, len[z]);
        }
        uint32_t pos = block_exclusive_scan<kPushThreads>(sum, part);
        if (t == kPushThreads - 1) sh = pos + sum;
        __syncthreads();
        const bool even = sh + (total - nmulti) + kPushWaves * longest <= (uint32_t)kPushEntries;
        if (!even) {
            sum = 0;
            for (int z = 0; z < kPushGroups; ++z) sum += len[z];
            pos = block_exclusive_scan<kPushThreads>(sum, part);
        }
        const uint32_t span_of = kWave * kPushGroups, piece = longest < span_of ? (span_of + 1 + even - longest) & ~1u : 2u;
        bool fits = longest < span_of;
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            const uint32_t k = t * kPushGroups + z, wave = pos / piece, f = pos % piece;
            if (!len[z]) continue;
            if (wave < (uint32_t)kPushWaves) {
                place[k] = wave | (f << 8);
                atomicMax(&many[wave], f + len[z]);
            } else {
                fits = false;
            }
            pos += even ? (len[z] + 1) & ~1u : len[z];
        }
        // (a hash that leaves no room for the others either needs shorter phases)
        if (!__syncthreads_and(fits)) {
            if (t == 0) atomicOr(status, 1u);
            return;
        }
    }
    for (int q = t; q < kPushEntries; q += kPushThreads) outw[q] = (uint32_t)(push_cells(win) + q / kPushGroups % kWave) << bshift;
    // the others fill the lanes that the shared buckets leave, in order, a wavefront's first words before its second
    const uint32_t singles = total - nmulti;
    if (t < kWave) {
        constexpr int kAll = kPushWaves * kPushGroups;
        const uint32_t room = t < kAll ? (uint32_t)kWave - (many[t / kPushGroups] + 1) / 2 : 0u;
        const uint32_t upto = wave_inclusive_scan(room);
        if (t < kAll) before[t + 1] = upto;
        if (t == 0) before[0] = 0u;
    }
    __syncthreads();
    if (before[kPushWaves * kPushGroups] < singles) {
        if (t == 0) atomicOr(status, 1u);
        return;
    }
    auto word_of = [&](uint32_t e) { return (push_cell(bucket(e)) << bshift) | (ent[e] & ((1u << bshift) - 1u)); };
    {
        uint32_t s = (uint32_t)(t * kPushGroups) - multi_before, group = 0;
#pragma unroll
        for (int z = 0; z < kPushGroups; ++z) {
            const uint32_t e = t * kPushGroups + z;
            if (e >= total || is_multi[z]) continue;
            while (before[group + 1] <= s) ++group;                  // there is room for all: the search ends
            const uint32_t wave = group / kPushGroups, lane = (many[wave] + 1) / 2 + s - before[group];
            outw[(wave * kWave + lane) * kPushGroups + group % kPushGroups] = word_of(e);
            ++s;
        }
    }
    for (uint32_t k = t; k < nmulti; k += kPushThreads) {
        const uint32_t n = nth[k], p = n ? place[place[k]] : place[k];
        outw[(p & 255u) * (kWave * kPushGroups) + (p >> 8) + n] = word_of(multi[k]) | (n ? 0x80000000u : 0u);
    }
    __syncthreads();
    for (int q = t; q < kPushEntries; q += kPushThreads)
        out[q] = outw[q];
}

// ------------------------------------------------------------------------------------------
// accumulation
// ------------------------------------------------------------------------------------------
struct PushArgs {
    const float *u;                   // [n][d], or the copies [ncopy][n][nph * span]
    const uint32_t *words;            // [r * nwin][nalloc][kPushWaves][64][kPushGroups]
    float *S;                         // [n][r][c]
    int64_t c, stride;                // floats between two workers' vectors
    int32_t n, r, nwin, win, span, nph, nalloc;
    int32_t share;                    // workers whose units take turns in the order of the units
    int8_t copy_of[SAMS_MAX_ROWS], row[SAMS_MAX_ROWS];     // a row's copy; the rows, those that take longest first
};

__device__ __forceinline__ void push_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float from_lane_before(float y)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(y), 0x138, 0xf, 0xf, false));
}

// The word and value rings are filled by unconditional loads in a fixed order, straight into the registers that the loop carries, so that
// the compiler waits for exactly the oldest; loads past the vector's end fetch padding words (nalloc), whose place is 0.
template <int PLACE>
__global__ void __launch_bounds__(kPushThreads)
k_sketch_push(PushArgs a)
{
    extern __shared__ float tbl[];                                   // [push_cells(win) + 64]
    // Units in the order row, window, worker; the 8 XCDs, to which workgroups are dealt round-robin, take `share` at a time: workers with the same words side
    // by side, and the windows of a row, which may take longer than others', on all XCDs.  Out of copies by 16 (25 million, n = 16, 10 x 100,000 with 1, 4 and
    // 16: 3,882, 3,907 and 3,539 us); out of the vectors, where the windows' workgroups read the same lines, by 4 (2.2 million, n = 83: with 8 and 16 up to 940
    // instead of 755).
    const int32_t slot = (int32_t)(blockIdx.x / 8), unit = (slot / a.share * 8 + (int32_t)(blockIdx.x % 8)) * a.share + slot % a.share;
    if (unit >= a.n * a.r * a.nwin) return;
    const int32_t i = unit % a.n, list = unit / a.n, j = a.row[list / a.nwin], jw = j * a.nwin + list % a.nwin;
    const int64_t b0 = (int64_t)(jw % a.nwin) * a.win;
    const float *ui = a.u + ((int64_t)a.copy_of[j] * a.n + i) * a.stride;
    const int t = threadIdx.x;
    constexpr int G = kPushGroups;
    constexpr uint32_t kPlaces = ((1u << PLACE) - 1u) << 2, kBuckets = ((1u << (30 - PLACE)) - 1u) << 2;
    typedef uint32_t vecw __attribute__((ext_vector_type(G)));
    vecw w[kPushRing];
    float v[kPushVals][G];
    const char *words = reinterpret_cast<const char *>(a.words + (int64_t)jw * a.nalloc * kPushEntries);
    uint32_t loff = (uint32_t)t * G * 4;                             // (a list is below 4 GB)
    const float *ucur = ui;
    int32_t vph = 0;
    auto load_words = [&](int z) {
        w[z] = *reinterpret_cast<const vecw *>(words + loff);
        loff += kPushEntries * 4;
        asm volatile("" : "+v"(loff));                               // one addition, not one of 64 bits for each phase of a turn
    };
    auto load_values = [&](int zv, int zw) {
        const char *base = reinterpret_cast<const char *>(vph < a.nph ? ucur : ui);
#pragma unroll
        for (int g = 0; g < G; ++g) v[zv][g] = *reinterpret_cast<const float *>(base + ((w[zw][g] << 1) & kPlaces));
        ucur += a.span;
        ++vph;
    };
    for (int32_t b = t; b < push_cells(a.win) + kWave; b += kPushThreads) tbl[b] = 0.f;
    // in the order in which the phases go on (or the first phases of a turn wait for values that are not theirs)
#pragma unroll
    for (int z = 0; z < kPushRing; ++z) {
        load_words(z);
        __builtin_amdgcn_sched_barrier(0);
        if (z >= kPushRing - kPushVals) load_values(z - (kPushRing - kPushVals), z - (kPushRing - kPushVals));
        __builtin_amdgcn_sched_barrier(0);
    }
    auto phase = [&](auto zc) {
        constexpr int z = zc;
        uint32_t ww[G];
        float vv[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            ww[g] = w[z][g];
            vv[g] = v[z % kPushVals][g];
            asm volatile("" : "+v"(ww[g]), "+v"(vv[g]));         // (or their use moves up, and with it the wait)
        }
        __builtin_amdgcn_sched_barrier(0);
        load_words(z);
        __builtin_amdgcn_sched_barrier(0);
        load_values(z % kPushVals, (z + kPushVals) % kPushRing);
        __builtin_amdgcn_sched_barrier(0);
        push_barrier();                                          // the phase before has been added
        float *cell[G], x[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            cell[g] = reinterpret_cast<float *>(reinterpret_cast<char *>(tbl) + ((ww[g] >> (PLACE - 1)) & kBuckets));
            vv[g] = __uint_as_float(__float_as_uint(vv[g]) ^ (ww[g] << 31));
            x[g] = *cell[g];
        }
        // a word that follows takes its bucket's sum from the word before: its lane's first word, or the second of the lane before
        static_assert(G == 2, "a lane's two words");
        const uint64_t first = __ballot((int)ww[0] < 0);
        const bool second = (int)ww[1] < 0;
        x[0] = x[0] + vv[0];
        const float x1 = second ? x[0] : x[1];
        if (!first) {
            *cell[0] = x[0];
            *cell[1] = x1 + vv[1];
            asm volatile("; in one lane" ::: "memory");              // (kept apart from the other case)
        } else {
            const uint64_t on = __ballot(second);
            const float r1 = x[1];
            x[1] = x1 + vv[1];
            // by one lane more each time; those that are there do the same again
            for (uint64_t far = first; far; far = first & (far & on) << 1) {
                const float y = from_lane_before(x[1]);
                x[0] = __builtin_amdgcn_inverse_ballot_w64(first) ? y + vv[0] : x[0];
                x[1] = (second ? x[0] : r1) + vv[1];
            }
            if (!second) *cell[0] = x[0];
            if (!__builtin_amdgcn_inverse_ballot_w64(first >> 1)) *cell[1] = x[1];
        }
    };
    // whole turns of the ring, with no way out in between (or the compiler waits for all loads at the turn's end), then what is left
    int32_t p = 0;
    for (; p + kPushRing <= a.nph; p += kPushRing) {
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
        phase(std::integral_constant<int, 4>{});
        phase(std::integral_constant<int, 5>{});
        phase(std::integral_constant<int, 6>{});
        phase(std::integral_constant<int, 7>{});
    }
    static_assert(kPushRing == 8, "the phases of a turn");
    if (p + 0 < a.nph) phase(std::integral_constant<int, 0>{});
    if (p + 1 < a.nph) phase(std::integral_constant<int, 1>{});
    if (p + 2 < a.nph) phase(std::integral_constant<int, 2>{});
    if (p + 3 < a.nph) phase(std::integral_constant<int, 3>{});
    if (p + 4 < a.nph) phase(std::integral_constant<int, 4>{});
    if (p + 5 < a.nph) phase(std::integral_constant<int, 5>{});
    if (p + 6 < a.nph) phase(std::integral_constant<int, 6>{});
    __syncthreads();
    const int32_t nb = a.c - b0 < a.win ? (int32_t)(a.c - b0) : a.win;
    float *out = a.S + ((int64_t)i * a.r + j) * a.c + b0;
    for (int32_t b = t; b < nb; b += kPushThreads) out[b] = tbl[push_cell((uint32_t)b)];
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static int push_place_bits(int32_t win) { return push_cells(win) + kWave <= 1 << 15 ? 15 : 14; }
static int32_t push_win(int64_t c, int32_t nwin) { return (int32_t)((c + nwin - 1) / nwin); }
static size_t push_lds(int32_t win) { return (size_t)(push_cells(win) + kWave) * 4; }
constexpr int32_t kPushTile = 1 << 14;        // most coordinates of a phase with copies: pass 1 holds one in LDS

// coordinates of a phase: its entries, a binomial number, stay below kPushEntries by `sigmas` deviations
static int32_t push_span(int64_t c, int32_t win, bool copies, double sigmas)
{
    const double f = (double)win / (double)c;
    double mean = kPushEntries;
    for (int it = 0; it < 20; ++it) mean = kPushEntries - sigmas * sqrt(mean * (1.0 - f) + 1.0);
    const int64_t span = (int64_t)(mean / f) / 32 * 32, most = copies ? kPushTile : ((int64_t)1 << push_place_bits(win)) - 32;
    return (int32_t)(span < most ? span : most);
}

// rows that a copy has room for: runs of a phase's coordinates that have everything they are sorted by in common keep 20 places
static int32_t push_rows(int32_t nwin, int32_t span)
{
    int64_t bins = 1;
    int32_t rows = 0;
    while (nwin > 1 && bins * nwin <= 1024 && span / (bins * nwin) >= 20) {
        bins *= nwin;
        ++rows;
    }
    return rows;
}

// The rows in the order of their workgroups, and in what copies: those whose buckets repeat first (they take longer), and a copy's rows side by side, so that
// what they read of it at about the same time comes from memory once.
static PushCopies push_copies(const sams_ctx *ctx, int32_t nwin, int32_t span, const uint32_t *repeat, int8_t *order)
{
    PushCopies pc = {};
    const int32_t most = push_rows(nwin, span);
    int32_t at = 0;
    if (most >= 1) pc.ncopy = (ctx->r + most - 1) / most;
    for (int repeats = 1; repeats >= 0; --repeats)
        for (int32_t j = 0; j < ctx->r; ++j) {
            if ((repeat[j] < (uint32_t)span) != (repeats == 1)) continue;
            const int32_t q = at * pc.ncopy / ctx->r;                // (as many rows in each, or one less)
            order[at++] = (int8_t)j;
            if (pc.ncopy) {
                pc.row[q][pc.rows[q]++] = (int8_t)j;
                pc.of[j] = (int8_t)q;
            }
        }
    return pc;
}

// What a sketch should take, in ns.  Workgroups run in rounds of 256, one per compute unit.  A phase out of the vectors takes the longer the more windows share
// their lines (cold caches; 310 to 400 with one window, 530 to 620 with two, up to 690 with four).  Out of copies it takes 320 at least and 340 to 430 with
// 1,870 entries where all units are busy, less where few are (of 51 timings 8 in 10 lie between 0.85 and 1.15 of what this says, the others
// between 0.81 and 1.35; out of the vectors of 29 between 0.73 and 1.10, and 0.70 and 1.31), and up to 500 where a copy has more than four
// rows, whose last ones read runs of 23 values; with rows that repeat 1.05 to 1.3 times that, also where a phase has dozens of entries for a bucket (0.94
// million, n = 54, 10 x 31,212 with a distance of 82 in phases of 2,016 469 us, by bins 1,016; 25 million, n = 16, 10 x 100,000 with 202 in 7,488 5.3 ms, by
// bins 7.5).  Copies are written at 5 TB/s, by the head at 4.0 to 5.
static double push_cost(const sams_ctx *ctx, int32_t nwin, bool copies, bool fused, const uint32_t *repeat)
{
    const int32_t win = push_win(ctx->c, nwin);
    const int32_t span = push_span(ctx->c, win, copies, 4.5);
    const double nph = (double)((ctx->d + span - 1) / span), entries = (double)span * win / ctx->c, nd = (double)ctx->n * ctx->d;
    const int64_t units = (int64_t)ctx->n * ctx->r * nwin, full = units / 256, rest = units % 256;
    double longer = 1.0;
    for (int32_t j = 0; j < ctx->r; ++j) {
        if (repeat[j] < (uint32_t)span / 64) return 1e30;            // (more of a phase's entries in a bucket than a wavefront has room for)
        if (repeat[j] < (uint32_t)span && longer < 1.2) longer = 1.2;
        if (repeat[j] < (uint32_t)span / 24) longer = 1.35;
    }
    if (!copies) {
        const double phase[] = {340, 560, 640, 690, 850};
        return 8000 + (full + (rest ? 1 : 0)) * nph * (nwin <= 5 ? phase[nwin - 1] : 350 + 100 * nwin) * longer;
    }
    const int32_t most = push_rows(nwin, span);
    if (most < 1) return 1e30;
    const int32_t ncopy = (ctx->r + most - 1) / most;
    const double one = 110 + 0.15 * entries > 320 ? 110 + 0.15 * entries : 320, last = rest ? 290 + 0.075 * entries * rest / 256 : 0;
    return 8000 + nph * (full * one + last + (most > 4 ? 80 * (full + 1) : 0)) * longer +
           (fused ? nd * ncopy * 4 / 4300.0 : 6000 + nd * (ncopy + 1) * 4 / 5000.0);
}

// Whether this shape may push: tables of 10,000 buckets (below, the lists of sams_pull.hip are the faster, and phases have dozens of coordinates for a bucket) to
// kPushMostWin windows, vectors of 2^18 coordinates (below, everything is launches and latencies) to 2^26 (the lists take gigabytes).
static bool push_shape(const sams_ctx *ctx, const Tunables &tun)
{
    if (tun.sketch_path != 0 || tun.estimate_path == 2 || tun.win_log2 || tun.tile_log2 || tun.chunk_log2 || tun.acc_threads || tun.stage_rows ||
        tun.stage_interleave || tun.run_pad != 16 || tun.acc_wide != 2 || tun.fuse_head == 1)
        return false;                                                // the caller asks for the binned path or for a shape of it
    if (ctx->c > kPushMostWin * (int64_t)kPushMaxWin || ctx->d > 1 << 26) return false;
    if (!tun.push_windows && ctx->c <= 1 << 15 && ctx->d > kOrderedSingleBinMaxD) return false;   // sums in parts, which the others give there, are more precise
    return tun.push_windows ? tun.push_windows > 0 : ctx->c > 10000 && ctx->d >= 1 << 18;
}

// the fastest number of windows, and whether out of copies; 1e30: none.  (Copies that only the head of Alg. 2 can write, as of a long vector whose length is
// no multiple of four, count as the head's: which update the context will have is not known yet.)
static double push_choose(const sams_ctx *ctx, const Tunables &tun, PushChoice *choice)
{
    const bool fused = head_form_fuses(tun, ctx->d, false);
    double best = 1e30;
    for (int mode = 0; mode < 2; ++mode)
        for (int32_t nwin = (int32_t)((ctx->c + kPushMaxWin - 1) / kPushMaxWin); nwin <= kPushMostWin; ++nwin) {
            if (tun.push_windows && tun.push_windows != mode * 100 + nwin) continue;
            const double cost = push_cost(ctx, nwin, mode == 1, fused, choice->repeat);
            if (cost >= best) continue;
            best = cost;
            choice->windows = nwin;
            choice->copies = mode == 1;
        }
    return best;
}

// Whether bins are taken to need more: 1.85 ns per thousand terms, which errs towards the bins: of 160 drawn shapes that could go either way (see above) all 93 on
// this side of the line take less by the lists, and of the 67 beyond it 50 would (1.02 to 1.74 times), six are alike and eleven take 1.01 to 1.32 times as long.
static bool push_pays(const sams_ctx *ctx, const Tunables &tun, double cost)
{
    return tun.push_windows ? cost < 1e30 : cost <= 10000 + (double)ctx->n * ctx->r * ctx->d * 1.85e-3;
}

// every row's repeat distance below 2^15, from the device (by way of the selection's scratch, which nothing uses yet)
static int push_repeats(sams_ctx *ctx, uint32_t *repeat)
{
    {
        ProfScope ps(ctx, KID_PLAN_BUILD);
        hipLaunchKernelGGL(k_push_repeat, dim3((unsigned)ctx->r), dim3(1024), 0, ctx->stream, ctx->hp, 1 << 15, ctx->sel_tile);
    }
    SAMS_HIP(hipGetLastError());
    SAMS_HIP(hipMemcpyAsync(repeat, ctx->sel_tile, (size_t)ctx->r * 4, hipMemcpyDeviceToHost, ctx->stream));
    SAMS_HIP(hipStreamSynchronize(ctx->stream));
    return SAMS_OK;
}

// Units that take turns (see the kernel): up to 16 workers' out of copies, 4 out of the vectors, but not so many that the XCD that has one turn more than others
// (32 of the 256 compute units) needs a round of workgroups more for it than units dealt one by one would.  Five workers, 50 lists: turns of five are 35 units
// for two of the XCDs (us, in turns of all workers and now: 11.2 million, n = 7, 5 x 55,872 753 and 429; 45 million, n = 6, 7 x 56,659 3,237 and 2,097; 2.4 million, n = 6,
// 7 x 150,527 148 and 98; bins need 884, about 4,000 and 211).
static int32_t push_share(int32_t n, int64_t units, bool copies)
{
    auto rounds = [&](int32_t share) { return (((units + share - 1) / share + 7) / 8 * share + 31) / 32; };
    const int32_t most = copies ? 16 : 4;
    int32_t share = n < most ? n : most;
    while (rounds(share) > rounds(1)) --share;
    return share;
}

// choice->ns: what a sketch should take this way (out of copies a little more: slices gain more from warm caches), 1e30 where bins are taken to need less or the
// shape cannot.  Slices (sams_pull.hip) go first where they are taken to
// need less.  Of 130 drawn shapes that could go by slices or this (see above) 21 take this: whole steps are 1.05 to 1.67 times as fast at 18, alike at one, and 1 and
// 2.5 % slower at two; of the 109 that keep the slices those are the faster at 74, up to 2.6 times, and at 31 this would be by 1.02 to 1.3 (us, sketches with cold
// caches: 2.1 million, n = 25, 7 x 29,263 770 and 353; 1.6 million, n = 6, 5 x 14,952 157 and 118; 0.57 million, n = 69, 3 x 21,015 159 and 127).
int push_estimate(sams_ctx *ctx, const Tunables &tun, PushChoice *choice)
{
    choice->ns = 1e30;
    if (!push_shape(ctx, tun)) return SAMS_OK;
    for (uint32_t &x : choice->repeat) x = 0x7fffffffu;
    if (!push_pays(ctx, tun, push_choose(ctx, tun, choice))) return SAMS_OK;   // not even with the best of hashes
    SAMS_TRY(push_repeats(ctx, choice->repeat));
    const double cost = push_choose(ctx, tun, choice);
    // (a head that writes copies is three launches, with the tail and the second moments on I_{t-1}; a context that pulls has one)
    const double launches = choice->copies && head_form_fuses(tun, ctx->d, false) ? 10000 : 0;
    if (push_pays(ctx, tun, cost)) choice->ns = tun.push_windows ? 0 : (choice->copies ? cost * 1.3 + launches : cost);
    return SAMS_OK;
}

int push_create(sams_ctx *ctx, const PushChoice &choice, bool *done)
{
    *done = false;
    PushPlan pp = {};
    PushCopies pc = {};
    const bool copies = choice.copies;
    uint32_t *status = ctx->sel_tile, h_status = 0;                  // (see push_repeats)
    int rc = SAMS_OK;
    pp.nwin = choice.windows;
    pp.share = push_share(ctx->n, (int64_t)ctx->n * ctx->r * pp.nwin, copies);
    do {
        hipError_t e;
        pp.win = push_win(ctx->c, pp.nwin);
        const int place_bits = copies ? 14 : push_place_bits(pp.win);
        pp.kernel = place_bits == 15 ? (const void *)k_sketch_push<15> : (const void *)k_sketch_push<14>;
        e = hipFuncSetAttribute((const void *)k_push_plan, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * push_bit_words(kPushMaxWin));
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_push_order, hipFuncAttributeMaxDynamicSharedMemorySize, kPushTile * 4);
        if (e == hipSuccess) e = hipFuncSetAttribute(pp.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)push_lds(kPushMaxWin));
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        if (copies && (rc = copies_create()) != SAMS_OK) break;
        for (double sigmas = 4.5; sigmas < 10; sigmas += 4.5) {
            pp.span = push_span(ctx->c, pp.win, copies, sigmas);
            pp.nph = (int32_t)((ctx->d + pp.span - 1) / pp.span);
            pp.nalloc = pp.nph + kPushRing;
            pp.word_bytes = (int64_t)ctx->r * pp.nwin * pp.nalloc * kPushEntries * 4;
            pc = push_copies(ctx, pp.nwin, pp.span, choice.repeat, pp.row);
            if (copies) {
                if (!pc.ncopy) break;
                pp.ncopy = pc.ncopy;
                memcpy(pp.copy_of, pc.of, sizeof(pp.copy_of));
                pp.order_bytes = (int64_t)pp.ncopy * pp.nph * pp.span * 2;
                pp.copy_words = (int64_t)pp.ncopy * ctx->n * pp.nph * pp.span;
                if (hipMalloc((void **)&pp.order, (size_t)pp.order_bytes) != hipSuccess) { pp.order = nullptr; break; }
            }
            if (hipMalloc((void **)&pp.words, (size_t)pp.word_bytes) != hipSuccess) { pp.words = nullptr; break; }
            rc = enqueue_fill_u32(ctx, status, 1, 0u);
            if (rc != SAMS_OK) break;
            {
                ProfScope ps(ctx, KID_PLAN_BUILD);
                if (copies) {
                    int32_t all = kPushThreads * 2;
                    while (all < pp.span) all *= 2;
                    hipLaunchKernelGGL(k_push_order, dim3((unsigned)pp.nph, (unsigned)pp.ncopy), dim3(kPushThreads), (size_t)all * 4, ctx->stream, ctx->hp,
                                       ctx->d, pc, pp.nwin, pp.win, pp.span, pp.nph, pp.order);
                }
                hipLaunchKernelGGL(k_push_plan, dim3((unsigned)pp.nalloc, (unsigned)(ctx->r * pp.nwin)), dim3(kPushThreads), (size_t)8 * push_bit_words(pp.win),
                                   ctx->stream, ctx->hp, ctx->d, pp.nwin, pp.win, pp.span, pp.nph, pp.nalloc, place_bits, pp.order, pc, pp.words,
                                   status);
            }
            e = hipMemcpyAsync(&h_status, status, 4, hipMemcpyDeviceToHost, ctx->stream);
            if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
            if (e == hipSuccess) e = hipGetLastError();
            if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
            if (!h_status) break;
            (void)hipFree(pp.words);
            if (pp.order) (void)hipFree(pp.order);
            pp.words = nullptr;
            pp.order = nullptr;
        }
        if (rc != SAMS_OK || !pp.words) break;
        *done = true;
        ctx->scratch_bytes += pp.word_bytes + pp.order_bytes;
    } while (0);
    (void)hipGetLastError();
    ctx->push = pp;
    if (!*done) push_destroy(ctx);
    return rc;
}

void push_destroy(sams_ctx *ctx)
{
    if (ctx->push.words) (void)hipFree(ctx->push.words);
    if (ctx->push.order) (void)hipFree(ctx->push.order);
    ctx->push = PushPlan{};
}

int enqueue_sketch_push(sams_ctx *ctx, const float *u, float *S_workers)
{
    const PushPlan &pp = ctx->push;
    if (pp.ncopy && ctx->plan.staged_u != u) {                       // not written by a fused head
        ctx->plan.staged_u = nullptr;                                // what it wrote is overwritten, also if an error follows
        SAMS_TRY(enqueue_sort_copies(ctx, u));
    }
    PushArgs a = {pp.ncopy ? ctx->plan.stg : u, pp.words, S_workers, ctx->c, pp.ncopy ? (int64_t)pp.nph * pp.span : ctx->d, ctx->n, ctx->r, pp.nwin,
                  pp.win, pp.span, pp.nph, pp.nalloc, 0, {0}, {0}};
    a.share = pp.share;
    memcpy(a.copy_of, pp.copy_of, sizeof(a.copy_of));
    memcpy(a.row, pp.row, sizeof(a.row));
    const int64_t units = (int64_t)ctx->n * ctx->r * pp.nwin, chunks = (units + a.share - 1) / a.share;
    void *args[] = {&a};
    ProfScope ps(ctx, KID_SKETCH_PUSH);
    SAMS_HIP(hipLaunchKernel(pp.kernel, dim3((unsigned)((chunks + 7) / 8 * 8 * a.share)), dim3(kPushThreads), args, push_lds(pp.win), ctx->stream));
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

}  // namespace sams

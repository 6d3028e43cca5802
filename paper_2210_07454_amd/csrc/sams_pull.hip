// Order-preserving Count Sketch accumulation (stage 1 of sams.h; Sec. II-C update rule) for narrow tables, without staging.
//
// The binned path (sams_plan.hip) writes every signed value to where its bucket's window will read it and reads it
// back: 8 bytes of memory traffic per (worker, row, coordinate), and a window that few workgroups share when the table
// is small.  A narrow table turns that round: the workgroups pull.  The vector is cut into tiles that fit in LDS; a
// workgroup has one worker, one row and a range of up to 56 slices of 64 buckets (a window), walks the worker's tiles in
// order, and every lane of a wavefront owns one bucket of each of its one, two or four slices, with the sum in a register.  Which
// coordinates of a tile a bucket takes is worked out once, at context creation: per (row, tile, slice) a list of steps,
// each of 64 entries, one per lane -- the coordinate inside the tile and its sign --, padded with an entry that points at a
// zero; the lists of a wavefront lie one after the other, as one stream.  A lane takes its entries in ascending
// coordinate order, so the sums are those of a sequential loop over the coordinates, bit for bit (adding the padding's
// zero changes nothing: a sum that starts at +0 is never -0; a value is added as fma(value, +-1, sum), which rounds
// once, like the addition).  No atomics, no exchange between lanes, one barrier per tile.
// Vectors of more than 2^22 coordinates, whose sums need not be in that order, may be cut into parts: workgroups of their
// own make a table of every part, and the tables are added up part after part, always the same way.
//
// Cost: every workgroup reads its worker's whole vector, or part (through the L2: the workgroups of one worker sit on one XCD
// and walk in step), so the vector is read rows x windows times; the lists, which all workers share, once per worker.
// Bound by what one compute unit takes in from the L2 (a tile of 52 KB in 0.5 us, 105 GB/s, whether the lines hit or not) and by the
// steps of the lists, 5 ns each (a wavefront's read of 64 scattered values of the tile).  Two tiles are under way while a third is
// added: that takes a barrier of its own (tile_barrier), since __syncthreads lets the loaders wait for all they have asked for,
// and one tile then took 0.65 us (in this kernel, 431,003 coordinates, n = 5, 4 x 9,001: 37.5 -> 29 us; 65,536, n = 4, 5 x 2,048: 9.0 ->
// 7.8; 25.6 million, n = 4, 5 x 10,000 with its sums and estimates: 0.99 -> 0.85 ms).  Counters in LDS in place of the barrier, so
// that the wavefronts need not walk in step, cost more than they give (29 -> 48 us: their latency is in every tile).
// What a list holds beyond its coordinates is by the row's hash: 1.5 to 3.1 entries per coordinate in 28 of 30 rows of 10,000
// buckets, 5.5 and 5.8 in the others; 2.7 with 9,001, 1.35 with 400.  A launch waits for its worst row.
// Measured on MI355X, both passes of the binned path before and this kernel: d = 60,000, n = 50, 5 x 400: 98 and 10 us; n = 100:
// 130 and 20 us; d = 65,536, n = 4, 5 x 2,048: 21 and 8 us; d = 431,003, n = 5, 4 x 9,001: 103 and 39 us; d = 25.6 million,
// n = 4, 5 x 10,000: 8.5 and 0.83 to 1.0 ms by the hash (2.4 with one slice per wavefront and the vector in one part: twelve
// windows that read it instead of three).  The lists are made in half the time of the plan: 0.13 ms at 65,536, 0.33 at
// 431,003, 5.3 at 25.6 million (0.26, 0.43 and 10); two waits for the stream and a sum over their lengths on the host are in it.
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
constexpr int kPullSpare = 64;                // words behind the last list, read ahead but not used
constexpr int kPullMaxList = 512;             // longest list of one bucket in one tile
// A word holds two consecutive steps of a lane: the first step's coordinate in bits 2-15 (so that it is a byte offset) and
// its sign in bit 0, the second's in bits 17-30 and 31.  Words come in groups of 1, 2 or 4 (PullOrder::group), which a lane
// reads with one load; bit 1 of a group's first word, in every lane: this group ends a tile's list.

// ------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------
// Where the lists are: wavefront w of the workgroup for (row, window, part of the tiles) has the per_wave slices from
// win * per_win + w * per_wave on; its lists, tile by tile and in a tile slice by slice, are one stream.
struct PullOrder {
    int32_t ntile, nslice, per_win, nwin, group, per_wave, parts, per_part;
};
__host__ __device__ __forceinline__ int64_t stream_number(const PullOrder &po, int j, int win, int part, int wave)
{
    return (((int64_t)j * po.nwin + win) * po.parts + part) * (po.per_win / po.per_wave) + wave;
}
__device__ __forceinline__ int64_t list_number(const PullOrder &po, int j, int tile, int s)
{
    const int in = s % po.per_win;
    return (stream_number(po, j, s / po.per_win, tile / po.per_part, in / po.per_wave) * po.per_part + tile % po.per_part) *
               po.per_wave + in % po.per_wave;
}
// slices that have lists: those of every wavefront that has a slice at all (its others are empty: one group of padding)
__host__ __device__ __forceinline__ int listed_slices(const PullOrder &po)
{
    return (po.nslice + po.per_wave - 1) / po.per_wave * po.per_wave;
}

// per (tile, row): groups of words of every list (the longest of its 64 columns, at least one group); *longest: the
// longest column
__global__ void __launch_bounds__(1024)
k_pull_count(HashParams hp, int64_t d, PullOrder po, uint32_t *__restrict__ len, uint32_t *__restrict__ longest)
{
    extern __shared__ uint32_t cnt[];                                // [nslice * 64]
    const int j = blockIdx.y, nslice = listed_slices(po);
    const int64_t l0 = (int64_t)blockIdx.x * kPullTile;
    const int lim = d - l0 < kPullTile ? (int)(d - l0) : kPullTile;
    for (int b = threadIdx.x; b < nslice * kWave; b += 1024) cnt[b] = 0;
    __syncthreads();
    for (int p = threadIdx.x; p < lim; p += 1024) atomicAdd(&cnt[bucket_of(hp, j, (uint32_t)(l0 + p))], 1u);
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t most = 0;
    for (int s = wave; s < nslice; s += 16) {
        uint32_t m = cnt[s * kWave + lane];
        for (int off = kWave / 2; off; off >>= 1) {
            const uint32_t o = __shfl_xor(m, off);
            m = o > m ? o : m;
        }
        const uint32_t steps = 2u * (uint32_t)po.group;
        if (lane == 0) len[list_number(po, j, blockIdx.x, s)] = m ? (m + steps - 1) / steps : 1u;
        most = m > most ? m : most;
    }
    if (lane == 0) atomicMax(longest, most);
}

// per (tile, row): the lists
__global__ void __launch_bounds__(1024)
k_pull_place(HashParams hp, int64_t d, PullOrder po, const uint32_t *__restrict__ off, uint32_t *__restrict__ lists)
{
    const int nslice = listed_slices(po);
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
        const int64_t o = list_number(po, j, blockIdx.x, s);
        const int b = s * kWave + lane;
        const uint32_t lo = b ? end[b - 1] : 0u, hi = end[b];
        const uint32_t words = (off[o + 1] - off[o]) * (uint32_t)po.group;
        uint32_t *out = lists + ((int64_t)off[o] * kWave + lane) * po.group;   // the words of a group are consecutive in a lane
        for (uint32_t q = 0; q < words; ++q) {
            const uint32_t e0 = lo + 2 * q < hi ? ent[lo + 2 * q] : (uint32_t)kPullZero,
                           e1 = lo + 2 * q + 1 < hi ? ent[lo + 2 * q + 1] : (uint32_t)kPullZero;
            const uint32_t g = q / po.group, z = q % po.group;
            const uint32_t end_flag = z == 0 && q + po.group >= words ? 2u : 0u;
            out[(int64_t)g * kWave * po.group + z] =
                ((e0 & 0x7fffu) << 2) | (e0 >> 15) | ((e1 & 0x7fffu) << 17) | ((e1 >> 15) << 31) | end_flag;
        }
    }
}

// ------------------------------------------------------------------------------------------
// accumulation
// ------------------------------------------------------------------------------------------
struct PullArgs {
    const float *u;
    const uint32_t *lists, *first;    // first[stream]: the stream's first group of words; [streams]: the end
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

// W: words per group; D: groups of words on their way ahead of the one being added.
// Three tile buffers: the loaders bring the next two tiles in while the adders work on the third.  The two kinds wait for
// their own loads only (a wavefront's loads come back in order: one that fetched both would wait for the whole next
// tile before each list).  The adders' loop is a stream of groups: one load is issued per group, unconditionally and
// straight into the registers that the loop carries, so that the compiler waits for exactly the oldest; the two to eight
// values of a group are read from LDS together and added in order.
// PW: slices per wavefront, whose sums take turns in x[0].
template <int W, int D, int PW>
__global__ void __launch_bounds__(kPullThreads)
k_sketch_pull(PullArgs a)
{
    extern __shared__ float buf[];                                   // [kPullBufs][kPullBuf], and 64 words nobody reads
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    // workgroups are dealt round-robin to the 8 XCDs: consecutive (worker, row, window) triples to one XCD
    const int64_t per = (int64_t)gridDim.x / 8, q = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    const PullOrder &po = a.po;
    const int32_t rw = a.r * po.nwin;                                // workgroups that walk the same tiles
    if (q >= (int64_t)a.n * po.parts * rw) return;
    const int32_t i = (int32_t)(q / rw) / po.parts, part = (int32_t)(q / rw) % po.parts;
    const int32_t j = (int32_t)(q % rw) / po.nwin, win = (int32_t)(q % rw) % po.nwin;
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
    const int32_t s = win * po.per_win + wave * PW;
    if (wave * PW >= po.per_win || s >= po.nslice) {                 // no slice: only the barriers
        for (int32_t tl = 0; tl < ntile; ++tl) tile_barrier();
        return;
    }
    typedef uint32_t vecw __attribute__((ext_vector_type(W)));
    const int64_t stream = stream_number(po, j, win, part, wave);
    const uint32_t g0 = a.first[stream], g1 = a.first[stream + 1];
    const vecw *src = reinterpret_cast<const vecw *>(a.lists) + (int64_t)g0 * kWave + lane;
    const int32_t ng = (int32_t)(g1 - g0);
    vecw ring[D];
#pragma unroll
    for (int z = 0; z < D; ++z) {
        ring[z] = src[(int64_t)z * kWave];                           // kPullSpare words end the array
        __builtin_amdgcn_sched_barrier(0);
    }
    src += (int64_t)D * kWave;
    float x[PW];
#pragma unroll
    for (int p = 0; p < PW; ++p) x[p] = 0.f;
    int32_t lists_left = PW;                                         // of the tile
    const char *base = reinterpret_cast<const char *>(buf + mis);
    int32_t left = kPullBufs;                                        // buffers until the first one again
    tile_barrier();                                                  // tile 0 is there
    for (int32_t m0 = 0; m0 < ng; m0 += D) {
#pragma unroll
        for (int z = 0; z < D; ++z) {
            const vecw w = ring[z];
            if (m0 + z < ng) {                                       // uniform; false only past the stream's end
                float v[2 * W], sg[2 * W];
#pragma unroll
                for (int p = 0; p < W; ++p) {
                    v[2 * p] = *reinterpret_cast<const float *>(base + (w[p] & 0xfffcu));
                    v[2 * p + 1] = *reinterpret_cast<const float *>(base + ((w[p] >> 15) & 0xfffcu));
                    sg[2 * p] = __uint_as_float(0x3f800000u | (w[p] << 31));
                    sg[2 * p + 1] = __uint_as_float(0x3f800000u | (w[p] & 0x80000000u));
                }
#pragma unroll
                for (int p = 0; p < 2 * W; ++p) x[0] = __builtin_fmaf(v[p], sg[p], x[0]);
                if (__builtin_amdgcn_readfirstlane((int)w[0]) & 2) { // the list ends
                    const float y = x[0];                            // after a tile's PW lists x[0] is the first slice's again
#pragma unroll
                    for (int p = 0; p + 1 < PW; ++p) x[p] = x[p + 1];
                    x[PW - 1] = y;
                    if (--lists_left == 0) {
                        lists_left = PW;
                        if (m0 + z + 1 < ng) tile_barrier();         // the next tile is there
                        base += kPullBuf * 4;
                        if (--left == 0) {
                            base -= kPullBufs * kPullBuf * 4;
                            left = kPullBufs;
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            ring[z] = src[(int64_t)z * kWave];
            __builtin_amdgcn_sched_barrier(0);
        }
        src += (int64_t)D * kWave;
    }
    float *out = a.S + (((int64_t)part * a.n + i) * a.r + j) * a.c;
#pragma unroll
    for (int p = 0; p < PW; ++p)
        if ((s + p) * kWave + lane < a.c) out[(s + p) * kWave + lane] = x[p];
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
// Whether this shape pulls (if its lists turn out short enough, see pull_slower), and into how many windows.  Tables of 128 to 2^14 buckets under vectors of up to 2^26
// coordinates.  With fewer buckets a bucket's list gets too long to sort by insertion at creation, with more the lists of a
// tile's 64 buckets get too uneven (on average one entry with 2^14 buckets, the longest of 64 four); the lists of
// longer vectors take gigabytes.
constexpr int64_t kPullLongD = 1000000;       // shorter vectors always pull: both paths are launches and latencies
static bool pull_shape(const sams_ctx *ctx, const Tunables &tun, PullPlan &pp)
{
    if (tun.sketch_path != 0 || tun.estimate_path == 2 || tun.win_log2 || tun.tile_log2 || tun.chunk_log2 || tun.acc_threads ||
        tun.stage_rows)
        return false;                                                // the caller asks for the binned path or for a shape of it
    if (ctx->c < 128 || ctx->c > (1 << 14) || ctx->d > ((int64_t)1 << 26) || (int64_t)ctx->n * ctx->d < 4) return false;
    pp.nslice = (int32_t)((ctx->c + kWave - 1) / kWave);
    pp.ntile = (int32_t)((ctx->d + kPullTile - 1) / kPullTile);
    // One workgroup per compute unit: the cost is taken to be tiles per workgroup (and about twelve that starting and ending takes)
    // times rounds of 256 workgroups.  Two or four slices per wavefront are fewer windows, and so fewer rounds; the vector is
    // cut into parts where the order of the additions is not promised (d > 2^22).  Ties go to fewer slices and parts.
    // The steps of the lists, whose number no choice here changes but which a workgroup with more slices has more of, are not
    // in it.
    const int64_t pairs = (int64_t)ctx->n * ctx->r;
    const int32_t most_parts = ctx->d > kOrderedSingleBinMaxD ? 128 : 1;
    int64_t best = INT64_MAX, nwin = 1;
    for (int32_t pw = 1; pw <= 4; pw *= 2) {
        const int64_t least = (pp.nslice + kPullAdders * pw - 1) / (kPullAdders * pw);
        for (int32_t parts = 1; parts <= most_parts; ++parts) {
            const int64_t rounds = (pairs * least * parts + 255) / 256, cost = rounds * ((pp.ntile + parts - 1) / parts + 12);
            if (cost >= best) continue;
            best = cost;
            pp.per_wave = pw;
            pp.parts = parts;
            nwin = parts == 1 ? rounds * 256 / pairs : least;        // as many windows as the rounds have room for
        }
    }
    if (nwin > pp.nslice) nwin = pp.nslice;
    pp.per_win = (int32_t)((pp.nslice + nwin - 1) / nwin);
    pp.per_win = (pp.per_win + pp.per_wave - 1) / pp.per_wave * pp.per_wave;
    pp.nwin = (pp.nslice + pp.per_win - 1) / pp.per_win;
    pp.per_part = (pp.ntile + pp.parts - 1) / pp.parts;
    pp.parts = (pp.ntile + pp.per_part - 1) / pp.per_part;           // none is empty
    // The binned path cuts a table of up to 2^12 buckets into windows of 2^7 until it has 1024 workgroups: with few pairs under
    // a long vector many short streams, where every puller has to take in the whole vector.  In ns: 820 per tile here; there a
    // base, 0.67 per position of a window's stream, 1.6 per thousand terms through staging.  Lists and bins (us), one pair of 4,096
    // buckets: d = 431,003 25 and 28, a million 67 and 40, four million 257 and 109; 2 x 3 of 3,000, four million 256 and
    // 174; 4 x 5 of 4,096, four million 290 and 256, a million 76 and 85; 2 x 5 of 2,000, four million 264 and 263.
    if (ctx->d >= kPullLongD && ctx->d <= kOrderedSingleBinMaxD && ctx->c <= (1 << 12)) {
        const int64_t bins = 25000 + 86 * ctx->d / ctx->c + pairs * ctx->d * 16 / 10000, here = best * 820;
        if (pairs * ((ctx->c + 127) / 128) < 2048 && bins < here) return false;
    }
    return true;
}

// Whether the other path is faster with lists of this many steps.  A tile takes a workgroup 0.64 us and 5.1 ns per step; with many
// pairs and more than 2^13 buckets, several rounds of workgroups with up to 56 slices each, that can exceed the 2 us per
// million terms of the binned path (or, above 2^22 coordinates, of LDS atomics).  Both (ms): 5 x 16,384, n = 50, d = four
// million 2.39 and 1.93, ten million 7.2 and 4.9; 5 x 9,001 (a row whose lists are half padding), n = 32, five million
// 2.79 and 2.21; 5 x 12,000, n = 50, four million 1.78 and 1.94.
static bool pull_slower(const sams_ctx *ctx, const PullPlan &pp, int64_t steps)
{
    const int64_t pairs = (int64_t)ctx->n * ctx->r;
    if (ctx->d < kPullLongD || ctx->c <= (1 << 13) || pairs < 160) return false;
    const int64_t rounds = (pairs * pp.nwin * pp.parts + 255) / 256;
    const int64_t here = rounds * pp.per_part * 640 + rounds * pp.per_part * 51 / 10 * steps / ((int64_t)ctx->r * pp.nwin * pp.ntile);
    return here > 25000 + 2 * pairs * ctx->d / 1000;
}

static PullOrder pull_order(const PullPlan &pp)
{
    return {pp.ntile, pp.nslice, pp.per_win, pp.nwin, pp.group, pp.per_wave, pp.parts, pp.per_part};
}

// SAMS_OK with *done saying whether the context pulls; device memory that cannot be had means it does not
int pull_create(sams_ctx *ctx, const Tunables &tun, bool *done)
{
    *done = false;
    PullPlan pp = {};
    if (!pull_shape(ctx, tun, pp)) return SAMS_OK;
    // Groups of eight steps where the lists of a tile are long (13308 / c entries on average, the longest of 64 decides),
    // else of four; of two where a wavefront has four lists per tile and the steps, padding among them, are what
    // bounds the kernel (5 x 10,000, n = 4, 25.6 million coordinates: 1.13 -> 1.00 ms)
    const int32_t group = ctx->c <= 4096 ? 4 : (pp.per_wave == 4 ? 1 : 2);
    pp.group = group;
    const void *const kernels[2][3] = {
        {(const void *)k_sketch_pull<2, 8, 1>, (const void *)k_sketch_pull<2, 8, 2>, (const void *)k_sketch_pull<1, 16, 4>},
        {(const void *)k_sketch_pull<4, 6, 1>, (const void *)k_sketch_pull<4, 6, 2>, (const void *)k_sketch_pull<4, 6, 4>}};
    pp.kernel = kernels[group == 4][pp.per_wave / 2];
    const PullOrder po = pull_order(pp);
    const int64_t streams = stream_number(po, ctx->r, 0, 0, 0), per_stream = (int64_t)pp.per_part * pp.per_wave,
                  lists = streams * per_stream;
    const int64_t part_bytes = pp.parts > 1 ? (int64_t)pp.parts * ctx->n * ctx->r * ctx->c * 4 : 0;
    uint32_t *longest = nullptr, *off = nullptr;                     // build-time only
    uint32_t *h_off = (uint32_t *)malloc((size_t)(lists + 1) * 4), *h_first = (uint32_t *)malloc((size_t)(streams + 1) * 4);
    int rc = SAMS_OK;
    do {
        if (!h_off || !h_first || hipMalloc((void **)&longest, 4) != hipSuccess || hipMalloc((void **)&off, (size_t)(lists + 1) * 4) != hipSuccess ||
            hipMalloc((void **)&pp.first, (size_t)(streams + 1) * 4) != hipSuccess)
            break;
        const dim3 grid((unsigned)pp.ntile, (unsigned)ctx->r);
        const int lds_count = listed_slices(po) * kWave * 4, lds_place = lds_count + kPullTile * 2;
        const int lds_max = kPullLds;                                // more than the other two kernels need
        hipError_t e = hipFuncSetAttribute((const void *)k_pull_count, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_pull_place, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e == hipSuccess) e = hipFuncSetAttribute(pp.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        rc = enqueue_fill_u32(ctx, longest, 1, 0u);
        if (rc == SAMS_OK) rc = enqueue_fill_u32(ctx, off, lists, 0u);   // lists that no slice has stay empty
        if (rc != SAMS_OK) break;
        {
            ProfScope ps(ctx, KID_PLAN_BUILD);
            hipLaunchKernelGGL(k_pull_count, grid, dim3(1024), (size_t)lds_count, ctx->stream, ctx->hp, ctx->d, po, off, longest);
        }
        uint32_t h_longest = 0;
        e = hipMemcpyAsync(h_off, off, (size_t)lists * 4, hipMemcpyDeviceToHost, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(&h_longest, longest, 4, hipMemcpyDeviceToHost, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        uint64_t run = 0;
        for (int64_t q = 0; q < lists; ++q) {
            const uint32_t len = h_off[q];
            if (q % per_stream == 0) h_first[q / per_stream] = (uint32_t)run;
            h_off[q] = (uint32_t)run;
            run += len;
        }
        // A hash that crowds a tile's coordinates into few buckets makes long or mostly empty lists: not for this path.
        const uint64_t steps = run * 2 * group * kWave, fair = 12ull * (uint64_t)ctx->r * (uint64_t)ctx->d + 8ull * kWave * lists;
        if (h_longest > kPullMaxList || steps > fair || run >= (1ull << 31) || pull_slower(ctx, pp, (int64_t)(run * 2 * group))) break;
        h_first[streams] = (uint32_t)run;
        h_off[lists] = (uint32_t)run;
        pp.list_bytes = (int64_t)(run * group + kPullSpare) * kWave * 4;
        if (hipMalloc((void **)&pp.lists, (size_t)pp.list_bytes) != hipSuccess) break;
        if (part_bytes && hipMalloc((void **)&pp.part_sums, (size_t)part_bytes) != hipSuccess) break;
        e = hipMemcpyAsync(off, h_off, (size_t)(lists + 1) * 4, hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(pp.first, h_first, (size_t)(streams + 1) * 4, hipMemcpyHostToDevice, ctx->stream);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        {
            ProfScope ps(ctx, KID_PLAN_BUILD);
            hipLaunchKernelGGL(k_pull_place, grid, dim3(1024), (size_t)lds_place, ctx->stream, ctx->hp, ctx->d, po, off, pp.lists);
        }
        e = hipStreamSynchronize(ctx->stream);                       // the host arrays are released below
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = SAMS_EHIP; break; }
        *done = true;
    } while (0);
    (void)hipGetLastError();
    free(h_off);
    free(h_first);
    if (longest) (void)hipFree(longest);
    if (off) (void)hipFree(off);
    ctx->pull = pp;
    if (*done) {
        ctx->plan.mode = pp.parts == 1 ? PLAN_BINNED : PLAN_LDS_ROW; // to the caller: whether the order is the coordinates'
        ctx->scratch_bytes += pp.list_bytes + (streams + 1) * 4 + part_bytes;
    } else {
        pull_destroy(ctx);
    }
    return rc;
}

void pull_destroy(sams_ctx *ctx)
{
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
                  ctx->r, pull_order(pp)};
    const int64_t wgs = (int64_t)ctx->n * ctx->r * pp.nwin * pp.parts;
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

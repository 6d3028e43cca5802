// Stage 5 (AMSGrad update with error feedback: tail and head of Alg. 2), stage 2 (mean of the worker
// sketches) and stage 4 (exact values of the selected coordinates) of the pipeline declared in sams.h.
#include "sams_ctx.h"

// Every formula below is evaluated as separate IEEE-754 binary32 operations, rounded to nearest:
// no fused multiply-add is formed (here and with -ffp-contract=off on the command line), and
// x / y and sqrtf(x) are the correctly rounded ones (hipcc's default; never build this file with
// -ffast-math or -fno-hip-fp32-correctly-rounded-divide-sqrt).
#pragma clang fp contract(off)

namespace sams {
// ------------------------------------------------------------------------------------------
// stage 5: tail (finish iteration t) and head (start iteration t+1) of Alg. 2
// ------------------------------------------------------------------------------------------
// The first position of the ascending idx[0..k) whose value is at least `want`, by one wavefront: 64 probes at a time, so
// two to four dependent loads for up to 2^24 entries.
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t *__restrict__ idx, int64_t k, int64_t want)
{
    const int lane = threadIdx.x & (kWave - 1);
    int64_t lo = 0, hi = k;                                          // the answer is in [lo, hi]
    while (hi > lo) {
        const int64_t step = (hi - lo + kWave - 1) / kWave, p = lo + lane * step;
        const int below = __popcll(__ballot(p < hi && (int64_t)idx[p < hi ? p : hi - 1] < want));   // a prefix of the probes
        if (below == 0) return lo;
        const int64_t next = lo + below * step;                      // the first probe that is not below, if any
        lo = lo + (below - 1) * step + 1;
        hi = next < hi ? next : hi;
    }
    return lo;
}

// range[0..2) (LDS) = positions of the index set's members in [l0, l1); complete after the next barrier.  The first two
// wavefronts search, one bound each.
__device__ __forceinline__ void member_range(const int32_t *__restrict__ idx, int64_t k, int64_t l0, int64_t l1, int64_t *range)
{
    const int wave = threadIdx.x / kWave;
    if (wave < 2) {
        const int64_t at = wave_lower_bound(idx, k, wave == 0 ? l0 : l1);
        if ((threadIdx.x & (kWave - 1)) == 0) range[wave] = at;
    }
}

// The tail for a head that reads the bitmap of I_t (the fused ones): a workgroup has 256 bitmap words, finds their
// members in the ascending idx, updates x there and writes the words whole -- no clearing pass, no atomics on memory.
// wordrank != null: also the rank in idx of the first member of every word that has one.
__global__ void __launch_bounds__(256)
k_tail(const int32_t *__restrict__ idx, const float *__restrict__ delta, int64_t k, int64_t words, float lr,
       float *__restrict__ x, uint32_t *__restrict__ bitmap, uint32_t *__restrict__ wordrank)
{
    __shared__ uint32_t bits[256];
    __shared__ int64_t range[2];
    const int t = threadIdx.x;
    const int64_t w0 = blockIdx.x * (int64_t)256;
    bits[t] = 0;
    member_range(idx, k, w0 * 32, (w0 + 256) * 32, range);
    __syncthreads();
    for (int64_t q = range[0] + t; q < range[1]; q += 256) {
        const int32_t l = idx[q];
        x[l] = (x[l] - (lr * delta[q]));
        atomicOr(&bits[(l >> 5) - (int)w0], 1u << (l & 31));
        if (wordrank && (q == 0 || (idx[q - 1] >> 5) != (l >> 5))) wordrank[l >> 5] = (uint32_t)q;
    }
    __syncthreads();
    if (w0 + t < words) bitmap[w0 + t] = bits[t];
}

// the tail when no head follows: x, and e[i][idx[q]] = 0
__global__ void k_tail_zero_e(const int32_t *__restrict__ idx, const float *__restrict__ delta, int64_t k, int32_t n, int64_t d,
                              float lr, float *__restrict__ x, float *__restrict__ e)
{
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= k) return;
    int64_t l = idx[q];
    x[l] = (x[l] - (lr * delta[q]));
    for (int32_t i = 0; i < n; ++i) e[(int64_t)i * d + l] = 0.0f;
}

// Tail and dense head in one launch, when the head is not fused with the first sketch pass.  Two kinds of workgroups:
//   dense   1024 coordinates of `wchunk` workers: m and u (over e), e taken as zero on I_t, whose members it finds in the
//           ascending idx; the workgroups of the first workers also have v and vhat off I_t, and on I_t if they have all
//           workers (ny = 1).  Alg. 1 (PA): v and vhat are per worker, and u = m / sqrt(vhat) + rho e.
//   sparse  the members of I_t: x, and (Alg. 2, ny > 1) h from all workers' g in ascending worker order, v, vhat; 32 lanes
//           share a member from kWideMinWorkers workers on (a chain of n memory latencies otherwise)
// Nothing that one workgroup writes is read by another.  VEC: 4 = 16-byte accesses (d a multiple of 4), 1 = a thread's
// four coordinates lie 256 apart.  The next worker's values are fetched while one is computed; the first ones while
// the members are searched for.
struct UpdateArgs {
    const float *g;
    float *m, *e, *v, *vhat, *x;
    const int32_t *idx;
    const float *delta;
    int64_t k, d, ntile;
    int32_t n, wchunk, ny;
    float beta1, omb1, beta2, omb2, rho, lr;
};

__device__ __forceinline__ void update_members(const UpdateArgs &a, int64_t block, bool pa, float *vals)
{
    const int t = threadIdx.x;
    const bool only_x = pa || a.ny == 1;
    if (only_x || a.n < kWideMinWorkers) {
        const int64_t q = block * 256 + t;
        if (q >= a.k) return;
        const int64_t l = a.idx[q];
        a.x[l] = (a.x[l] - (a.lr * a.delta[q]));
        if (only_x) return;
        float gs = 0.0f;
        for (int32_t i0 = 0; i0 < a.n; i0 += 8) {                    // eight loads in flight, added in worker order
            float val[8];
#pragma unroll
            for (int z = 0; z < 8; ++z) val[z] = a.g[(int64_t)(i0 + z < a.n ? i0 + z : a.n - 1) * a.d + l];
#pragma unroll
            for (int z = 0; z < 8; ++z)
                if (i0 + z < a.n) gs = (i0 + z == 0) ? val[z] : (gs + val[z]);
        }
        const float h = (gs / (float)a.n);
        const float vv = ((a.beta2 * a.v[l]) + (a.omb2 * (h * h)));
        a.v[l] = vv;
        if (vv > a.vhat[l]) a.vhat[l] = vv;
        return;
    }
    const int ql = t >> 5, wl = t & 31;
    const int64_t q = block * kWideCoords + ql;
    const int64_t l = q < a.k ? a.idx[q] : 0;
    float gs = 0.0f;
    for (int32_t i0 = 0; i0 < a.n; i0 += 256) {                      // 256 workers at a time through LDS [8][256]
        const int32_t lim = a.n - i0 < 256 ? a.n - i0 : 256;
        if (q < a.k)
            for (int32_t i = wl; i < lim; i += 32) vals[ql * 256 + i] = a.g[(int64_t)(i0 + i) * a.d + l];
        __syncthreads();
        if (wl == 0)
            for (int32_t i = 0; i < lim; ++i) gs = (i0 + i == 0) ? vals[ql * 256] : (gs + vals[ql * 256 + i]);
        __syncthreads();
    }
    if (q < a.k && wl == 0) {
        a.x[l] = (a.x[l] - (a.lr * a.delta[q]));
        const float h = (gs / (float)a.n);
        const float vv = ((a.beta2 * a.v[l]) + (a.omb2 * (h * h)));
        a.v[l] = vv;
        if (vv > a.vhat[l]) a.vhat[l] = vv;
    }
}

template <int VEC, bool PA>
__global__ void __launch_bounds__(256)
k_update(UpdateArgs a)
{
    __shared__ float vals[kWideCoords * 256];
    __shared__ uint32_t bits[32];
    __shared__ int64_t range[2];
    const int t = threadIdx.x;
    const int64_t dense = a.ntile * a.ny;
    if (blockIdx.x >= dense) {
        update_members(a, (int64_t)blockIdx.x - dense, PA, vals);
        return;
    }
    const int64_t l0 = (blockIdx.x % a.ntile) * 1024;
    const int32_t y = (int32_t)(blockIdx.x / a.ntile);
    const int32_t i0 = y * a.wchunk, i1 = i0 + a.wchunk < a.n ? i0 + a.wchunk : a.n;
    // this thread's coordinates: l0 + at(z), z < 4
    auto at = [&](int z) { return VEC == 4 ? t * 4 + z : t + 256 * z; };
    auto in = [&](int z) { return l0 + at(z) < a.d; };
    auto load = [&](const float *p, float *o) {
        if (VEC == 4) {
            float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
            if (in(0)) q = *reinterpret_cast<const float4 *>(p + t * 4);
            o[0] = q.x; o[1] = q.y; o[2] = q.z; o[3] = q.w;
        } else {
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = in(z) ? p[t + 256 * z] : 0.f;
        }
    };
    auto store = [&](float *p, const float *o) {
        if (VEC == 4) {
            if (in(0)) *reinterpret_cast<float4 *>(p + t * 4) = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int z = 0; z < 4; ++z)
                if (in(z)) p[t + 256 * z] = o[z];
        }
    };
    constexpr int A = PA ? 5 : 3;                                    // g, m, e (v, vhat) of the worker at hand and of the next
    float cur[A][4], nxt[A][4];
    auto load_worker = [&](int32_t i, float (&o)[A][4]) {
        const int64_t off = (int64_t)i * a.d + l0;
        load(a.g + off, o[0]);
        load(a.m + off, o[1]);
        load(a.e + off, o[2]);
        if constexpr (PA) {
            load(a.v + off, o[3]);
            load(a.vhat + off, o[4]);
        }
    };
    load_worker(i0, cur);
    uint32_t sel = 0;                                                // bit z: the thread's coordinate z is in I_t
    if (a.k > 0) {                                                   // uniform over the launch
        if (t < 32) bits[t] = 0;
        member_range(a.idx, a.k, l0, l0 + 1024, range);
        __syncthreads();
        for (int64_t q = range[0] + t; q < range[1]; q += 256) {
            const int p = (int)(a.idx[q] - l0);
            atomicOr(&bits[p >> 5], 1u << (p & 31));
        }
        __syncthreads();
#pragma unroll
        for (int z = 0; z < 4; ++z) sel |= ((bits[at(z) >> 5] >> (at(z) & 31)) & 1u) << z;
    }
    float gs[4];
    for (int32_t i = i0; i < i1; ++i) {
        if (i + 1 < i1) load_worker(i + 1, nxt);
        float mo[4], uo[4];
        if constexpr (!PA) {
#pragma unroll
            for (int z = 0; z < 4; ++z) gs[z] = i == i0 ? cur[0][z] : (gs[z] + cur[0][z]);
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const float gv = cur[0][z];
            const float mm = ((a.beta1 * cur[1][z]) + (a.omb1 * gv));
            const float ein = ((sel >> z) & 1u) ? 0.0f : cur[2][z];  // e_t is zero on I_t
            mo[z] = mm;
            if constexpr (PA) {
                const float v2 = ((a.beta2 * cur[3][z]) + (a.omb2 * (gv * gv)));
                cur[3][z] = v2;
                if (v2 > cur[4][z]) cur[4][z] = v2;
                uo[z] = ((mm / sqrtf(cur[4][z])) + (a.rho * ein));
            } else {
                uo[z] = (mm + (a.rho * ein));
            }
        }
        const int64_t off = (int64_t)i * a.d + l0;
        store(a.m + off, mo);
        store(a.e + off, uo);
        if constexpr (PA) {
            store(a.v + off, cur[3]);
            store(a.vhat + off, cur[4]);
        }
#pragma unroll
        for (int q = 0; q < A; ++q)
#pragma unroll
            for (int z = 0; z < 4; ++z) cur[q][z] = nxt[q][z];
    }
    if constexpr (!PA) {
        if (y == 0) {                                                // v and vhat off I_t, where h = 0
            float vv[4], vh[4];
            load(a.v + l0, vv);
            load(a.vhat + l0, vh);
            bool moved = false;
            const bool all = a.ny == 1;                              // of the workers have been here: members as well
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const float h = all && ((sel >> z) & 1u) ? (gs[z] / (float)a.n) : 0.0f;
                vv[z] = ((a.beta2 * vv[z]) + (a.omb2 * (h * h)));
                if (vv[z] > vh[z]) { vh[z] = vv[z]; moved = true; }
            }
            if (all || sel == 0u) {
                store(a.v + l0, vv);
                if (moved) store(a.vhat + l0, vh);
            } else {                                                 // the members belong to a sparse workgroup
#pragma unroll
                for (int z = 0; z < 4; ++z)
                    if (in(z) && !((sel >> z) & 1u)) {
                        a.v[l0 + at(z)] = vv[z];
                        a.vhat[l0 + at(z)] = vh[z];
                    }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// stage 2: mean of the worker sketches (Alg. 2, master)
// ------------------------------------------------------------------------------------------
// VEC = 4: four consecutive cells per thread with 16-byte loads (needs r*c to be a multiple of 4, so that
// every worker's table starts on a 16-byte boundary)
__device__ __forceinline__ float4 ld4_stream(const float *p)
{
    typedef float vec4f __attribute__((ext_vector_type(4)));
    const vec4f t = __builtin_nontemporal_load(reinterpret_cast<const vec4f *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}

// AHEAD: tables whose loads a thread has in flight
template <int VEC, int AHEAD>
__global__ void __launch_bounds__(256)
k_reduce(const float *__restrict__ S_w, float *__restrict__ S_mean, int32_t n, int64_t rc)
{
    int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * VEC;
    const int64_t st = (int64_t)gridDim.x * blockDim.x * VEC;
    const float fn = (float)n;
    for (; t < rc; t += st) {
        if constexpr (VEC == 4) {
            float4 acc = ld4_stream(S_w + t);                        // every table is read once: streaming loads
            for (int32_t i0 = 1; i0 < n; i0 += 8) {                  // eight tables' loads in flight, added in worker order
                float4 b[8];
#pragma unroll
                for (int z = 0; z < AHEAD; ++z) {
                    const int32_t i = (i0 + z < n) ? (i0 + z) : (n - 1);
                    b[z] = ld4_stream(S_w + (int64_t)i * rc + t);
                }
#pragma unroll
                for (int z = 0; z < AHEAD; ++z) {
                    if (i0 + z < n) {
                        acc.x = (acc.x + b[z].x);
                        acc.y = (acc.y + b[z].y);
                        acc.z = (acc.z + b[z].z);
                        acc.w = (acc.w + b[z].w);
                    }
                }
            }
            *reinterpret_cast<float4 *>(S_mean + t) = make_float4((acc.x / fn), (acc.y / fn), (acc.z / fn), (acc.w / fn));
        } else {
            float acc = S_w[t];
            for (int32_t i0 = 1; i0 < n; i0 += AHEAD) {
                float b[AHEAD];
#pragma unroll
                for (int z = 0; z < AHEAD; ++z) b[z] = S_w[(int64_t)(i0 + z < n ? i0 + z : n - 1) * rc + t];
#pragma unroll
                for (int z = 0; z < AHEAD; ++z)
                    if (i0 + z < n) acc = (acc + b[z]);
            }
            S_mean[t] = (acc / fn);
        }
    }
}

// ------------------------------------------------------------------------------------------
// stage 4: exact values of the selected coordinates (second round, Sec. III-A)
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_gather(const float *__restrict__ u, const float *__restrict__ vhat, const int32_t *__restrict__ idx,
         int64_t k, int32_t n, int64_t d, float *__restrict__ U_w, float *__restrict__ delta)
{
    int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= k) return;
    int64_t l = idx[q];
    float acc = 0.0f;
    // eight workers' values are fetched before the first is used (with many workers and few coordinates the
    // kernel is a chain of memory latencies otherwise); they are still added in worker order
    for (int32_t i0 = 0; i0 < n; i0 += 8) {
        float val[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const int32_t i = (i0 + z < n) ? (i0 + z) : (n - 1);
            val[z] = u[(int64_t)i * d + l];
        }
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            if (i0 + z < n) {
                U_w[(int64_t)(i0 + z) * k + q] = val[z];
                acc = (i0 + z == 0) ? val[z] : (acc + val[z]);
            }
        }
    }
    float mean = (acc / (float)n);
    delta[q] = vhat ? (mean / sqrtf(vhat[l])) : mean;
}

// The same for many workers: 32 lanes share a coordinate and fetch its n values side by side; they meet in LDS
// and one lane adds them in worker order.  With n in the tens and k in the hundreds the one-thread-per-
// coordinate kernel is a chain of n memory latencies on a handful of compute units.
__global__ void __launch_bounds__(256)
k_gather_wide(const float *__restrict__ u, const float *__restrict__ vhat, const int32_t *__restrict__ idx,
              int64_t k, int32_t n, int64_t d, float *__restrict__ U_w, float *__restrict__ delta)
{
    __shared__ float vals[kWideCoords * kMaxWorkers];
    const int ql = threadIdx.x >> 5, wl = threadIdx.x & 31;
    const int64_t q = blockIdx.x * (int64_t)kWideCoords + ql;
    const int64_t l = q < k ? idx[q] : 0;
    if (q < k) {
        for (int32_t i = wl; i < n; i += 32) {
            const float val = u[(int64_t)i * d + l];
            U_w[(int64_t)i * k + q] = val;
            vals[ql * n + i] = val;
        }
    }
    __syncthreads();
    if (q < k && wl == 0) {
        float acc = vals[ql * n];
        for (int32_t i = 1; i < n; ++i) acc = (acc + vals[ql * n + i]);
        const float mean = (acc / (float)n);
        delta[q] = vhat ? (mean / sqrtf(vhat[l])) : mean;
    }
}

int enqueue_tail_only(sams_ctx *ctx, float *e_u, float *x, const int32_t *idx, const float *delta, int64_t k_sel, float lr)
{
    if (k_sel == 0) return SAMS_OK;
    SAMS_LAUNCH(ctx, KID_TAIL_ZERO_E, k_tail_zero_e, grid_for(k_sel, 256), 256, idx, delta, k_sel, ctx->n, ctx->d, lr, x, e_u);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

int enqueue_tail(sams_ctx *ctx, float *x, const int32_t *idx, const float *delta, int64_t k_sel, float lr)
{
    const int64_t words = (ctx->d + 31) / 32;
    SAMS_LAUNCH(ctx, KID_TAIL, k_tail, grid_for(words, 256), 256, idx, delta, k_sel, words, lr, x, ctx->bitmap, ctx->wordrank);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

constexpr int64_t kUpdateLong = (int64_t)1 << 25;    // entries of g
int enqueue_update(sams_ctx *ctx, const float *g, float *m, float *e_u, float *v, float *vhat, float *x, const int32_t *idx,
                   const float *delta, int64_t k_sel, float beta1, float beta2, float lr, float rho, bool pa)
{
    const int64_t ntile = (ctx->d + 1023) / 1024;
    // Enough workgroups for a few per compute unit: the workers of a tile are shared out when there are few tiles.  A worker is
    // also traffic enough for the search to be hidden with per-worker second moments (n = 8, d = 11.2 million: 589 us, 635 with all
    // workers of a tile in one workgroup), and once g, m and e are more than the 256 MB Infinity Cache: the workgroups under
    // way then go through one worker's arrays instead of all (n = 8: 11.2 million 380 and 440 us, 124 million 4.2 and 4.8 ms;
    // n = 33, three million 376 and 416 us; n = 3, 11.2 million 182 and 189 us; below, n = 8, 103 and 95 us at three million).
    int64_t ny = (2048 + ntile - 1) / ntile;
    if (ny > ctx->n || pa || ctx->n * ctx->d >= kUpdateLong) ny = ctx->n;
    // With more than 1 in 64 coordinates in I_t the sparse workgroups' gathers of g, a memory line per value, cost more than that:
    // all workers in one workgroup, which has h of its members by itself.  Shared out and by itself: n = 8, d = 11.2 million, 1 % of
    // the coordinates 414 and 422 us, 2 % 449 and 441, 10 % 515 and 449; n = 4, 60 million, 2 % 1.38 and 1.30 ms; n = 16, 200,001
    // (196 tiles), 2 % 13 and 15 us.
    if (!pa && k_sel > ctx->d / 64 && ntile >= 256) ny = 1;
    const int32_t wchunk = (int32_t)((ctx->n + ny - 1) / ny);
    ny = (ctx->n + wchunk - 1) / wchunk;
    const int64_t per_sparse = pa || ny == 1 || ctx->n < kWideMinWorkers ? 256 : kWideCoords;
    const int64_t blocks = ntile * ny + (k_sel + per_sparse - 1) / per_sparse;
    const UpdateArgs a = {g, m, e_u, v, vhat, x, idx, delta, k_sel, ctx->d, ntile, ctx->n, wchunk, (int32_t)ny, beta1, 1.0f - beta1,
                          beta2, 1.0f - beta2, rho, lr};
    const bool vec = (ctx->d & 3) == 0;
    ProfScope ps(ctx, pa ? KID_HEAD_PA : KID_HEAD);
    const auto kernel = pa ? (vec ? k_update<4, true> : k_update<1, true>) : (vec ? k_update<4, false> : k_update<1, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, ctx->stream, a);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

int enqueue_reduce(sams_ctx *ctx, const float *S_workers, float *S_mean)
{
    const int64_t rc = (int64_t)ctx->r * ctx->c;
    // one cell per thread for small tables: with four, a table of 2,000 cells would be two workgroups, each a chain of n / 8
    // memory latencies (n = 100: 14 us)
    if ((rc & 3) == 0 && rc >= 4 * 256 * 256)
        SAMS_LAUNCH(ctx, KID_REDUCE, (k_reduce<4, 8>), grid_for(rc / 4, 256, 1 << 16), 256, S_workers, S_mean, ctx->n, rc);
    else {
        // about as many tables in flight as there are: in place of those past the last one it is read again (n = 2, 7 x 262,143 4.2
        // and 7.7 us with one and eight, n = 10, 5 x 1,048,577 37 and 54 us with 16 and 32)
        const auto kernel = ctx->n <= 2 ? k_reduce<1, 1> : ctx->n <= 3 ? k_reduce<1, 2> : ctx->n <= 9 ? k_reduce<1, 8>
                            : ctx->n <= 17 ? k_reduce<1, 16> : k_reduce<1, 32>;
        SAMS_LAUNCH(ctx, KID_REDUCE, kernel, grid_for(rc, 256, 1 << 16), 256, S_workers, S_mean, ctx->n, rc);
    }
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

int enqueue_gather(sams_ctx *ctx, const float *u, const float *vhat, const int32_t *idx,
                   float *U_workers, float *delta)
{
    if (ctx->n >= kWideMinWorkers)
        SAMS_LAUNCH(ctx, KID_GATHER, k_gather_wide, (unsigned)((ctx->k + kWideCoords - 1) / kWideCoords), 256, u, vhat,
                    idx, ctx->k, ctx->n, ctx->d, U_workers, delta);
    else
        SAMS_LAUNCH(ctx, KID_GATHER, k_gather, grid_for(ctx->k, 256), 256, u, vhat, idx, ctx->k, ctx->n,
                    ctx->d, U_workers, delta);
    SAMS_HIP(hipGetLastError());
    return SAMS_OK;
}

}  // namespace sams

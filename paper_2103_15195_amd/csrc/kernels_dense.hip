// Dense-code compressors (EF-Sign, QSGD, TernGrad, FP16) and their
// decompress-and-sum, for gfx950.  One launch covers a whole merged group
// (Section 4.1 of the paper: the tensors of a group are compressed in one
// operation); tensors are reached through the segment table, nothing is copied.
//
// All kernels are HBM-streaming: each operand is touched once per pass with
// lane-consecutive 4-byte accesses (256 contiguous bytes per wave instruction),
// sign / ternary planes are packed with 64-lane ballots, group scalars are
// reduced per block in LDS and combined by the kernel itself: in groups of at most 64 tiles by the block that arrives last, in
// others by a block that waits for them (OneBit, and very large groups: a one-block kernel after it).
#include <algorithm>
#include <cstddef>

#include "mc_internal.h"

namespace mc {

// ---------------------------------------------------------------------------
// pointer-table upload: the per-call list of tensor addresses travels in the
// kernel argument buffer, so no host staging memory has to outlive the call.
// ---------------------------------------------------------------------------
__global__ void upload_ptrs_k(PtrChunk chunk, uintptr_t *dst, uint32_t count)
{
    uint32_t i = threadIdx.x;
    if (i < count) dst[i] = chunk.p[i];
}

void launch_upload_ptrs(const LaunchCtx &lc, const uintptr_t *host, uintptr_t *dev, uint32_t count)
{
    for (uint32_t done = 0; done < count; done += 256) {
        PtrChunk ch;
        uint32_t m = count - done < 256 ? count - done : 256;
        for (uint32_t i = 0; i < 256; ++i) ch.p[i] = i < m ? host[done + i] : 0;
        prof_begin(lc, K_UPLOAD);
        MC_LAUNCH(upload_ptrs_k, dim3(1), dim3(256), lc, ch, dev + done, m);
        prof_end(lc, K_UPLOAD);
    }
}

// Per-chunk address table of a freshly uploaded tensor address list: the address of
// the chunk's first element when all 1024 elements lie in one tensor, else 2 s + 1 with s the tensor of its first element.
__global__ __launch_bounds__(kBlock) void expand_ptrs_k(GroupView g, uintptr_t *chunk_addr)
{
    const uint32_t nchunks = (g.n + (uint32_t)kChunk - 1u) / (uint32_t)kChunk;
    const uint32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= nchunks) return;
    const uint32_t base = c * (uint32_t)kChunk;
    const uint32_t s = g.chunk_seg[c];
    const uint32_t beg = g.seg_off[s], end = g.seg_off[s + 1];
    uintptr_t a = ((uintptr_t)s << 1) | 1u;            // not an address: where the loop over the chunk's tensors starts
    if (g.n - base >= (uint32_t)kChunk && end - base >= (uint32_t)kChunk) a = g.ptrs[s] + (uintptr_t)(base - beg) * sizeof(float);
    chunk_addr[c] = a;
}

void launch_expand_ptrs(const LaunchCtx &lc, const GroupView &g, uintptr_t *chunk_addr)
{
    if (g.n == 0) return;
    const uint32_t nchunks = (uint32_t)(((uint64_t)g.n + kChunk - 1) / kChunk);
    prof_begin(lc, K_UPLOAD);
    MC_LAUNCH(expand_ptrs_k, dim3((nchunks + kBlock - 1) / kBlock), dim3(kBlock), lc, g, chunk_addr);
    prof_end(lc, K_UPLOAD);
}

// The same for the chunks of all groups (tb.list and the tables are on the device already).
__global__ __launch_bounds__(kBlock) void expand_all_k(GroupTable tb, uint32_t tiles, uintptr_t *chunk_addr)
{
    const uint32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= tiles * (uint32_t)kWavesPerBlock) return;
    const GroupConst &G = tb.groups[tb.block_group[BLK_TILE][c / kWavesPerBlock]];
    const uint32_t local = c - G.first[BLK_TILE] * (uint32_t)kWavesPerBlock, base = local * (uint32_t)kChunk;
    if (base >= G.n) return;                           // the last tile of a group may have fewer than four chunks
    const uint32_t s = G.chunk_seg[local];
    const uint32_t beg = G.seg_off[s], end = G.seg_off[s + 1];
    uintptr_t a = ((uintptr_t)s << 1) | 1u;
    if (G.n - base >= (uint32_t)kChunk && end - base >= (uint32_t)kChunk) a = tb.list[G.first_ptr + s] + (uintptr_t)(base - beg) * sizeof(float);
    chunk_addr[c] = a;
}

void launch_expand_all(const LaunchCtx &lc, const GroupTable &tb, uint32_t tiles, uintptr_t *chunk_addr)
{
    if (tiles == 0) return;
    prof_begin(lc, K_UPLOAD);
    MC_LAUNCH(expand_all_k, dim3((tiles * kWavesPerBlock + kBlock - 1) / kBlock), dim3(kBlock), lc, tb, tiles, chunk_addr);
    prof_end(lc, K_UPLOAD);
}

// ---------------------------------------------------------------------------
// The one-bit schemes, single pass: one sign bit per element of a vector p.
//   SIGN_EF       EF-Sign: delta = (||p||_1 / n) sign(p), p = g + e, e <- p - delta
//   SIGN_MEANS    OneBit: delta = mean of the class (p >= 0 / p < 0) of the element, same residual rule
//   SIGN_PLAIN    SignSGD: p = g, nothing is remembered
//   SIGN_MOMENTUM SigNUM: p = m <- beta m + (1 - beta) g, the momentum is the state
// The bits of the first two do not depend on their group scalars, so the residual is
// not written: the state keeps p and the scalars of the call that produced it, and
// the residual of the previous call is re-derived on the fly as
//     e = p_prev - (p_prev >= 0 ? hi_prev : lo_prev)          (EF-Sign: hi = s, lo = -s)
// with the same fp32 operations an explicit update would have used.
// Traffic per element: read g, read p_prev, write p, 1/8 byte of sign bits.
// Per-block partials: EF-Sign sum |p|; OneBit sum of the upper class, sum of the lower
// class, size of the upper class (three arrays of gridDim.x doubles).
// ---------------------------------------------------------------------------
// header of a payload whose group scalar needs no reduction (written by one thread of the compress kernel itself)
__device__ __forceinline__ void put_plain_header(PayloadHeader *hdr, uint32_t algo, uint32_t n, float scale, float scale_lo = 0.0f, uint32_t levels = 0u)
{
    PayloadHeader h;
    h.magic = kMagic; h.algo = algo; h.n = n; h.k = 0; h.scale = scale; h.levels = levels;
    for (int i = 0; i < 24; ++i) h.pad[i] = 0;
    h.pad[0] = __float_as_uint(scale_lo);
    *hdr = h;
}
// the group scalars from the combined partials (fp64, rounded once)
__device__ __forceinline__ float mean_abs(double sum, uint32_t n) { return (float)(sum / (double)n); }
__device__ __forceinline__ void class_means(double sum_hi, double sum_lo, double n_hi, uint32_t n, float &hi, float &lo)
{
    const double n_lo = (double)n - n_hi;
    hi = n_hi > 0.0 ? (float)(sum_hi / n_hi) : 0.0f;
    lo = n_lo > 0.0 ? (float)(sum_lo / n_lo) : 0.0f;
}

// ---- small groups: partial sums combined inside the kernel -------------------------------------------------------
// A block's partial goes past the die's cache, and when it is there the block adds one to the group's count, which is
// never reset: call c of a group of N tiles takes it from c N to (c + 1) N.
__device__ __forceinline__ void put_partial(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// one thread of the block that put its partials: the count before
__device__ __forceinline__ uint64_t arrive_at(uint64_t *count)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);             // the partials are written through before the count says so
    return __hip_atomic_fetch_add(count, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The other end: after the count has been seen complete, before the partials are read.  (They bypass the caches, so nothing
// has to be invalidated; but relaxed loads of different addresses are otherwise free to be moved before the count's.)
__device__ __forceinline__ void all_arrived() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); }
// the wavefront that put the block's partials: whether all of the group's blocks have put theirs
__device__ __forceinline__ bool arrives_last(const CompressJob &job)
{
    uint64_t before = 0;
    if (threadIdx.x == 0) before = arrive_at(job.arrive);
    before = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)before) |
             ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(before >> 32)) << 32);
    if (before % job.ntiles != job.ntiles - 1u) return false;
    all_arrived();
    return true;
}
// one wavefront, N <= 64 partials: their sum (maximum) in the order of scalar_finalize_k, in all lanes
template <bool MAX>
__device__ __forceinline__ double combine_partials(const double *partial, uint32_t N)
{
    const uint32_t lane = threadIdx.x & 63u;
    double acc = lane < N ? __hip_atomic_load(partial + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const double o = __shfl_xor(acc, m, 64);
        acc = MAX ? fmax(acc, o) : acc + o;
    }
    return acc;
}

// ---- launches with larger groups: collectors -------------------------------------------------------------------------
// A launch's last blocks wait for the partials of the groups of more than 64 tiles and combine them as scalar_finalize_k would.  The partials are stored
// past the die's cache, each into a slot that is empty (all ones, which no sum is) until its tile's block has filled it, and the collector empties it
// again, so that there is nothing to count.  It looks at the last tiles first, which are the first to be done, and when the last
// block has stored its partial it takes about two trips to memory more, where a kernel of its own took a boundary, a start and the loads of all
// partials.  Groups of up to 64 tiles in such a launch are combined by the block that arrives last, and nobody waits.
// (Compress and decompress-and-sum, that kernel -> collectors: 25.6 M elements, EF-Sign 79.8 -> 78.2 us, in 161 groups 79.6 -> 78.1, QSGD
// in three groups 123.9 -> 122.3; 44.5 M, 16 workers, EF-Sign 142.3 -> 140.5; 10 M, TernGrad 46.5 -> 45.6.  Compress of 400 groups of 1000 elements / 2000 of
// 256, and one of 1.6 M: EF-Sign, that kernel 13.8 / 28.0 us, collectors for all groups 22.0 / 72.5, now 10.2 / 14.9; QSGD 21.3 / 38.4, 29.6 / 81.7, 17.5 / 25.3.)
// A collector waits for blocks that start before it, and which wait for nothing.  Should that not come to an end all the same, it
// leaves after `looks` looks and flags it: from then on slots may hold what a call before has left, and no call on such groups sends a valid header
// until mc_last_device_status has reported it and emptied the slots.
constexpr uint64_t kEmptySlot = ~0ull;
__device__ __forceinline__ void fill_slot(double *p, double v)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), x == kEmptySlot ? 0x7FF8000000000000ull : x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kFinalThreads = 1024;
// The sum (maximum) of n slots, in scalar_finalize_k's order: what each of its threads adds is added by itself, THREADS of the
// block's threads standing for kFinalThreads.  False: not to be had.
template <int THREADS, bool MAX>
__device__ __forceinline__ bool collect(const CompressJob &job, int *status, uint32_t limit, double *red /* LDS, a word per wavefront of kFinalThreads */,
                                        bool *vain /* LDS */, double &sum)
{
    constexpr int kEach = kFinalThreads / THREADS, kLoads = 4;
    uint64_t *const from = reinterpret_cast<uint64_t *>(job.slots);
    const uint32_t n = job.ntiles;
    const int flagged = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (looked at behind the partials)
    double acc[kEach];
#pragma unroll
    for (int v = 0; v < kEach; ++v) acc[v] = 0.0;
    uint32_t looks = *vain ? limit + 1u : 0u;
    for (uint32_t top = (n + kFinalThreads - 1u) / kFinalThreads; top > 0u; top = top > (uint32_t)(kLoads / kEach) ? top - (uint32_t)(kLoads / kEach) : 0u) {
        uint64_t x[kLoads];
        auto at = [&](int l) {                   // load l: round (the highest first), share; n and more: none
            const uint32_t r = (uint32_t)(l / kEach), i = (top - 1u - r) * (uint32_t)kFinalThreads + (uint32_t)(l % kEach * THREADS) + threadIdx.x;
            return r < top ? i : n;
        };
        for (;;) {
            bool missing = false;
#pragma unroll
            for (int l = 0; l < kLoads; ++l) x[l] = at(l) < n ? __hip_atomic_load(from + at(l), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
#pragma unroll
            for (int l = 0; l < kLoads; ++l) missing = missing || x[l] == kEmptySlot;
            if (!missing || looks > limit) break;
            if (looks++ == limit) { raise_flag(status, FLAG_GAVE_UP); break; }
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int l = 0; l < kLoads; ++l) {
            if (at(l) < n) from[at(l)] = kEmptySlot;
            const double y = __builtin_bit_cast(double, x[l]);
            acc[l % kEach] = MAX ? fmax(acc[l % kEach], y) : acc[l % kEach] + y;
        }
    }
#pragma unroll
    for (int v = 0; v < kEach; ++v) {
        double s = acc[v];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const double o = __shfl_xor(s, m, 64);
            s = MAX ? fmax(s, o) : s + o;
        }
        if ((threadIdx.x & 63u) == 0) red[v * (THREADS / 64) + (int)(threadIdx.x >> 6)] = s;
    }
    if (__builtin_amdgcn_ballot_w64(flagged == FLAG_GAVE_UP || looks > limit) != 0ull) *vain = true;
    __syncthreads();
    sum = red[0];
#pragma unroll 4
    for (int w = 1; w < kFinalThreads / 64; ++w) sum = MAX ? fmax(sum, red[w]) : sum + red[w];
    return !*vain;
}
// body(group's job, sum, or not valid) for the groups of this collector, the last ones first
template <int THREADS, bool MAX, class SRC, class Body>
__device__ __forceinline__ void each_collected(const SRC &src, Body body)
{
    __shared__ double red[kFinalThreads / 64];
    __shared__ bool vain;                        // whether a scalar was not to be had: no later one is, then
    if (threadIdx.x == 0) vain = false;
    __syncthreads();
    const uint32_t collectors = gridDim.x - src.tiles(), y = src.collected();
    for (uint32_t q = blockIdx.x - src.tiles(); q < y; q += collectors) {
        const CompressJob job = src.collected_job(q);
        double sum = 0.0;
        const bool valid = collect<THREADS, MAX>(job, src.status, src.looks, red, &vain, sum);
        body(job, sum, valid);
        __syncthreads();                         // (red)
    }
}
// A tile's partial is there, in the block's first thread.  True, in one wavefront, if this block has the group's scalar to write.
template <bool MAX>
__device__ __forceinline__ bool hand_in(const CompressJob &job, double mine, double &sum)
{
    if (job.ntiles > kSmallTiles) {
        if (threadIdx.x == 0) fill_slot(job.slots + job.tile, mine);
        return false;
    }
    if (threadIdx.x >= 64u) return false;
    if (threadIdx.x == 0) put_partial(job.partial + job.tile, mine);
    if (!arrives_last(job)) return false;
    sum = combine_partials<MAX>(job.partial, job.ntiles);
    return true;
}
// the header of a payload whose scalar is not to be had: no payload's
__device__ __forceinline__ void put_no_header(PayloadHeader *hdr) { *hdr = PayloadHeader{}; }

// HOW = COMBINE_LAST: the group's last block to arrive combines the partials and writes the headers, instead of a kernel after this one.
// (EF-Sign compress, 1 .. 64 tiles: 8.0 -> 5.6 .. 5.9 us, OneBit 8.6 .. 9.2 -> 6.2 .. 7.5: a launch and a kernel boundary less.
// With the tile spread over more threads, 33 / 34 000 / 262 000 elements: EF-Sign 5.9 / 5.9 / 6.0 -> 4.8 / 5.4 / 5.8, OneBit 7.4 / 7.5 / 8.0 ->
// 6.2 / 6.8 / 7.5, SignSGD 3.4 / 3.6 / 3.7 -> 2.2 / 2.4 / 2.6.)
// S: elements per lane, 16, or 4 on a launch of few tiles (kSpread threads per tile).
template <int MODE, bool EF, class SRC, int HOW = COMBINE_AFTER, int S = kSteps>
__global__ __launch_bounds__(kTile / S) void sign_compress_k(SRC src, float beta, uint32_t algo)
{
    constexpr int kWaves = kTile / S / kWave;
    __shared__ uint64_t stage[kWaves][S];
    __shared__ double red[kWaves];
    __shared__ double red3[MODE == SIGN_MEANS ? 3 : 1][kWaves];
    constexpr bool kHeld = S != kSteps && (MODE == SIGN_EF || MODE == SIGN_MEANS);
    __shared__ float held[kHeld ? kTile : 1];    // p of the tile, to be summed in the order of the other form
    auto publish = [&](const CompressJob &of, double sum, bool valid) {
        if (threadIdx.x) return;
        if (!valid) { put_no_header(of.hdr); return; }
        const float scale = mean_abs(sum, of.g.n);
        put_plain_header(of.hdr, algo, of.g.n, scale);
        if (EF) of.state_header()->scale = scale;        // (every block of the group has read the last call's)
    };
    if constexpr (HOW == COMBINE_COLLECT) {
        static_assert(MODE == SIGN_EF, "one sum");
        if (blockIdx.x >= src.tiles()) { each_collected<kTile / S, false>(src, publish); return; }
    }
    const CompressJob job = src.job();
    const GroupView &g = job.g;
    float *st = job.st;
    uint32_t *words = reinterpret_cast<uint32_t *>(job.body());
    const uint32_t nwords = (g.n + 31u) >> 5;
    const Chunk c = my_chunk<S>(g.n, job.tile);
    // SignSGD, SigNUM: the decoded values are +-1, no finalize kernel follows
    if ((MODE == SIGN_PLAIN || MODE == SIGN_MOMENTUM) && job.tile == job.ntiles - 1u && threadIdx.x == 0) put_plain_header(job.hdr, algo, g.n, 1.0f);
    double acc = 0.0, acc_lo = 0.0, cnt_hi = 0.0;
    if (c.base < g.n) {
        float p[S];
        load_seg(g, c, p);
        if (MODE == SIGN_MOMENTUM) {
            const float omb = 1.0f - beta;
            float q[S];
            load_flat(st, c, g.n, q, 0.0f);
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const float bm = beta * q[j], og = omb * p[j];
                p[j] = bm + og;
            }
            store_flat(st, c, g.n, p);
        } else if (EF && MODE != SIGN_PLAIN) {
            const StateHeader *prev = job.state_header();
            const float hi = prev->scale, lo = MODE == SIGN_MEANS ? prev->scale_lo : -hi;
            float q[S];
            load_flat(st, c, g.n, q, 0.0f);
#pragma unroll
            for (int j = 0; j < S; ++j) {
                float d = q[j] >= 0.0f ? hi : lo;
                float e = q[j] - d;
                p[j] = p[j] + e;
            }
            store_flat(st, c, g.n, p);
        }
        uint64_t b[S];
#pragma unroll
        for (int j = 0; j < S; ++j) {
            bool valid = c.full || (c.base + 64 * j + c.lane < g.n);
            const bool up = valid && p[j] >= 0.0f;
            b[j] = __builtin_amdgcn_ballot_w64(up);
            if (kHeld) { held[c.base % (uint32_t)kTile + 64 * j + c.lane] = p[j]; continue; }
            if (MODE == SIGN_EF) acc += valid ? fabs((double)p[j]) : 0.0;
            if (MODE == SIGN_MEANS) {
                acc += up ? (double)p[j] : 0.0;
                acc_lo += valid && !up ? (double)p[j] : 0.0;
            }
        }
        if (MODE == SIGN_MEANS) {
#pragma unroll
            for (int j = 0; j < S; ++j) if (c.lane == 0) cnt_hi += (double)__popcll(b[j]);
        }
        store_plane(words, nwords, c, b, stage[threadIdx.x >> 6]);
    }
    if (kHeld) {
        __syncthreads();
        const uint32_t left = g.n - job.tile * (uint32_t)kTile;
        if (threadIdx.x < (uint32_t)kBlock) {
#pragma unroll
            for (int j = 0; j < kSteps; ++j) {
                const uint32_t i = threadIdx.x / 64u * (uint32_t)kChunk + 64u * j + c.lane;
                const bool valid = i < left;
                const float x = held[i];
                const bool up = valid && x >= 0.0f;
                if (MODE == SIGN_EF) acc += valid ? fabs((double)x) : 0.0;
                else { acc += up ? (double)x : 0.0; acc_lo += valid && !up ? (double)x : 0.0; }
            }
        }
    }
    if (MODE == SIGN_EF) {
        double t = block_sum<kWaves>(acc, red);
        if constexpr (HOW == COMBINE_COLLECT) {
            double sum;
            if (hand_in<false>(job, t, sum)) publish(job, sum, true);
        } else if (threadIdx.x == 0) {
            if (HOW == COMBINE_LAST) put_partial(job.partial + job.tile, t); else job.partial[job.tile] = t;
        }
    }
    if (MODE == SIGN_MEANS) {       // the three sums behind one pair of barriers, each combined in block_sum's order
        acc = wave_sum(acc); acc_lo = wave_sum(acc_lo); cnt_hi = wave_sum(cnt_hi);
        if ((threadIdx.x & 63) == 0) { red3[0][threadIdx.x >> 6] = acc; red3[1][threadIdx.x >> 6] = acc_lo; red3[2][threadIdx.x >> 6] = cnt_hi; }
        __syncthreads();
        if (threadIdx.x < 3) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; w += 4) {
                const double four = (red3[threadIdx.x][w] + red3[threadIdx.x][w + 1]) + (red3[threadIdx.x][w + 2] + red3[threadIdx.x][w + 3]);
                t = w ? t + four : four;
            }
            const uint32_t at = threadIdx.x * job.ntiles + job.tile;
            if (HOW == COMBINE_LAST) put_partial(job.partial + at, t); else job.partial[at] = t;
        }
    }
    if (HOW == COMBINE_LAST && threadIdx.x < 64) {             // the wavefront that put the partials
        if (!arrives_last(job)) return;
        const uint32_t N = job.ntiles, n = g.n;
        const double a = combine_partials<false>(job.partial, N);
        float hi, lo = 0.0f;
        if (MODE == SIGN_MEANS) {
            const double b = combine_partials<false>(job.partial + N, N), n_hi = combine_partials<false>(job.partial + 2 * N, N);
            class_means(a, b, n_hi, n, hi, lo);
        } else hi = mean_abs(a, n);
        if (threadIdx.x == 0) {
            put_plain_header(job.hdr, algo, n, hi, lo);
            if (EF) { job.state_header()->scale = hi; if (MODE == SIGN_MEANS) job.state_header()->scale_lo = lo; }
        }
    }
}

// a collector for each group of more than 64 tiles, or for every kCollectors-th
template <class SRC>
static uint32_t collectors(const SRC &src) { return std::min(src.collected(), kCollectors); }

template <int MODE, bool EF, int HOW, class SRC>
static void sign_compress_t(const LaunchCtx &lc, const SRC &src, uint32_t tiles, float beta, uint32_t algo)
{
    constexpr uint32_t most = MODE == SIGN_EF || MODE == SIGN_MEANS ? kSpreadSumTiles : kSpreadTiles;
    const dim3 grid(tiles + (HOW == COMBINE_COLLECT ? collectors(src) : 0u));
    if (tiles <= most) MC_LAUNCH((sign_compress_k<MODE, EF, SRC, HOW, kSpreadSteps>), grid, dim3(kSpread), lc, src, beta, algo);
    else MC_LAUNCH((sign_compress_k<MODE, EF, SRC, HOW>), grid, dim3(kBlock), lc, src, beta, algo);
}
template <int MODE, bool EF, class SRC>
static void sign_compress_sums(const LaunchCtx &lc, const SRC &src, uint32_t tiles, uint32_t algo, bool small)
{
    if (small) { sign_compress_t<MODE, EF, COMBINE_LAST>(lc, src, tiles, 0.0f, algo); return; }
    if constexpr (MODE == SIGN_EF) if (src.slots) { sign_compress_t<MODE, EF, COMBINE_COLLECT>(lc, src, tiles, 0.0f, algo); return; }
    sign_compress_t<MODE, EF, COMBINE_AFTER>(lc, src, tiles, 0.0f, algo);
}

template <class SRC>
void launch_sign_compress(const LaunchCtx &lc, int mode, const SRC &src, uint32_t tiles, bool ef, float beta, uint32_t algo, bool small)
{
    if (tiles == 0) return;
    prof_begin(lc, K_EFSIGN_COMPRESS);
    switch (mode) {
    case SIGN_EF:
        if (ef) sign_compress_sums<SIGN_EF, true>(lc, src, tiles, algo, small);
        else sign_compress_sums<SIGN_EF, false>(lc, src, tiles, algo, small);
        break;
    case SIGN_MEANS:
        if (ef) sign_compress_sums<SIGN_MEANS, true>(lc, src, tiles, algo, small);
        else sign_compress_sums<SIGN_MEANS, false>(lc, src, tiles, algo, small);
        break;
    case SIGN_PLAIN:
        sign_compress_t<SIGN_PLAIN, false, COMBINE_AFTER>(lc, src, tiles, beta, algo);
        break;
    default:
        sign_compress_t<SIGN_MOMENTUM, true, COMBINE_AFTER>(lc, src, tiles, beta, algo);
        break;
    }
    prof_end(lc, K_EFSIGN_COMPRESS);
}
template void launch_sign_compress<OneCompress>(const LaunchCtx &, int, const OneCompress &, uint32_t, bool, float, uint32_t, bool);
template void launch_sign_compress<AllCompress>(const LaunchCtx &, int, const AllCompress &, uint32_t, bool, float, uint32_t, bool);

// ---------------------------------------------------------------------------
// One block per group: combine the per-block partials in a fixed order (bit-reproducible
// whatever the launch geometry of the producer was), derive the group scalar,
// write the payload header (and, for EF-Sign, the scale kept in the state).
//   RED_MEAN_ABS: scale = (float)(sum / n)      RED_L2: norm = (float)sqrt(sum)
//   RED_MAX_ABS : max of the partials (exact)   mode < 0: header only
//   RED_ONE     : scale = 1 (SignSGD, SigNUM: the decoded values are +-1)
//   RED_MEANS   : three partial arrays (sum of the upper class, of the lower class, size of the
//                 upper class) -> scale = mean of the upper class, second scalar = mean of the lower
// ---------------------------------------------------------------------------
template <class SRC>
__global__ __launch_bounds__(kFinalThreads) void scalar_finalize_k(SRC src, int mode, uint32_t algo, uint32_t levels, int keep)
{
    __shared__ double red[kFinalThreads / 64];
    const CompressJob job = src.group_job(blockIdx.x);
    const double *partial = job.partial;
    const uint32_t nblocks = job.ntiles, n = job.g.n;
    PayloadHeader *hdr = job.hdr;
    // where the state keeps the scalar(s) of this call (EF-Sign: one float, OneBit: two)
    float *state_scale = keep && n > 0 ? &job.state_header()->scale : nullptr;
    if (mode == RED_MEANS) {
        // the three sums side by side (their loads in flight together, one barrier), each in the fixed order of the
        // single-sum case
        __shared__ double red3[3][kFinalThreads / 64];
        double acc3[3] = {0.0, 0.0, 0.0};
        for (uint32_t rounds = (nblocks + 8u * kFinalThreads - 1u) / (8u * kFinalThreads); rounds-- > 0u;) {
            double v[3][8];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t i = (8u * rounds + 7u - (uint32_t)u) * (uint32_t)kFinalThreads + threadIdx.x;
                    v[a][u] = i < nblocks ? partial[(size_t)a * nblocks + i] : 0.0;
                }
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int u = 0; u < 8; ++u) acc3[a] += v[a][u];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) acc3[a] += __shfl_xor(acc3[a], m, 64);
            if ((threadIdx.x & 63) == 0) red3[a][threadIdx.x >> 6] = acc3[a];
        }
        __syncthreads();
        double S[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double T = red3[a][0];
            for (int w = 1; w < kFinalThreads / 64; ++w) T += red3[a][w];
            S[a] = T;
        }
        if (threadIdx.x == 0) {
            float hi, lo;
            class_means(S[0], S[1], S[2], n, hi, lo);
            put_plain_header(hdr, algo, n, hi, lo, levels);
            if (state_scale) { state_scale[0] = hi; state_scale[1] = lo; }
        }
        return;
    }
    double acc = 0.0;
    if (mode >= 0 && mode != RED_ONE) {
        // eight independent loads in flight per thread and round (one round up to 8192 partials);
        // the order of additions, a collector's (the last tiles are the first to be done), depends on nblocks only
        for (uint32_t rounds = (nblocks + 8u * kFinalThreads - 1u) / (8u * kFinalThreads); rounds-- > 0u;) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t i = (8u * rounds + 7u - (uint32_t)u) * (uint32_t)kFinalThreads + threadIdx.x;
                v[u] = i < nblocks ? partial[i] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = mode == RED_MAX_ABS ? fmax(acc, v[u]) : acc + v[u];
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        double o = __shfl_xor(acc, m, 64);
        acc = mode == RED_MAX_ABS ? fmax(acc, o) : acc + o;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double S = red[0];
        for (int w = 1; w < kFinalThreads / 64; ++w) S = mode == RED_MAX_ABS ? fmax(S, red[w]) : S + red[w];
        float scale = 0.0f;
        if (n > 0) {
            if (mode == RED_MEAN_ABS) scale = mean_abs(S, n);
            else if (mode == RED_L2) scale = (float)sqrt(S);
            else if (mode == RED_MAX_ABS) scale = (float)S;
        }
        if (mode == RED_ONE) scale = 1.0f;
        put_plain_header(hdr, algo, n, scale, 0.0f, levels);
        if (state_scale) *state_scale = scale;
    }
}

// keep: the state remembers the scalar(s)
template <class SRC>
void launch_scalar_finalize(const LaunchCtx &lc, const SRC &src, uint32_t groups, int mode, uint32_t algo, uint32_t levels, bool keep)
{
    prof_begin(lc, K_SCALAR_FINALIZE);
    MC_LAUNCH(scalar_finalize_k<SRC>, dim3(groups), dim3(kFinalThreads), lc, src, mode, algo, levels, keep ? 1 : 0);
    prof_end(lc, K_SCALAR_FINALIZE);
}
template void launch_scalar_finalize<OneCompress>(const LaunchCtx &, const OneCompress &, uint32_t, int, uint32_t, uint32_t, bool);
template void launch_scalar_finalize<AllCompress>(const LaunchCtx &, const AllCompress &, uint32_t, int, uint32_t, uint32_t, bool);

// The two stochastic quantizers, one element: what is sent and what the receiver reconstructs from it.
// QSGD with a = |p| s / norm:  level = floor(a) + [u < a - floor(a)], code = sgn(p) level, d = code * (norm / s).
// The two per-group divisions are taken in fp64 and rounded once, which equals the correctly rounded
// fp32 quotient of two fp32 numbers.
struct QsgdScale {
    float norm, sf, r, q;
    int levels;
    __device__ __forceinline__ QsgdScale(float norm_, uint32_t levels_)
        : norm(norm_), sf((float)levels_), r(norm_ > 0.0f ? (float)((double)(float)levels_ / (double)norm_) : 0.0f),
          q((float)((double)norm_ / (double)(float)levels_)), levels((int)levels_) {}
};
__device__ __forceinline__ int qsgd_code(const QsgdScale &k, float p, float u)
{
    int xi = 0;
    if (k.norm > 0.0f) {
        // a >= s (or not a number) means level s: clamped to s, the steps below give exactly that (floor s, fraction 0,
        // and no u lies below 0), and below s the level cannot exceed s -- one minimum instead of a compare, a select
        // and a second clamp
        const float a = fminf(fabsf(p) * k.r, k.sf);
        const float l = floorf(a);
        const float f = a - l;
        xi = (int)l + (u < f ? 1 : 0);
    }
    return p < 0.0f ? -xi : xi;
}
__device__ __forceinline__ float qsgd_decode(const QsgdScale &k, int code) { return (float)code * k.q; }
// TernGrad: nz = [u * smax < |p|] (Bernoulli(|p| / smax) without a division), d = +-smax or 0
__device__ __forceinline__ float tern_decode(float smax, float p, float u, bool valid, bool &nz, bool &neg)
{
    nz = valid && (u * smax < fabsf(p));
    neg = nz && p < 0.0f;
    return nz ? (neg ? -smax : smax) : 0.0f;
}

// ---------------------------------------------------------------------------
// Pass A of the two-pass quantizers: p = g + e, kept in the state; per-block partial of
// sum p^2 (QSGD) or max |p| (TernGrad).
// The state never holds e itself: what pass B sends is a function of p, of the group
// scalar and of the random stream (worker, iteration) alone, so the residual of the last
// call is re-derived here as  e = p_prev - d(p_prev)  by quantizing p_prev again with the
// scalar and the stream that the state header recorded -- the same fp32 operations an
// explicit update would have used.  Pass B then writes no residual (17 instead of 21
// bytes per element over the two passes).  A zero-filled or imported state has scalar 0,
// for which d = 0 and e = p.
// ---------------------------------------------------------------------------
// p = g + e of a chunk (zeros past the end of the group), kept in the state
template <bool EF, int MODE>
__device__ __forceinline__ void accumulate(const CompressJob &job, const Chunk &c, uint32_t levels, uint64_t seed, float (&p)[kSteps])
{
    const GroupView &g = job.g;
    if (c.base >= g.n) {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) p[j] = 0.0f;
        return;
    }
    load_seg(g, c, p);
    if (EF) {
        const StateHeader *prev = job.state_header();
        const float sprev = prev->scale;
        const uint32_t wprev = prev->prev_worker, iprev = prev->prev_iter;
        float q[kSteps], uni[kSteps];
        // an ordinary load: the state is written here and read once more by the encode pass.  (Compress of 25.6 M elements,
        // QSGD 75.9 -> 71.9 us, TernGrad 72.7 -> 69.7; also for the gradient 78.3, also in the encode pass 73.6.  In
        // the one-pass schemes an ordinary load of the state costs 5 us of 54.)
        load_flat<float, false>(job.st, c, g.n, q, 0.0f);
        chunk_uniforms(seed, wprev, iprev, g.goff + c.base, c.lane, uni);
        const QsgdScale ks(MODE == RED_L2 ? sprev : 0.0f, levels);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            float d;
            if (MODE == RED_L2) d = qsgd_decode(ks, qsgd_code(ks, q[j], uni[j]));
            else { bool nz, neg; d = tern_decode(sprev, q[j], uni[j], true, nz, neg); }
            const float e = q[j] - d;
            // past the end of the group there is nothing (QSGD with a subnormal norm decodes even a 0 to +-norm there)
            p[j] = c.full || c.base + 64 * j + c.lane < g.n ? p[j] + e : 0.0f;
        }
        store_flat(job.st, c, g.n, p);
    }
}

template <bool EF, int MODE, class SRC, int HOW>
__global__ __launch_bounds__(kBlock) void accum_reduce_k(SRC src, uint32_t levels, uint64_t seed)
{
    __shared__ double red[kWavesPerBlock];
    __shared__ float redf[kWavesPerBlock];
    auto publish = [&](const CompressJob &of, double x, bool valid) {
        if (threadIdx.x) return;
        if (valid) put_plain_header(of.hdr, MODE == RED_L2 ? MC_ALGO_QSGD : MC_ALGO_TERNGRAD, of.g.n, MODE == RED_L2 ? (float)sqrt(x) : (float)x, 0.0f, levels);
        else put_no_header(of.hdr);
    };
    if constexpr (HOW == COMBINE_COLLECT) {
        if (blockIdx.x >= src.tiles()) { each_collected<kBlock, MODE == RED_MAX_ABS>(src, publish); return; }
    }
    const CompressJob job = src.job();
    const Chunk c = my_chunk(job.g.n, job.tile);
    double acc = 0.0;
    float mx = 0.0f;
    if (c.base < job.g.n) {
        float p[kSteps];
        accumulate<EF, MODE>(job, c, levels, seed, p);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {   // elements past n are 0 and add nothing
            if (MODE == RED_L2) acc += (double)p[j] * (double)p[j];
            else mx = fmaxf(mx, fabsf(p[j]));
        }
    }
    const double t = MODE == RED_L2 ? block_sum(acc, red) : (double)block_max(mx, redf);
    if constexpr (HOW == COMBINE_COLLECT) {
        double x;
        if (hand_in<MODE == RED_MAX_ABS>(job, t, x)) publish(job, x, true);
    } else if (threadIdx.x == 0) job.partial[job.tile] = t;
}

template <bool EF, int MODE, class SRC>
static void accum_reduce_t(const LaunchCtx &lc, const SRC &src, uint32_t tiles, uint32_t levels, uint64_t seed)
{
    if (src.slots) MC_LAUNCH((accum_reduce_k<EF, MODE, SRC, COMBINE_COLLECT>), dim3(tiles + collectors(src)), dim3(kBlock), lc, src, levels, seed);
    else MC_LAUNCH((accum_reduce_k<EF, MODE, SRC, COMBINE_AFTER>), dim3(tiles), dim3(kBlock), lc, src, levels, seed);
}
template <class SRC>
void launch_accum_reduce(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, int mode, uint32_t levels, uint64_t seed)
{
    if (tiles == 0) return;
    prof_begin(lc, K_ACCUM_REDUCE);
    if (mode == RED_L2) {
        if (ef) accum_reduce_t<true, RED_L2>(lc, src, tiles, levels, seed);
        else accum_reduce_t<false, RED_L2>(lc, src, tiles, levels, seed);
    } else {
        if (ef) accum_reduce_t<true, RED_MAX_ABS>(lc, src, tiles, levels, seed);
        else accum_reduce_t<false, RED_MAX_ABS>(lc, src, tiles, levels, seed);
    }
    prof_end(lc, K_ACCUM_REDUCE);
}
template void launch_accum_reduce<OneCompress>(const LaunchCtx &, const OneCompress &, uint32_t, bool, int, uint32_t, uint64_t);
template void launch_accum_reduce<AllCompress>(const LaunchCtx &, const AllCompress &, uint32_t, bool, int, uint32_t, uint64_t);

// p of pass B: from the state (where pass A left it) or, without error feedback, the gradient itself
template <bool EF>
__device__ __forceinline__ void load_p(const GroupView &g, const float *st, const Chunk &c, float (&p)[kSteps])
{
    if (EF) load_flat(st, c, g.n, p, 0.0f);
    else load_seg(g, c, p);
}

// Store one one-byte code per element of a chunk.  Codes are staged through LDS so that each lane
// writes 16 contiguous bytes (a wave store of 64 single bytes covers only half a cache line, and
// measured slower; the two-byte codes of FP16 cover a whole line and are stored directly).
template <typename T>
__device__ __forceinline__ void store_codes(T *codes, uint32_t n, uint32_t n_padded, const Chunk &c,
                                            const T (&v)[kSteps], uint4 *stage /* room for kChunk entries, wave-private; read 16 bytes at a time */)
{
    static_assert(alignof(uint4) == 16, "the stage is read with 16-byte LDS loads");
    if (c.full) {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) reinterpret_cast<T *>(stage)[64 * j + c.lane] = v[j];
        __builtin_amdgcn_wave_barrier();
        constexpr int kVec = (int)(kChunk * sizeof(T) / 16 / kWave);     // 16-byte vectors per lane
        uint4 *dst = reinterpret_cast<uint4 *>(codes + c.base);
#pragma unroll
        for (int r = 0; r < kVec; ++r) dst[r * 64 + c.lane] = stage[r * 64 + c.lane];
        __builtin_amdgcn_wave_barrier();
    } else {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            uint32_t i = c.base + 64 * j + c.lane;
            if (i < n) codes[i] = v[j];
            else if (i < n_padded) codes[i] = (T)0;      // zero padding up to a multiple of 4 bytes
        }
    }
}

// ---------------------------------------------------------------------------
// Pass B of the two-pass quantizers: the codes of p.  With error feedback p stays in the state
// as it is, and one thread records the group scalar and the random stream of this call in the
// state header, from which the next call's pass A re-derives the residual (see there).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void remember_call(const CompressJob &job, float scale, uint32_t worker, uint32_t iter_lo)
{
    if (job.tile == job.ntiles - 1u && threadIdx.x == 0) {
        StateHeader *sh = job.state_header();
        sh->scale = scale; sh->scale_lo = 0.0f; sh->prev_worker = worker; sh->prev_iter = iter_lo;
    }
}

// Can a chunk be encoded four consecutive elements per lane, and from where?  With error feedback p lies in the state,
// without, in one tensor.  This form computes a Philox block in the lane that needs its four words (wide_words), and what
// the lane has of a chunk is a word of codes, or a nibble of either plane: no words handed round, no LDS stage.  The pass
// was bound by the vector ALU and is now bound by memory: QSGD encode of 25.6 M elements 31 -> 21 us (6.1 TB/s for its
// 128 MB), TernGrad of 10 M 14.0 -> 8.1.  Chunks that are not whole, start inside a Philox block (a group after an odd
// number of elements) or, without error feedback, straddle tensors take the form below it.  (Pass A in the same form
// measured the same to 0.4 us slower: there the draws hide behind 12 bytes per element.)
template <bool EF>
__device__ __forceinline__ const float *wide_source(const GroupView &g, const float *st, const Chunk &c)
{
    if (!wide_random(c, g.goff + c.base)) return nullptr;
    if (EF) return st + c.base;
    const uintptr_t entry = chunk_entry(g, c);
    return entry & 1u ? nullptr : reinterpret_cast<const float *>(entry);
}

template <bool EF, class SRC>
__global__ __launch_bounds__(kBlock) void qsgd_encode_k(SRC src, uint32_t levels, uint64_t seed, uint32_t worker, uint32_t iter_lo)
{
    __shared__ uint4 stage[kWavesPerBlock][kChunk / 16];
    const CompressJob job = src.job();
    const GroupView &g = job.g;
    const float *st = job.st;
    int8_t *codes = reinterpret_cast<int8_t *>(job.body());
    const Chunk c = my_chunk(g.n, job.tile);
    const float norm = job.hdr->scale;
    if (EF) remember_call(job, norm, worker, iter_lo);
    if (c.base >= g.n) return;
    const QsgdScale ks(norm, levels);
    if (const float *src4 = wide_source<EF>(g, st, c)) {
        float4v p[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) p[m] = EF ? load_wide(src4, c.lane, m) : load_wide_unaligned(src4, c.lane, m);
        uint32_t *dst = reinterpret_cast<uint32_t *>(codes + c.base);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            uint32_t x[4], word = 0;
            wide_words(seed, worker, iter_lo, g.goff + c.base, c.lane, m, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) word |= ((uint32_t)qsgd_code(ks, p[m][e], u01(x[e])) & 0xFFu) << (8 * e);
            st_stream(dst + 64 * m + c.lane, word);
        }
        return;
    }
    float p[kSteps];
    load_p<EF>(g, st, c, p);
    float uni[kSteps];
    chunk_uniforms(seed, worker, iter_lo, g.goff + c.base, c.lane, uni);
    int8_t code[kSteps];
#pragma unroll
    for (int j = 0; j < kSteps; ++j) code[j] = (int8_t)qsgd_code(ks, p[j], uni[j]);
    store_codes<int8_t>(codes, g.n, (g.n + 3u) & ~3u, c, code, stage[threadIdx.x >> 6]);
}

template <class SRC>
void launch_qsgd_encode(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, uint32_t levels, uint64_t seed, uint32_t worker, uint32_t iter_lo)
{
    if (tiles == 0) return;
    dim3 grid(tiles), block(kBlock);
    prof_begin(lc, K_QSGD_ENCODE);
    if (ef) MC_LAUNCH((qsgd_encode_k<true, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo);
    else MC_LAUNCH((qsgd_encode_k<false, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo);
    prof_end(lc, K_QSGD_ENCODE);
}
template void launch_qsgd_encode<OneCompress>(const LaunchCtx &, const OneCompress &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t);
template void launch_qsgd_encode<AllCompress>(const LaunchCtx &, const AllCompress &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t);

// or of a value over each eight lanes (0..7, 8..15, ...), in all of them
__device__ __forceinline__ uint32_t or_of_eight(uint32_t x)
{
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);      // quad_perm 1 0 3 2
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);      // quad_perm 2 3 0 1
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, true);     // row_half_mirror: lane i of eight <- lane 7 - i
    return x;
}

// the two planes of a chunk, one element per lane and step
__device__ __forceinline__ void tern_planes(const Chunk &c, uint32_t n, float smax, const float (&p)[kSteps], const float (&uni)[kSteps],
                                            uint64_t (&bnz)[kSteps], uint64_t (&bng)[kSteps])
{
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        bool nz, neg;
        (void)tern_decode(smax, p[j], uni[j], c.full || c.base + 64 * j + c.lane < n, nz, neg);
        bnz[j] = __builtin_amdgcn_ballot_w64(nz);
        bng[j] = __builtin_amdgcn_ballot_w64(neg);
    }
}

// TernGrad: two bit planes (non-zero, negative)
template <bool EF, class SRC>
__global__ __launch_bounds__(kBlock) void tern_encode_k(SRC src, uint64_t seed, uint32_t worker, uint32_t iter_lo)
{
    __shared__ uint64_t stage[kWavesPerBlock][kSteps];
    const CompressJob job = src.job();
    const GroupView &g = job.g;
    const float *st = job.st;
    uint32_t *planes = reinterpret_cast<uint32_t *>(job.body());
    const uint32_t nwords = (g.n + 31u) >> 5;
    const Chunk c = my_chunk(g.n, job.tile);
    const float smax = job.hdr->scale;
    if (EF) remember_call(job, smax, worker, iter_lo);
    if (c.base >= g.n) return;
    if (const float *src4 = wide_source<EF>(g, st, c)) {
        float4v p[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) p[m] = EF ? load_wide(src4, c.lane, m) : load_wide_unaligned(src4, c.lane, m);
        uint32_t wz = 0, wg = 0;                 // the word of the plane that this lane stores, if any
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            uint32_t x[4], z = 0, s = 0;         // the lane's four bits of either plane, element e in bit e
            wide_words(seed, worker, iter_lo, g.goff + c.base, c.lane, m, x);
#pragma unroll
            for (int e = 3; e >= 0; --e) {
                bool nz, neg;
                (void)tern_decode(smax, p[m][e], u01(x[e]), true, nz, neg);
                z = 2u * z + (nz ? 1u : 0u);
                s = __builtin_amdgcn_alignbit(s, __float_as_uint(p[m][e]), 31);      // sign bits shifted in
            }
            // eight lanes' bits make a word: or-ed inside the quads, then between the two quads of eight lanes
            const uint32_t at = 4u * (c.lane & 7u);
            z = or_of_eight(z << at);
            s = or_of_eight(s << at) & z;        // (a negative zero is never sent as non-zero)
            if ((c.lane & 3u) == (uint32_t)m) { wz = z; wg = s; }
        }
        // word 8 m + q of the chunk's 32 is in lanes 8 q .. 8 q + 7: lane 8 q + m stores the one of the first plane, lane
        // 8 q + 4 + m of the second
        const uint32_t m = c.lane & 3u, q = c.lane >> 3;
        const bool second = (c.lane & 4u) != 0u;
        uint32_t *dst = planes + (c.base >> 5) + (second ? nwords : 0u);
        st_stream(dst + 8u * m + q, second ? wg : wz);
        return;
    }
    float p[kSteps];
    load_p<EF>(g, st, c, p);
    float uni[kSteps];
    chunk_uniforms(seed, worker, iter_lo, g.goff + c.base, c.lane, uni);
    uint64_t bnz[kSteps], bng[kSteps];
    tern_planes(c, g.n, smax, p, uni, bnz, bng);
    store_plane(planes, nwords, c, bnz, stage[threadIdx.x >> 6]);
    store_plane(planes + nwords, nwords, c, bng, stage[threadIdx.x >> 6]);
}

template <class SRC>
void launch_tern_encode(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, uint64_t seed, uint32_t worker, uint32_t iter_lo)
{
    if (tiles == 0) return;
    dim3 grid(tiles), block(kBlock);
    prof_begin(lc, K_TERN_ENCODE);
    if (ef) MC_LAUNCH((tern_encode_k<true, SRC>), grid, block, lc, src, seed, worker, iter_lo);
    else MC_LAUNCH((tern_encode_k<false, SRC>), grid, block, lc, src, seed, worker, iter_lo);
    prof_end(lc, K_TERN_ENCODE);
}
template void launch_tern_encode<OneCompress>(const LaunchCtx &, const OneCompress &, uint32_t, bool, uint64_t, uint32_t, uint32_t);
template void launch_tern_encode<AllCompress>(const LaunchCtx &, const AllCompress &, uint32_t, bool, uint64_t, uint32_t, uint32_t);

// ---------------------------------------------------------------------------
// The two-pass quantizers on a small group, in one kernel: p stays in registers between the passes, and in place of the two
// kernel boundaries the group's blocks (64 at most, which start one after the other and fit a fraction of the device)
// wait until all have put their partial.
// (Against a kernel per pass, before a tile was spread over more threads: QSGD compress, 1 .. 64 tiles, 11.7 .. 13.2 -> 8.6 ..
// 10.0 us, TernGrad 11.8 -> 9.2 .. 10.3.)
// No block has to be running for another to finish: one that has looked `looks` times in vain (the rest of the group has
// found no room on the device for about a millisecond) hands its tile over and leaves, and the block that arrives last,
// which never waits, encodes what was handed over besides its own.  (That a block may go round for another tile costs
// 0.03 us a call; the encode written out a second time for it 0.25 with TernGrad.)
// ---------------------------------------------------------------------------
// One thread of a block that gives up: the tiles it still has to encode (its own, or none).  The last block looks at the word
// after its own arrival, and takes it if it is not 0: if the count is not complete after the hand-over, the tile will be
// found; if it is, the tile is taken back unless the last block was faster.  Either way the word is 0 when all have left.
__device__ __forceinline__ uint64_t hand_over(const CompressJob &job, uint64_t all)
{
    const uint64_t bit = 1ull << job.tile;
    release_to_device();                         // (p in the state has to be seen with it)
    (void)__hip_atomic_fetch_or(job.handed_over(), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    release_to_device();                         // (done before the count is looked at)
    if (__hip_atomic_load(job.arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all) return 0;
    return __hip_atomic_fetch_and(job.handed_over(), ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit;
}

// The chip is nearly idle on such groups and a block takes as long as one wavefront's instructions do, so a tile is spread over
// 1024 threads, four consecutive elements each: one Philox block per draw of a thread, a word of codes or a nibble of either
// plane to store, and a quarter of the instructions that 16 elements per lane took.  The draws of the call itself are
// made while the partials travel.  (Compress, 1025 / 34 000 / 262 000 elements: QSGD
// 10.3 / 10.4 / 10.5 -> 5.2 / 6.0 / 6.4 us, TernGrad 10.1 / 10.5 / 10.6 -> 4.8 / 5.5 / 5.9; 40 tensors in 1025 elements 30.6 -> 7.3; 272 000 in
// eight groups, QSGD 13.0 -> 7.1; 6 M in 64 groups, TernGrad 35.0 -> 28.9.)
struct Four { float x[4]; };
__device__ __forceinline__ void load_four(const float *st, uint32_t i0, uint32_t n, Four &v)
{
    const global_ptr<const float> p = in_global(st) + i0;
    if (i0 < n && n - i0 >= 4u) { const float4v f = *(global_ptr<const float4v>)p; v = {f.x, f.y, f.z, f.w}; }
    else
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) v.x[e] = i0 + e < n ? p[e] : 0.0f;
}
// the same of the gradient; the elements of the wavefront lie in one chunk
__device__ __forceinline__ void load_four(const GroupView &g, uint32_t i0, Four &v)
{
    v = {0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t lane = threadIdx.x & 63u, span = (uint32_t)__builtin_amdgcn_readfirstlane((int)i0);
    if (span >= g.n) return;
    Chunk c;
    c.base = span & ~(uint32_t)(kChunk - 1);
    c.lane = lane;
    c.full = g.n - c.base >= (uint32_t)kChunk;
    const uintptr_t entry = chunk_entry(g, c);
    if (!(entry & 1u)) {
        const float4u f = *(global_ptr<const float4u>)(in_global(reinterpret_cast<const float *>(entry)) + (i0 - c.base));
        v = {f.x, f.y, f.z, f.w};
        return;
    }
    const uint32_t s0 = (uint32_t)(entry >> 1), lim = chunk_end(g, c);
    uintptr_t at[4];
    if (each_span_of_chunk<4>(tensors_of_chunk(g, s0), i0, min(span + 256u, lim), lim, at)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v.x[e] = *in_global(reinterpret_cast<const float *>(at[e]));
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) v.x[e] = i0 + e < g.n ? v.x[e] : 0.0f;
        return;
    }
    for_each_tensor_of_chunk(g, c, s0, [&](uint32_t beg, uint32_t end, uintptr_t ptr) {
        const global_ptr<const float> p = in_global(reinterpret_cast<const float *>(ptr));
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) if (i0 + e >= beg && i0 + e < end) v.x[e] = p[i0 + e - beg];
    });
}
// the words of the random stream for four elements from model-wide index at on
__device__ __forceinline__ void four_words(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t at, uint32_t off /* at % 4, uniform */, uint32_t (&x)[4])
{
    philox4x32_10(seed, worker, iter_lo, at >> 2, x);
    if (off) {                                   // the group starts inside a block: the rest is in the next one
        uint32_t y[4];
        philox4x32_10(seed, worker, iter_lo, (at >> 2) + 1u, y);
        const uint32_t w[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t one = e + 1 < 4 ? w[(e + 1) & 3] : y[(e + 1) & 3], two = e + 2 < 4 ? w[(e + 2) & 3] : y[(e + 2) & 3],
                           three = e + 3 < 4 ? w[(e + 3) & 3] : y[(e + 3) & 3];
            x[e] = off == 1u ? one : off == 2u ? two : three;
        }
    }
}

template <bool EF, int MODE, class SRC>
__global__ __launch_bounds__(kSpread) void quantize_small_k(SRC src, uint32_t levels, uint64_t seed, uint32_t worker, uint32_t iter_lo, uint32_t looks)
{
    constexpr int kWaves = kSpread / kWave;
    __shared__ double red[kWaves];
    __shared__ float scalar;
    __shared__ uint64_t todo;                    // the tiles that this block encodes, one bit each
    __shared__ __attribute__((aligned(16))) float held[MODE == RED_L2 ? kTile : 4];      // p of the tile
    CompressJob job = src.job();
    const GroupView &g = job.g;
    const uint32_t n = g.n, nwords = (n + 31u) >> 5, t = threadIdx.x, off = (uint32_t)g.goff & 3u;
    uint32_t i0 = job.tile * (uint32_t)kTile + 4u * t;
    // ---- p = g + e (zeros past the end of the group), kept in the state: see accumulate
    Four p;
    if (EF) {
        const StateHeader *prev = job.state_header();
        const float sprev = prev->scale;
        const uint32_t wprev = prev->prev_worker, iprev = prev->prev_iter;
        Four q;
        load_four(job.st, i0, n, q);
        load_four(g, i0, p);
        uint32_t x[4];
        four_words(seed, wprev, iprev, g.goff + i0, off, x);
        const QsgdScale ks(MODE == RED_L2 ? sprev : 0.0f, levels);
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) {
            float d;
            if (MODE == RED_L2) d = qsgd_decode(ks, qsgd_code(ks, q.x[e], u01(x[e])));
            else { bool nz, neg; d = tern_decode(sprev, q.x[e], u01(x[e]), true, nz, neg); }
            const float r = q.x[e] - d;
            p.x[e] = i0 + e < n ? p.x[e] + r : 0.0f;
        }
        const global_ptr<float> to = in_global(job.st) + i0;
        if (i0 < n && n - i0 >= 4u) *(global_ptr<float4v>)to = float4v{p.x[0], p.x[1], p.x[2], p.x[3]};
        else
#pragma unroll
            for (uint32_t e = 0; e < 4u; ++e) if (i0 + e < n) to[e] = p.x[e];
    } else load_four(g, i0, p);
    // ---- this tile's partial
    double part = 0.0;                           // (wavefront 0)
    if (MODE == RED_L2) {                        // summed in the order of accum_reduce_k: the same norm to the last bit
        *reinterpret_cast<float4v *>(&held[4u * t]) = float4v{p.x[0], p.x[1], p.x[2], p.x[3]};
        __syncthreads();
        if (t < (uint32_t)kBlock) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < kSteps; ++j) {   // elements past n are 0 and add nothing
                const float v = held[t / 64u * (uint32_t)kChunk + 64u * j + (t & 63u)];
                acc += (double)v * (double)v;
            }
            acc = wave_sum(acc);
            if ((t & 63u) == 0) red[t >> 6] = acc;
        }
        __syncthreads();
        part = (red[0] + red[1]) + (red[2] + red[3]);
    } else {
        const float mx = wave_max(fmaxf(fmaxf(fmaxf(fmaxf(0.0f, fabsf(p.x[0])), fabsf(p.x[1])), fabsf(p.x[2])), fabsf(p.x[3])));
        if ((t & 63u) == 0) red[t >> 6] = (double)mx;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) part = fmax(part, red[w]);
    }
    uint32_t x[4];                               // the draws of this call
    if (t < 64u) {
        uint64_t before = 0;
        if (t == 0) {
            put_partial(job.partial + job.tile, part);
            before = arrive_at(job.arrive);
        }
        four_words(seed, worker, iter_lo, g.goff + i0, off, x);
        uint64_t mine = 1ull << job.tile, handed = 0;
        if (t == 0) {
            const uint64_t all = (before / job.ntiles + 1u) * job.ntiles;
            // (looked at first, in the shadow of the partials: taking it is an atomic's round trip, 0.1 us of a call)
            if (before + 1u == all) handed = __hip_atomic_load(job.handed_over(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
                for (uint32_t look = 0; __hip_atomic_load(job.arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all; ++look) {
                    if (look >= looks) { mine = hand_over(job, all); break; }
                    __builtin_amdgcn_s_sleep(4);
                }
        }
        all_arrived();
        const double S = combine_partials<MODE == RED_MAX_ABS>(job.partial, job.ntiles);       // (after a hand-over: of no use)
        if (t == 0) {
            if (handed) mine |= __hip_atomic_exchange(job.handed_over(), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            scalar = MODE == RED_L2 ? (float)sqrt(S) : (float)S;
            todo = mine;
        }
    } else four_words(seed, worker, iter_lo, g.goff + i0, off, x);
    __syncthreads();
    const float scale = scalar;
    uint64_t left = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)todo) |
                    ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(todo >> 32)) << 32);
    if (!left) return;
    for (;;) {                                   // its own tile, then those handed over
        if (job.tile == job.ntiles - 1u && t == 0)
            put_plain_header(job.hdr, MODE == RED_L2 ? MC_ALGO_QSGD : MC_ALGO_TERNGRAD, n, scale, 0.0f, MODE == RED_L2 ? levels : 0u);
        if (EF) remember_call(job, scale, worker, iter_lo);
        if (MODE == RED_L2) {
            const QsgdScale ks(scale, levels);
            uint32_t word = 0;
#pragma unroll
            for (uint32_t e = 0; e < 4u; ++e) word |= (i0 + e < n ? (uint32_t)qsgd_code(ks, p.x[e], u01(x[e])) & 0xFFu : 0u) << (8u * e);
            if (i0 < n) in_global(reinterpret_cast<uint32_t *>(job.body()))[i0 >> 2] = word;        // (the body ends on a multiple of four codes)
        } else {
            uint32_t z = 0, s = 0;               // the thread's four bits of either plane
#pragma unroll
            for (uint32_t e = 0; e < 4u; ++e) {
                bool nz, neg;
                (void)tern_decode(scale, p.x[e], u01(x[e]), i0 + e < n, nz, neg);
                z |= (nz ? 1u : 0u) << e;
                s |= (neg ? 1u : 0u) << e;
            }
            const uint32_t nibble = 4u * (t & 7u), w = i0 >> 5;
            z = or_of_eight(z << nibble);
            s = or_of_eight(s << nibble);
            if ((t & 7u) < 2u && w < nwords) in_global(reinterpret_cast<uint32_t *>(job.body()))[(t & 1u ? nwords : 0u) + w] = t & 1u ? s : z;
        }
        left &= ~(1ull << job.tile);
        if (!left) return;
        job.tile = (uint32_t)__builtin_ctzll(left);
        i0 = job.tile * (uint32_t)kTile + 4u * t;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");      // p of that tile, as the block that left it stored it
        if (EF) load_four(job.st, i0, n, p); else load_four(g, i0, p);
        four_words(seed, worker, iter_lo, g.goff + i0, off, x);
    }
}

template <class SRC>
void launch_quantize_small(const LaunchCtx &lc, int mode, const SRC &src, uint32_t tiles, bool ef, uint32_t levels, uint64_t seed, uint32_t worker,
                           uint32_t iter_lo, uint32_t looks)
{
    if (tiles == 0) return;
    dim3 grid(tiles), block(kSpread);
    const int slot = mode == RED_L2 ? K_QSGD_ENCODE : K_TERN_ENCODE;
    prof_begin(lc, slot);
    if (mode == RED_L2) {
        if (ef) MC_LAUNCH((quantize_small_k<true, RED_L2, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo, looks);
        else MC_LAUNCH((quantize_small_k<false, RED_L2, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo, looks);
    } else {
        if (ef) MC_LAUNCH((quantize_small_k<true, RED_MAX_ABS, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo, looks);
        else MC_LAUNCH((quantize_small_k<false, RED_MAX_ABS, SRC>), grid, block, lc, src, levels, seed, worker, iter_lo, looks);
    }
    prof_end(lc, slot);
}
template void launch_quantize_small<OneCompress>(const LaunchCtx &, int, const OneCompress &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t, uint32_t);
template void launch_quantize_small<AllCompress>(const LaunchCtx &, int, const AllCompress &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t, uint32_t);

// ---------------------------------------------------------------------------
// FP16, single pass: h = binary16(p) round-to-nearest-even, e <- p - (float)h.  S: see sign_compress_k (33 / 34 000 / 262 000
// elements: 4.1 / 4.0 / 4.1 -> 2.4 / 2.7 / 3.1 us).
// ---------------------------------------------------------------------------
template <bool EF, class SRC, int S = kSteps>
__global__ __launch_bounds__(kTile / S) void fp16_compress_k(SRC src)
{
    const CompressJob job = src.job();
    const GroupView &g = job.g;
    float *st = job.st;
    uint16_t *halves = reinterpret_cast<uint16_t *>(job.body());
    const Chunk c = my_chunk<S>(g.n, job.tile);
    if (job.tile == job.ntiles - 1u && threadIdx.x == 0) put_plain_header(job.hdr, MC_ALGO_FP16, g.n, 0.0f);
    if (c.base >= g.n) return;
    float p[S];
    load_seg(g, c, p);
    if (EF) {
        float e[S];
        load_flat(st, c, g.n, e, 0.0f);
#pragma unroll
        for (int j = 0; j < S; ++j) p[j] = p[j] + e[j];
    }
    uint16_t h[S];
    float e[S];
#pragma unroll
    for (int j = 0; j < S; ++j) {
        _Float16 hv = (_Float16)p[j];                 // v_cvt_f16_f32: round to nearest even, keeps subnormals
        h[j] = __builtin_bit_cast(uint16_t, hv);
        e[j] = p[j] - (float)hv;
    }
    if (EF) store_flat(st, c, g.n, e);
    // 64 lanes x 2 bytes: one whole 128-byte line per wave store (the body of a payload starts on a line), which
    // measured faster than 16-byte stores out of an LDS stage (58.6 against 65.0 us for the kernel's call)
    if (c.full) {
        uint16_t *dst = halves + c.base + c.lane;
#pragma unroll
        for (int j = 0; j < S; ++j) st_stream(dst + 64 * j, h[j]);
    } else {
        const uint32_t n_padded = (g.n + 1u) & ~1u;       // zero padding up to a multiple of 4 bytes
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const uint32_t i = c.base + 64 * j + c.lane;
            if (i < g.n) halves[i] = h[j];
            else if (i < n_padded) halves[i] = (uint16_t)0;
        }
    }
}

template <class SRC>
void launch_fp16_compress(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef)
{
    if (tiles == 0) return;
    dim3 grid(tiles), block(kBlock);
    prof_begin(lc, K_FP16_COMPRESS);
    if (tiles <= kSpreadTiles) {
        if (ef) MC_LAUNCH((fp16_compress_k<true, SRC, kSpreadSteps>), grid, dim3(kSpread), lc, src);
        else MC_LAUNCH((fp16_compress_k<false, SRC, kSpreadSteps>), grid, dim3(kSpread), lc, src);
    } else if (ef) MC_LAUNCH((fp16_compress_k<true, SRC>), grid, block, lc, src);
    else MC_LAUNCH((fp16_compress_k<false, SRC>), grid, block, lc, src);
    prof_end(lc, K_FP16_COMPRESS);
}
template void launch_fp16_compress<OneCompress>(const LaunchCtx &, const OneCompress &, uint32_t, bool);
template void launch_fp16_compress<AllCompress>(const LaunchCtx &, const AllCompress &, uint32_t, bool);

// ---------------------------------------------------------------------------
// Decompress-and-sum of dense codes (Algorithm 1: g~ = aggregate(C^-1(Delta))):
// out_i = alpha * (((0 + d_0,i) + d_1,i) + ...), workers in ascending order, one
// pass, every payload read once, the dense result written once through the
// segment table.
// ---------------------------------------------------------------------------
// Workers are taken in batches: all loads of a batch (header scalars and codes)
// are issued before the first is used, so a wavefront pays the HBM latency once
// per batch instead of once per worker.
//
// Two lane mappings.  Wide (QSGD, a full chunk inside one tensor whose address is 16-byte aligned):
// lane l holds four consecutive elements in each of four steps, element (256 m + 4 l + rot) mod 1024
// onward, so the codes of a worker arrive in 4 loads of 4 bytes per lane instead of 16 loads of one
// byte, and the sums leave as 16-byte stores; rot puts the stores on the output's 128-byte lines.
// Plain (FP16, and any other chunk): the usual element 64 j + l per step.  The work is elementwise,
// so the mapping changes no result: every element still adds its workers' values in worker order.
// (Measured, 8 workers, 25.6 M elements: QSGD 62.9 -> 54.6 us.  The same mapping with 8-byte loads
// made FP16 slower, 80.3 -> 82.5..85 us with 2, 4 or 8 workers per batch, so FP16 stays plain.)
// S: elements per lane, 16, or 4 on a launch of few tiles (kSpreadDecodeTiles).  Those are bound by one wavefront's chain of instructions and
// waits: a quarter of the additions each, and with the registers that frees, eight workers in a batch -- every batch waits for its scales and
// codes anew.  (Device time, 1 / 120 / 238 tiles in one tensor: QSGD, 1 worker 2.8 / 3.1 / 3.4 -> 2.8 / 3.2 / 3.5 us, 4 workers 3.0 / 3.7 / 4.0 -> 3.1 / 3.8 / 4.0,
// 8 workers 3.8 / 5.0 / 5.2 -> 3.7 / 4.3 / 4.7, 16 workers 5.5 / 7.4 / 7.9 -> 5.3 / 6.2 / 6.7; FP16, 1 worker 2.8 / 3.3 / 3.6 -> 3.0 / 3.3 / 3.6, 8 workers 4.2 / 6.1 / 6.7
// -> 3.4 / 4.8 / 5.3.  238 tiles in 60 tensors: QSGD, 1 / 8 workers 5.0 / 8.3 -> 4.3 / 6.3.  The rule does not look at the tenth of a microsecond that one
// worker's codes lose in one tensor.)
template <int ALGO, class SRC, int S = kSteps>
__global__ __launch_bounds__(kTile / S) void dense_decompress_k(SRC src, int W, float alpha, uint32_t levels, int *status)
{
    static_assert(ALGO == MC_ALGO_QSGD || ALGO == MC_ALGO_FP16, "one code per element");
    constexpr int kBatch = S == kSteps ? 4 : 8, kWords = S / 4;
    if (blockIdx.x < SRC::kCheckers) { if (S == kSteps || threadIdx.x < (uint32_t)kBlock) src.check({ALGO, false, false}, W, status); return; }
    const auto job = src.template job<BLK_TILE>();
    const GroupView &out = job.out;
    const Chunk c = my_chunk<S>(out.n, job.block);
    if (c.base >= out.n) return;
    const uintptr_t entry = chunk_entry(out, c);
    if (ALGO == MC_ALGO_QSGD && !(entry & 15u)) {               // an address (even), and 16-byte aligned
        const uint32_t rot = chunk_rotation(entry);             // a multiple of 4 here
        const uint32_t part = c.base & (uint32_t)(kChunk - 1), chunk = c.base - part;      // (part: 0 unless a wavefront holds a quarter)
        uint32_t at[kWords];                                    // first of the lane's four elements in step m
#pragma unroll
        for (int m = 0; m < kWords; ++m) at[m] = (part + 256u * m + 4u * c.lane + rot) & (uint32_t)(kChunk - 1);
        float acc[kWords][4];
#pragma unroll
        for (int m = 0; m < kWords; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[m][e] = 0.0f;
        for (int w0 = 0; w0 < W; w0 += kBatch) {
            const uint8_t *pl[kBatch];
            job.template payloads<kBatch>(w0, W, pl);
            float scale[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                scale[b] = 0.0f;
                if (w0 + b < W) scale[b] = ld_uniform(&reinterpret_cast<const PayloadHeader *>(pl[b])->scale);
            }
            uint32_t cw[kBatch][kWords];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const global_ptr<const uint8_t> codes = in_global(pl[b]) + kHeaderBytes + chunk;
#pragma unroll
                for (int m = 0; m < kWords; ++m) cw[b][m] = w0 + b < W ? __builtin_nontemporal_load((global_ptr<const uint32_t>)(codes + at[m])) : 0u;
            }
            hold(scale);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (w0 + b < W) {
                    const float q = (float)((double)scale[b] / (double)(float)levels);
#pragma unroll
                    for (int m = 0; m < kWords; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[m][e] = acc[m][e] + (float)(int8_t)(cw[b][m] >> (8 * e)) * q;
                }
            }
        }
        const global_ptr<float> p = in_global(reinterpret_cast<float *>(entry));
#pragma unroll
        for (int m = 0; m < kWords; ++m) {
            float4v v = {alpha * acc[m][0], alpha * acc[m][1], alpha * acc[m][2], alpha * acc[m][3]};
            __builtin_nontemporal_store(v, (global_ptr<float4v>)(p + at[m]));
        }
        return;
    }
    float acc[S];
#pragma unroll
    for (int j = 0; j < S; ++j) acc[j] = 0.0f;
    for (int w0 = 0; w0 < W; w0 += kBatch) {
        const uint8_t *pl[kBatch];
        job.template payloads<kBatch>(w0, W, pl);
        float scale[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            scale[b] = 0.0f;
            if (w0 + b < W) scale[b] = ld_uniform(&reinterpret_cast<const PayloadHeader *>(pl[b])->scale);
        }
        if (ALGO == MC_ALGO_QSGD) {
            int8_t cd[kBatch][S];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (w0 + b < W) load_flat<int8_t>(reinterpret_cast<const int8_t *>(pl[b] + kHeaderBytes), c, out.n, cd[b], (int8_t)0);
            }
            hold(scale);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (w0 + b < W) {
                    const float q = (float)((double)scale[b] / (double)(float)levels);
#pragma unroll
                    for (int j = 0; j < S; ++j) acc[j] = acc[j] + (float)cd[b][j] * q;
                }
            }
        } else {   // FP16
            _Float16 hv[kBatch][S];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (w0 + b < W) load_flat<_Float16>(reinterpret_cast<const _Float16 *>(pl[b] + kHeaderBytes), c, out.n, hv[b], (_Float16)0.0f);
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (w0 + b < W) {
#pragma unroll
                    for (int j = 0; j < S; ++j) acc[j] = acc[j] + (float)hv[b][j];
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < S; ++j) acc[j] = alpha * acc[j];
    store_seg(out, c, acc, entry);
}

// ---------------------------------------------------------------------------
// EF-Sign / TernGrad decompress-and-sum.  With W sign planes the per-element work of the
// generic kernel (extract bit, select +-scale, add; W times) exceeds what the
// vector ALUs can do at HBM speed, so this kernel works on whole words:
//   * the sum of the first (up to) 8 workers takes one of 2^8 values per group;
//     every block tabulates them in LDS with the very same sequence of fp32
//     additions  ((0 + d_0) + d_1) + ... , so a lookup returns the exact result;
//   * a lane owns 32 consecutive elements, i.e. one word of every worker's plane;
//     four 8x8 bit-matrix transposes turn its 8 words into 32 table indices;
//   * further workers (W > 8) are added one by one in order;
//   * results go through a skewed LDS stage so that the global stores are the
//     usual 256 contiguous bytes per wave instruction.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t transpose8x8(uint64_t x)
{
    // bit (8 r + c) <-> bit (8 c + r): three rounds of masked swaps
    uint64_t t;
    t = 0x0f0f0f0f00000000ull & (x ^ (x << 28)); x ^= t ^ (t >> 28);
    t = 0x3333000033330000ull & (x ^ (x << 14)); x ^= t ^ (t >> 14);
    t = 0x5500550055005500ull & (x ^ (x << 7));  x ^= t ^ (t >> 7);
    return x;
}

constexpr int kPlaneBatch = 8;                             // workers whose planes are asked for together
constexpr int kSignWaveElems = 2048;                       // 64 lanes x 32 elements
constexpr int kSignTile = kSignWaveElems * kWavesPerBlock; // 8192 elements per block
static_assert(kSignTile == 2 * kTile, "blocks of the bit-plane decode (BLK_PLANE)");

// bytes of 8 words (one per worker) -> per element the 8 workers' bits: word q byte -> 8 table indices
__device__ __forceinline__ uint64_t gather_transpose(const uint32_t (&wd)[8], int q)
{
    uint32_t lo = ((wd[0] >> (8 * q)) & 0xFFu) | (((wd[1] >> (8 * q)) & 0xFFu) << 8) |
                  (((wd[2] >> (8 * q)) & 0xFFu) << 16) | (((wd[3] >> (8 * q)) & 0xFFu) << 24);
    uint32_t hi = ((wd[4] >> (8 * q)) & 0xFFu) | (((wd[5] >> (8 * q)) & 0xFFu) << 8) |
                  (((wd[6] >> (8 * q)) & 0xFFu) << 16) | (((wd[7] >> (8 * q)) & 0xFFu) << 24);
    return transpose8x8((uint64_t)lo | ((uint64_t)hi << 32));
}

// TERN = false: the one-plane schemes (2^8 sums of the first 8 workers' +-level).  TERN = true: TernGrad (non-zero and
// negative planes; a worker contributes 0, +s or -s): no table, every worker is added by itself (add_terns).
// what a set / clear bit of worker w decodes to (one-plane schemes)
__device__ __forceinline__ void plane_levels(float scale, float scale_lo, int kind, float &hi, float &lo)
{
    hi = kind == PLANE_VOTE ? 1.0f : scale;
    lo = kind == PLANE_MEANS ? scale_lo : -hi;
}
__device__ __forceinline__ float vote_of(float tally) { return tally > 0.0f ? 1.0f : (tally < 0.0f ? -1.0f : 0.0f); }

// kind (one-plane schemes only): PLANE_SCALE  EF-Sign, a bit decodes to +-scale
//                                PLANE_MEANS  OneBit, to the mean of its class
//                                PLANE_VOTE   SignSGD / SigNUM, to +-1, and the sum becomes its sign (majority vote)
// Bit e of a TernGrad worker's two plane words -> what the worker adds to element e: 0, +s or -s, as bit
// operations on s (a one-bit field, sign-extended, is the mask).  The masks pass through an empty asm so that the
// compiler does not turn them back into compares and selects (9 issue slots with their wait states instead of 5).
__device__ __forceinline__ float tern_term(uint32_t nzw, uint32_t ngw, int e, float sc)
{
    uint32_t mx = (uint32_t)__builtin_amdgcn_sbfe((int)nzw, e, 1), my = (uint32_t)__builtin_amdgcn_sbfe((int)ngw, e, 1);
    asm("" : "+v"(mx));
    asm("" : "+v"(my));
    return __uint_as_float((__float_as_uint(sc) ^ (my & 0x80000000u)) & mx);
}

// bit e of a one-plane worker's word -> the level it decodes to, the same way
__device__ __forceinline__ float plane_term(uint32_t word, int e, float hi, float lo)
{
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)word, e, 1);
    asm("" : "+v"(m));
    return __uint_as_float((__float_as_uint(hi) & m) | (__float_as_uint(lo) & ~m));
}

// A worker's word added to the sums of its 32 elements.  Where the two levels are +s and -s, bits e and e + 16 are made the
// signs of two halves +-1.0 (a shift and one three-input bit operation for both), and each sum is one mixed-precision
// multiply-add, half x float + float: the product +-s is exact, so the one rounding is that of the addition.  (s goes to a
// vector register: an operand from a scalar one makes most vector instructions take twice the cycles on this part.)
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void add_signs(float (&acc)[32], uint32_t word, float s)
{
    asm("" : "+v"(s));
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const half2v h = __builtin_bit_cast(half2v, (~(word << (15 - e)) & 0x80008000u) | 0x3C003C00u);
        acc[e] = __builtin_fmaf((float)h.x, s, acc[e]);
        acc[e + 16] = __builtin_fmaf((float)h.y, s, acc[e + 16]);
    }
}
// TernGrad's two words the same way: the half of an element is its non-zero bit as bit 14 -- 2.0, or 0 -- and its negative
// bit as the sign, multiplied by s / 2.  The bits of even elements are laid next to each other in one word, those of odd ones
// in another, so that here too one shift and one mask make two halves.
__device__ __forceinline__ void add_terns(float (&acc)[32], uint32_t nz, uint32_t ng, float half_s)
{
    asm("" : "+v"(half_s));
    const uint32_t even = (nz & 0x55555555u) | ((ng << 1) & 0xAAAAAAAAu), odd = ((nz >> 1) & 0x55555555u) | (ng & 0xAAAAAAAAu);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const half2v h = __builtin_bit_cast(half2v, (e & 1 ? odd << (15 - e) : even << (14 - e)) & 0xC000C000u);
        acc[e] = __builtin_fmaf((float)h.x, half_s, acc[e]);
        acc[e + 16] = __builtin_fmaf((float)h.y, half_s, acc[e + 16]);
    }
}
// Whether that gives what an addition of 0, +s or -s gives: s / 2 has to be exact, and 0 times it has to be 0.
__device__ __forceinline__ bool halves_exactly(float s) { return 0.5f * s + 0.5f * s == s && fabsf(s) < __builtin_inff(); }

// MORE: more than kPlaneBatch workers, in a kernel of its own (80 registers, 6 wavefronts per SIMD, only when asked for; with both in one kernel 81,
// and the sums of up to eight workers 1 to 3 % slower).
template <bool TERN, bool MORE, class SRC>
__attribute__((amdgpu_waves_per_eu(TERN ? 4 : 6)))
__global__ __launch_bounds__(kBlock) void plane_decompress_k(SRC src, int W, float alpha, int *status, int algo, int kind)
{
    __shared__ float table[TERN ? 1 : 256];
    __shared__ float stage[kWavesPerBlock][kChunk + 32];
    const uint32_t t = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63u;
    if (blockIdx.x < SRC::kCheckers) { src.check({(uint32_t)algo, false, false}, W, status); return; }
    const auto job = src.template job<BLK_PLANE>();
    const GroupView &out = job.out;
    const uint32_t wbase = job.block * (uint32_t)kSignTile + wave * (uint32_t)kSignWaveElems;
    const uint32_t nwords = (out.n + 31u) >> 5;
    const uint32_t wi = (wbase >> 5) + lane;
    // What is needed of the eight workers from w0 on, asked for together: the header's scalars on the scalar path (as vector
    // loads they would queue behind the compute unit's stores), the words of the planes on the vector path.
    struct Batch { const uint8_t *pl[kPlaneBatch]; float scale[kPlaneBatch], scale_lo[kPlaneBatch]; uint32_t word[kPlaneBatch], second[kPlaneBatch]; };
    auto fetch = [&](int w0, Batch &x) {
        job.template payloads<kPlaneBatch>(w0, W, x.pl);
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            const PayloadHeader *h = reinterpret_cast<const PayloadHeader *>(x.pl[b]);
            x.scale[b] = x.scale_lo[b] = 0.0f;
            if (w0 + b < W) {
                if (TERN || kind != PLANE_VOTE) x.scale[b] = ld_uniform(&h->scale);
                if (!TERN && kind == PLANE_MEANS) x.scale_lo[b] = __uint_as_float(ld_uniform(&h->pad[0]));
            }
        }
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            x.word[b] = x.second[b] = 0u;
            if (w0 + b < W && wi < nwords) {
                const global_ptr<const uint32_t> plane = in_global(reinterpret_cast<const uint32_t *>(x.pl[b] + kHeaderBytes));
                // (ordinary loads for TernGrad: 25.6 M elements, 8 workers 37.6 -> 32.1 us; with one plane 27.2 against 28.1)
                x.word[b] = TERN ? plane[wi] : __builtin_nontemporal_load(plane + wi);
                if (TERN) x.second[b] = plane[nwords + wi];
            }
        }
        hold(x.scale);
        if (!TERN) hold(x.scale_lo);
    };
    Batch x;
    fetch(0, x);
    float acc[32];
    if (!TERN) {
        // the table takes the first eight workers
        float sum = 0.0f;
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            float hi, lo;
            plane_levels(x.scale[b], x.scale_lo[b], kind, hi, lo);
            sum = b < W ? sum + (((t >> b) & 1u) ? hi : lo) : sum;
        }
        if (!MORE && kind == PLANE_VOTE) sum = vote_of(sum);
        table[t] = MORE ? sum : alpha * sum;
        __syncthreads();
        if (wbase >= out.n) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // byte q of the words -> rows of an 8x8 bit matrix (row = worker, column = element 8q + c)
            const uint64_t m = gather_transpose(x.word, q);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[8 * q + e] = table[(uint32_t)(m >> (8 * e)) & 0xFFu];
        }
    } else {
        if (wbase >= out.n) return;
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[e] = 0.0f;
    }
    // the further workers (TernGrad: all), one by one
#pragma unroll 1
    for (int w0 = TERN ? 0 : kPlaneBatch; w0 < (MORE ? W : TERN ? 1 : 0); w0 += kPlaneBatch) {
        if (w0) fetch(w0, x);
        // (One decision for the batch: with one per worker every worker's sums were copied to other registers, half a
        // move per element, next to two instructions that add it.)
        if (TERN) {
            bool exact = true;
#pragma unroll
            for (int b = 0; b < kPlaneBatch; ++b) exact = exact && halves_exactly(x.scale[b]);
            if (exact) {
#pragma unroll
                for (int b = 0; b < kPlaneBatch; ++b) if (w0 + b < W) add_terns(acc, x.word[b], x.second[b], 0.5f * x.scale[b]);
            } else {
#pragma unroll
                for (int b = 0; b < kPlaneBatch; ++b) {
                    if (w0 + b >= W) break;
#pragma unroll
                    for (int e = 0; e < 32; ++e) acc[e] = acc[e] + tern_term(x.word[b], x.second[b], e, x.scale[b]);
                }
            }
        } else {
            bool signs = kind != PLANE_MEANS;
            if (kind == PLANE_SCALE)
#pragma unroll
                for (int b = 0; b < kPlaneBatch; ++b) signs = signs && x.scale[b] == x.scale[b];      // (a NaN would keep its sign)
            if (signs) {
#pragma unroll
                for (int b = 0; b < kPlaneBatch; ++b) if (w0 + b < W) add_signs(acc, x.word[b], kind == PLANE_VOTE ? 1.0f : x.scale[b]);
            } else {
#pragma unroll
                for (int b = 0; b < kPlaneBatch; ++b) {
                    if (w0 + b >= W) break;
                    float hi, lo;
                    plane_levels(x.scale[b], x.scale_lo[b], kind, hi, lo);
#pragma unroll
                    for (int e = 0; e < 32; ++e) acc[e] = acc[e] + plane_term(x.word[b], e, hi, lo);
                }
            }
        }
    }
    if (MORE || TERN) {
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[e] = alpha * (!TERN && kind == PLANE_VOTE ? vote_of(acc[e]) : acc[e]);
    }
    // two halves of 1024 elements through one skewed LDS stage (lanes 32 h .. 32 h + 31 own the elements of
    // half h), so that the global stores are 256 contiguous bytes per wave instruction
    float *mine = stage[wave];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __builtin_amdgcn_wave_barrier();
        if ((lane >> 5) == (uint32_t)half) {
#pragma unroll
            for (int e = 0; e < 32; ++e) mine[33 * (lane & 31u) + e] = acc[e];     // element 32 (lane % 32) + e, skewed
        }
        __builtin_amdgcn_wave_barrier();
        Chunk c;
        c.base = wbase + half * (uint32_t)kChunk;
        c.lane = lane;
        c.full = c.base < out.n && out.n - c.base >= (uint32_t)kChunk;
        if (c.base < out.n) {
            const uintptr_t entry = chunk_entry(out, c);
            const uint32_t rot = TERN ? 0u : chunk_rotation(entry);     // measured: no gain for TernGrad, whose decode is bound by the vector ALU
            float v[kSteps];
#pragma unroll
            for (int j = 0; j < kSteps; ++j) {
                const uint32_t i = rotated(j, lane, rot);                // element of this half, rotated onto the lines
                v[j] = mine[i + (i >> 5)];
            }
            store_seg_rot(out, c, v, entry, rot);
        }
    }
}

// The same on few tiles, where the time is one wavefront's chain: four times as many wavefronts, a lane holds eight elements, one byte of every
// worker's plane, and one transpose; every term is added as what it is.  (Device time, 1 / 120 / 238 blocks in one tensor: EF-Sign, 1 worker 4.1 / 4.8 / 5.1 -> 3.7 / 4.3 /
// 4.7 us, 4 workers 4.2 / 4.8 / 5.0 -> 3.9 / 4.5 / 4.8, 8 workers 4.3 / 4.8 / 5.2 -> 4.3 / 4.9 / 5.3, 16 workers 6.3 / 6.9 / 7.3 -> 5.9 / 6.6 / 7.0; TernGrad, 1 worker 3.6 / 4.2 / 4.5 ->
// 3.2 / 3.8 / 4.1, 4 workers 4.0 / 4.6 / 4.9 -> 3.8 / 4.4 / 4.8, 8 workers 4.5 / 5.1 / 5.4 -> 4.6 / 5.2 / 5.5, 16 workers 6.4 / 7.0 / 7.3 -> 6.7 / 7.4 / 7.6.  One block of 60 tensors, where a
// wavefront of 2048 elements walks over the tensors of its two chunks one after the other: EF-Sign, 1 / 8 / 16 workers 6.6 / 6.8 / 8.9 -> 4.9 / 5.5 / 7.2, TernGrad
// 6.1 / 7.1 / 9.0 -> 4.3 / 5.9 / 8.2.  The rule does not look at what many workers' planes lose in one tensor.)
constexpr int kByteSteps = 8, kByteWave = 64 * kByteSteps, kByteThreads = kSignTile / kByteSteps;
template <bool TERN, class SRC>
__global__ __launch_bounds__(kByteThreads) void plane_spread_k(SRC src, int W, float alpha, int *status, int algo, int kind)
{
    __shared__ float table[TERN ? 1 : 256];
    __shared__ float stage[kByteThreads / 64][kByteWave + 64];
    const uint32_t t = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63u;
    if (blockIdx.x < SRC::kCheckers) { if (t < (uint32_t)kBlock) src.check({(uint32_t)algo, false, false}, W, status); return; }
    const auto job = src.template job<BLK_PLANE>();
    const GroupView &out = job.out;
    const uint32_t wbase = job.block * (uint32_t)kSignTile + wave * (uint32_t)kByteWave;
    const uint32_t nbytes = 4u * ((out.n + 31u) >> 5);
    const uint32_t at = (wbase >> 3) + lane;
    float scale[kPlaneBatch], scale_lo[kPlaneBatch];
    uint32_t bits[kPlaneBatch], second[kPlaneBatch];
    auto fetch = [&](int w0) {
        const uint8_t *pl[kPlaneBatch];
        job.template payloads<kPlaneBatch>(w0, W, pl);
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            const PayloadHeader *h = reinterpret_cast<const PayloadHeader *>(pl[b]);
            scale[b] = scale_lo[b] = 0.0f;
            if (w0 + b < W) {
                if (TERN || kind != PLANE_VOTE) scale[b] = ld_uniform(&h->scale);
                if (!TERN && kind == PLANE_MEANS) scale_lo[b] = __uint_as_float(ld_uniform(&h->pad[0]));
            }
        }
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            bits[b] = second[b] = 0u;
            if (w0 + b < W && at < nbytes) {
                const global_ptr<const uint8_t> plane = in_global(pl[b]) + kHeaderBytes;
                bits[b] = plane[at];
                if (TERN) second[b] = plane[nbytes + at];
            }
        }
        hold(scale);
        if (!TERN) hold(scale_lo);
    };
    fetch(0);
    float acc[kByteSteps];
    if (!TERN) {
        if (t < 256u) {
            float sum = 0.0f;
#pragma unroll
            for (int b = 0; b < kPlaneBatch; ++b) {
                float hi, lo;
                plane_levels(scale[b], scale_lo[b], kind, hi, lo);
                sum = b < W ? sum + (((t >> b) & 1u) ? hi : lo) : sum;
            }
            table[t] = sum;
        }
        __syncthreads();
        if (wbase >= out.n) return;
        const uint32_t lo = bits[0] | bits[1] << 8 | bits[2] << 16 | bits[3] << 24, hi = bits[4] | bits[5] << 8 | bits[6] << 16 | bits[7] << 24;
        const uint64_t m = transpose8x8((uint64_t)lo | (uint64_t)hi << 32);      // (row = worker, column = element)
#pragma unroll
        for (int e = 0; e < kByteSteps; ++e) acc[e] = table[(uint32_t)(m >> (8 * e)) & 0xFFu];
    } else {
        if (wbase >= out.n) return;
#pragma unroll
        for (int e = 0; e < kByteSteps; ++e) acc[e] = 0.0f;
    }
#pragma unroll 1
    for (int w0 = TERN ? 0 : kPlaneBatch; w0 < W; w0 += kPlaneBatch) {
        if (w0) fetch(w0);
#pragma unroll
        for (int b = 0; b < kPlaneBatch; ++b) {
            if (w0 + b >= W) break;
            float hi, lo;
            plane_levels(scale[b], scale_lo[b], kind, hi, lo);
#pragma unroll
            for (int e = 0; e < kByteSteps; ++e) acc[e] = acc[e] + (TERN ? tern_term(bits[b], second[b], e, scale[b]) : plane_term(bits[b], e, hi, lo));
        }
    }
    // through LDS, skewed, so that the stores are 256 contiguous bytes per wave instruction
    float *mine = stage[wave];
#pragma unroll
    for (int e = 0; e < kByteSteps; ++e) mine[(kByteSteps + 1) * lane + e] = alpha * (!TERN && kind == PLANE_VOTE ? vote_of(acc[e]) : acc[e]);
    __builtin_amdgcn_wave_barrier();
    const Chunk c{wbase, lane, out.n - wbase >= (uint32_t)kByteWave};
    float v[kByteSteps];
#pragma unroll
    for (int j = 0; j < kByteSteps; ++j) {
        const uint32_t i = 64u * j + lane;
        v[j] = mine[i + i / kByteSteps];
    }
    store_seg(out, c, v, chunk_entry(out, c));
}

template <class SRC>
static void dense_decompress_t(const LaunchCtx &lc, int algo, const SRC &src, uint32_t blocks, int W, float alpha, uint32_t levels, int *status)
{
    dim3 grid(blocks + SRC::kCheckers), block(kBlock);           // (the first ones check the headers)
    prof_begin(lc, K_DENSE_DECOMPRESS);
    switch (algo) {
    case MC_ALGO_EFSIGN:
    case MC_ALGO_ONEBIT:
    case MC_ALGO_SIGNSGD:
    case MC_ALGO_SIGNUM:
    {
        const int kind = algo == MC_ALGO_EFSIGN ? PLANE_SCALE : algo == MC_ALGO_ONEBIT ? PLANE_MEANS : PLANE_VOTE;
        if (blocks <= kSpreadPlanes) { MC_LAUNCH((plane_spread_k<false, SRC>), grid, dim3(kByteThreads), lc, src, W, alpha, status, algo, kind); break; }
        if constexpr (SRC::kRoom > kPlaneBatch) if (W > kPlaneBatch) { MC_LAUNCH((plane_decompress_k<false, true, SRC>), grid, block, lc, src, W, alpha, status, algo, kind); break; }
        MC_LAUNCH((plane_decompress_k<false, false, SRC>), grid, block, lc, src, W, alpha, status, algo, kind);
        break;
    }
    case MC_ALGO_TERNGRAD:
        if (blocks <= kSpreadPlanes) { MC_LAUNCH((plane_spread_k<true, SRC>), grid, dim3(kByteThreads), lc, src, W, alpha, status, algo, PLANE_SCALE); break; }
        if constexpr (SRC::kRoom > kPlaneBatch) if (W > kPlaneBatch) { MC_LAUNCH((plane_decompress_k<true, true, SRC>), grid, block, lc, src, W, alpha, status, algo, PLANE_SCALE); break; }
        MC_LAUNCH((plane_decompress_k<true, false, SRC>), grid, block, lc, src, W, alpha, status, algo, PLANE_SCALE);
        break;
    case MC_ALGO_QSGD:
        if (blocks <= kSpreadDecodeTiles) MC_LAUNCH((dense_decompress_k<MC_ALGO_QSGD, SRC, kSpreadSteps>), grid, dim3(kSpread), lc, src, W, alpha, levels, status);
        else MC_LAUNCH((dense_decompress_k<MC_ALGO_QSGD, SRC>), grid, block, lc, src, W, alpha, levels, status);
        break;
    default:
        if (blocks <= kSpreadDecodeTiles) MC_LAUNCH((dense_decompress_k<MC_ALGO_FP16, SRC, kSpreadSteps>), grid, dim3(kSpread), lc, src, W, alpha, levels, status);
        else MC_LAUNCH((dense_decompress_k<MC_ALGO_FP16, SRC>), grid, block, lc, src, W, alpha, levels, status);
        break;
    }
    prof_end(lc, K_DENSE_DECOMPRESS);
}
template <class SRC>
void launch_dense_decompress(const LaunchCtx &lc, int algo, const SRC &src, uint32_t blocks, int W, float alpha, uint32_t levels, int *status)
{
    if (blocks == 0) return;
    if constexpr (std::is_same_v<SRC, OneDecompress>) if (W <= kFewRoom) { dense_decompress_t(lc, algo, with_few(src), blocks, W, alpha, levels, status); return; }
    dense_decompress_t(lc, algo, src, blocks, W, alpha, levels, status);
}
template void launch_dense_decompress<OneDecompress>(const LaunchCtx &, int, const OneDecompress &, uint32_t, int, float, uint32_t, int *);
template void launch_dense_decompress<AllDecompress>(const LaunchCtx &, int, const AllDecompress &, uint32_t, int, float, uint32_t, int *);

// ---------------------------------------------------------------------------
// State <-> plain residual.  EF-Sign, OneBit, QSGD and TernGrad keep p and the scalars
// of the last call instead of the residual; the other algorithms copy (SigNUM: the momentum).
// ---------------------------------------------------------------------------
// One thread per element of the group (a launch holds fewer than 2^32 threads, and DGC's two vectors together
// may hold more floats than that): the thread of element i converts float i of every vector.
__global__ __launch_bounds__(kBlock) void state_convert_k(int algo, int to_residual, uint32_t n, const uint8_t *src, uint8_t *dst,
                                                          uint32_t levels, uint64_t seed, uint64_t goff)
{
    // plain side: n floats (DGC: v[n] then u[n]); opaque side: header, then the same floats (DGC: u from dgc_u_offset(n))
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const size_t uoff = dgc_u_offset(n);
    if (to_residual) {
        const StateHeader *h = reinterpret_cast<const StateHeader *>(src);
        const float *f = reinterpret_cast<const float *>(src + kHeaderBytes);
        float *e = reinterpret_cast<float *>(dst);
        if (i < n) {
            float v = f[i];
            if (algo == MC_ALGO_EFSIGN) { float sp = h->scale; v = v - (v >= 0.0f ? sp : -sp); }
            if (algo == MC_ALGO_ONEBIT) v = v - (v >= 0.0f ? h->scale : h->scale_lo);
            if (algo == MC_ALGO_QSGD || algo == MC_ALGO_TERNGRAD) {
                // what the last call sent of p is quantized once more, with its scalar and its random stream
                uint32_t w[4];
                philox4x32_10(seed, h->prev_worker, h->prev_iter, (goff + i) >> 2, w);
                const uint32_t word = (goff + i) & 3u;
                const float u = u01(word == 0 ? w[0] : word == 1 ? w[1] : word == 2 ? w[2] : w[3]);
                float d;
                if (algo == MC_ALGO_QSGD) { const QsgdScale ks(h->scale, levels); d = qsgd_decode(ks, qsgd_code(ks, v, u)); }
                else { bool nz, neg; d = tern_decode(h->scale, v, u, true, nz, neg); }
                v = v - d;
            }
            // Top-k, DGC: what the last call sent above its threshold key is masked by the next streaming pass, not zeroed
            const bool sent = (algo == MC_ALGO_TOPK || algo == MC_ALGO_DGC) && (__float_as_uint(v) & 0x7FFFFFFFu) > h->sent_key;
            e[i] = sent ? 0.0f : v;
            if (algo == MC_ALGO_DGC) e[(size_t)n + i] = sent ? 0.0f : f[uoff + i];
        }
    } else {
        const float *e = reinterpret_cast<const float *>(src);
        float *f = reinterpret_cast<float *>(dst + kHeaderBytes);
        if (i < n) {
            f[i] = e[i];                      // EF-Sign, OneBit, QSGD, TernGrad: p = e with scalars 0 re-derives exactly e
            if (algo == MC_ALGO_DGC) f[uoff + i] = e[(size_t)n + i];
        }
        // a cleared header; for the sparsifiers sent_key = all ones: nothing of an imported residual counts as sent
        if (i < kHeaderBytes / 4)
            reinterpret_cast<uint32_t *>(dst)[i] = i == offsetof(StateHeader, sent_key) / 4 && (algo == MC_ALGO_TOPK || algo == MC_ALGO_DGC || algo == MC_ALGO_RANDK) ? 0xFFFFFFFFu : 0u;
        if (algo == MC_ALGO_DGC && i >= n && i < uoff) f[i] = 0.0f;                       // the gap between v and u
    }
}

void launch_state_convert(const LaunchCtx &lc, int algo, bool to_residual, uint32_t n, const void *src, void *dst, uint32_t levels,
                          uint64_t seed, uint64_t goff)
{
    // the header is cleared too, and so is DGC's gap (fewer than 32 floats past n)
    const size_t work = (size_t)n + 32u > (size_t)kHeaderBytes / 4 ? (size_t)n + 32u : (size_t)kHeaderBytes / 4;
    prof_begin(lc, K_STATE_CONVERT);
    MC_LAUNCH(state_convert_k, dim3((uint32_t)((work + kBlock - 1) / kBlock)), dim3(kBlock), lc, algo,
                       to_residual ? 1 : 0, n, (const uint8_t *)src, (uint8_t *)dst, levels, seed, goff);
    prof_end(lc, K_STATE_CONVERT);
}

}  // namespace mc

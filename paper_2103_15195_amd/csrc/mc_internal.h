// Host <-> kernel-launcher interface of the library (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>
#include <type_traits>

#include "../../include/mergecomp.h"
#include "mc_device.h"

namespace mc {

constexpr uint32_t kMagic = 0x3150434Du;
constexpr int kHeaderBytes = 128;     // bodies of payload and state start on a 128-byte cache line
constexpr int kMaxWorkers = 64;

struct PayloadHeader {          // one cache line, see the layout in mergecomp.h
    uint32_t magic, algo;
    uint64_t n, k;
    float scale;
    uint32_t levels;
    uint32_t pad[24];           // pad[0]: OneBit's mean of the negative class; the rest zero
};
static_assert(sizeof(PayloadHeader) == kHeaderBytes, "payload header is one 128-byte line");

struct StateHeader {            // one cache line in front of the error-feedback floats
    float scale;                // EF-Sign: scale of the last call; OneBit: mean of its upper class (0 after zero-fill / import)
    float scale_lo;             // OneBit: mean of the lower class of the last call
    uint32_t prev_worker, prev_iter;   // QSGD / TernGrad: whose random stream the last call drew from (scale: its norm / max)
    uint32_t sent_key;          // Top-k, DGC: elements of the last call whose key exceeds this were sent and count as 0 (see sparse_accum_k)
    uint32_t pad[27];
};
static_assert(sizeof(StateHeader) == kHeaderBytes, "state header is one 128-byte line");

// DGC keeps two vectors in the state: v[n] first, then u[n] from the next multiple of 32 floats on, so that both start
// on a 128-byte line (a chunk's stores then cover whole lines).
__host__ __device__ inline size_t dgc_u_offset(uint32_t n) { return ((size_t)n + 31u) & ~(size_t)31u; }

// What the kernels leave for mc_last_device_status.  The larger one stays: a call that gave up waiting leaves a payload that a
// decompress-and-sum then finds wrong, and a state of which the caller has to know.
enum DeviceFlag { FLAG_PAYLOAD = 1, FLAG_GAVE_UP = 2 };
__device__ __forceinline__ void raise_flag(int *status, DeviceFlag f) { atomicMax(status, (int)f); }

struct PtrChunk { uintptr_t p[256]; };

// ---- which group a block works on -----------------------------------------------------------------------------
// A kernel covers one group (mc_compress, mc_decompress_sum), whose addresses then travel as kernel arguments, or all
// groups of a context in one launch (the _groups calls).  In the second case the blocks of all groups are numbered
// one group after the other, a table says which group a block belongs to, and what the group's blocks need to know
// is split into a table that is fixed when the context is created (GroupConst) and a list of the call's addresses.
// Kernels take the difference as a template parameter: both forms hand out the same job.
// (Measured, compress and decompress-sum of a rank with 8 workers, launch by launch / all groups at once: 161 groups of
// one tensor each, 25.6 M elements, EF-Sign 3170 -> 82 us, what the same elements take as one group; 270 000 elements
// in four groups, Top-k 108 -> 32 us, in eight, QSGD 174 -> 34; two groups of 12.8 M, DGC 152 -> 133, three, QSGD 171 -> 134.
// A table costs a kernel one more level of scalar loads: the merged model as one group keeps its arguments.)
enum BlockKind { BLK_TILE = 0, BLK_PLANE = 1, BLK_SELECT = 2, BLK_EMIT = 3, BLK_KINDS = 4 };   // 4096 elements; 8192; 16 tiles; 4 tiles
struct GroupConst {
    const uint32_t *seg_off, *chunk_seg;
    uint64_t goff, k;
    uint32_t n, nseg;
    uint32_t first[BLK_KINDS];    // number of the group's first block, per kind of block (BLK_TILE: its first tile)
    uint32_t first_ptr;           // its first tensor in the list of addresses
    uint32_t first_sub;           // sparsifiers: its first sublist of keys in the threshold's bin
};
struct GroupTable {
    const GroupConst *groups;
    const uint32_t *block_group[BLK_KINDS];
    const uintptr_t *list;        // addresses of the call: tensors of all groups (the non-empty ones), then what the call needs per group
    const uintptr_t *chunk_addr;  // per chunk of all groups' tiles
    uint32_t live;                // tensors in the list
    uint32_t y;
};

__device__ __forceinline__ GroupView view_of(const GroupTable &tb, const GroupConst *c)
{
    GroupView g;
    g.seg_off = ld_uniform(&c->seg_off);
    g.chunk_seg = ld_uniform(&c->chunk_seg);
    g.ptrs = tb.list + ld_uniform(&c->first_ptr);
    g.chunk_addr = tb.chunk_addr + (size_t)ld_uniform(&c->first[BLK_TILE]) * kWavesPerBlock;
    g.nseg = ld_uniform(&c->nseg);
    g.n = ld_uniform(&c->n);
    g.goff = ld_uniform(&c->goff);
    return g;
}
// Groups of at most this many tiles (262 144 elements) combine their blocks' partial sums inside the compressing kernel, by
// counting arrivals: 64 of them at one address take about a microsecond (256 blocks that wait for each other took 6 to 7,
// thousands far longer than the launch of a kernel that combines them), and 64 partials are one per lane of the
// wavefront that adds them, in that kernel's order.
constexpr uint32_t kSmallTiles = 64;
constexpr int kArriveStride = 16;             // 64-bit words between the groups' counts (a line each)
constexpr uint32_t kWaitLooks = 1u << 10;     // looks of about a microsecond each before a waiting quantizer's block leaves its tile to the last one
// Launches of at most this many tiles, of all their groups, spread a tile over kSpread threads: two such blocks fit a compute
// unit, 512 the card, so that up to here all of them run at once.  Compress of 256 / 500 / 800 / 1200 / 2000 tiles, 16 elements per lane
// and spread: SigNUM 4.9 / 5.7 / 8.1 / 10.3 / 16.4 and 4.3 / 5.0 / 7.4 / 10.2 / 16.6 us, FP16 4.6 / 5.6 / 8.6 / 11.4 / 18.9 and 4.5 / 5.5 / 7.8 / 11.2 /
// 18.7, Top-k 17.6 / 19.0 / 21.8 / 24.8 / 32.9 and 16.4 / 17.9 / 21.5 / 24.8 / 32.5, SignSGD 4.2 / 4.3 / 4.5 / 5.1 / 6.9 and 4.3 / 4.2 / 4.4 / 5.7 / 8.6.
// (The spread form is still ahead up to about 900 tiles and clearly behind from 1200 on only where next to nothing is read besides the
// gradient: the line is on the safe side of all of them.)
constexpr uint32_t kSpreadTiles = 512;
// ... and EF-Sign and OneBit, which sum p in the order of the other form: 400 000 / 1 M / 2 M elements, EF-Sign 8.1 / 8.7 / 10.0 and
// 7.8 / 8.8 / 10.4, OneBit 9.8 / 10.5 / 11.8 and 9.6 / 10.5 / 13.0.
constexpr uint32_t kSpreadSumTiles = 128;
// ... and the decompress-and-sum of one code per element: a block per compute unit.  Of 256 / 400 / 500 tiles in one tensor, QSGD, 1 worker 4.1 / 4.3 /
// 4.4 and 3.9 / 4.6 / 5.2 us, 8 workers 7.4 / 7.6 / 7.5 and 5.2 / 6.7 / 7.1; FP16, 1 worker 4.1 / 4.5 / 4.5 and 4.2 / 4.2 / 4.3, 8 workers 6.8 /
// 8.1 / 8.6 and 5.3 / 7.1 / 7.6.
constexpr uint32_t kSpreadDecodeTiles = 256;
// ... and of bit planes, in blocks of 8192 elements, with the blocks that check the headers one per compute unit.  Of 128 / 250 / 300 / 400 blocks in one
// tensor, EF-Sign, 1 worker 5.3 / 5.5 / 6.2 / 6.5 and 4.6 / 4.8 / 6.4 / 6.8 us, 8 workers 5.7 / 6.4 / 6.6 / 7.1 and 5.3 / 6.0 / 7.8 / 8.2; TernGrad, 8 workers
// 5.9 / 6.3 / 6.9 / 6.9 and 5.8 / 6.0 / 7.8 / 7.8.
constexpr uint32_t kSpreadPlanes = 240;
__host__ __device__ inline uint32_t tiles_in(uint32_t n) { return (uint32_t)(((uint64_t)n + kTile - 1) / kTile); }

// How the blocks' partial sums become the group's scalars: by a kernel after this one; by the block of a small group that arrives last; by that one, or
// in a larger group by a block of the same launch that waits for them (a collector).
enum Combine { COMBINE_AFTER = 0, COMBINE_LAST = 1, COMBINE_COLLECT = 2 };
// Blocks of a launch that collect, each for every kCollectors-th of the larger groups: few enough that the collectors of a good number of launches side
// by side leave room for what they wait for.
constexpr uint32_t kCollectors = 64;
// They are used where the largest group has at most so many tiles.  A collector reads 1024 partials at a time, each time with a wait of its own among
// the other blocks' traffic, and falls behind on a larger group.  (Compress of 8000 / 10 864 / 20 000 / 40 000 tiles, a kernel after the pass and a
// collector: EF-Sign without error feedback 24.9 / 32.3 / 56.5 / 112.2 and 24.4 / 32.6 / 59.6 / 121.6 us, with it, from 10 864, 86.5 / 154.3 / 306.6 and 84.8 / 154.6 /
// 311.8; TernGrad without 47.3 / 64.2 / 111.0 / 216.5 and 46.8 / 63.8 / 113.7 / 223.9, with it 112.3 / 200.6 / 423.0 and 110.5 / 199.6 / 435.1.)
constexpr uint32_t kCollectTiles = 12288;
constexpr uint32_t kCollectLooks = 1u << 21;     // looks of about a microsecond before a collector gives up: no launch that has the device comes near it

// A dense compressor's job.  The state's header lies in front of st, the payload's body behind hdr.
struct CompressJob {
    GroupView g;
    float *st;                    // null when the scheme keeps no state
    PayloadHeader *hdr;
    double *partial;              // one double per tile (OneBit: three arrays of one per tile)
    uint64_t *arrive;             // the group's count of blocks that have their partial ready (small groups); the word behind it: handed_over
    double *slots;                // one double per tile, empty between calls: partials on their way to a collector
    uint32_t tile, ntiles;
    __device__ __forceinline__ StateHeader *state_header() const { return reinterpret_cast<StateHeader *>(st) - 1; }
    __device__ __forceinline__ uint8_t *body() const { return reinterpret_cast<uint8_t *>(hdr) + kHeaderBytes; }
    __device__ __forceinline__ uint64_t *handed_over() const { return arrive + 1; }      // tiles that a waiting quantizer left to the last block; 0 between calls
};
struct OneCompress {
    GroupView g;
    float *st;
    PayloadHeader *hdr;
    double *partial;
    uint64_t *arrive;             // null: the call may not rely on what an earlier one left (mc_compress_static)
    double *slots;                // null: a kernel after this one combines the partials
    int *status;
    uint32_t looks;
    __device__ __forceinline__ uint32_t tiles() const { return tiles_in(g.n); }
    __host__ __device__ __forceinline__ uint32_t collected() const { return 1u; }
    __device__ __forceinline__ CompressJob group_job(uint32_t) const { return {g, st, hdr, partial, arrive, slots, 0u, tiles()}; }
    __device__ __forceinline__ CompressJob collected_job(uint32_t) const { return group_job(0u); }
    __device__ __forceinline__ CompressJob job() const { return {g, st, hdr, partial, arrive, slots, tiles() - 1u - blockIdx.x, tiles()}; }
};
struct AllCompress {              // list: tensors, then y states, then y payloads
    GroupTable tb;
    double *partial;
    uint64_t *arrive;             // kArriveStride words per group
    double *slots;
    int *status;
    uint32_t looks;
    uint32_t all_tiles, large_groups;
    const uint32_t *large;        // the groups of more than kSmallTiles tiles, the last ones first
    __device__ __forceinline__ uint32_t tiles() const { return all_tiles; }
    __host__ __device__ __forceinline__ uint32_t collected() const { return large_groups; }
    __device__ __forceinline__ CompressJob collected_job(uint32_t q) const { return group_job(ld_uniform(large + q)); }
    __device__ __forceinline__ CompressJob group_job(uint32_t q) const
    {
        CompressJob j;
        const GroupConst *c = tb.groups + q;
        j.g = view_of(tb, c);
        const uintptr_t state = ld_uniform(tb.list + tb.live + q);
        j.st = state ? reinterpret_cast<float *>(state + kHeaderBytes) : nullptr;
        j.hdr = reinterpret_cast<PayloadHeader *>(ld_uniform(tb.list + tb.live + tb.y + q));
        j.partial = partial + 3u * (size_t)ld_uniform(&c->first[BLK_TILE]);
        j.arrive = arrive + (size_t)q * kArriveStride;
        j.slots = slots + ld_uniform(&c->first[BLK_TILE]);
        j.tile = 0u;
        j.ntiles = tiles_in(j.g.n);
        return j;
    }
    __device__ __forceinline__ CompressJob job() const
    {
        const uint32_t block = all_tiles - 1u - blockIdx.x, q = ld_uniform(tb.block_group[BLK_TILE] + block);
        CompressJob j = group_job(q);
        j.tile = block - ld_uniform(&tb.groups[q].first[BLK_TILE]);
        return j;
    }
};

// What the header of a payload has to say.  The first blocks of a decompress-and-sum do nothing but look at them, a header per
// thread: in the block of a tile, field by field in front of its work, they were four memory latencies in a row, most of what a
// block of a small group takes, and read ahead of the work and compared after it their registers cost the sparse kernel a
// wavefront per SIMD (25.6 M elements, 8 workers: 0.6 us of 22).  (One block that went through the headers of all groups was
// the last to finish where there are many: 100 000 elements in 161 / 300 groups, 16 workers, Top-k 9.6 / 15.9 -> 5.8 / 5.8 us, EF-Sign
// 8.4 / 13.8 -> 7.0 / 7.2; 300 groups, 64 workers 62 -> 18 and 51 -> 19.)
struct Expected {
    uint32_t algo;
    bool sparse, capped;          // the number of kept entries is fixed by the group, or at most what there is room for
    __device__ __forceinline__ void check(const uint8_t *payload, uint32_t n, uint64_t k, int *status) const
    {
        const PayloadHeader *h = reinterpret_cast<const PayloadHeader *>(payload);
        const uint64_t n_sent = h->n, k_sent = h->k;      // (all asked for before the first is looked at)
        const uint32_t magic = h->magic, of = h->algo, levels = h->levels;
        const bool fits = !sparse | (capped ? (k_sent <= k) & (levels == (uint32_t)k) : k_sent == k);
        if ((magic != kMagic) | (of != algo) | (n_sent != (uint64_t)n) | !fits) raise_flag(status, FLAG_PAYLOAD);
    }
};

// A decompress-and-sum's job: the output, the payloads of the group, and this block's number among the group's.  kRoom: the most workers that the
// source may have.
// ROOM: payloads that there is room for.  The arguments of a launch are written across the bus: those for 64 workers took a call 0.6 us
// longer than those for eight (3.3 instead of 2.7 us for the launch of a kernel that does nothing).
constexpr int kFewRoom = 8;
template <int ROOM>
struct DecompressOf {
    GroupView out;
    const uint8_t *pl[ROOM];
    uint64_t k;
    struct Job {
        GroupView out;
        const DecompressOf *src;
        uint64_t k;
        uint32_t block;
        // the payloads of workers w0 .. w0 + N - 1 (w0: a multiple of N); behind the last worker's some other one
        template <int N> __device__ __forceinline__ void payloads(int w0, int, const uint8_t *(&p)[N]) const
        {
#pragma unroll
            for (int b = 0; b < N; ++b) p[b] = src->pl[w0 + b];
            hold(p);
        }
    };
    template <int KIND> __device__ __forceinline__ Job job() const { return {out, this, k, my_tile_index()}; }
    static constexpr int kRoom = ROOM;
    static constexpr uint32_t kCheckers = 1;      // blocks that look at the headers
    __device__ __forceinline__ void check(const Expected &e, int W, int *status) const
    {
        if ((int)threadIdx.x < W) e.check(pl[threadIdx.x], out.n, k, status);
    }
};
using OneDecompress = DecompressOf<kMaxWorkers>;
inline DecompressOf<kFewRoom> with_few(const OneDecompress &src)
{
    DecompressOf<kFewRoom> few{src.out, {}, src.k};
    for (int w = 0; w < kFewRoom; ++w) few.pl[w] = src.pl[w];
    return few;
}
struct AllDecompress {            // list: tensors, then the W payloads of group 0, of group 1, ...
    GroupTable tb;
    int W;
    static constexpr int kRoom = kMaxWorkers;
    struct Job {
        GroupView out;
        const uintptr_t *pl;
        uint64_t k;
        uint32_t block;
        template <int N> __device__ __forceinline__ void payloads(int w0, int W, const uint8_t *(&p)[N]) const
        {
#pragma unroll
            for (int b = 0; b < N; ++b) p[b] = reinterpret_cast<const uint8_t *>(ld_uniform(pl + (w0 + b < W ? w0 + b : 0)));
            hold(p);
        }
    };
    template <int KIND> __device__ __forceinline__ Job job() const
    {
        Job j;
        const uint32_t b = my_tile_index(), q = ld_uniform(tb.block_group[KIND] + b);
        const GroupConst *c = tb.groups + q;
        j.out = view_of(tb, c);
        j.pl = tb.list + tb.live + (size_t)q * W;
        j.k = ld_uniform(&c->k);
        j.block = b - ld_uniform(&c->first[KIND]);
        return j;
    }
    // A constant: computed from the number of headers, every block would have to wait for its arguments before it knows that
    // it is a tile's, 0.25 us of a call on small groups.
    static constexpr uint32_t kCheckers = 16;
    __device__ __forceinline__ void check(const Expected &e, int, int *status) const
    {
        for (uint32_t i = blockIdx.x * (uint32_t)kBlock + threadIdx.x; i < tb.y * (uint32_t)W; i += kCheckers * (uint32_t)kBlock) {
            const GroupConst &c = tb.groups[i / (uint32_t)W];
            const uintptr_t payload = tb.list[tb.live + i];
            const uint64_t k = c.k;
            if (c.n) e.check(reinterpret_cast<const uint8_t *>(payload), c.n, k, status);
        }
    }
};

// radix-select state carried between the passes of the exact top-k
struct SelectState {
    uint32_t lo;         // the threshold key lies in [lo, lo + range of the levels still to resolve)
    uint32_t mode;       // what the seed kernel found (fast / refill flags)
    uint64_t need;       // entries still to take among the keys of that range
};

// profiling slots
enum KernelId {
    K_UPLOAD = 0, K_EFSIGN_COMPRESS, K_SCALAR_FINALIZE, K_ACCUM_REDUCE, K_QSGD_ENCODE, K_TERN_ENCODE,
    K_FP16_COMPRESS, K_DENSE_DECOMPRESS, K_SPARSE_ACCUM, K_SPARSE_SEED, K_CAND_HIST2, K_CAND_HIST3, K_CAND_COUNT,
    K_CAND_EMIT, K_SPARSE_DECOMPRESS, K_STATE_CONVERT, K_LEAN_SELECT, K_LEAN_EMIT, K_COUNT
};

// reduction kinds of the two-pass quantizers
enum ReduceMode { RED_MEAN_ABS = 0, RED_L2 = 1, RED_MAX_ABS = 2, RED_ONE = 3, RED_MEANS = 4 };
// the one-bit compressors (one kernel) and what their single plane decodes to
enum SignMode { SIGN_EF = 0, SIGN_MEANS = 1, SIGN_PLAIN = 2, SIGN_MOMENTUM = 3 };
enum PlaneKind { PLANE_SCALE = 0, PLANE_MEANS = 1, PLANE_VOTE = 2 };

struct LaunchCtx {               // what a launcher needs besides its arguments
    hipStream_t stream;
    void *prof;                  // opaque: profiling recorder or null
    mutable hipEvent_t ev_a = nullptr, ev_b = nullptr;   // set by prof_begin when the next launch is to be timed
};
// prof_begin arms the next MC_LAUNCH with a start / stop event pair (if that kernel slot is being timed);
// the events are attached to the dispatch itself, so they bracket the kernel's execution only.
void prof_begin(const LaunchCtx &lc, int id);
void prof_end(const LaunchCtx &lc, int id);
// A launch by the runtime's call itself: the triple-bracket form hands the configuration through a stack of the runtime's
// first (3.3 -> 3.1 us of host time, and a small group's call takes the host as long as the GPU).
template <class... P>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t stream, std::common_type_t<P>... args)
{
    void *at[] = {static_cast<void *>(&args)...};
    (void)hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, at, 0, stream);      // (an error is what hipGetLastError says)
}
#define MC_LAUNCH(kernel, grid, block, lc, ...)                                                                       \
    do {                                                                                                              \
        if ((lc).ev_a) hipExtLaunchKernelGGL(kernel, grid, block, 0, (lc).stream, (lc).ev_a, (lc).ev_b, 0, __VA_ARGS__); \
        else mc::launch(kernel, grid, block, (lc).stream, __VA_ARGS__);                                               \
    } while (0)

// ---- dense kernels (kernels_dense.hip) -----------------------------------------
// The launchers of the path come in the two forms of a job source; `tiles` is the number of blocks of 4096 elements
// that the launch covers (of all its groups), `groups` the number of groups.
void launch_upload_ptrs(const LaunchCtx &lc, const uintptr_t *host, uintptr_t *dev, uint32_t count);
void launch_expand_ptrs(const LaunchCtx &lc, const GroupView &g, uintptr_t *chunk_addr);
void launch_expand_all(const LaunchCtx &lc, const GroupTable &tb, uint32_t tiles, uintptr_t *chunk_addr);
// small: every group has at most kSmallTiles tiles and src.arrive counts.  src.slots: otherwise COMBINE_COLLECT
template <class SRC> void launch_sign_compress(const LaunchCtx &lc, int mode, const SRC &src, uint32_t tiles, bool ef, float beta, uint32_t algo, bool small);
template <class SRC> void launch_quantize_small(const LaunchCtx &lc, int mode, const SRC &src, uint32_t tiles, bool ef, uint32_t levels, uint64_t seed,
                                                uint32_t worker, uint32_t iter_lo, uint32_t looks);
template <class SRC> void launch_scalar_finalize(const LaunchCtx &lc, const SRC &src, uint32_t groups, int mode, uint32_t algo, uint32_t levels,
                                                 bool keep);
template <class SRC> void launch_accum_reduce(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, int mode, uint32_t levels, uint64_t seed);
template <class SRC> void launch_qsgd_encode(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, uint32_t levels, uint64_t seed,
                                             uint32_t worker, uint32_t iter_lo);
template <class SRC> void launch_tern_encode(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef, uint64_t seed, uint32_t worker, uint32_t iter_lo);
template <class SRC> void launch_fp16_compress(const LaunchCtx &lc, const SRC &src, uint32_t tiles, bool ef);
template <class SRC> void launch_dense_decompress(const LaunchCtx &lc, int algo, const SRC &src, uint32_t blocks /* of 8192 elements for the bit planes */,
                                                  int W, float alpha, uint32_t levels, int *status);
inline uint32_t plane_blocks(uint32_t n) { return (uint32_t)(((uint64_t)n + 2 * kTile - 1) / (2 * kTile)); }
void launch_state_convert(const LaunchCtx &lc, int algo, bool to_residual, uint32_t n, const void *src, void *dst, uint32_t levels,
                          uint64_t seed, uint64_t goff);

// ---- sparse kernels (kernels_sparse.hip) ----------------------------------------
constexpr int kHintWorkers = 64;                         // hints kept per group, one per worker id modulo this
constexpr int kHintWords = 4;                            // words of a hint record (filter key, halvings of the margin, calls it is held after a miss, cap on the halvings)
constexpr int kWinCopies = 8;                                // copies of the window histogram (a block adds to the copy of its index)
constexpr int kHistWords = 2048 * kWinCopies + 2048 + 1024 + 2048 + 64;   // bins of the window and of the three radix levels, copies of the window's open bin

// The keys that share the threshold's window bin (the only candidates whose fate the window does not settle) are
// handed from the select kernel to the emit kernel as an unordered list, appended to by wave-wide atomic adds.
// Adds to one address queue up behind each other, so the list is kept in kUSub sublists (a wavefront appends to the
// one of its tile index) whose counters sit on cache lines of their own.
constexpr int kUSub = 64;
constexpr uint32_t kUCap = 4096;      // keys in the threshold's window bin that the two-kernel route takes; a sublist holds as many
constexpr int kUCountStride = 32;     // words between sublist counters (one 128-byte line each)
struct UEntry { uint32_t idx, bits; };       // group-relative index, candidate bits
// Candidate slots behind the last chunk of the scratch.  A chunk's 1024 slots are read as a head of 64 and units of 256,
// masked after the load: a chunk with more than 64 + 3 * 256 candidates reads up to slot 64 + 4 * 256 - 1, of the chunk
// after it, and the scratch's last chunk into these.
constexpr int kCandHead = 64, kCandUnit = 256;
constexpr int kCandPad = kCandHead + (kChunk - kCandHead + kCandUnit - 1) / kCandUnit * kCandUnit - kChunk;

struct SparseScratch {
    uint32_t *hist;        // kHistWords counters; each level is cleared by a later kernel of the same call
    SelectState *sel;      // [0]: after the seed, [1..3]: after each radix level
    uint32_t *hint;        // this (group, worker)'s hint record; word 0: keys >= it are candidates (0 = everything)
    uint32_t *cand_bits;   // candidate values (fp32 bit patterns), 1024 slots per chunk, filled from the front
    uint16_t *cand_loc;    // candidate positions inside their chunk
    uint64_t *tile_runs;   // candidates of the four chunks of every tile, 16 bits each
    uint32_t *tile_cnt;    // per tile: candidates above (low 16 bits) / equal to (high 16 bits) the threshold
    uint32_t *blk_cnt;     // the same per block of four tiles
    UEntry *ulist;         // kUSub sublists of kUCap entries: the candidates in the threshold's window bin
    uint32_t *ucount;      // their lengths, kUCountStride words apart; cleared by the streaming pass of the next call
    uint32_t *arrive;      // arrivals at the grid-wide barriers of the slow routes (cleared by the streaming pass), a line of its own
    uint32_t *sync;        // [32..36): calls per route; [40], [41]: what mc_select_stats reports of the most recent call
    uint32_t spin_limit;   // polls after which a block gives up waiting at such a barrier (mc_set_barrier_spin_limit)
};
// The part of the scratch that group number q of a launch over all groups works in: every group has its own, laid out
// one after the other (hint records: of the worker that `all` was set up for).
__host__ __device__ inline SparseScratch scratch_of(const SparseScratch &all, uint32_t q, uint32_t first_tile, uint32_t first_sub)
{
    SparseScratch s = all;
    s.hist += (size_t)q * kHistWords;
    s.sel += (size_t)q * 4;
    s.hint += (size_t)q * kHintWorkers * kHintWords;
    s.cand_bits += (size_t)first_tile * kTile;
    s.cand_loc += (size_t)first_tile * kTile;
    s.tile_runs += first_tile;
    s.tile_cnt += first_tile;
    s.blk_cnt += first_tile;
    s.ulist += (size_t)first_sub * kUCap;
    s.ucount += (size_t)q * kUSub * kUCountStride;
    s.arrive += (size_t)q * kUCountStride;
    return s;
}
constexpr int kSelTiles = 16, kEmitTiles = kWavesPerBlock;     // tiles per block of the select and the emit kernel
// Blocks of a group that lean_small_k, which is both for small groups, runs the slow routes on.  (Up to 8 tiles one block, which needs
// no barriers, is ahead: 8 tiles, a refill and a rise in turn, Top-k 41.7 us, two blocks 45.2; 16 tiles 54.4, four blocks 49.1.)
constexpr uint32_t kOneBlockTiles = 8;
__host__ __device__ constexpr uint32_t small_sel_blocks(uint32_t tiles) { return tiles == 0u ? 0u : tiles <= kOneBlockTiles ? 1u : (tiles + kEmitTiles - 1u) / kEmitTiles; }
constexpr int kArriveWindow = 1;                               // word behind SparseScratch::arrive: blocks of lean_small_k that have read the window
constexpr int kArriveDone = 2;                                 // ... of sparse_accum_k, where the selection follows, that are done (0 between calls)

// A sparsifier's job: `block` is this block's number among the group's `blocks` of its kind (tiles: handed out last first).
struct SparseJob {
    GroupView g;
    float *st;
    PayloadHeader *hdr;
    uint64_t k;
    SparseScratch sc;
    uint32_t block, blocks;
    bool reports;                 // this group's counts are what mc_select_stats shows as the most recent call's
};
struct OneSparse {
    GroupView g;
    float *st;
    PayloadHeader *hdr;
    uint64_t k;
    SparseScratch sc;
    template <int KIND> __device__ __forceinline__ SparseJob job() const
    {
        return {g, st, hdr, k, sc, KIND == BLK_TILE ? my_tile_index() : blockIdx.x, gridDim.x, true};
    }
    __device__ __forceinline__ SparseJob small_job() const { return {g, st, hdr, k, sc, blockIdx.x, gridDim.x, true}; }
};
struct AllSparse {                // list: tensors, then y states, then y payloads
    GroupTable tb;
    SparseScratch all;
    uint32_t last_group;          // the last one that holds elements
    bool one_each;                // lean_small_k: one block for each group, so that none has to look its group up
    __device__ __forceinline__ SparseJob group_job(uint32_t q) const
    {
        const GroupConst *c = tb.groups + q;
        const uintptr_t state = ld_uniform(tb.list + tb.live + q);
        return {view_of(tb, c), state ? reinterpret_cast<float *>(state + kHeaderBytes) : nullptr,
                reinterpret_cast<PayloadHeader *>(ld_uniform(tb.list + tb.live + tb.y + q)), ld_uniform(&c->k),
                scratch_of(all, q, ld_uniform(&c->first[BLK_TILE]), ld_uniform(&c->first_sub)), 0u, 0u, q == last_group};
    }
    template <int KIND> __device__ __forceinline__ SparseJob job() const
    {
        const uint32_t b = KIND == BLK_TILE ? my_tile_index() : blockIdx.x, q = ld_uniform(tb.block_group[KIND] + b);
        constexpr uint32_t per = KIND == BLK_SELECT ? kSelTiles : KIND == BLK_EMIT ? kEmitTiles : 1;
        SparseJob j = group_job(q);
        j.block = b - ld_uniform(&tb.groups[q].first[KIND]);
        j.blocks = (tiles_in(j.g.n) + per - 1u) / per;
        return j;
    }
    __device__ __forceinline__ SparseJob small_job() const
    {
        SparseJob j = one_each ? group_job(blockIdx.x) : job<BLK_EMIT>();
        j.blocks = small_sel_blocks(tiles_in(j.g.n));
        return j;
    }
};
// What a sparsifier needs besides its groups.  sync_blocks: how many blocks of 1024 threads the device surely holds at once (one per
// compute unit): the slow routes of the selection run on that many blocks with grid-wide barriers between their steps.
struct SparseCall {
    float momentum;
    uint64_t seed;
    uint32_t worker, iter_lo, sync_blocks;
    int *status;
    uint32_t sample_stride = 0, sample_first = 0;      // DGC with a sampled threshold (one group only)
    uint64_t sample_need = 0;
};
// Groups whose selection one block finishes (lean_small_k).  A block of 1024 threads holds 16384 candidates; under the filter's
// rules there are about 2 k, 2.5 leave room.  (At both limits together, 32 tiles and 6029 kept, Top-k compress 18.0 us against 21.4 with
// the two kernels.)
constexpr int kSmallSelTiles = 32;
constexpr uint32_t kSmallKept = 6144;
inline bool selects_small(uint32_t n, uint64_t k) { return tiles_in(n) <= (uint32_t)kSmallSelTiles && k <= kSmallKept; }
// Tiles of a launch of sparse_accum_k with the selection.  (Beyond, a compute unit has room for one of its blocks, or for two of the streaming pass: Top-k compress of
// 64 groups of 1 / 3 / 5 tiles, two kernels 16.4 / 13.6 / 15.2 us, one 14.8 / 14.2 / 21.0.)
constexpr uint32_t kSameTiles = 64;
struct SparseBlocks {             // blocks of each kind that the launches cover
    uint32_t tiles, select, emit;
    uint32_t small = 0;           // those of lean_small_k, if all groups are such
    bool same = false;            // ... and sparse_accum_k does their work
};
inline SparseBlocks sparse_blocks(uint32_t n)
{
    const uint32_t t = tiles_in(n);
    return {t, (t + kSelTiles - 1) / kSelTiles, (t + kEmitTiles - 1) / kEmitTiles};
}
template <class SRC> void launch_sparse_compress(const LaunchCtx &lc, int algo, const SRC &src, const SparseBlocks &nb, bool ef, const SparseCall &call);
template <class SRC> void launch_sparse_decompress(const LaunchCtx &lc, int algo, const SRC &src, uint32_t tiles, int W, float alpha, int *status,
                                                   bool capped);

}  // namespace mc

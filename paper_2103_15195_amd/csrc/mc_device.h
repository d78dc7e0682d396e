// Device-side building blocks shared by the gfx950 kernels: the wave-chunk
// element mapping, segment-table addressing, reductions and Philox.
//
// Element mapping.  A block of 256 threads (4 wavefronts of 64) owns a tile of
// 4096 consecutive flat elements of a merged group; wavefront w owns the
// 1024-element chunk starting at tile + 1024 w, and in step j (0..15) lane l
// holds flat element  chunk + 64 j + l.  A wave instruction therefore touches 256
// contiguous bytes whatever the alignment of the tensors behind the flat index,
// and a 64-bit ballot of step j is exactly two consecutive 32-bit words of a
// packed bit plane.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mc {

constexpr int kBlock = 256;
constexpr int kWave = 64;
constexpr int kSteps = 16;                  // elements per lane per chunk
constexpr int kChunk = kWave * kSteps;      // 1024 elements per wavefront
constexpr int kTile = kBlock * kSteps;      // 4096 elements per block
constexpr int kWavesPerBlock = kBlock / kWave;

// A merged group as the kernels see it: the flat index space [0, n) laid over
// `nseg` non-empty tensors.  seg_off[s] is the flat index of the first element
// of tensor s (strictly increasing, seg_off[nseg] = n); ptrs[s] its address.
struct GroupView {
    const uint32_t *seg_off;
    const uint32_t *chunk_seg;   // tensor that holds the first element of each 1024-element chunk
    const uintptr_t *ptrs;
    const uintptr_t *chunk_addr; // per chunk: its address if the whole chunk lies in one tensor, else 2 * first tensor + 1 (chunk_entry)
    uint32_t nseg;
    uint32_t n;
    uint64_t goff;   // model-global flat index of element 0 (random streams only)
};

// Small groups leave most of the chip idle, and their kernels take as long as one wavefront's instructions do: they spread a
// tile over four times as many wavefronts.  What a wavefront holds is then a quarter of a chunk, kSpreadSteps elements
// per lane, and kSteps in what follows is whatever the array has that an element is held in.
constexpr int kSpreadSteps = 4;
constexpr int kSpread = kTile / kSpreadSteps;       // threads per tile

struct Chunk {
    uint32_t base;   // flat index of the wavefront's first element (wave-uniform)
    uint32_t lane;
    bool full;       // all of the wavefront's elements lie below n
};

// Tiles are handed out last first (block 0 takes the last tile).  The chunks that straddle tensors are the slow
// ones, and in a model's gradient list they crowd where the small tensors are -- at the end, when the list is in
// the order the gradients become ready, the first layers last.  Started first, they are hidden behind the rest
// (read-only pass over the ResNet-50 list: 18.0 us instead of 19.5; 17.1 with no such chunk at all).
// (A decompress-and-sum's grid has more blocks, the first ones, which get numbers behind the last tile's: Expected.)
__device__ __forceinline__ uint32_t my_tile_index() { return gridDim.x - 1u - blockIdx.x; }

template <int S = kSteps>
__device__ __forceinline__ Chunk my_chunk(uint32_t n, uint32_t tile)
{
    Chunk c;
    uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    c.base = tile * (uint32_t)kTile + wave * (uint32_t)(kWave * S);
    c.lane = threadIdx.x & 63u;
    c.full = c.base < n && n - c.base >= (uint32_t)(kWave * S);
    return c;
}
__device__ __forceinline__ Chunk my_chunk(uint32_t n) { return my_chunk(n, my_tile_index()); }

// A load whose address is the same for the whole wavefront, forced onto the scalar path (constant address
// space).  In a kernel that streams stores, loads on the vector path queue behind those stores; the scalar
// cache does not.  (Measured: the same 16 table loads per wavefront cost the sparse decompress 5-7 us more
// when the compiler happened to issue them as vector loads.)  Only for data no thread of this kernel writes.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T *p)
{
    typedef const T __attribute__((address_space(4))) *const_ptr;
    return *(const_ptr)(uintptr_t)p;
}

// Values that are the same for the wavefront, all there from here on.  Asked for under conditions of their own ("if
// there is a worker b"), scalar loads are waited for one after the other, a memory latency each; loaded without condition
// and passed through here they travel together.  (One address, scale and directory entry per worker after the other, decompress-and-sum of 25.6 M
// elements and 8 workers: Rand-k 26.0 us, then 22.1; TernGrad 32.0, then 28.3; 16 workers, EF-Sign of 44.5 M 65, then 55.)
template <typename T>
__device__ __forceinline__ void hold(T (&x)[4]) { asm volatile("" : "+s"(x[0]), "+s"(x[1]), "+s"(x[2]), "+s"(x[3])); }
template <typename T>
__device__ __forceinline__ void hold(T (&x)[8])
{
    asm volatile("" : "+s"(x[0]), "+s"(x[1]), "+s"(x[2]), "+s"(x[3]), "+s"(x[4]), "+s"(x[5]), "+s"(x[6]), "+s"(x[7]));
}

// An address that came out of a table or through hold() as one in device memory.  Of a generic one the compiler does not
// know that it is not in LDS: every access then counts as an LDS access too, and waiting for either waits for both.
template <typename T>
using global_ptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> in_global(T *p) { return (global_ptr<T>)(uintptr_t)p; }

template <typename T>
__device__ __forceinline__ T ld_stream(const T *p) { return __builtin_nontemporal_load(p); }
template <typename T>
__device__ __forceinline__ void st_stream(T *p, T v) { __builtin_nontemporal_store(v, p); }

// ---- flat (contiguous) buffers -------------------------------------------
// (STREAM: non-temporal, which is faster for what is read once)
template <typename T, bool STREAM = true, int S>
__device__ __forceinline__ void load_flat(const T *buf, const Chunk &c, uint32_t n, T (&v)[S], T fill)
{
    const global_ptr<const T> p = in_global(buf) + c.base + c.lane;
    if (c.full) {
#pragma unroll
        for (int j = 0; j < S; ++j) v[j] = STREAM ? __builtin_nontemporal_load(p + 64 * j) : p[64 * j];
    } else {
#pragma unroll
        for (int j = 0; j < S; ++j) v[j] = (c.base + 64 * j + c.lane < n) ? p[64 * j] : fill;
    }
}

template <typename T, int S>
__device__ __forceinline__ void store_flat(T *buf, const Chunk &c, uint32_t n, const T (&v)[S])
{
    const global_ptr<T> p = in_global(buf) + c.base + c.lane;
    if (c.full) {
#pragma unroll
        for (int j = 0; j < S; ++j) __builtin_nontemporal_store(v[j], p + 64 * j);
    } else {
#pragma unroll
        for (int j = 0; j < S; ++j) if (c.base + 64 * j + c.lane < n) p[64 * j] = v[j];
    }
}

// ---- rotated chunks ----------------------------------------------------------
// Stores are sensitive to where a wave instruction's 256 bytes start: on this part the plane decompress
// kernel takes 27 us when they start on 128-byte lines, 32 us when they are 32 bytes off (separately
// allocated tensors whose sizes are not multiples of 32 elements put every chunk of the flat grid off the
// lines), and 30.4 us when they only start on 64-byte boundaries.  A kernel that takes its output from
// LDS may permute a chunk's elements among its lanes freely, so it can rotate the mapping by `rot`
// elements: in step j lane l holds element (64 j + l + rot) mod 1024 of the chunk, with rot chosen such
// that element `rot` lies on a line boundary.  Every wave store then covers two whole lines; only step 15
// wraps round to the chunk's first `rot` elements.  (Measured in the library: the one-plane decompress
// gains 2.4-3 us of 32, the sparse decompress 0.2-0.9; both store that way.  The TernGrad decompress
// loses 1.5 us, QSGD and FP16 lose up to 8 us when their code loads are rotated too (they then straddle
// lines) and gain or lose about 1 us when only the sums are rotated with ds_bpermute: those keep the plain mapping.)
constexpr uint32_t kLineElems = 32;        // 128-byte cache line
__device__ __forceinline__ uint32_t chunk_rotation(uintptr_t entry)       // 0 for a chunk without an address of its own
{
    return (entry & 1u) ? 0u : (kLineElems - (uint32_t)((entry >> 2) & (kLineElems - 1u))) & (kLineElems - 1u);
}
__device__ __forceinline__ uint32_t rotated(int j, uint32_t lane, uint32_t rot)
{
    const uint32_t i = 64u * (uint32_t)j + lane + rot;       // below 1024 except, possibly, in the last step
    return j == kSteps - 1 ? i & (uint32_t)(kChunk - 1) : i;
}

// The per-chunk table entry: the address of the chunk's first element when all 1024 elements lie in one
// tensor (even: tensors are 4-byte aligned), else 2 s + 1 with s the tensor that holds the chunk's first
// element (where the loop over the chunk's tensors starts).  Never 0.  A kernel that has other loads to
// wait for before it stores fetches this first, so that the two latencies overlap.
__device__ __forceinline__ uintptr_t chunk_entry(const GroupView &g, const Chunk &c) { return ld_uniform(g.chunk_addr + (c.base >> 10)); }

// ---- segmented (per-tensor) buffers ------------------------------------------
// Fast path: the chunk lies inside one tensor and its address was tabulated when
// the tensor address list was uploaded (one scalar load, then the data).
// Otherwise (the chunk straddles tensors, or is the ragged last one) the wavefront
// fetches the table entries of up to 64 tensors from the chunk's first one on, one per
// lane (tensors_of_chunk).  Their bounds and addresses then come out of the lanes: a walk over
// the chunk's steps, one uniform comparison a step and tensor, gives every element's address, so that
// the data of all tensors is asked for at once, 16 accesses of the wavefront whatever the number of tensors.
// (Tensor by tensor, with a condition around every access, a wavefront waited for each tensor's data in turn, which
// is what a small group's kernels took longest for.  Compress / decompress-and-sum of 1025 elements in eight tensors, 8
// workers: EF-Sign 8.9 / 7.8 -> 5.8 / 4.6 us, QSGD 13.5 / 8.0 -> 10.1 / 5.5, Top-k 20.1 / 7.1 -> 16.6 / 4.6; 272 000 elements
// in 65 tensors and four groups, Top-k 28.6 -> 25.5 for both.)
// (A walk of the table by every lane, two dependent loads per tensor boundary, made the ~100 such chunks of the
// ResNet-50 list the last to finish: 21 instead of 17 us for a read-only pass over the 102 MB.)
struct ChunkTensors { uint32_t beg, end; uintptr_t ptr; };      // of the tensor that this lane holds: flat bounds, address
__device__ __forceinline__ ChunkTensors tensors_of_chunk(const GroupView &g, uint32_t s0)
{
    const uint32_t t = s0 + (threadIdx.x & 63u);
    return {g.seg_off[t < g.nseg ? t : g.nseg], g.seg_off[t < g.nseg ? t + 1u : g.nseg],      // seg_off has nseg + 1 entries, the last is n
            g.ptrs[t < g.nseg ? t : g.nseg - 1u]};
}
template <int S = kSteps>
__device__ __forceinline__ uint32_t chunk_end(const GroupView &g, const Chunk &c) { return g.n - c.base >= (uint32_t)(kWave * S) ? c.base + (uint32_t)(kWave * S) : g.n; }
// (readlane returns int: through uint32_t, or the low word's bit 31 would smear over the high word)
__device__ __forceinline__ uintptr_t lane_addr(uintptr_t x, int k)
{
    return (uintptr_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, k) | ((uintptr_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), k) << 32);
}
// body(j, address of the lane's element of step j) for the 16 steps (STOP: for those that have elements), if the chunk holds
// at most 64 tensors (else false).  A lane behind the end of the group gets the group's last element.
template <bool STOP, int S, typename Body>
__device__ __forceinline__ bool each_step_of_chunk(const GroupView &g, const Chunk &c, const ChunkTensors &ts, Body body)
{
    const uint32_t lim = chunk_end<S>(g, c);
    if ((uint32_t)__builtin_amdgcn_readlane((int)ts.end, 63) < lim) return false;
    const uintptr_t from = ts.ptr - sizeof(float) * (uintptr_t)ts.beg;               // where the group's element 0 would be
    int k = 0;
    uintptr_t cur = lane_addr(from, 0);
    uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)ts.end, 0);
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const uint32_t first = c.base + 64u * (uint32_t)j;
        if (STOP && first >= lim) break;
        const uint32_t hi = min(first + 64u, lim), i = min(first + c.lane, lim - 1u);
        uintptr_t at = cur;
        while (end < hi) {                       // another tensor starts among the step's elements
            const uint32_t beg = end;
            ++k;
            cur = lane_addr(from, k);
            end = (uint32_t)__builtin_amdgcn_readlane((int)ts.end, k);
            at = i >= beg ? cur : at;
        }
        body(j, at + sizeof(float) * (uintptr_t)i);
    }
    return true;
}
// The same for N consecutive elements per lane, i0 the lane's first, hi the end of the wavefront's: their addresses.
template <int N>
__device__ __forceinline__ bool each_span_of_chunk(const ChunkTensors &ts, uint32_t i0, uint32_t hi, uint32_t lim, uintptr_t (&at)[N])
{
    if ((uint32_t)__builtin_amdgcn_readlane((int)ts.end, 63) < lim) return false;
    const uintptr_t from = ts.ptr - sizeof(float) * (uintptr_t)ts.beg;
    uintptr_t cur = lane_addr(from, 0);
    uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)ts.end, 0);
#pragma unroll
    for (int e = 0; e < N; ++e) at[e] = cur;
    for (int k = 1; end < hi; ++k) {
        const uint32_t beg = end;
        cur = lane_addr(from, k);
        end = (uint32_t)__builtin_amdgcn_readlane((int)ts.end, k);
#pragma unroll
        for (int e = 0; e < N; ++e) at[e] = min(i0 + (uint32_t)e, lim - 1u) >= beg ? cur : at[e];
    }
#pragma unroll
    for (int e = 0; e < N; ++e) at[e] += sizeof(float) * (uintptr_t)min(i0 + (uint32_t)e, lim - 1u);
    return true;
}
// body(first element, end, address) for the tensors of a chunk, one after the other, however many
template <int S = kSteps, typename Body>
__device__ __forceinline__ void for_each_tensor_of_chunk(const GroupView &g, const Chunk &c, uint32_t s0, Body body)
{
    const uint32_t lim = chunk_end<S>(g, c);
    for (;;) {
        const ChunkTensors ts = tensors_of_chunk(g, s0);
        for (int k = 0; k < 64; ++k) {
            const uint32_t b = __builtin_amdgcn_readlane(ts.beg, k), e = __builtin_amdgcn_readlane(ts.end, k);
            if (b >= lim) return;                                                // past the chunk (or past the last tensor: b = n)
            body(b, e, lane_addr(ts.ptr, k));
        }
        s0 += 64u;
    }
}

template <int S>
__device__ __forceinline__ void load_seg(const GroupView &g, const Chunk &c, float (&v)[S])
{
    const uintptr_t entry = chunk_entry(g, c);
    if (!(entry & 1u)) {
        const global_ptr<const float> p = in_global(reinterpret_cast<const float *>(entry)) + (S == kSteps ? 0u : c.base & (uint32_t)(kChunk - 1)) + c.lane;
#pragma unroll
        for (int j = 0; j < S; ++j) v[j] = __builtin_nontemporal_load(p + 64 * j);
    } else {
        const uint32_t s0 = (uint32_t)(entry >> 1);
        if (each_step_of_chunk<false, S>(g, c, tensors_of_chunk(g, s0), [&](int j, uintptr_t at) { v[j] = *in_global(reinterpret_cast<const float *>(at)); })) {
            if (!c.full)
#pragma unroll
                for (int j = 0; j < S; ++j) v[j] = c.base + 64 * j + c.lane < g.n ? v[j] : 0.0f;
            return;
        }
#pragma unroll
        for (int j = 0; j < S; ++j) v[j] = 0.0f;
        for_each_tensor_of_chunk<S>(g, c, s0, [&](uint32_t beg, uint32_t end, uintptr_t ptr) {
            const global_ptr<const float> p = in_global(reinterpret_cast<const float *>(ptr));
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const uint32_t i = c.base + 64 * j + c.lane;
                if (i >= beg && i < end) v[j] = p[i - beg];
            }
        });
    }
}

// (Measured on this part: stores whose 256-byte wave windows miss a 64-byte boundary are slower -- a bare
// 102 MB fill takes 16 us aligned and 22 us not, the plane decompress kernel 27 and 32 us -- while loads
// are not sensitive.  Rotating lanes to aligned windows did not pay in these kernels.  Tensors whose flat
// offset is a multiple of 16 elements keep the aligned rate.)
template <int S>
__device__ __forceinline__ void store_seg(const GroupView &g, const Chunk &c, const float (&v)[S], uintptr_t entry)
{
    if (!(entry & 1u)) {
        const global_ptr<float> p = in_global(reinterpret_cast<float *>(entry)) + (S == kSteps ? 0u : c.base & (uint32_t)(kChunk - 1)) + c.lane;
#pragma unroll
        for (int j = 0; j < S; ++j) __builtin_nontemporal_store(v[j], p + 64 * j);
    } else {
        const uint32_t s0 = (uint32_t)(entry >> 1);
        if (each_step_of_chunk<true, S>(g, c, tensors_of_chunk(g, s0), [&](int j, uintptr_t at) {
                if (c.base + 64 * j + c.lane < g.n) *in_global(reinterpret_cast<float *>(at)) = v[j];
            })) return;
        for_each_tensor_of_chunk<S>(g, c, s0, [&](uint32_t beg, uint32_t end, uintptr_t ptr) {
            const global_ptr<float> p = in_global(reinterpret_cast<float *>(ptr));
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const uint32_t i = c.base + 64 * j + c.lane;
                if (i >= beg && i < end) p[i - beg] = v[j];
            }
        });
    }
}
__device__ __forceinline__ void store_seg(const GroupView &g, const Chunk &c, const float (&v)[kSteps])
{
    store_seg(g, c, v, chunk_entry(g, c));
}
// v in the rotated mapping, rot = chunk_rotation(entry) (0 when the chunk has no address of its own)
__device__ __forceinline__ void store_seg_rot(const GroupView &g, const Chunk &c, const float (&v)[kSteps], uintptr_t entry, uint32_t rot)
{
    if (!(entry & 1u)) {
        // steps 0..14 at constant offsets from one address (they fold into the instructions), step 15 may wrap
        const global_ptr<float> p = in_global(reinterpret_cast<float *>(entry)), q = p + (c.lane + rot);
#pragma unroll
        for (int j = 0; j < kSteps - 1; ++j) __builtin_nontemporal_store(v[j], q + 64 * j);
        __builtin_nontemporal_store(v[kSteps - 1], p + rotated(kSteps - 1, c.lane, rot));
    } else {
        store_seg(g, c, v, entry);
    }
}

// ---- packed bit planes -------------------------------------------------------
// Store the ballots of a wavefront's steps (two words each) to a plane of `nwords` words.
// `stage` is one uint64 of LDS per step, private to the calling wavefront.
template <int S>
__device__ __forceinline__ void store_plane(uint32_t *plane, uint32_t nwords, const Chunk &c,
                                            const uint64_t (&ballots)[S], uint64_t *stage)
{
#pragma unroll
    for (int j = 0; j < S; ++j) if (c.lane == (uint32_t)j) stage[j] = ballots[j];
    __builtin_amdgcn_wave_barrier();
    if (c.lane < 2 * S) {
        uint32_t w = (c.base >> 5) + c.lane;
        if (w < nwords) plane[w] = reinterpret_cast<const uint32_t *>(stage)[c.lane];
    }
    __builtin_amdgcn_wave_barrier();
}

// ---- reductions ----------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}
__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
    return x;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// Inclusive prefix sum over the 64 lanes with data-parallel-primitive moves inside the vector ALU (three shifts by one,
// two and three lanes, shifts by four and eight inside the rows of 16, then the row totals handed on: seven adds) instead
// of six rounds through the LDS crossbar that a shuffle-based scan takes: about 30 against 600 cycles of latency, which
// counts in kernels that do little else than wait.  All 64 lanes must be active.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x)
{
    uint32_t v = x;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);      // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);      // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x113, 0xf, 0xf, true);      // row_shr:3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xe, true);      // row_shr:4, lanes 4..15 of a row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xc, true);      // row_shr:8, lanes 8..15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, true);      // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, true);      // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t wave_total(uint32_t incl) { return (uint32_t)__builtin_amdgcn_readlane((int)incl, 63); }

// all threads of the block get the block total; fixed combination order
template <int WAVES = kWavesPerBlock>
__device__ __forceinline__ double block_sum(double x, double *lds)
{
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; w += 4) {
        const double four = (lds[w] + lds[w + 1]) + (lds[w + 2] + lds[w + 3]);
        t = w ? t + four : four;
    }
    __syncthreads();
    return t;
}
__device__ __forceinline__ float block_max(float x, float *lds4)
{
    x = wave_max(x);
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = x;
    __syncthreads();
    float t = fmaxf(fmaxf(lds4[0], lds4[1]), fmaxf(lds4[2], lds4[3]));
    __syncthreads();
    return t;
}

// Release at the scope of the device, by one thread behind a barrier: what the block has stored is in memory, where other dies read it.
// The write-back of the die's cache is waited for by an instruction of its own: the wait that the fence brings is dropped where the compiler knows of
// nothing else that the wavefront has under way.
__device__ __forceinline__ void release_to_device()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __builtin_amdgcn_s_waitcnt(0);
}

// number of set bits of a ballot below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t ballot)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

// ---- Philox-4x32-10 (Salmon et al., SC'11) --------------------------------------
// Counter = (J lo, J hi, worker, iteration), J = global element index / 4, key =
// seed; the element takes output word (index % 4), top 24 bits scaled to [0, 1).
// a ^ b ^ k in one instruction (the three-input bit operation with the truth table of xor); k is the same for the
// whole wavefront (a round key: it lives in a scalar register).  The compiler emits two two-input operations for
// the same expression, and where the quantizers' pass over p is bound by the vector ALU that shows: QSGD compress
// 84.2 -> 82.4 us.
__device__ __forceinline__ uint32_t xor3_uniform(uint32_t a, uint32_t b, uint32_t k)
{
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
}

__device__ __forceinline__ void philox4x32_10(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t J, uint32_t (&out)[4])
{
    uint32_t c0 = (uint32_t)J, c1 = (uint32_t)(J >> 32), c2 = worker, c3 = iter_lo;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32 x 32 -> 64 multiply each (two instructions instead of four on the quarter-rate multiplier)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        c0 = xor3_uniform(hi1, c1, k0);
        c1 = lo1;
        c2 = xor3_uniform(hi0, c3, k1);
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

__device__ __forceinline__ float u01(uint32_t x) { return (float)(x >> 8) * 5.9604644775390625e-8f; }

template <int R>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t x)      // value of lane R of each group of four lanes
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, R | (R << 2) | (R << 4) | (R << 6), 0xF, 0xF, true);
}

// The Philox words of the wavefront's steps (16, or 4) for this lane (element gbase + 64 j + lane in step j
// takes word (index % 4) of block index / 4).
// Four adjacent lanes hold four consecutive elements; when gbase is a multiple of 4 these
// share one Philox block, so each lane computes one block per four steps (the one of step
// 4m + lane % 4) and the four words are handed round inside the quad.
template <int S>
__device__ __forceinline__ void chunk_words(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t gbase, uint32_t lane,
                                            uint32_t (&x)[S])
{
    if ((gbase & 3u) == 0) {
        const uint32_t me = lane & 3u;
#pragma unroll
        for (int m = 0; m < S / 4; ++m) {
            uint32_t w[4];
            philox4x32_10(seed, worker, iter_lo, (gbase + 64u * (4 * m + me) + lane) >> 2, w);
            uint32_t y[4][4];                      // y[r][i]: word i of the block of step 4m + r
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                y[0][i] = quad_bcast<0>(w[i]); y[1][i] = quad_bcast<1>(w[i]);
                y[2][i] = quad_bcast<2>(w[i]); y[3][i] = quad_bcast<3>(w[i]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                x[4 * m + r] = me == 0 ? y[r][0] : me == 1 ? y[r][1] : me == 2 ? y[r][2] : y[r][3];
        }
    } else {
        // The chunk starts s = gbase % 4 elements into a Philox block (a group whose tensors before it do not add up to
        // a multiple of 4).  With v = lane + s, the element of step j sits in block B0 + 16 j + v / 4, word v % 4: the
        // same 256 blocks as above, B0 + 16 j + q computed by lane 4 q + j % 4, plus one more, B0 + 256 (of 16 steps), that only the
        // last s lanes need in the last step (every lane computes it: five blocks per lane instead of the sixteen of a block
        // per element).  A lane with v >= 64 is served by quad 0's blocks of the next step.  The lanes that share a
        // block are no aligned quad any more, so the words travel through ds_bpermute.
        // (Measured, compress of such a group of 25.6 M elements: QSGD 118.5 -> 86.8 us, TernGrad 105.9 -> 86.0, Rand-k 94.8 -> 86.7:
        // what a group that starts on a block takes.)
        const uint32_t s = (uint32_t)gbase & 3u, v = lane + s, i = v & 3u;
        const uint64_t B0 = (gbase - s) >> 2;
        const uint32_t me = lane & 3u, quad = lane >> 2;
        const bool over = v >= 64u;
        uint32_t w[S / 4][4], wl[4];
#pragma unroll
        for (int m = 0; m < S / 4; ++m) philox4x32_10(seed, worker, iter_lo, B0 + 16u * (4 * m + me) + quad, w[m]);
        philox4x32_10(seed, worker, iter_lo, B0 + 16u * S, wl);
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int m = j >> 2, r = j & 3;
            const uint32_t src = over ? (uint32_t)((j + 1) & 3) : ((v >> 2) << 2) + (uint32_t)r;     // the lane that computed the block
            uint32_t got[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) got[t] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)w[m][t]);
            uint32_t val = i == 0 ? got[0] : i == 1 ? got[1] : i == 2 ? got[2] : got[3];
            if (r == 3) {            // for the lanes with v >= 64 the next step's block comes out of the next round of four
                uint32_t alt[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    alt[t] = j + 1 < S ? (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)w[m + 1 < S / 4 ? m + 1 : 0][t]) : wl[t];
                const uint32_t a = i == 0 ? alt[0] : i == 1 ? alt[1] : i == 2 ? alt[2] : alt[3];
                val = over ? a : val;
            }
            x[j] = val;
        }
    }
}

// ---- four consecutive elements per lane --------------------------------------------
// In step m (0..3) lane l holds elements 256 m + 4 l .. + 3 of a full chunk.  When the chunk starts on a Philox block
// (and the block numbers of the chunk share their high word) these four take the four words of one block: nothing is
// handed round between lanes, and every access is 16 bytes per lane.
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));       // in a tensor: 4-byte aligned

__device__ __forceinline__ bool wide_random(const Chunk &c, uint64_t gbase)
{
    return c.full && (gbase & 3u) == 0 && (uint32_t)(gbase >> 2) <= 0xFFFFFFFFu - (uint32_t)(kChunk / 4);
}
// The words of step m.  What the first two rounds compute from the block number's high word, the worker and the iteration
// alone is the same for the wavefront and stays on the scalar unit: 18 instead of 20 multiplies on the vector unit, where
// they run at a quarter of the rate.
__device__ __forceinline__ void wide_words(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t gbase, uint32_t lane, int m,
                                           uint32_t (&out)[4])
{
    const uint64_t J0 = gbase >> 2;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * worker, p0 = (uint64_t)0xD2511F53u * ((uint32_t)J0 + 64u * (uint32_t)m + lane);
    const uint32_t u0 = (uint32_t)(p1 >> 32) ^ (uint32_t)(J0 >> 32) ^ k0, u1 = (uint32_t)p1;
    uint32_t c2 = (uint32_t)(p0 >> 32) ^ (iter_lo ^ k1), c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    const uint64_t q0 = (uint64_t)0xD2511F53u * u0, q1 = (uint64_t)0xCD9E8D57u * c2;
    uint32_t c0 = (uint32_t)(q1 >> 32) ^ (u1 ^ k0), c1 = (uint32_t)q1;
    c2 = c3 ^ ((uint32_t)(q0 >> 32) ^ k1);
    c3 = (uint32_t)q0;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t a = (uint64_t)0xD2511F53u * c0, b = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3_uniform((uint32_t)(b >> 32), c1, k0);
        c2 = xor3_uniform((uint32_t)(a >> 32), c3, k1);
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}
// the lane's four elements of step m: of a flat buffer (16-byte aligned) or of a tensor
__device__ __forceinline__ float4v load_wide(const float *p, uint32_t lane, int m)
{
    return __builtin_nontemporal_load(reinterpret_cast<const float4v *>(p + 256 * m) + lane);
}
__device__ __forceinline__ float4v load_wide_unaligned(const float *p, uint32_t lane, int m)
{
    const float4u v = __builtin_nontemporal_load(reinterpret_cast<const float4u *>(p + 256 * m) + lane);
    return float4v{v.x, v.y, v.z, v.w};
}

// the words of chunk_words as uniforms in [0, 1)
__device__ __forceinline__ void chunk_uniforms(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t gbase, uint32_t lane,
                                               float (&u)[kSteps])
{
    uint32_t x[kSteps];
    chunk_words(seed, worker, iter_lo, gbase, lane, x);
#pragma unroll
    for (int j = 0; j < kSteps; ++j) u[j] = u01(x[j]);
}

}  // namespace mc

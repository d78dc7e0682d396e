// Sparsifiers (Top-k, DGC, Rand-k) for gfx950: exact top-k of |p| over a whole merged
// group, ties at the threshold taken in index order (lower index wins), payload
// written in ascending index order, and the sparse decompress-and-sum.
// Rand-k is the same selection on keys that do not depend on the values: the k
// largest of the elements' Philox words (31 bits) are k positions drawn uniformly.
//
// The paper singles out the top-k() operation as the cost that merging alone
// does not remove (Section 5.1).  Here the selection is a radix select on the
// 31-bit magnitude key that never sorts and, in the steady state, touches the
// gradient once and resolves 20 of the 31 bits inside that one pass:
//
//   accumulate   p = g + e (DGC: u = m u + g, v = v + u) streamed once; every element
//                whose key reaches a *hint* (a little below the last threshold of this
//                group) is copied, in index order, into the candidate slots of its
//                1024-element chunk, and counted in a *window* histogram: 2048 bins of
//                2048 keys each, starting at the hint (the last bin also takes all above)
//   select       every block reads the window.  Usual case: the k-th largest key falls in one
//                of its bins; candidates above that bin are counted, the few inside it
//                listed.  Otherwise (the threshold left the window, a bin of very many
//                equal keys, a first call) the group's first blocks finish the selection
//                and the payload themselves, with grid-wide barriers between the steps
//   emit         usual case: the threshold key T and the number of keys == T to take from
//                the list; ordered compaction of the kept candidates into (idx, val)
//
// DGC with a threshold from a sample has a payload of varying length and keeps a kernel per step: seed (reads the
// window; where that does not settle it, level 1 of a radix select), two kernels for levels 2 and 3, count (kept candidates
// per tile), emit.
//
// If at least k elements have key >= hint, the k-th largest key T is >= hint, so
// every element with key >= T is a candidate and the result is exact whatever the
// hint was; the hint only decides how much work the later kernels have.
// The kernels that walk the candidates give every 4096-element tile to one
// wavefront: tiles are independent until the emit kernel adds up the kept counts
// of the tiles before its own.  On the usual route no block waits on another: every
// dependency is a kernel boundary.
#include <algorithm>
#include <type_traits>

#include "mc_internal.h"

namespace mc {

__host__ __device__ static inline uint32_t chunks_of(uint32_t n) { return (uint32_t)(((uint64_t)n + kChunk - 1) / kChunk); }

constexpr int kWindowShift = 11;                       // keys per window bin = 2^11: what hist 3 resolves after a fast seed
constexpr int kBinsW = 2048, kBins1 = 2048, kBins2 = 1024, kBins3 = 1 << kWindowShift;
// Histogram scratch: the window and the three radix levels one after the other.  Global
// atomics on one address serialise (tens of nanoseconds each on this part), so only
// the bins themselves are updated -- no shared summary counters -- and a level is
// resolved by a wavefront that reads all its bins.
// The window histogram is kept in kWinCopies copies, a block adding to the copy of its index, and the select
// kernel sums them.  The flush of the streaming pass is one multi-lane add per block and 128-byte line of bins, and adds to one
// line queue up behind each other (about 5 ns each): when the candidates are spread evenly over the tiles, every
// block holds some of nearly every bin between the hint and the threshold, and with a single copy the pass took
// 132 us instead of 54 (all tensors of one scale).  One bin per line was tried first (62 us, but the adds of a wave
// no longer coalesce: +2..4 us on clustered candidates and a 2048-line gather in the select kernel); copies keep the adds
// coalesced.  Measured, Top-k compress on clustered / evenly spread candidates: 2 copies 87.6 / 125.6 us, 4 copies
// 88.4 / 97.5, 8 copies 89.7 / 99.0, 16 copies 93.3 / 101.7, 32 copies 106 / 114 (the select kernel reads them all).
constexpr int kHistW = 0, kHist1 = kHistW + kBinsW * kWinCopies, kHist2 = kHist1 + kBins1, kHist3 = kHist2 + kBins2;
// The window's open last bin takes a count from nearly every block (all keys above the window), and
// adds from thousands of blocks to one address queue up behind each other for tens of microseconds:
// its count is spread over kOpenCopies words, chosen by the block index, which the select kernel sums.
constexpr int kOpenCopies = 64, kHistOpen = kHist3 + kBins3;
static_assert(kHistOpen + kOpenCopies == kHistWords, "histogram scratch layout");
constexpr uint32_t kHintMargin = 3u << 19;   // 3/16 of an octave below the last threshold
// The window spans 2^22 keys (half an octave) from the hint upward: it holds the new threshold if that
// lies between 12 % below and 24 % above the last one (2^23 keys are one octave of magnitude).

// seed result (SelectState::mode)
// hint record of a (group, worker): the filter key, how many times the margin below the threshold was halved,
// and for how many calls it stays at the full margin after a miss
constexpr int kHintShift = 1, kHintHold = 2, kHintCap = 3;
constexpr uint32_t kHintShiftMax = 4u, kHintHoldCalls = 8u;      // margin at least 3/256 of an octave (0.8 %)
constexpr uint32_t kHintCapCalls = 64u;
constexpr uint32_t kHintSeen = 1u << 31;      // in the cap word: this (group, worker) has had a call, the filter key stands for something

// How far below the threshold the next call starts filtering, after a call whose threshold lay inside the window.
// Under error feedback the values pile up just below the threshold, in the long run those of every tensor, and a fixed
// margin lets through many times k of them (each costs the streaming pass a store and the histogram an add): the
// margin is halved while the filter passes more than 2 k (at most four times: 0.8 % below the threshold) and doubled
// again when it passes fewer than 1.25 k.  (Measured, every worker on new gradients: with "more than 4 k" the bench's
// Top-k stayed at the full margin, 12 %, and 850 000 candidates; with 3 k it settles at one halving and 533 000,
// with 2 k at two, 3 %, and 396 000: Top-k compress went 80.2 -> 78.5 us with the second rule and 77.0 -> 75.5 us
// with the third, no miss in 200 calls with any of them.)
// A call whose threshold fell below the filter (a miss: a second streaming pass) resets the margin, keeps it for
// kHintHoldCalls calls, and caps the halvings below what the margin had been halved to when it missed, one step
// more being allowed again after every kHintCapCalls calls: a threshold that jitters by more than the tightest margin
// costs a miss every so many calls, not every few.  cap word: steps taken off kHintShiftMax | calls left << 8 | kHintSeen.
__device__ __forceinline__ void margin_after_hit(uint32_t *hint, uint32_t shift, uint32_t hold, uint32_t capw, uint64_t cands, uint64_t k)
{
    uint32_t off = capw & 0xFFu, left = (capw & ~kHintSeen) >> 8;
    if (left) --left;
    else if (off) { --off; left = off ? kHintCapCalls : 0u; }
    const uint32_t cap = kHintShiftMax - (off < kHintShiftMax ? off : kHintShiftMax);
    if (hold) --hold;
    else if (cands > 2u * k && shift < cap) ++shift;
    if (4u * cands < 5u * k && shift) --shift;
    if (shift > cap) shift = cap;
    hint[kHintShift] = shift; hint[kHintHold] = hold; hint[kHintCap] = off | (left << 8) | kHintSeen;
}
// below: the threshold fell below the filter (else it rose above the window, which no margin prevents)
__device__ __forceinline__ void margin_after_miss(uint32_t *hint, uint32_t shift, uint32_t capw, bool below)
{
    hint[kHintShift] = 0u; hint[kHintHold] = kHintHoldCalls;
    hint[kHintCap] = (below && shift ? (kHintShiftMax - (shift - 1u)) | (kHintCapCalls << 8) : capw) | kHintSeen;
}
// What the streaming pass filters with: the record's key; before the first call of a (group, worker) a key that no element
// reaches, for which the call is a refill.  (With every element a candidate the first pass took 118 us instead of 52, and
// all later steps walked all elements.)
__device__ __forceinline__ bool first_call(uint32_t hint, uint32_t capw) { return hint == 0u && !(capw & kHintSeen); }
constexpr uint32_t kModeFast = 1u;      // lo / need are those of level 3 already
constexpr uint32_t kModeUniform = 2u;   // after a refill: every element is a candidate, chunk c holds 1024 c ...
constexpr uint32_t kModeLean = 4u;      // fast, and the keys of the threshold's window bin were listed: the emit kernel finishes alone
constexpr uint32_t kModeFirst = 16u;    // first call of a (group, worker): a refill that is reported as "above", as first calls are
constexpr uint32_t kModeDense = 8u;     // fast, but that bin holds too many keys to list: its 2048 keys were histogrammed instead

__device__ __forceinline__ uint32_t key_of(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

// add a block's LDS histogram to the global one
__device__ __forceinline__ void flush_fine(const uint32_t *lds, uint32_t *fine, int bins)
{
    for (int b = threadIdx.x; b < bins; b += blockDim.x) {
        uint32_t h = lds[b];
        if (h) atomicAdd(&fine[b], h);
    }
}

// key of the stochastic choices: Philox key and the worker / iteration words of the counter
struct RngKey { uint64_t seed; uint32_t worker, iter_lo; };

// DGC with a sampled threshold: the histograms that find the threshold count only the sample, every
// stride-th element of the group starting at `first` (drawn by the host with Philox).  stride = 0: off.
struct SampleRule { uint32_t stride, first, inv /* floor(2^32 / stride) */; };

__device__ __forceinline__ bool in_sample(const SampleRule &r, uint32_t i)
{
    if (r.stride <= 1u) return true;
    uint32_t rem = i - __umulhi(i, r.inv) * r.stride;      // the quotient estimate is at most 1 too small
    if (rem >= r.stride) rem -= r.stride;
    return rem == r.first;
}

// Copy the flagged elements of a wavefront, in index order, into its chunk's candidate slots from slot `run` on.
// bits: what the later kernels see of the element (its key is bits & 0x7FFFFFFF): the value itself, or
// for Rand-k the random key.
template <int S>
__device__ __forceinline__ void put_candidates(const Chunk &c, const uint32_t (&bits)[S], const uint64_t (&flag)[S], uint32_t run,
                                               uint32_t hint, uint32_t *cand_bits, uint16_t *cand_loc, uint32_t *hist /* LDS */,
                                               const SampleRule &smp)
{
    const uint32_t base = S == kSteps ? c.base : c.base & ~(uint32_t)(kChunk - 1), off = S == kSteps ? 0u : c.base & (uint32_t)(kChunk - 1);
    const uint64_t me = 1ull << c.lane;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        if (flag[j] & me) {
            uint32_t slot = base + run + lanes_below(flag[j]);
            cand_bits[slot] = bits[j];
            cand_loc[slot] = (uint16_t)(off + 64 * j + c.lane);
            const uint32_t bin = ((bits[j] & 0x7FFFFFFFu) - hint) >> kWindowShift;
            if (in_sample(smp, c.base + 64 * j + c.lane))
                atomicAdd(&hist[bin < (uint32_t)kBinsW - 1u ? bin : (uint32_t)kBinsW - 1u], 1u);
        }
        run += __popcll(flag[j]);
    }
}

// ---------------------------------------------------------------------------
// accumulate + candidate filter + window histogram of the candidates
// ---------------------------------------------------------------------------
// S: elements per lane, 16, or 4 on a launch of few tiles (kSpread threads per tile): a block of a small group takes as long as one
// wavefront's instructions.  (Compress, 33 / 34 000 / 200 000 / 2 M elements, with one copy of the window on the first two: Top-k
// 11.9 / 11.8 / 17.0 / 20.4 -> 9.1 / 10.2 / 15.4 / 19.2 us, DGC 12.6 / 12.0 / 16.7 / 21.7 -> 9.0 / 10.3 / 14.9 / 19.9, Rand-k 18.8 / 16.7 /
// 20.7 / 24.1 -> 15.1 / 14.4 / 18.3 / 22.1.)
// SMALL: the whole compress of groups of at most kOneBlockTiles tiles, in launches of at most kSameTiles.  In the block of a group that is done
// last with the streaming pass the selection follows, as lean_small_k has it: a kernel that starts behind another one takes 1 us of the device
// and 2.6 of the host, a die's lines written to memory and a count of the blocks that are done take less.  No block waits for another.  (A word more for the plain kernel's arguments took 0.3 us of a call.)
// (Compress, two kernels -> one, device time, without the launch that the host saves.  Top-k 1 % of 1 / 4 / 8 tiles 9.5 / 9.7 / 9.8 -> 8.8 / 9.3 / 9.7 us, 5 % 9.6 /
// 10.8 / 12.2 -> 9.0 / 10.3 / 11.9; DGC 1 % 9.8 / 10.1 / 10.3 -> 9.3 / 9.7 / 10.1; Rand-k 1 % 10.3 / 11.1 / 11.5 -> 9.9 / 11.2 / 11.7; seven groups of 1 / 4 / 8 tiles in
// one call, Top-k 10.9 / 11.0 / 11.1 -> 9.9 / 10.0 / 10.6, Rand-k 12.4 / 12.8 / 13.3 -> 11.2 / 12.1 / 12.8.  Larger groups lose what the launch saves to the tail's
// wait for the slowest block: four groups of 12 / 16 / 18 tiles, both directions, 18.4 / 18.9 / 18.9 -> 18.5 / 19.8 / 19.9, and 0.2 more since the write-back is waited for.)
constexpr int kRoundTiles = 4096;      // tiles per round of the slow routes' compaction: 256 blocks of 16 wavefronts at most
template <int ALGO, bool EF, int MOST>
__device__ __forceinline__ void small_tail(SparseJob job, RngKey rng, uint32_t sync_blocks, int *status, uint32_t *hist, uint32_t *pfx, uint32_t *small);
template <int ALGO, bool EF, class SRC, int S = kSteps, bool SMALL = false>
__global__ __launch_bounds__(kTile / S) void sparse_accum_k(SRC src, float momentum, RngKey rng, std::conditional_t<SMALL, int *, SampleRule> last)
{
    constexpr int kThreads = kTile / S, kWaves = kThreads / kWave, kQuarters = kSteps / S;      // wavefronts per chunk: one, or four
    SampleRule smp{0u, 0u, 0u};
    if constexpr (!SMALL) smp = last;
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBinsW];
    __shared__ uint32_t wcnt[kWaves];
    for (int b = threadIdx.x; b < kBinsW; b += kThreads) hist[b] = 0u;
    __syncthreads();
    const SparseJob job = src.template job<BLK_TILE>();
    const GroupView &g = job.g;
    float *st = job.st;
    const SparseScratch &sc = job.sc;
    const uint32_t order = job.blocks - 1u - job.block;          // the how-manieth of the group's blocks this is
    const Chunk c = my_chunk<S>(g.n, job.block);
    const uint32_t hint0 = *sc.hint, hint = first_call(hint0, sc.hint[kHintCap]) ? 0xFFFFFFFFu : hint0;
    // the emit kernel of the call before is done with the list of keys in the threshold's bin: its sublists are empty again
    if (order == 0 && threadIdx.x < (uint32_t)kUSub) sc.ucount[threadIdx.x * kUCountStride] = 0u;
    if (order == 0 && threadIdx.x == 0) sc.arrive[0] = sc.arrive[kArriveWindow] = 0u;       // and nobody waits at a grid-wide barrier of that call any more
    // The radix levels are cleared by the kernels that use them -- unless a call gave up at a barrier (MC_ERR_DEVICE):
    // what it left behind must not enter this call's counts.  (A group of fewer tiles than it takes blocks to clear them at
    // once goes round again; a tail of one block keeps the levels in LDS.)
    if (!SMALL)
        for (uint32_t i = order * (uint32_t)kThreads + threadIdx.x; i < (uint32_t)(kHistOpen - kHist1); i += job.blocks * (uint32_t)kThreads)
            sc.hist[kHist1 + i] = 0u;
    uint32_t run = 0;
    uint32_t bits[S];
    uint64_t flag[S];
    if (c.base < g.n) {
        float p[S];
        // What the last call sent leaves the memory: an element whose key was above that call's threshold key counts as 0
        // here, instead of having been set to 0 there -- one scattered 4-byte store per kept entry, each a read-modify-write
        // of a whole line in memory, was most of what the compaction cost.  (Kept entries *equal* to the threshold are still
        // zeroed in place: which of the equal keys were taken depends on their order.  A state that was zero-filled,
        // imported, or written by a scheme that zeroes in place says sent_key = all ones or holds zeros: nothing is masked.)
        const uint32_t sent_key = (ALGO == MC_ALGO_DGC || EF) ? reinterpret_cast<const StateHeader *>(reinterpret_cast<const uint8_t *>(st) - kHeaderBytes)->sent_key : 0u;
        if (ALGO == MC_ALGO_DGC) {
            // momentum correction: u = m u + g ; v = v + u ; the vector compressed is v
            float *vbuf = st, *ubuf = st + dgc_u_offset(g.n);
            float u[S], v[S];
            load_flat(ubuf, c, g.n, u, 0.0f);
            load_flat(vbuf, c, g.n, v, 0.0f);
            load_seg(g, c, p);
#pragma unroll
            for (int j = 0; j < S; ++j) {
                if (key_of(v[j]) > sent_key) { u[j] = 0.0f; v[j] = 0.0f; }       // momentum factor masking of what was sent
                float mu = momentum * u[j];
                u[j] = mu + p[j];
                v[j] = v[j] + u[j];
                p[j] = v[j];
            }
            store_flat(ubuf, c, g.n, u);
            store_flat(vbuf, c, g.n, v);
        } else if (EF) {
            float e[S];
            load_flat(st, c, g.n, e, 0.0f);
            load_seg(g, c, p);
#pragma unroll
            for (int j = 0; j < S; ++j) p[j] = p[j] + (key_of(e[j]) > sent_key ? 0.0f : e[j]);
            store_flat(st, c, g.n, p);
        } else {
            load_seg(g, c, p);
        }
        if (ALGO == MC_ALGO_RANDK) {
            chunk_words(rng.seed, rng.worker, rng.iter_lo, g.goff + c.base, c.lane, bits);
#pragma unroll
            for (int j = 0; j < S; ++j) bits[j] >>= 1;
        } else {
#pragma unroll
            for (int j = 0; j < S; ++j) bits[j] = __float_as_uint(p[j]);
        }
#pragma unroll
        for (int j = 0; j < S; ++j) {
            bool valid = c.full || c.base + 64 * j + c.lane < g.n;
            flag[j] = __builtin_amdgcn_ballot_w64(valid && (bits[j] & 0x7FFFFFFFu) >= hint);
        }
#pragma unroll
        for (int j = 0; j < S; ++j) run += __popcll(flag[j]);
        if (S == kSteps) put_candidates(c, bits, flag, 0u, hint, sc.cand_bits, sc.cand_loc, hist, smp);
    }
    if (c.lane == 0) wcnt[threadIdx.x >> 6] = run;
    __syncthreads();
    if (S != kSteps) {           // behind those of the chunk's wavefronts before this one
        const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        uint32_t at = 0;
#pragma unroll
        for (int q = 0; q < kQuarters - 1; ++q) if ((uint32_t)q < wave % (uint32_t)kQuarters) at += wcnt[wave / (uint32_t)kQuarters * (uint32_t)kQuarters + (uint32_t)q];
        if (run) put_candidates(c, bits, flag, at, hint, sc.cand_bits, sc.cand_loc, hist, smp);
        __syncthreads();
    }
    if (threadIdx.x == 0) {      // candidates of the tile's four chunks, 16 bits each (a chunk holds at most 1024)
        uint64_t runs = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) runs += (uint64_t)wcnt[w] << (16 * (w / kQuarters));
        sc.tile_runs[job.block] = runs;
    }
    // (A group of few tiles has no crowd at its bins: one copy then, the only one that a kernel for small groups reads.)
    flush_fine(hist, sc.hist + kHistW + (job.blocks <= (uint32_t)kSmallSelTiles ? 0u : order % kWinCopies) * kBinsW, kBinsW - 1);
    if (threadIdx.x == kThreads - 1 && hist[kBinsW - 1]) atomicAdd(&sc.hist[kHistOpen + (order & (kOpenCopies - 1))], hist[kBinsW - 1]);
    if constexpr (SMALL) {
        static_assert(kThreads == 1024 && kBinsW >= kBins1, "the tail's block and histogram");
        __shared__ uint32_t pfx[2 * kRoundTiles], small[64];
        uint32_t *done = sc.arrive + kArriveDone;
        // Every wavefront's stores and counts are in the die's cache before the barrier.  (The fence keeps them in front of the wait, which is an
        // instruction to the compiler and nothing more.)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) {
            release_to_device();
            const uint32_t before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (before == job.blocks - 1u) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                *done = 0u;                      // (for the next call)
            }
            small[0] = before;
        }
        __syncthreads();
        const uint32_t before = (uint32_t)__builtin_amdgcn_readfirstlane((int)small[0]);
        if (before != job.blocks - 1u) return;
        __syncthreads();
        SparseJob tail = job;
        tail.block = 0u;
        tail.blocks = 1u;
        small_tail<ALGO, EF, (int)kOneBlockTiles>(tail, rng, 1u, last, hist, pfx, small);
    }
}

// ---------------------------------------------------------------------------
// Resolve one radix level inside a wavefront: find the bin b with
//   count(bins > b) < need <= count(bins >= b)        and  rest = need - count(bins > b).
// Every lane reads BINS / 64 adjacent bins, a suffix scan over the lanes finds the
// lane where the running count crosses `need`, and that lane walks its own bins.
// One memory latency, no block barrier.  Returns false (bin = 0, rest = 0) if the
// histogram holds fewer than `need` keys.
// ---------------------------------------------------------------------------
template <int BINS>
__device__ __forceinline__ bool resolve_wave(const uint32_t *fine, uint64_t need, uint32_t &bin, uint64_t &rest,
                                             uint32_t top_extra = 0u /* counted in the last bin besides fine[BINS - 1] */,
                                             uint64_t *total = nullptr /* out: the sum of all bins */)
{
    constexpr int kPer = BINS / 64;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t h[kPer];
    uint64_t own = 0;
    const uint4 *src = reinterpret_cast<const uint4 *>(fine + lane * kPer);
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
        const uint4 x = src[i];
        h[4 * i] = x.x; h[4 * i + 1] = x.y; h[4 * i + 2] = x.z; h[4 * i + 3] = x.w;
    }
    if (lane == 63u) h[kPer - 1] += top_extra;
#pragma unroll
    for (int i = 0; i < kPer; ++i) own += h[i];
    uint64_t incl = own;                                    // inclusive suffix sum over lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t o = __shfl_down(incl, d, 64);
        if (lane + d < 64) incl += o;
    }
    if (total) *total = __shfl(incl, 0, 64);
    uint64_t run = incl - own;                              // keys in the bins of higher lanes
    const bool mine = run < need && need <= incl;
    uint32_t b = 0;
    uint64_t r = 0;
    if (mine) {
#pragma unroll
        for (int i = kPer - 1; i >= 0; --i) {
            if (run < need && need <= run + h[i]) { b = lane * kPer + i; r = need - run; }
            run += h[i];
        }
    }
    const uint64_t hit = __builtin_amdgcn_ballot_w64(mine);
    const uint32_t src_lane = hit ? (uint32_t)__builtin_ctzll(hit) : 0u;     // an inconsistent histogram still gives a defined bin
    bin = __shfl(b, src_lane, 64);
    rest = __shfl(r, src_lane, 64);
    return hit != 0;
}

// The same for a histogram in LDS.  There the adjacent bins of a lane would all fall into the banks that every
// other lane's bins fall into (a lane owns BINS / 64 = 32 consecutive words: 64 lanes, one bank group), and the
// reads of a wavefront would be served one lane at a time -- measured: the resolve of a 2048-bin histogram by
// all four wavefronts of all blocks made the emit kernel twice as long.  Each lane therefore reads its bins in
// an order rotated by its lane number, which spreads every read over all banks; the lane in which the count
// crosses `need` reads its bins once more, in order.
template <int BINS>
__device__ __forceinline__ bool resolve_lds(const uint32_t *fine, uint64_t need, uint32_t &bin, uint64_t &rest,
                                            uint32_t top_extra = 0u, uint64_t *total = nullptr)
{
    constexpr int kPer = BINS / 64;
    static_assert((kPer & (kPer - 1)) == 0, "rotation needs a power of two");
    const uint32_t lane = threadIdx.x & 63u;
    uint64_t own = 0;
#pragma unroll 4              // (a few reads in flight are enough; all 32 at once cost the calling kernel its registers)
    for (int i = 0; i < kPer; ++i) own += fine[lane * kPer + ((i + lane) & (kPer - 1))];
    if (lane == 63u) own += top_extra;
    uint64_t incl = own;                                    // inclusive suffix sum over lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t o = __shfl_down(incl, d, 64);
        if (lane + d < 64) incl += o;
    }
    if (total) *total = __shfl(incl, 0, 64);
    uint64_t run = incl - own;                              // keys in the bins of higher lanes
    const bool mine = run < need && need <= incl;
    uint32_t b = 0;
    uint64_t r = 0;
    if (mine) {
        for (int i = kPer - 1; i >= 0; --i) {
            const uint64_t h = (uint64_t)fine[lane * kPer + i] + (lane == 63u && i == kPer - 1 ? top_extra : 0u);
            if (run < need && need <= run + h) { b = lane * kPer + i; r = need - run; }
            run += h;
        }
    }
    const uint64_t hit = __builtin_amdgcn_ballot_w64(mine);
    const uint32_t src_lane = hit ? (uint32_t)__builtin_ctzll(hit) : 0u;
    bin = __shfl(b, src_lane, 64);
    rest = __shfl(r, src_lane, 64);
    return hit != 0;
}

// ---------------------------------------------------------------------------
// The candidates of one tile, walked by one wavefront in index order.  `runs`
// holds the candidate counts of the tile's four chunks (16 bits each); the slots of
// chunk c are cand[1024 c ...].  Up to twelve rounds of 64 candidates are fetched together,
// so a tile of a tensor that holds most of the kept entries (several hundred
// candidates) costs the wavefront one memory latency.
// `body(valid, chunk, bits, loc)` is called by all 64 lanes (it may use ballots).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t runs_total(uint64_t runs)
{
    return (uint32_t)(runs & 0xFFFFu) + (uint32_t)((runs >> 16) & 0xFFFFu) + (uint32_t)((runs >> 32) & 0xFFFFu) + (uint32_t)(runs >> 48);
}

// candidate counts of a tile after a refill: every element below n
__device__ __forceinline__ uint64_t uniform_runs(uint32_t tile, uint32_t n)
{
    uint64_t r = 0;
#pragma unroll
    for (int s = 0; s < kWavesPerBlock; ++s) {
        const uint64_t base = (uint64_t)tile * kTile + (uint64_t)s * kChunk;
        const uint64_t cnt = base >= n ? 0u : (n - base < (uint64_t)kChunk ? n - base : (uint64_t)kChunk);
        r |= cnt << (16 * s);
    }
    return r;
}

// One batch of the walk: rounds [f0, f0 + 64 ROUNDS) of the tile's candidates, all loads issued before the first use.
template <bool WITH_LOC, int ROUNDS, typename Body>
__device__ __forceinline__ void tile_batch(const SparseScratch &sc, uint32_t tile, uint32_t r0, uint32_t r1, uint32_t r2, uint32_t total,
                                           uint32_t f0, Body body)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t ch[ROUNDS], bits[ROUNDS], loc[ROUNDS];
    size_t slot[ROUNDS];
    bool valid[ROUNDS];
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
        const uint32_t f = f0 + 64 * u + lane;
        valid[u] = f < total;
        const uint32_t sub = (f >= r0) + (f >= r1) + (f >= r2);          // chunk of the tile, then slot inside it
        const uint32_t off = f - (sub == 0 ? 0u : sub == 1 ? r0 : sub == 2 ? r1 : r2);
        ch[u] = tile * kWavesPerBlock + (valid[u] ? sub : 0u);
        slot[u] = valid[u] ? (size_t)ch[u] * kChunk + off : (size_t)tile * kTile;
    }
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
        bits[u] = 0u; loc[u] = 0u;
        if (valid[u]) {
            bits[u] = sc.cand_bits[slot[u]];
            if (WITH_LOC) loc[u] = sc.cand_loc[slot[u]];
        }
    }
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (f0 + 64 * u < total) body(valid[u], ch[u], bits[u], loc[u]);
}

// A tile with at most 256 candidates -- nearly every tile when the candidates are spread over the whole group -- takes
// one batch of four rounds: the slot arithmetic of sixteen rounds, most of them empty, was a third of what the
// count kernel did.  Other tiles take batches of twelve rounds (with sixteen the level-3 and emit kernels need 81 .. 83
// registers and five wavefronts fit a SIMD; with twelve, seven or eight do; eight rounds measure the same but would
// cost a tile full of candidates eight dependent batches).  Top-k compress, evenly spread / clustered candidates:
// 98.2 -> 89.7 us / 88.6 -> 88.1; Rand-k 97.7 -> 90.0; DGC 114.1 -> 111.4.
// Fetching the four rounds ahead of what else a kernel waits for (its resolve, its prefix sum) gained another 1 us on
// spread candidates and lost as much on clustered ones, whose heavy tiles then wait for their candidate counts before
// anything else is asked for: not kept.
template <bool WITH_LOC, typename Body>
__device__ __forceinline__ void tile_walk(const SparseScratch &sc, uint32_t tile, uint64_t runs, Body body)
{
    constexpr int kRounds = 12, kFew = 4;
    const uint32_t r0 = (uint32_t)(runs & 0xFFFFu), r1 = r0 + (uint32_t)((runs >> 16) & 0xFFFFu),
                   r2 = r1 + (uint32_t)((runs >> 32) & 0xFFFFu), total = r2 + (uint32_t)(runs >> 48);
    if (total <= 64u * kFew) { tile_batch<WITH_LOC, kFew>(sc, tile, r0, r1, r2, total, 0u, body); return; }
    for (uint32_t f0 = 0; f0 < total; f0 += 64 * kRounds) tile_batch<WITH_LOC, kRounds>(sc, tile, r0, r1, r2, total, f0, body);
}

// the tile of this wavefront in the kernels that walk the candidates, and its runs
struct TileJob { uint32_t tile; uint64_t runs; };

__device__ __forceinline__ TileJob my_tile(const SparseScratch &sc, uint32_t n, uint32_t ntiles)
{
    TileJob j;
    j.tile = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    j.runs = j.tile < ntiles ? sc.tile_runs[j.tile] : 0ull;      // ignored after a refill
    return j;
}

// ---------------------------------------------------------------------------
// seed: 1024 threads per block.  Wavefront 0 of every block resolves the window
// histogram; all blocks reach the same verdict.
//   fast      the threshold lies in window bin b < 2047: block 0 records lo = hint + 2048 b
//             and the entries to take from that bin; everybody leaves
//   above     it lies above the window: all blocks histogram bits 30..20 of key - lo of
//             the candidates with key >= lo = hint + 2048 * 2047
//   refill    fewer than k candidates: every element becomes a candidate (chunk c holds
//             candidates 1024 c ...) and joins the level-1 histogram of the plain keys
// ---------------------------------------------------------------------------
constexpr int kSeedThreads = 1024;

__global__ __launch_bounds__(kSeedThreads) void sparse_seed_k(uint32_t n, const float *v, uint64_t k, SparseScratch sc, SampleRule smp)
{
    __shared__ uint32_t hist[kBins1];
    __shared__ __attribute__((aligned(16))) uint32_t wbins[kBinsW];
    __shared__ uint32_t verdict[6];              // found, bin, rest lo, rest hi, candidates lo, hi
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    // everything the verdict and its record need is asked for up front: one memory latency, not three in a row
    const uint32_t hint = *sc.hint, hint_shift = sc.hint[kHintShift], hint_hold = sc.hint[kHintHold], hint_cap = sc.hint[kHintCap];
    uint32_t open = wave == 0 ? sc.hist[kHistOpen + lane] : 0u;
    for (int b = t; b < kBinsW; b += kSeedThreads) {          // the window: the sum of its copies
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < kWinCopies; ++r) sum += sc.hist[kHistW + r * kBinsW + b];
        wbins[b] = sum;
    }
    __syncthreads();
    if (wave == 0) {
        uint32_t bin;
        uint64_t rest;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) open += __shfl_xor(open, d, 64);
        uint64_t cands;
        const bool found = resolve_lds<kBinsW>(wbins, k, bin, rest, open, &cands);
        if (lane == 0) {
            verdict[0] = found; verdict[1] = bin; verdict[2] = (uint32_t)rest; verdict[3] = (uint32_t)(rest >> 32);
            verdict[4] = (uint32_t)cands; verdict[5] = (uint32_t)(cands >> 32);
        }
    }
    for (int b = t; b < kBins1; b += kSeedThreads) hist[b] = 0u;
    __syncthreads();
    const bool found = verdict[0] != 0u;
    const uint32_t bin = verdict[1];
    if (found && bin < (uint32_t)kBinsW - 1u) {
        if (blockIdx.x == 0 && t == 0) {
            SelectState s;
            s.lo = hint + (bin << kWindowShift); s.mode = kModeFast; s.need = (uint64_t)verdict[2] | ((uint64_t)verdict[3] << 32);
            sc.sel[0] = s;
            margin_after_hit(sc.hint, hint_shift, hint_hold, hint_cap, (uint64_t)verdict[4] | ((uint64_t)verdict[5] << 32), k);
        }
        return;
    }
    // missed: the next calls filter with the full margin again, and keep it for a while
    if (blockIdx.x == 0 && t == 0) margin_after_miss(sc.hint, hint_shift, hint_cap, !found && !first_call(hint, hint_cap));
    const uint32_t ntiles = (n + (uint32_t)kTile - 1u) / (uint32_t)kTile;
    const uint32_t uwave = __builtin_amdgcn_readfirstlane(wave), waves = kSeedThreads / 64;
    if (found) {
        // ---- above the window
        const uint32_t lo = hint + (((uint32_t)kBinsW - 1u) << kWindowShift);
        for (uint32_t tile = blockIdx.x * waves + uwave; tile < ntiles; tile += gridDim.x * waves) {
            tile_walk<true>(sc, tile, sc.tile_runs[tile], [&](bool valid, uint32_t chunk, uint32_t bits, uint32_t loc) {
                const uint32_t key = bits & 0x7FFFFFFFu;
                if (valid && key >= lo && in_sample(smp, chunk * (uint32_t)kChunk + loc)) atomicAdd(&hist[(key - lo) >> 20], 1u);
            });
        }
        __syncthreads();
        flush_fine(hist, sc.hist + kHist1, kBins1);
        if (blockIdx.x == 0 && t == 0) {
            SelectState s;
            s.lo = lo; s.mode = 0u; s.need = k;
            sc.sel[0] = s;
        }
        return;
    }
    // ---- refill
    const uint32_t nch = (n + (uint32_t)kChunk - 1u) / (uint32_t)kChunk;
    for (uint32_t ch = blockIdx.x * waves + uwave; ch < nch; ch += gridDim.x * waves) {
        Chunk c;
        c.base = ch * (uint32_t)kChunk;
        c.lane = lane;
        c.full = n - c.base >= (uint32_t)kChunk;
        float x[kSteps];
        load_flat(v, c, n, x, 0.0f);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            uint32_t i = c.base + 64 * j + c.lane;
            if (c.full || i < n) {
                sc.cand_bits[i] = __float_as_uint(x[j]);
                sc.cand_loc[i] = (uint16_t)(64 * j + c.lane);
                if (in_sample(smp, i)) atomicAdd(&hist[key_of(x[j]) >> 20], 1u);
            }
        }
    }
    __syncthreads();
    flush_fine(hist, sc.hist + kHist1, kBins1);
    if (blockIdx.x == 0 && t == 0) {
        SelectState s;
        s.lo = 0u; s.mode = kModeUniform; s.need = k;
        sc.sel[0] = s;
    }
}

// ---------------------------------------------------------------------------
// level 2 / level 3 histogram over the candidates, one tile per wavefront
//   LEVEL 2: nothing to do after a fast seed.  Otherwise resolves level 1 (2048 bins of
//            2^20 keys above the seed's lo) and histograms bits 19..10 of key - lo
//   LEVEL 3: after a fast seed lo / need come from the seed; otherwise resolves level 2.
//            Histograms the last 10 bits
// Block 0 records the resolved state for the next kernel and clears the histogram
// that the previous kernel has finished reading.
// ---------------------------------------------------------------------------
template <int LEVEL>
__global__ __launch_bounds__(kBlock) void cand_hist_k(uint32_t n, uint32_t ntiles, SparseScratch sc, SampleRule smp)
{
    constexpr int kBins = LEVEL == 2 ? kBins2 : kBins3;
    __shared__ uint32_t hist[kBins];
    const SelectState s0 = sc.sel[0];
    if (LEVEL == 2) {
        // the seed is done with the window: all blocks clear it together (one block alone is the whole duration of
        // this kernel on the fast route: 1.5 us)
        for (uint32_t b = blockIdx.x * kBlock + threadIdx.x; b < (uint32_t)(kWinCopies * kBinsW + kOpenCopies); b += gridDim.x * kBlock)
            sc.hist[b < (uint32_t)(kWinCopies * kBinsW) ? kHistW + b : kHistOpen - kWinCopies * kBinsW + b] = 0u;
        if (s0.mode & kModeFast) return;
    }
    const bool uniform = (s0.mode & kModeUniform) != 0u;
    TileJob job = my_tile(sc, n, ntiles);
    for (int b = threadIdx.x; b < kBins; b += kBlock) hist[b] = 0u;
    uint32_t lo;
    uint64_t need;
    if (LEVEL == 2) {
        uint32_t bin;
        resolve_wave<kBins1>(sc.hist + kHist1, s0.need, bin, need);
        lo = s0.lo + (bin << 20);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            SelectState s;
            s.lo = lo; s.mode = s0.mode; s.need = need;
            sc.sel[1] = s;
        }
    } else {
        if (s0.mode & kModeFast) { lo = s0.lo; need = s0.need; }
        else {
            const SelectState s1 = sc.sel[1];
            uint32_t bin;
            resolve_wave<kBins2>(sc.hist + kHist2, s1.need, bin, need);
            lo = s1.lo + (bin << 10);
        }
        if (blockIdx.x == 0) {
            if (threadIdx.x == 0) {
                SelectState s;
                s.lo = lo; s.mode = s0.mode; s.need = need;
                sc.sel[2] = s;
            }
            for (int b = threadIdx.x; b < kBins1; b += kBlock) sc.hist[kHist1 + b] = 0u;   // level 2 is done with level 1
        }
    }
    __syncthreads();
    if (uniform) job.runs = job.tile < ntiles ? uniform_runs(job.tile, n) : 0ull;
    // keys still undecided: level 2 leaves 2^10 to level 3; a fast seed leaves a whole window bin
    const uint32_t kRange = LEVEL == 2 ? 1u << 20 : (s0.mode & kModeFast) ? 1u << kWindowShift : 1u << 10;
    constexpr int kShift = LEVEL == 2 ? 10 : 0;
    uint32_t any = 0;
    tile_walk<true>(sc, job.tile, job.runs, [&](bool valid, uint32_t chunk, uint32_t bits, uint32_t loc) {
        const uint32_t d = (bits & 0x7FFFFFFFu) - lo;       // wraps to a large number for keys below lo
        if (valid && d < kRange && in_sample(smp, chunk * (uint32_t)kChunk + loc)) { atomicAdd(&hist[d >> kShift], 1u); any = 1u; }
    });
    if (__syncthreads_or((int)any)) flush_fine(hist, sc.hist + (LEVEL == 2 ? kHist2 : kHist3), kBins);
}

// ---------------------------------------------------------------------------
// count: resolve level 3 -> threshold key T and `need` (keys == T to take, in
// index order); candidates above / equal to T per tile and per block of four tiles.
// ---------------------------------------------------------------------------
// (six wavefronts per SIMD hold all tiles of the ResNet-50 buffer at once; left alone the compiler takes 102 registers: four)
__attribute__((amdgpu_waves_per_eu(6, 6)))
__global__ __launch_bounds__(kBlock) void cand_count_k(uint32_t n, uint32_t ntiles, SparseScratch sc)
{
    __shared__ uint32_t wgt[kWavesPerBlock], weq[kWavesPerBlock];
    __shared__ uint32_t res[3];
    TileJob job = my_tile(sc, n, ntiles);
    const SelectState s2 = sc.sel[2];
    const uint32_t hint_shift = sc.hint[kHintShift];        // (asked for now: block 0 would wait for it later)
    // one wavefront reads the bins for the block: every wavefront doing so would move the histogram
    // once per tile of the group
    if (threadIdx.x < 64) {
        uint32_t b;
        uint64_t r;
        resolve_wave<kBins3>(sc.hist + kHist3, s2.need, b, r);
        if (threadIdx.x == 0) { res[0] = b; res[1] = (uint32_t)r; res[2] = (uint32_t)(r >> 32); }
    }
    __syncthreads();
    const uint32_t bin = res[0];
    const uint64_t rest = (uint64_t)res[1] | ((uint64_t)res[2] << 32);
    const uint32_t T = s2.lo + bin;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            SelectState s;
            s.lo = T; s.mode = s2.mode; s.need = rest;
            sc.sel[3] = s;
            const uint32_t margin = kHintMargin >> hint_shift;
            *sc.hint = T > margin ? T - margin : 0u;                // where the next call starts filtering
        }
        for (int b = threadIdx.x; b < kBins2; b += kBlock) sc.hist[kHist2 + b] = 0u;   // level 3 is done with level 2
    }
    if (s2.mode & kModeUniform) job.runs = job.tile < ntiles ? uniform_runs(job.tile, n) : 0ull;
    uint32_t ngt = 0, neq = 0;
    tile_walk<false>(sc, job.tile, job.runs, [&](bool valid, uint32_t, uint32_t bits, uint32_t) {
        uint32_t key = bits & 0x7FFFFFFFu;
        ngt += __popcll(__builtin_amdgcn_ballot_w64(valid && key > T));
        neq += __popcll(__builtin_amdgcn_ballot_w64(valid && key == T));
    });
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) {
        wgt[wave] = ngt; weq[wave] = neq;
        if (job.tile < ntiles) sc.tile_cnt[job.tile] = ngt | (neq << 16);     // a tile holds at most 4096 candidates
    }
    __syncthreads();
    if (threadIdx.x == 0)                                                      // a block at most 16384
        sc.blk_cnt[blockIdx.x] = (wgt[0] + wgt[1] + wgt[2] + wgt[3]) | ((weq[0] + weq[1] + weq[2] + weq[3]) << 16);
}

// ---------------------------------------------------------------------------
// emit: ordered compaction.  A candidate is kept if its key is above T, or equal
// to T and among the first `need` such keys in index order.  Its slot is
//   (#kept before it) = (#above before it) + min(#equal before it, need).
// Every block adds up the counts of the blocks before it; nothing waits.
// ---------------------------------------------------------------------------
// The directory that ends a sparse payload: entry t = kept entries with index below 4096 t, t = 0 .. tiles (the paper
// gives no payload format; this one lets the receiver find a payload's share of a tile without searching).  It follows
// the index and value lists, which have room for `cap` entries each.
__device__ __forceinline__ uint32_t *payload_directory(PayloadHeader *hdr, uint64_t cap)
{
    return reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(hdr) + kHeaderBytes + 8u * cap);
}

// What the compaction does to the memory of an entry it keeps.  Top-k and DGC leave entries above the threshold key to the
// next call's streaming pass (StateHeader::sent_key) and zero only kept entries equal to it; Rand-k, whose choice does not
// depend on the values, zeroes in place.
template <int ALGO, bool EF>
__device__ __forceinline__ void drop_sent(float *st, uint32_t n, uint32_t i, bool equal)
{
    if (ALGO == MC_ALGO_RANDK) st[i] = 0.0f;
    else if (ALGO == MC_ALGO_DGC) { if (equal) { st[i] = 0.0f; st[dgc_u_offset(n) + i] = 0.0f; } }      // momentum factor masking
    else if (EF) { if (equal) st[i] = 0.0f; }
}
// ... and what it tells the next call (one thread)
template <int ALGO, bool EF>
__device__ __forceinline__ void record_sent_key(float *st, uint32_t T)
{
    if (ALGO == MC_ALGO_DGC || EF)
        reinterpret_cast<StateHeader *>(reinterpret_cast<uint8_t *>(st) - kHeaderBytes)->sent_key = ALGO == MC_ALGO_RANDK ? 0xFFFFFFFFu : T;
}

// DGC with a sampled threshold: T comes from the sample, so the number of keys >= T varies.
// cap is the payload's capacity: all keys above T are kept in index order while there is room, then
// keys equal to T; the header records how many entries were kept and unused entries are zeroed.
__global__ __launch_bounds__(kBlock) void cand_emit_k(uint32_t n, uint32_t ntiles, float *st, PayloadHeader *hdr, uint64_t cap,
                                                      SparseScratch sc)
{
    __shared__ uint64_t sgt[kWavesPerBlock], seq[kWavesPerBlock], stg[kWavesPerBlock], ste[kWavesPerBlock];
    TileJob job = my_tile(sc, n, ntiles);
    const SelectState s3 = sc.sel[3];
    const uint32_t T = s3.lo;
    uint32_t *idx = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(hdr) + kHeaderBytes);
    float *val = reinterpret_cast<float *>(idx + cap);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    // kept-before of this wavefront inside the block
    uint64_t wg = 0, we = 0;
    if (lane < wave && job.tile < ntiles) {          // then the tiles before it in the block exist too
        const uint32_t x = sc.tile_cnt[blockIdx.x * kWavesPerBlock + lane];
        wg = x & 0xFFFFu; we = x >> 16;
    }
    // kept-before of this block: sum over the blocks before it, and over all blocks, eight loads in flight per thread
    uint64_t ag = 0, ae = 0, tg = 0, te = 0;
    for (uint32_t b0 = 0; b0 < gridDim.x; b0 += 8 * kBlock) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t b = b0 + u * kBlock + threadIdx.x;
            x[u] = b < gridDim.x ? sc.blk_cnt[b] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t b = b0 + u * kBlock + threadIdx.x;
            if (b < blockIdx.x) { ag += x[u] & 0xFFFFu; ae += x[u] >> 16; }
            tg += x[u] & 0xFFFFu; te += x[u] >> 16;
        }
    }
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b < kBins3; b += kBlock) sc.hist[kHist3 + b] = 0u;   // count is done with level 3
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        ag += __shfl_xor(ag, m, 64); ae += __shfl_xor(ae, m, 64);
        wg += __shfl_xor(wg, m, 64); we += __shfl_xor(we, m, 64);
        tg += __shfl_xor(tg, m, 64); te += __shfl_xor(te, m, 64);
    }
    if (lane == 0) { sgt[wave] = ag; seq[wave] = ae; stg[wave] = tg; ste[wave] = te; }
    __syncthreads();
    uint64_t gt_before = (sgt[0] + sgt[1]) + (sgt[2] + sgt[3]) + wg;
    uint64_t eq_before = (seq[0] + seq[1]) + (seq[2] + seq[3]) + we;
    const uint64_t all_gt = (stg[0] + stg[1]) + (stg[2] + stg[3]), all_eq = (ste[0] + ste[1]) + (ste[2] + ste[3]);
    const uint64_t kept_gt = all_gt < cap ? all_gt : cap, need = all_eq < cap - kept_gt ? all_eq : cap - kept_gt, kept = kept_gt + need;
    // entries of the payload that stay unused are zero
    for (uint64_t pos = kept + (uint64_t)blockIdx.x * kBlock + threadIdx.x; pos < cap; pos += (uint64_t)gridDim.x * kBlock) {
        idx[pos] = 0u;
        val[pos] = 0.0f;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        PayloadHeader h;
        h.magic = kMagic; h.algo = MC_ALGO_DGC; h.n = n; h.k = kept; h.scale = 0.0f; h.levels = (uint32_t)cap;
        for (int i = 0; i < 24; ++i) h.pad[i] = 0;
        *hdr = h;
        // this kernel zeroes what it keeps in place: the next streaming pass has nothing to mask
        reinterpret_cast<StateHeader *>(reinterpret_cast<uint8_t *>(st) - kHeaderBytes)->sent_key = 0xFFFFFFFFu;
    }
    if (s3.mode & kModeUniform) job.runs = job.tile < ntiles ? uniform_runs(job.tile, n) : 0ull;
    if (lane == 0 && job.tile < ntiles) {
        uint32_t *dir = payload_directory(hdr, cap);
        const uint64_t at = gt_before + (eq_before < need ? eq_before : need);      // (there may be no room for all of them)
        dir[job.tile] = (uint32_t)(at < kept ? at : kept);
        if (job.tile == ntiles - 1u) dir[ntiles] = (uint32_t)kept;
    }
    // the tile's candidates: gt_before / eq_before are the numbers of keys above / equal to T among all candidates before them
    tile_walk<true>(sc, job.tile, job.runs, [&](bool valid, uint32_t chunk, uint32_t b, uint32_t loc) {
        const uint32_t key = b & 0x7FFFFFFFu;
        const bool is_gt = valid && key > T, is_eq = valid && key == T;
        const uint64_t bgt = __builtin_amdgcn_ballot_w64(is_gt), beq = __builtin_amdgcn_ballot_w64(is_eq);
        const uint64_t gtb = gt_before + lanes_below(bgt), eqb = eq_before + lanes_below(beq);
        if (is_gt || (is_eq && eqb < need)) {
            const uint64_t pos = gtb + (eqb < need ? eqb : need);
            const uint32_t i = chunk * (uint32_t)kChunk + loc;
            if (pos < cap && i < n) {                // while there is room
                idx[pos] = i;
                val[pos] = __uint_as_float(b);
                st[i] = 0.0f; st[dgc_u_offset(n) + i] = 0.0f;      // momentum factor masking
            }
        }
        gt_before += __popcll(bgt);
        eq_before += __popcll(beq);
    });
}

// ---------------------------------------------------------------------------
// The two-kernel tail (everything but DGC with a sampled threshold).
//
//   select   every block (16 wavefronts, one 4096-element tile each) resolves the window on its own -- no
//            kernel in between just to reduce 2048 bins -- and all blocks reach the same verdict:
//     lean     the threshold lies in window bin b, which holds at most kUCap keys.  Every key above the
//              bin is kept whatever the threshold turns out to be: their number per tile and per block is
//              all the emit kernel needs of them.  The keys inside the bin -- a few hundred out of
//              millions -- are appended to a list.
//     dense    bin b holds more than kUCap keys (heavy ties, or a pile of values just under the
//              threshold): the blocks histogram its 2048 keys, as level 3 of a radix select
//     above    the threshold lies above the window: level 1 (bits 30..20 above the window's top) over
//              the candidates
//     refill   fewer than k candidates: levels 1 and 2 over all elements; those in or above level 1's bin
//              become the candidates
//   emit     lean: every block reads the whole list (it is small), finds the threshold key T and the
//            number of keys equal to T to take with a histogram in LDS, counts the list's kept keys
//            that lie before each of its tiles, adds the kept counts of the blocks before it, and
//            compacts its tiles' kept candidates into the payload.  One kernel after the select: no
//            level-3 pass, no counting pass.
//            On the other routes the radix levels still open, the per-tile counts and the compaction run as steps of
//            the select kernel's first blocks, at most one per compute unit, separated by grid-wide barriers; the
//            emit kernel then only clears the window.  Written for the 57 registers that the select kernel may take
//            without losing wavefronts (64), they cost the usual route no launch of their own: an idle slot
//            between the two kernels was 1.2 us of 80.8 (Top-k compress, 25.6 M elements) and, with four groups, 4
//            of 269.  Measured there without error feedback, whole call, before / after: first call 484 / 176 us,
//            refill 398 / 174, above 241 / 196, dense 120 / 120.
// Both kernels are bound by memory latency, not by traffic, so each asks for its tile's candidates as soon
// as it knows how many there are, before it waits for anything else.
// ---------------------------------------------------------------------------
constexpr int kSelThreads = 1024, kSelWaves = kSelTiles;      // select: 16 tiles per block (the window is read once per block)
constexpr int kEmitThreads = kBlock, kEmitWaves = kEmitTiles;    // emit: 4 tiles per block
constexpr int kSyncRoutes = 32, kSyncLastBin = 40, kSyncLastCands = 41;     // words of SparseScratch::sync (mc_api.hip reads the last three)

// Select.  The keys inside the threshold's bin [lo, lo + 2048) -- rarely more than a few per tile -- are collected
// in a buffer of the wavefront's own in LDS and appended to sublist `sub` with one atomic add per tile (per 64
// entries when there are more): an add per batch of candidates put its latency between the batches.
constexpr int kMemberBuf = 64;
struct MemberBuf { UEntry *buf; uint32_t held; };

__device__ __forceinline__ void flush_members(const SparseScratch &sc, MemberBuf &m, uint32_t sub)
{
    if (!m.held) return;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&sc.ucount[sub * kUCountStride], m.held);
    base = __builtin_amdgcn_readfirstlane(base);
    __builtin_amdgcn_wave_barrier();
    if (lane < m.held && base + lane < kUCap) sc.ulist[(size_t)sub * kUCap + base + lane] = m.buf[lane];   // (always in range: the bin holds at most kUCap keys)
    __builtin_amdgcn_wave_barrier();
    m.held = 0u;
}

__device__ __forceinline__ void put_sparse_header(PayloadHeader *hdr, uint32_t algo, uint32_t n, uint64_t k)
{
    PayloadHeader h;
    h.magic = kMagic; h.algo = algo; h.n = n; h.k = k; h.scale = 0.0f; h.levels = 0u;
    for (int i = 0; i < 24; ++i) h.pad[i] = 0;
    *hdr = h;
}
// where the next call of this (group, worker) starts filtering: a margin below this call's threshold key
__device__ __forceinline__ void publish_hint(const SparseScratch &sc, uint32_t T)
{
    const uint32_t margin = kHintMargin >> sc.hint[kHintShift];
    *sc.hint = T > margin ? T - margin : 0u;
}

// Grid-wide barrier of the slow routes, for the first `blocks` blocks of the grid, all of which the device
// holds at once (one per compute unit at most): arrivals are counted in one word (cleared by the streaming pass),
// the `round`-th barrier is passed when it reaches round * blocks.  The release / acquire pair makes what every
// block wrote before the barrier visible to every block after it.  The wait is bounded: should the count never
// come (it always does when the blocks are resident together), the block flags the failure and leaves, and so
// does every later wait.
// A single block (blocks = 1) has only its own wavefronts to wait for.
__device__ __forceinline__ bool grid_barrier(uint32_t *arrive, uint32_t blocks, uint32_t round, uint32_t *dead /* LDS */, int *status, uint32_t limit)
{
    __syncthreads();
    if (blocks == 1u) return true;
    if (threadIdx.x == 0 && !*dead) {
        release_to_device();
        __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t target = round * blocks;
        uint32_t spins = 0;
        // polled without acquire semantics: an acquire at agent scope invalidates the die's L2, and two hundred waiting
        // blocks doing that every few hundred cycles starve the blocks still at work (phases of 60-120 us instead of 10)
        while (__hip_atomic_load(arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(32);
            if (spins++ >= limit) { *dead = 1u; raise_flag(status, FLAG_GAVE_UP); break; }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return *dead == 0u;
}

// A radix level resolved by a block of 1024 threads, one or two adjacent bins each: the bin b with
//   count(bins > b) < need <= count(bins >= b)   and   rest = need - count(bins > b)
// (the counts stay below 2^32, there being fewer elements than that).  sums: 16 words of LDS, res: 2 words.
template <int BINS>
__device__ __forceinline__ void resolve_block(const uint32_t *fine, uint64_t need, uint32_t &bin, uint64_t &rest, uint32_t *res, uint32_t *sums)
{
    constexpr int kPer = BINS / 1024;
    static_assert(kPer == 1 || kPer == 2, "one or two bins per thread");
    const uint32_t t = threadIdx.x, wave = t >> 6;
    uint2 own = {0u, 0u};                        // the lower and the upper bin
    if (kPer == 2) own = *reinterpret_cast<const uint2 *>(fine + 2u * t);
    else own.x = fine[t];
    const uint32_t both = own.x + own.y, incl = wave_scan_incl(both), total = wave_total(incl);
    if ((t & 63u) == 0) sums[wave] = total;
    if (t == 0) { res[0] = 0u; res[1] = 0u; }    // (an inconsistent histogram still gives a defined bin)
    __syncthreads();
    uint32_t above = total - incl;               // keys in the bins of higher threads
#pragma unroll
    for (int w = 0; w < 16; ++w) if ((uint32_t)w > wave) above += sums[w];
    if ((uint64_t)above < need && need <= (uint64_t)above + both) {
        const bool upper = kPer == 2 && need <= (uint64_t)above + own.y;
        res[0] = (uint32_t)kPer * t + (upper ? 1u : 0u);
        res[1] = (uint32_t)need - above - (kPer == 2 && !upper ? own.y : 0u);
    }
    __syncthreads();
    bin = res[0];
    rest = res[1];
    __syncthreads();
}

// ---- access to the candidate slots of a tile ---------------------------------------------------------------
// A chunk's candidates sit at the front of its 1024 slots, in index order.  They are read as a *head* -- the first
// 64, one per lane -- and up to four *units* of 256 -- a lane takes four consecutive candidates with one 16-byte
// load of values and one 8-byte load of positions.  The kernels below live on memory latency, not on traffic: the
// heads of a tile's four chunks are asked for before the number of candidates is known (what lies beyond it is
// masked out afterwards; most chunks hold fewer than 64), and a crowded chunk costs one more round of loads, not
// one per 64 candidates.  Candidate number o >= 64 of a chunk is held by lane ((o - 64) % 256) / 4 of unit (o - 64) / 256.
constexpr int kHead = kCandHead, kUnit = kCandUnit;
__device__ __forceinline__ uint32_t load_head_bits(const SparseScratch &sc, uint32_t chunk)
{
    return sc.cand_bits[(size_t)chunk * kChunk + (threadIdx.x & 63u)];
}
__device__ __forceinline__ uint32_t load_head_loc(const SparseScratch &sc, uint32_t chunk)
{
    return sc.cand_loc[(size_t)chunk * kChunk + (threadIdx.x & 63u)];
}
__device__ __forceinline__ uint4 load_bits4(const SparseScratch &sc, uint32_t chunk, uint32_t v)
{
    return *reinterpret_cast<const uint4 *>(sc.cand_bits + (size_t)chunk * kChunk + kHead + v * kUnit + (threadIdx.x & 63u) * 4u);
}
__device__ __forceinline__ uint2 load_loc4(const SparseScratch &sc, uint32_t chunk, uint32_t v)
{
    return *reinterpret_cast<const uint2 *>(sc.cand_loc + (size_t)chunk * kChunk + kHead + v * kUnit + (threadIdx.x & 63u) * 4u);
}
// x[q] for a q that is only known at run time, without putting the array into scratch memory
__device__ __forceinline__ uint32_t pick4(const uint32_t (&x)[4], uint32_t q) { return q == 0 ? x[0] : q == 1 ? x[1] : q == 2 ? x[2] : x[3]; }
__device__ __forceinline__ uint32_t elem4(const uint4 &x, int j) { return j == 0 ? x.x : j == 1 ? x.y : j == 2 ? x.z : x.w; }
__device__ __forceinline__ uint32_t loc4(const uint2 &x, int j) { return ((j < 2 ? x.x : x.y) >> (16 * (j & 1))) & 0xFFFFu; }
// is candidate (unit v, lane, j) of a chunk with cnt candidates there?  (head: candidates before unit 0)
__device__ __forceinline__ bool in_unit(uint32_t cnt, uint32_t v, int j, uint32_t head = kHead) { return head + v * (uint32_t)kUnit + 4u * (threadIdx.x & 63u) + (uint32_t)j < cnt; }

// The units of a tile, numbered in chunk order: unit e is unit v of chunk q.
struct TileUnits {
    uint32_t per[kWavesPerBlock], total;
    __device__ __forceinline__ TileUnits(const uint32_t (&cnt)[kWavesPerBlock])
    {
        total = 0;
#pragma unroll
        for (int q = 0; q < kWavesPerBlock; ++q) { per[q] = cnt[q] > (uint32_t)kHead ? (cnt[q] - (uint32_t)kHead + (uint32_t)kUnit - 1u) / (uint32_t)kUnit : 0u; total += per[q]; }
    }
    __device__ __forceinline__ void locate(uint32_t e, uint32_t &q, uint32_t &v) const
    {
        q = 0;
#pragma unroll
        for (int i = 0; i < kWavesPerBlock - 1; ++i) if (q == (uint32_t)i && e >= per[i]) { e -= per[i]; ++q; }
        v = e;
    }
};

// Select: counts the keys above the threshold's bin, buffers those inside it (with the tile's first index: all that
// the emit kernel needs of a listed key's position is its tile).
__device__ __forceinline__ uint32_t select_one(const SparseScratch &sc, uint32_t bits, bool valid, uint32_t tile, uint32_t lo, uint32_t sub,
                                               MemberBuf &m)
{
    const uint32_t key = bits & 0x7FFFFFFFu;
    const bool reach = valid && key >= lo;
    const bool inside = reach && key - lo < (1u << kWindowShift);
    const uint64_t mb = __builtin_amdgcn_ballot_w64(inside);
    if (mb) {
        const uint32_t c = __popcll(mb);
        if (m.held + c > (uint32_t)kMemberBuf) flush_members(sc, m, sub);
        if (inside) { UEntry e; e.idx = tile * (uint32_t)kTile; e.bits = bits; m.buf[m.held + lanes_below(mb)] = e; }
        m.held += c;
    }
    return __popcll(__builtin_amdgcn_ballot_w64(reach && key - lo >= (1u << kWindowShift)));
}

// What a wavefront of the select kernel asks for of one tile before it knows the verdict.
struct TileAhead {
    uint32_t tile, cnt[kWavesPerBlock], head[kWavesPerBlock], uq[4], uv[4], units;
    uint4 ub[4];
};
__device__ __forceinline__ void look_ahead(const SparseScratch &sc, uint32_t tile, bool live, TileAhead &a)
{
    a.tile = tile;
    const uint64_t runs = live ? sc.tile_runs[tile] : 0ull;
    // the first 64 slots of each chunk, without waiting for the counts
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) a.head[q] = live ? load_head_bits(sc, tile * kWavesPerBlock + q) : 0u;
    // ... and, as soon as the counts are there, the first four units of a tile with crowded chunks (nearly always all it has)
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) a.cnt[q] = (uint32_t)(runs >> (16 * q)) & 0xFFFFu;
    const TileUnits tu(a.cnt);
    a.units = tu.total;
    if (tu.total) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tu.locate((uint32_t)i < tu.total ? (uint32_t)i : 0u, a.uq[i], a.uv[i]);
            a.ub[i] = load_bits4(sc, tile * kWavesPerBlock + a.uq[i], a.uv[i]);
        }
    }
}
// ... and what it does with it on the lean route: the tile's keys above the threshold's bin are counted, those inside listed
__device__ __forceinline__ uint32_t select_tile(const SparseScratch &sc, TileAhead &a, uint32_t lo, uint32_t sub, MemberBuf &mb)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t above = 0;
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) if (a.cnt[q]) above += select_one(sc, a.head[q], lane < a.cnt[q], a.tile, lo, sub, mb);
    if (a.units) {
        const TileUnits tu(a.cnt);
        for (uint32_t e0 = 0; e0 < tu.total; e0 += 4u) {
            if (e0) {                            // (more than four units: the next four)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    tu.locate(e0 + i < tu.total ? e0 + i : e0, a.uq[i], a.uv[i]);
                    a.ub[i] = load_bits4(sc, a.tile * kWavesPerBlock + a.uq[i], a.uv[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (e0 + i >= tu.total) break;
#pragma unroll
                for (int j = 0; j < 4; ++j) above += select_one(sc, elem4(a.ub[i], j), in_unit(pick4(a.cnt, a.uq[i]), a.uv[i], j), a.tile, lo, sub, mb);
            }
        }
    }
    if (lane == 0) sc.tile_cnt[a.tile] = above;
    return above;
}

// Emit, lean route.  One candidate per lane (a chunk's head): gt0 / eq0 count the keys above / equal to T before it
// in the whole group; they are advanced past these 64.  Returns whether the lane's candidate was kept.
template <int ALGO, bool EF>
__device__ __forceinline__ bool emit_head(uint32_t bits, uint32_t loc, bool valid, uint32_t chunk, uint32_t n, uint32_t k, float *st,
                                          uint32_t *idx, float *val, uint32_t T, uint32_t need, uint32_t &gt0, uint32_t &eq0)
{
    const uint32_t key = bits & 0x7FFFFFFFu;
    const bool is_gt = valid && key > T, is_eq = valid && key == T;
    const uint64_t bgt = __builtin_amdgcn_ballot_w64(is_gt), beq = __builtin_amdgcn_ballot_w64(is_eq);
    const uint32_t gtb = gt0 + lanes_below(bgt);
    const uint32_t eqb = eq0 + lanes_below(beq);
    const bool keep = is_gt || (is_eq && eqb < need);
    if (keep) {
        const uint32_t pos = gtb + (eqb < need ? eqb : need);
        const uint32_t i = chunk * (uint32_t)kChunk + loc;
        if (pos < k && i < n) {                  // always true for consistent scratch
            idx[pos] = i;
            if (ALGO == MC_ALGO_RANDK) val[pos] = st[i];      // the candidate slot holds the random key: the value is p
            else val[pos] = __uint_as_float(bits);
            drop_sent<ALGO, EF>(st, n, i, is_eq);
        }
    }
    gt0 += __popcll(bgt); eq0 += __popcll(beq);
    return keep;
}

// ... four consecutive candidates per lane (a unit; it holds at most 256 keys above T and as many equal to it)
template <int ALGO, bool EF, int HEAD = kHead>
__device__ __forceinline__ void emit_unit(const uint4 &bits, const uint2 &loc, uint32_t cnt, uint32_t v, uint32_t chunk, uint32_t n,
                                          uint32_t k, float *st, uint32_t *idx, float *val, uint32_t T, uint32_t need, uint32_t &gt0, uint32_t &eq0)
{
    bool isg[4], ise[4];
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t key = elem4(bits, j) & 0x7FFFFFFFu;
        const bool valid = in_unit(cnt, v, j, HEAD);
        isg[j] = valid && key > T; ise[j] = valid && key == T;
        mine += (isg[j] ? 1u : 0u) + (ise[j] ? 0x10000u : 0u);
    }
    const uint32_t inc = wave_scan_incl(mine);
    const uint32_t tot = wave_total(inc);
    uint32_t gtb = gt0 + ((inc - mine) & 0xFFFFu);
    uint32_t eqb = eq0 + ((inc - mine) >> 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (isg[j] || (ise[j] && eqb < need)) {
            const uint32_t pos = gtb + (eqb < need ? eqb : need);
            const uint32_t i = chunk * (uint32_t)kChunk + loc4(loc, j);
            if (pos < k && i < n) {
                idx[pos] = i;
                if (ALGO == MC_ALGO_RANDK) val[pos] = st[i];
                else val[pos] = __uint_as_float(elem4(bits, j));
                drop_sent<ALGO, EF>(st, n, i, ise[j]);
            }
        }
        gtb += isg[j] ? 1u : 0u; eqb += ise[j] ? 1u : 0u;
    }
    gt0 += tot & 0xFFFFu; eq0 += tot >> 16;
}

// ---- the slow routes -------------------------------------------------------------------------------------------
// A chunk's candidates in units of 256 from its first slot on, 16 bytes per lane and load.
template <typename Body>
__device__ __forceinline__ void each_of_chunk(const SparseScratch &sc, uint32_t chunk, uint32_t cnt, Body body)
{
    const uint32_t at = 4u * (threadIdx.x & 63u);
    const uint4 *src = reinterpret_cast<const uint4 *>(sc.cand_bits + (size_t)chunk * kChunk) + (threadIdx.x & 63u);
#pragma unroll 1
    for (uint32_t v = 0; v < cnt; v += (uint32_t)kUnit) {
        const uint4 x = src[v / 4u];
#pragma unroll
        for (int j = 0; j < 4; ++j) body(v + at + j < cnt, elem4(x, j));
    }
}
// All candidates of the group, chunks gw, gw + nw, ... to a wavefront; in no order.
template <typename Body>
__device__ __forceinline__ void walk_chunks(const SparseScratch &sc, uint32_t nch, uint32_t gw, uint32_t nw, Body body)
{
    const uint16_t *runs = reinterpret_cast<const uint16_t *>(sc.tile_runs);
    for (uint32_t ch = gw; ch < nch; ch += nw)
        each_of_chunk(sc, ch, (uint32_t)__builtin_amdgcn_readfirstlane((int)runs[ch]), body);
}
// body(valid, bits, position in the chunk) for the elements of a chunk, in index order from call to call.  Written for few
// registers: Rand-k's words are drawn one element at a time (a block each), a chunk that straddles tensors tensor by tensor.
template <bool FROM_STATE, bool RANDOM, typename Body>
__device__ __forceinline__ void each_key(const GroupView &g, const float *st, const RngKey &rng, const Chunk &c, Body body)
{
    const uintptr_t entry = FROM_STATE || RANDOM ? 0u : chunk_entry(g, c);
    if (RANDOM) {
#pragma unroll 1
        for (uint32_t at = c.lane; at < (uint32_t)kChunk; at += 64u) {
            uint32_t w[4];
            const uint64_t i = g.goff + c.base + at;
            philox4x32_10(rng.seed, rng.worker, rng.iter_lo, i >> 2, w);
            body(c.full || c.base + at < g.n, pick4(w, (uint32_t)i & 3u) >> 1, at);
        }
    } else if (!(entry & 1u)) {
        float v[kSteps];
        if (FROM_STATE) load_flat(st, c, g.n, v, 0.0f);
        else {
            const float *p = reinterpret_cast<const float *>(entry) + c.lane;
#pragma unroll
            for (int j = 0; j < kSteps; ++j) v[j] = ld_stream(p + 64 * j);
        }
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            body(c.full || c.base + 64 * j + c.lane < g.n, __float_as_uint(v[j]), 64u * j + c.lane);
            __builtin_amdgcn_sched_barrier(0);       // (one step after the other: side by side they need more registers than there are)
        }
    } else {
        for_each_tensor_of_chunk(g, c, (uint32_t)(entry >> 1), [&](uint32_t beg, uint32_t end, uintptr_t ptr) {
            const float *p = reinterpret_cast<const float *>(ptr);
#pragma unroll 1
            for (uint32_t at = c.lane; at < (uint32_t)kChunk; at += 64u) {
                const uint32_t i = c.base + at;
                const bool in = i >= beg && i < end;
                body(in, in ? __float_as_uint(p[i - beg]) : 0u, at);
            }
        });
    }
}


// The routes that need more than the window: all radix levels still open, the per-tile counts and the ordered
// compaction, as steps of the first `blocks` blocks of the group's select blocks (which the device holds at once).
// `mode`: what the window said (kModeFast | kModeDense: the threshold's bin [lo, lo + 2048) is known but too full to
// list; 0: the threshold lies above lo, the window's top; kModeUniform: too few candidates.  Then the elements
// themselves are streamed twice more, for level 1 and for level 2, and the second time those that reach the bin of
// level 1 -- an eighth of an octave -- become the candidates of the later steps.)
template <int ALGO, bool EF, bool FROM_STATE, bool RANDOM>
__device__ __forceinline__ void slow_routes(const SparseJob &job, const RngKey &rng, uint32_t mode, uint32_t lo, uint64_t need, uint32_t blocks,
                                            int *status, uint32_t *hist /* 2048 words of LDS */, uint32_t *pfx /* 2 * kRoundTiles words of LDS */,
                                            uint32_t *small /* 64 words of LDS */)
{
    uint32_t *res = small, *dead = small + 4, *wsum = small + 8;      // wsum: 2 * kSelWaves words
    const SparseScratch &sc = job.sc;
    const GroupView &g = job.g;
    float *st = job.st;
    PayloadHeader *hdr = job.hdr;
    const uint32_t k = (uint32_t)job.k;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = __builtin_amdgcn_readfirstlane(t >> 6), me = job.block;
    const uint32_t n = g.n, ntiles = tiles_in(n), nch = chunks_of(n);
    const uint32_t nw = blocks * kSelWaves, gw = me * kSelWaves + wave;
    const bool refill = (mode & kModeUniform) != 0u;
    if (t == 0) *dead = 0u;
    uint32_t round = 0, T, bin;
    // A block's counts of a level go to the group's, which are resolved behind a barrier; a single block resolves its own, in
    // LDS.  (Top-k compress of a group of at most sixteen tiles on these routes, a refill and a rise in turn, n = 64 / 4104 /
    // 62 000: 36.0 / 49.5 / 70.9 us with the detour and the fences it takes to see one's own atomics, 21.4 / 35.1 / 55.9.)
    const bool alone = blocks == 1u;
    auto publish = [&](uint32_t *level, int bins) { if (!alone) flush_fine(hist, level, bins); };
    for (int b = t; b < kBins1; b += kSelThreads) hist[b] = 0u;
    __syncthreads();
    if (!(mode & kModeFast)) {
        // ---- level 1: bits 30..20 of key - lo
        if (!refill) {
            walk_chunks(sc, nch, gw, nw, [&](bool valid, uint32_t bits) {
                const uint32_t key = bits & 0x7FFFFFFFu;
                if (valid && key >= lo) atomicAdd(&hist[(key - lo) >> 20], 1u);
            });
        } else {
            for (uint32_t ch = gw; ch < nch; ch += nw) {
                const Chunk c{ch * (uint32_t)kChunk, lane, n - ch * (uint32_t)kChunk >= (uint32_t)kChunk};
                each_key<FROM_STATE, RANDOM>(g, st, rng, c, [&](bool valid, uint32_t bits, uint32_t) {
                    if (valid) atomicAdd(&hist[(bits & 0x7FFFFFFFu) >> 20], 1u);
                });
            }
        }
        __syncthreads();
        publish(sc.hist + kHist1, kBins1);
        if (!grid_barrier(sc.arrive, blocks, ++round, dead, status, sc.spin_limit)) return;
        resolve_block<kBins1>(alone ? hist : sc.hist + kHist1, need, bin, need, res, wsum);
        lo += bin << 20;
        // ---- level 2: bits 19..10
        for (int b = t; b < kBins2; b += kSelThreads) hist[b] = 0u;
        __syncthreads();
        if (!refill) {
            walk_chunks(sc, nch, gw, nw, [&](bool valid, uint32_t bits) {
                const uint32_t key = bits & 0x7FFFFFFFu;
                if (valid && key >= lo && key - lo < (1u << 20)) atomicAdd(&hist[(key - lo) >> 10], 1u);
            });
        } else {
            for (uint32_t ch = gw; ch < nch; ch += nw) {
                const Chunk c{ch * (uint32_t)kChunk, lane, n - ch * (uint32_t)kChunk >= (uint32_t)kChunk};
                uint32_t run = 0;
                each_key<FROM_STATE, RANDOM>(g, st, rng, c, [&](bool valid, uint32_t bits, uint32_t at) {
                    const uint32_t key = bits & 0x7FFFFFFFu;
                    const bool in = valid && key >= lo;
                    const uint64_t flag = __builtin_amdgcn_ballot_w64(in);
                    if (in) {
                        const uint32_t slot = c.base + run + lanes_below(flag);
                        sc.cand_bits[slot] = bits;
                        sc.cand_loc[slot] = (uint16_t)at;
                        if (key - lo < (1u << 20)) atomicAdd(&hist[(key - lo) >> 10], 1u);
                    }
                    run += __popcll(flag);
                });
                if (lane == 0) reinterpret_cast<uint16_t *>(sc.tile_runs)[ch] = (uint16_t)run;
            }
        }
        __syncthreads();
        publish(sc.hist + kHist2, kBins2);
        if (!grid_barrier(sc.arrive, blocks, ++round, dead, status, sc.spin_limit)) return;
        if (me == 0 && !alone) for (int b = t; b < kBins1; b += kSelThreads) sc.hist[kHist1 + b] = 0u;    // every block has resolved level 1
        resolve_block<kBins2>(alone ? hist : sc.hist + kHist2, need, bin, need, res, wsum);
        lo += bin << 10;
        for (int b = t; b < kBins3; b += kSelThreads) hist[b] = 0u;
        __syncthreads();
    }
    // ---- level 3: the bits still open (10 after level 2, the 11 of a window bin otherwise)
    const uint32_t open = (mode & kModeFast) ? 1u << kWindowShift : 1u << 10;
    walk_chunks(sc, nch, gw, nw, [&](bool valid, uint32_t bits) {
        const uint32_t key = bits & 0x7FFFFFFFu;
        if (valid && key >= lo && key - lo < open) atomicAdd(&hist[key - lo], 1u);
    });
    __syncthreads();
    publish(sc.hist + kHist3, kBins3);
    if (!grid_barrier(sc.arrive, blocks, ++round, dead, status, sc.spin_limit)) return;
    if (!(mode & kModeFast) && me == 0 && !alone) for (int b = t; b < kBins2; b += kSelThreads) sc.hist[kHist2 + b] = 0u;
    resolve_block<kBins3>(alone ? hist : sc.hist + kHist3, need, bin, need, res, wsum);
    T = lo + bin;
    // ---- kept candidates per tile
    for (uint32_t tile = gw; tile < ntiles; tile += nw) {
        const uint64_t runs = sc.tile_runs[tile];
        uint32_t both = 0;                                     // above T, and equal to T << 16 (a lane holds 64 of the tile's)
#pragma unroll 1
        for (int q = 0; q < kWavesPerBlock; ++q) {
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(runs >> (16 * q)) & 0xFFFFu));
            each_of_chunk(sc, tile * kWavesPerBlock + q, cnt, [&](bool valid, uint32_t bits) {
                const uint32_t key = bits & 0x7FFFFFFFu;
                both += (valid && key > T ? 1u : 0u) + (valid && key == T ? 0x10000u : 0u);
            });
        }
        both = wave_total(wave_scan_incl(both));               // a tile holds at most 4096 of either
        if (lane == 0) sc.tile_cnt[tile] = both;
    }
    if (!grid_barrier(sc.arrive, blocks, ++round, dead, status, sc.spin_limit)) return;
    if (me == 0 && !alone) for (int b = t; b < kBins3; b += kSelThreads) sc.hist[kHist3 + b] = 0u;
    uint32_t *idx = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(hdr) + kHeaderBytes);
    float *val = reinterpret_cast<float *>(idx + k);
    if (me == 0 && t == 0) {
        put_sparse_header(hdr, ALGO, n, k);
        SelectState s;
        s.lo = T; s.mode = mode; s.need = need;
        sc.sel[3] = s;
        publish_hint(sc, T);
        record_sent_key<ALGO, EF>(st, T);
    }
    // ---- ordered compaction, kRoundTiles tiles at a time: every block scans the round's counts (in LDS) for the
    // keys kept before each tile, and carries the totals of the rounds before
    uint32_t base_gt = 0, base_eq = 0;                                       // (numbers of elements: below 2^32, as k is)
    constexpr int kPer = kRoundTiles / kSelThreads;
    for (uint32_t r0 = 0; r0 < ntiles; r0 += kRoundTiles) {
        uint32_t x[kPer], sg = 0, se = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t tile = r0 + t * kPer + i;
            x[i] = tile < ntiles ? sc.tile_cnt[tile] : 0u;
            sg += x[i] & 0xFFFFu; se += x[i] >> 16;
        }
        const uint32_t ig = wave_scan_incl(sg), ie = wave_scan_incl(se);     // inclusive scans over the wavefront
        if (lane == 63u) { wsum[wave] = ig; wsum[kSelWaves + wave] = ie; }
        __syncthreads();
        // (the sixteen wavefronts' totals, scanned in the lanes)
        const uint32_t vg = lane < (uint32_t)kSelWaves ? wsum[lane] : 0u, ve = lane < (uint32_t)kSelWaves ? wsum[kSelWaves + lane] : 0u;
        const uint32_t pg = wave_scan_incl(vg), pe = wave_scan_incl(ve);
        const uint32_t wg = (uint32_t)__builtin_amdgcn_readlane((int)(pg - vg), (int)wave), we = (uint32_t)__builtin_amdgcn_readlane((int)(pe - ve), (int)wave);
        const uint32_t tg = wave_total(pg), te = wave_total(pe);
        uint32_t xg = wg + ig - sg, xe = we + ie - se;                       // kept before this thread's first tile, inside the round
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            pfx[t * kPer + i] = xg; pfx[kRoundTiles + t * kPer + i] = xe;
            xg += x[i] & 0xFFFFu; xe += x[i] >> 16;
        }
        __syncthreads();
        for (uint32_t p = gw; p < (uint32_t)kRoundTiles && r0 + p < ntiles; p += nw) {
            const uint32_t tile = r0 + p;
            const uint64_t runs = sc.tile_runs[tile];
            uint32_t gtb = base_gt + pfx[p], eqb = base_eq + pfx[kRoundTiles + p];
            if (lane == 0) {
                uint32_t *dir = payload_directory(hdr, k);
                dir[tile] = gtb + (eqb < (uint32_t)need ? eqb : (uint32_t)need);
                if (tile == ntiles - 1u) dir[ntiles] = k;
            }
#pragma unroll 1
            for (int q = 0; q < kWavesPerBlock; ++q) {
                const uint32_t cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(runs >> (16 * q)) & 0xFFFFu));
                const uint32_t chunk = tile * kWavesPerBlock + q;
                const uint4 *src = reinterpret_cast<const uint4 *>(sc.cand_bits + (size_t)chunk * kChunk) + lane;
                const uint2 *locs = reinterpret_cast<const uint2 *>(sc.cand_loc + (size_t)chunk * kChunk) + lane;
#pragma unroll 1
                for (uint32_t v = 0; v * kUnit < cnt; ++v)
                    emit_unit<ALGO, EF, 0>(src[64 * v], locs[64 * v], cnt, v, chunk, n, k, st, idx, val, T, (uint32_t)need, gtb, eqb);
            }
        }
        base_gt += tg; base_eq += te;
        __syncthreads();
    }
}

// ---- the verdict of the window, by a block of 1024 threads --------------------------------------------------------
// The bin b with  count(bins > b) < k <= count(bins >= b), by a suffix scan over the block's threads, two bins each (the
// counts stay below 2^32, there being fewer elements than that).
struct WindowPart { uint32_t lower, upper, above; };      // the thread's two bins; they and all above in its wavefront
// open: the copies of the open last bin, one per lane of the last wavefront.  A small group's counts are all in the first copy.
// Behind a barrier wtot holds the wavefronts' sums.
__device__ __forceinline__ WindowPart read_window(const SparseScratch &sc, uint32_t open, uint32_t *wtot)
{
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    uint2 w = *reinterpret_cast<const uint2 *>(sc.hist + kHistW + 2 * t);       // window bins 2 t and 2 t + 1
    if (wave == kSelWaves - 1) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) open += __shfl_xor(open, d, 64);
        if (lane == 63u) w.y += open;            // the last bin also counts every key above the window
    }
    const uint32_t pair = w.x + w.y;
    const uint32_t pre = wave_scan_incl(pair);
    const uint32_t suf = wave_total(pre) - pre + pair;  // inclusive suffix sum: this thread's bins and all above
    if (lane == 0) wtot[wave] = suf;
    return {w.x, w.y, suf};
}
__device__ __forceinline__ void clear_window(const SparseScratch &sc)
{
    const uint32_t t = threadIdx.x;
    *reinterpret_cast<uint2 *>(sc.hist + kHistW + 2 * t) = uint2{0u, 0u};
    if (t >= (uint32_t)(kSelThreads - kOpenCopies)) sc.hist[kHistOpen + (t & 63u)] = 0u;
}
// verdict (8 words of LDS; [0] is 0): found, bin, entries to take from it (64 bits), candidates (64 bits), keys in the bin
__device__ __forceinline__ void find_bin(const WindowPart &part, uint64_t k, const uint32_t *wtot, uint32_t *verdict)
{
    const uint32_t t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), pair = part.lower + part.upper;
    uint32_t suf = part.above, higher = 0, all = 0;      // candidates in the wavefronts after this one; all candidates
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) { if ((uint32_t)w > wave) higher += wtot[w]; all += wtot[w]; }
    suf += higher;
    if ((uint64_t)suf >= k && (uint64_t)(suf - pair) < k) {      // the count crosses k in one of this thread's two bins
        const uint32_t above = suf - pair;
        const bool upper = (uint64_t)above + part.upper >= k;
        const uint64_t rest = k - above - (upper ? 0u : part.upper);
        verdict[0] = 1u; verdict[1] = 2u * t + (upper ? 1u : 0u); verdict[2] = (uint32_t)rest; verdict[3] = 0u;
        verdict[6] = upper ? part.upper : part.lower;
    }
    if (t == 0) { verdict[4] = all; verdict[5] = 0u; }
}
// The route, where it starts and how many entries it has to find; the group's first thread writes down what the next calls need.
__device__ __forceinline__ void record_verdict(const SparseJob &job, const uint32_t *verdict, uint32_t hint, uint32_t hint_shift, uint32_t hint_hold,
                                               uint32_t hint_cap, uint32_t &mode, uint32_t &lo, uint64_t &need)
{
    const SparseScratch &sc = job.sc;
    const uint64_t k = job.k;
    const bool found = verdict[0] != 0u;
    const uint32_t bin = verdict[1];
    const bool first = job.block == 0 && threadIdx.x == 0, fresh = first_call(hint, hint_cap);
    if (first && job.reports) {
        sc.sync[kSyncLastBin] = fresh ? job.g.n : found ? verdict[6] : 0u;          // diagnostics (mc_select_stats); before a first call
        sc.sync[kSyncLastCands] = fresh ? job.g.n : verdict[4];                     // nothing is filtered out
    }
    mode = found ? 0u : kModeUniform | (fresh ? kModeFirst : 0u);
    lo = found ? hint + (((uint32_t)kBinsW - 1u) << kWindowShift) : 0u;
    need = k;
    if (found && bin < (uint32_t)kBinsW - 1u) {
        lo = hint + (bin << kWindowShift);
        need = (uint64_t)verdict[2] | ((uint64_t)verdict[3] << 32);
        const bool lean = verdict[6] <= kUCap;
        mode = kModeFast | (lean ? kModeLean : kModeDense);
        if (first) margin_after_hit(sc.hint, hint_shift, hint_hold, hint_cap, (uint64_t)verdict[4] | ((uint64_t)verdict[5] << 32), k);
    } else if (first) {
        // missed: the next calls filter with the full margin again, and keep it for a while
        margin_after_miss(sc.hint, hint_shift, hint_cap, !found && !fresh);
    }
    if (first) {
        SelectState s;
        s.lo = lo; s.mode = mode; s.need = need;
        sc.sel[0] = s;
        const uint32_t route = (mode & kModeLean) ? MC_SELECT_FAST : (mode & kModeDense) ? MC_SELECT_DENSE : found || fresh ? MC_SELECT_ABOVE : MC_SELECT_REFILL;
        atomicAdd(&sc.sync[kSyncRoutes + route], 1u);
    }
}

// The select kernel: sixteen tiles per block, one wavefront each; the window is read once per block.  When the window does
// not settle the selection, the group's first blocks go on with the slow routes, which wait for one another: blocks
// start in the order of their numbers, so at most `sync_blocks` of them -- one per compute unit -- are held at once whatever
// the size of the group, and of several groups the earliest that is not done has all of its own running.
template <int ALGO, bool EF, class SRC>
__attribute__((amdgpu_waves_per_eu(8, 8)))
__global__ __launch_bounds__(kSelThreads) void lean_select_k(SRC src, RngKey rng, uint32_t sync_blocks, int *status)
{
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins1];      // (these three: slow routes)
    __shared__ uint32_t pfx[2 * kRoundTiles];
    __shared__ uint32_t small[64];
    __shared__ uint32_t wtot[kSelWaves];
    __shared__ uint32_t verdict[8];              // found, bin, rest lo, rest hi, candidates lo, hi, keys in the bin
    __shared__ UEntry members[kSelWaves][kMemberBuf];
    __shared__ uint32_t wabove[kSelWaves];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const SparseJob job = src.template job<BLK_SELECT>();
    const SparseScratch &sc = job.sc;
    const uint64_t k = job.k;
    const uint32_t ntiles = tiles_in(job.g.n);
    const uint32_t tile = job.block * kSelWaves + wave;
    // everything is asked for up front: what there is to know of the tile, the hint record, the window
    TileAhead a0;
    look_ahead(sc, tile, tile < ntiles, a0);
    const uint32_t hint = *sc.hint, hint_shift = sc.hint[kHintShift], hint_hold = sc.hint[kHintHold], hint_cap = sc.hint[kHintCap];
    uint32_t open = wave == kSelWaves - 1 ? sc.hist[kHistOpen + lane] : 0u;      // (the wavefront that holds the window's last bin)
    // (As in read_window, find_bin and record_verdict, written out here: called, they cost this kernel its last registers, and
    // with them a spill that the runtime answers with an allocation of its own on the first launch, a millisecond.)
    uint2 wsum = {0u, 0u};                       // window bins 2 t and 2 t + 1
#pragma unroll
    for (int r = 0; r < kWinCopies; ++r) {
        const uint2 x = *reinterpret_cast<const uint2 *>(sc.hist + kHistW + r * kBinsW + 2 * t);
        wsum.x += x.x; wsum.y += x.y;
    }
    // ---- the verdict: the bin b with  count(bins > b) < k <= count(bins >= b), by a suffix scan over the block's
    // threads (two bins each; the counts stay below 2^32, there being fewer elements than that)
    if (wave == kSelWaves - 1) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) open += __shfl_xor(open, d, 64);
        if (lane == 63u) wsum.y += open;         // the last bin also counts every key above the window
    }
    const uint32_t pair = wsum.x + wsum.y;
    const uint32_t pre = wave_scan_incl(pair);
    uint32_t suf = wave_total(pre) - pre + pair;  // inclusive suffix sum: this thread's bins and all above
    if (lane == 0) wtot[wave] = suf;
    if (t == 0) verdict[0] = 0u;
    __syncthreads();
    uint32_t higher = 0, all = 0;                // candidates in the wavefronts after this one; all candidates
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) { if ((uint32_t)w > wave) higher += wtot[w]; all += wtot[w]; }
    suf += higher;
    if ((uint64_t)suf >= k && (uint64_t)(suf - pair) < k) {      // the count crosses k in one of this thread's two bins
        const uint32_t above = suf - pair;
        const bool upper = (uint64_t)above + wsum.y >= k;
        const uint64_t rest = k - above - (upper ? 0u : wsum.y);
        verdict[0] = 1u; verdict[1] = 2u * t + (upper ? 1u : 0u); verdict[2] = (uint32_t)rest; verdict[3] = 0u;
        verdict[6] = upper ? wsum.y : wsum.x;
    }
    if (t == 0) { verdict[4] = all; verdict[5] = 0u; }
    __syncthreads();
    const bool found = verdict[0] != 0u;
    const uint32_t bin = verdict[1];
    const bool first = job.block == 0 && t == 0, fresh = first_call(hint, hint_cap);
    if (first && job.reports) {
        sc.sync[kSyncLastBin] = fresh ? job.g.n : found ? verdict[6] : 0u;          // diagnostics (mc_select_stats); before a first call
        sc.sync[kSyncLastCands] = fresh ? job.g.n : verdict[4];                     // nothing is filtered out
    }
    uint32_t mode = found ? 0u : kModeUniform | (fresh ? kModeFirst : 0u), lo = found ? hint + (((uint32_t)kBinsW - 1u) << kWindowShift) : 0u;
    uint64_t need = k;
    if (found && bin < (uint32_t)kBinsW - 1u) {
        lo = hint + (bin << kWindowShift);
        need = (uint64_t)verdict[2] | ((uint64_t)verdict[3] << 32);
        const bool lean = verdict[6] <= kUCap;
        mode = kModeFast | (lean ? kModeLean : kModeDense);
        if (first) margin_after_hit(sc.hint, hint_shift, hint_hold, hint_cap, (uint64_t)verdict[4] | ((uint64_t)verdict[5] << 32), k);
    } else if (first) {
        // missed: the next calls filter with the full margin again, and keep it for a while
        margin_after_miss(sc.hint, hint_shift, hint_cap, !found && !fresh);
    }
    if (first) {
        SelectState s;
        s.lo = lo; s.mode = mode; s.need = need;
        sc.sel[0] = s;
        const uint32_t route = (mode & kModeLean) ? MC_SELECT_FAST : (mode & kModeDense) ? MC_SELECT_DENSE : found || fresh ? MC_SELECT_ABOVE : MC_SELECT_REFILL;
        atomicAdd(&sc.sync[kSyncRoutes + route], 1u);
    }
    if (mode & kModeLean) {
        uint32_t above = 0;
        if (tile < ntiles) {
            const uint32_t sub = tile & (uint32_t)(kUSub - 1);
            MemberBuf mb{members[wave], 0u};
            above = select_tile(sc, a0, lo, sub, mb);
            flush_members(sc, mb, sub);
        }
        // keys above the bin in this block's sixteen tiles
        if (lane == 0) wabove[wave] = above;
        __syncthreads();
        if (t == 0) {
            uint32_t sum = 0;
#pragma unroll
            for (int w = 0; w < kSelWaves; ++w) sum += wabove[w];
            sc.blk_cnt[job.block] = sum;                          // sixteen tiles hold at most 65536 candidates
        }
        return;
    }
    const uint32_t blocks = job.blocks < sync_blocks ? job.blocks : sync_blocks;
    if (job.block < blocks)
        slow_routes<ALGO, EF, ALGO == MC_ALGO_DGC || EF, ALGO == MC_ALGO_RANDK>(job, rng, mode, lo, need, blocks, status, hist, pfx, small);
}

// Emit: four tiles per block, one wavefront each.  Every block reads the whole list of the keys in the threshold's
// bin (it is small), finds the threshold key T and the number of keys equal to T to take with a histogram in LDS,
// counts the list's kept keys that lie before each of its tiles, adds the keys above the bin in the tiles before,
// and compacts its tiles' kept candidates into the payload.  The heads of the tile's chunks and the first entries
// of every sublist are asked for together with everything else, so the usual tile costs one memory latency.
// Consecutive entries that a thread of an emit block fetches before the sublists' lengths are known, four threads per
// sublist: a list of a few hundred keys (9 per sublist) is then complete after the first level of loads.  Measured
// with 1 / 2 / 4 / 8: emit 13.6 / 13.5 / 13.0 / 13.8 us on the bench's Top-k, whole compress 82.7 / 82.1 / 80.1 / 78.0
// where the bin holds 2500 keys (tensors of one scale), DGC and Rand-k +1 us with 8 (68 registers instead of 60).
constexpr int kUPer = 4;
constexpr int kUSpec = 4 * kUPer;      // ... which covers the first kUSpec entries of every sublist
static_assert(4 * kUSub == kEmitThreads, "four threads per sublist");

template <int ALGO, bool EF, class SRC>
__global__ __launch_bounds__(kEmitThreads) void lean_emit_k(SRC src)
{
    __shared__ uint32_t hist[kBins3], coarse[64];          // the listed keys' 11 open bits, and the same 32 bins at a time
    __shared__ uint32_t small[4];
    __shared__ uint32_t ulen[kUSub], upre[kUSub + 1];
    __shared__ uint32_t cgt[kEmitWaves + 1], ceq[kEmitWaves + 1];
    __shared__ uint32_t red[kEmitWaves];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const SparseJob job = src.template job<BLK_EMIT>();
    const SparseScratch &sc = job.sc;
    float *st = job.st;
    PayloadHeader *hdr = job.hdr;
    const uint32_t k = (uint32_t)job.k;
    const uint32_t n = job.g.n, ntiles = tiles_in(n);
    const uint32_t tile = job.block * kEmitWaves + wave;
    const bool live = tile < ntiles;
    // ---- everything that needs no other load to be located is asked for now
    const uint64_t runs = live ? sc.tile_runs[tile] : 0ull;
    const SelectState s0 = sc.sel[0];
    const uint32_t ucnt = wave == 0 ? sc.ucount[lane * kUCountStride] : 0u;
    // entries (t % 4) kUPer ... of sublist t / 4, if it has that many.  (A group of fewer tiles than kUSub has as many
    // sublists as tiles; what is read past them, of the next groups' or of the padding behind the last, is not used.
    // A condition around these loads cost the kernel 0.8 us of 11.)
    UEntry spec[kUPer];
#pragma unroll
    for (int i = 0; i < kUPer; ++i) spec[i] = sc.ulist[(size_t)(t / 4u) * kUCap + (t % 4u) * kUPer + i];
    uint32_t hb[kWavesPerBlock], hl[kWavesPerBlock];
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) {
        hb[q] = live ? load_head_bits(sc, tile * kWavesPerBlock + q) : 0u;
        hl[q] = live ? load_head_loc(sc, tile * kWavesPerBlock + q) : 0u;
    }
    // ... and, as soon as the counts are there, the first four units of a tile with crowded chunks (nearly always all it has)
    uint32_t cnt[kWavesPerBlock];
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) cnt[q] = (uint32_t)(runs >> (16 * q)) & 0xFFFFu;
    const TileUnits tu(cnt);
    uint4 kb[4];
    uint2 kl[4];
    uint32_t kq[4], kv[4];
    if (tu.total) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tu.locate((uint32_t)i < tu.total ? (uint32_t)i : 0u, kq[i], kv[i]);
            kb[i] = load_bits4(sc, tile * kWavesPerBlock + kq[i], kv[i]);
            kl[i] = load_loc4(sc, tile * kWavesPerBlock + kq[i], kv[i]);
        }
    }
    // keys above the bin in the select blocks (sixteen tiles each) before this tile's, then in the tiles before it in its own
    const uint32_t sblock = tile / (uint32_t)kSelWaves, sfirst = sblock * (uint32_t)kSelWaves;
    uint32_t before = 0;
    for (uint32_t b = t; b < job.block / (uint32_t)(kSelWaves / kEmitWaves); b += kEmitThreads) before += sc.blk_cnt[b];
    uint32_t mine = live && sfirst + lane < tile ? sc.tile_cnt[sfirst + lane] : 0u;
    // the select kernel is done with the window: all blocks clear it together
    for (uint32_t b = job.block * kEmitThreads + t; b < (uint32_t)(kWinCopies * kBinsW + kOpenCopies); b += job.blocks * kEmitThreads)
        sc.hist[b < (uint32_t)(kWinCopies * kBinsW) ? kHistW + b : kHistOpen - kWinCopies * kBinsW + b] = 0u;
    if (!(s0.mode & kModeLean)) return;                 // (the slow routes have written the payload themselves)
    const uint32_t lo = s0.lo;
    // ---- the list
    if (wave == 0) {
        const uint32_t len = min(ucnt, kUCap);
        ulen[lane] = len;
        const uint32_t inc = wave_scan_incl(len > (uint32_t)kUSpec ? len - (uint32_t)kUSpec : 0u);      // entries beyond the speculative ones, scanned
        upre[lane + 1] = inc;
        if (lane == 0) upre[0] = 0u;
    }
    for (int b = t; b < kBins3; b += kEmitThreads) hist[b] = 0u;
    if (t < 64u) coarse[t] = 0u;
    if (t <= (uint32_t)kEmitWaves) { cgt[t] = 0u; ceq[t] = 0u; }
    __syncthreads();
    const uint32_t spec_n = ulen[t / 4u] > (t % 4u) * kUPer ? min(ulen[t / 4u] - (t % 4u) * kUPer, (uint32_t)kUPer) : 0u;      // of spec[], this many exist
    const uint32_t more = min(upre[kUSub], kUCap);       // (nothing, when no sublist holds more than kUSpec entries)
    // further entry e: entry kUSpec + (e - upre[s]) of the sublist s that is the last to start at or before e
    auto further = [&](uint32_t e) {
        uint32_t sl = 0;
#pragma unroll
        for (int step = kUSub / 2; step >= 1; step >>= 1) if (upre[sl + step] <= e) sl += step;
        return sc.ulist[(size_t)sl * kUCap + kUSpec + (e - upre[sl])];
    };
    auto tally = [&](uint32_t bits) {
        const uint32_t d = (bits & 0x7FFFFFFFu) - lo;
        if (d < (uint32_t)kBins3) { atomicAdd(&hist[d], 1u); atomicAdd(&coarse[d >> 5], 1u); }
    };
#pragma unroll
    for (int i = 0; i < kUPer; ++i) if ((uint32_t)i < spec_n) tally(spec[i].bits);
    for (uint32_t e0 = t; e0 < more; e0 += 4 * kEmitThreads) {        // (four loads in flight)
        UEntry x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) if (e0 + i * kEmitThreads < more) x[i] = further(e0 + i * kEmitThreads);
#pragma unroll
        for (int i = 0; i < 4; ++i) if (e0 + i * kEmitThreads < more) tally(x[i].bits);
    }
    __syncthreads();
    // threshold key and the number of keys equal to it to take: the key at which the count from the top reaches
    // s0.need, first among the 64 coarse bins, then among the 32 keys of that one
    if (wave == 0) {
        const uint32_t want = (uint32_t)s0.need;           // (at most kUCap)
        const uint32_t c = coarse[lane];
        const uint32_t cpre = wave_scan_incl(c);
        const uint32_t suf = wave_total(cpre) - cpre + c;          // from the top
        const uint64_t hit = __builtin_amdgcn_ballot_w64(suf >= want && suf - c < want);
        uint32_t b = 0, r = 0;
        if (hit) {
            const uint32_t cl = (uint32_t)__builtin_ctzll(hit);
            const uint32_t left = want - (__shfl(suf, cl, 64) - __shfl(c, cl, 64));      // to take inside the coarse bin
            const uint32_t f = lane < 32u ? hist[32u * cl + lane] : 0u;
            const uint32_t fpre = wave_scan_incl(f);
            const uint32_t fs = wave_total(fpre) - fpre + f;
            const uint64_t hit2 = __builtin_amdgcn_ballot_w64(lane < 32u && fs >= left && fs - f < left);
            if (hit2) {
                const uint32_t fl = (uint32_t)__builtin_ctzll(hit2);
                b = 32u * cl + fl;
                r = left - (__shfl(fs, fl, 64) - __shfl(f, fl, 64));
            }
        }
        if (lane == 0) { small[0] = b; small[1] = r; }       // (an inconsistent list: T = lo, nothing equal taken)
    }
    __syncthreads();
    const uint32_t T = lo + small[0], need = small[1];
    // the list's kept keys, by where they lie: before this block, or in its tile j (bucket j + 1)
    const uint32_t first = job.block * (uint32_t)(kEmitWaves * kTile);
    auto classify = [&](const UEntry &x) {
        const uint32_t key = x.bits & 0x7FFFFFFFu;
        if (key >= T) {
            const uint32_t bucket = x.idx < first ? 0u : ((x.idx - first) >> 12) + 1u;
            if (bucket <= (uint32_t)kEmitWaves) atomicAdd(key > T ? &cgt[bucket] : &ceq[bucket], 1u);
        }
    };
#pragma unroll
    for (int i = 0; i < kUPer; ++i) if ((uint32_t)i < spec_n) classify(spec[i]);
    for (uint32_t e0 = t; e0 < more; e0 += 4 * kEmitThreads) {
        UEntry x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) if (e0 + i * kEmitThreads < more) x[i] = further(e0 + i * kEmitThreads);
#pragma unroll
        for (int i = 0; i < 4; ++i) if (e0 + i * kEmitThreads < more) classify(x[i]);
    }
    before = wave_total(wave_scan_incl(before));          // (sums of candidates: below 2^32)
    mine = wave_total(wave_scan_incl(mine));
    if (lane == 0) red[wave] = before;
    __syncthreads();
    if (job.block == 0 && t == 0) { put_sparse_header(hdr, ALGO, n, k); publish_hint(sc, T); record_sent_key<ALGO, EF>(st, T); }
    if (!live) return;
    uint32_t gt0 = mine;
    uint32_t eq0;
#pragma unroll
    for (int w = 0; w < kEmitWaves; ++w) gt0 += red[w];
    {
        uint32_t g2 = 0, e2 = 0;                            // the list's kept keys before this tile: buckets 0 .. wave
#pragma unroll
        for (int b = 0; b <= kEmitWaves; ++b) if ((uint32_t)b <= wave) { g2 += cgt[b]; e2 += ceq[b]; }
        gt0 += g2; eq0 = e2;
    }
    uint32_t *idx = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(hdr) + kHeaderBytes);
    float *val = reinterpret_cast<float *>(idx + k);
    if (lane == 0) {
        uint32_t *dir = payload_directory(hdr, k);
        dir[tile] = gt0 + (eq0 < need ? eq0 : need);
        if (tile == ntiles - 1u) dir[ntiles] = k;              // (the selection keeps exactly k)
    }
    if (tu.total == 0) {
        // the usual tile: no chunk holds more than 64 candidates, and they are all here
#pragma unroll
        for (int q = 0; q < kWavesPerBlock; ++q)
            if (cnt[q]) emit_head<ALGO, EF>(hb[q], hl[q], lane < cnt[q], tile * kWavesPerBlock + q, n, k, st, idx, val, T, need, gt0, eq0);
        return;
    }
    // A tile with crowded chunks: its pieces -- the head of chunk 0, its units, the head of chunk 1, ... -- are placed in
    // index order, the counts of kept keys running along.  Up to four units, nearly every such tile, were fetched at
    // the start; a tile with more fetches them four at a time.  One copy of the unit's code in a loop that is not
    // unrolled: sixteen unrolled copies were 2 us slower (code size), and counting all pieces first, scanning the counts
    // and fetching the units of a very crowded tile a second time 1.3 us slower (Top-k emit 13.0 -> 11.7 us).
    uint32_t e = 0;                                         // next unit of the tile
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) {
        const uint32_t cq = cnt[q];
        if (!cq) continue;
        emit_head<ALGO, EF>(hb[q], hl[q], lane < cq, tile * kWavesPerBlock + q, n, k, st, idx, val, T, need, gt0, eq0);
        const uint32_t nu = tu.per[q];
#pragma unroll 1
        for (uint32_t v = 0; v < nu; ++v, ++e) {
            if (e >= 4u && (e & 3u) == 0u) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    tu.locate(e + i < tu.total ? e + i : e, kq[i], kv[i]);
                    kb[i] = load_bits4(sc, tile * kWavesPerBlock + kq[i], kv[i]);
                    kl[i] = load_loc4(sc, tile * kWavesPerBlock + kq[i], kv[i]);
                }
            }
            // unit e % 4 of the four in registers, chosen word by word (an array indexed at run time would live in scratch memory)
            const uint32_t s = e & 3u;
            auto sel = [s](uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) { return s == 0u ? a0 : s == 1u ? a1 : s == 2u ? a2 : a3; };
            uint4 b;
            b.x = sel(kb[0].x, kb[1].x, kb[2].x, kb[3].x); b.y = sel(kb[0].y, kb[1].y, kb[2].y, kb[3].y);
            b.z = sel(kb[0].z, kb[1].z, kb[2].z, kb[3].z); b.w = sel(kb[0].w, kb[1].w, kb[2].w, kb[3].w);
            uint2 l;
            l.x = sel(kl[0].x, kl[1].x, kl[2].x, kl[3].x); l.y = sel(kl[0].y, kl[1].y, kl[2].y, kl[3].y);
            emit_unit<ALGO, EF>(b, l, cq, v, tile * kWavesPerBlock + q, n, k, st, idx, val, T, need, gt0, eq0);
        }
    }
}

// ---------------------------------------------------------------------------
// Select and emit of a small group (kSmallSelTiles tiles, kSmallKept entries) in one kernel.  On such a
// group the two kernels do next to nothing but start, read the window and wait for two levels of loads, each.  One
// block can hold all candidates, 16 per thread in index order, and needs no list and no counts in memory: the
// window's verdict, a histogram of the threshold's bin in LDS, a scan over the block's wavefronts, and the entries are
// written.  The candidates are asked for as soon as the chunks' counts are known, while the verdict is found.
// (Compress, the streaming pass included, two kernels -> one.  Top-k 1 % of 1 / 8 / 17 / 32 tiles: 15.3 / 14.9 / 14.9 /
// 14.9 -> 9.6 / 10.0 / 10.6 / 11.9 us, 4 % 18.2 / 19.2 / 19.8 / 20.0 -> 9.8 / 11.6 / 13.6 / 16.8, 131 of 32 tiles 14.5 -> 10.0, 6029 of them
// 21.4 -> 18.0; DGC 0.1 % of 16 tiles 14.8 -> 10.3; Rand-k 1 % of 1 / 16 / 32 tiles 26.1 / 25.4 / 21.2 -> 19.8 / 16.4 / 16.7.)
// What the window does not settle, or more candidates than the block holds, goes the way of the slow routes, on
// small_sel_blocks() blocks, which on the usual route do nothing but read the window.  (By the group's first block alone, as up
// to 8 tiles, a group of 17 to 32 tiles took longer there than with the two kernels.  First call of a context, 17 / 24 / 32 tiles, Top-k:
// two kernels 51.5 / 55.5 / 61.3 us, one block 55.3 / 66.7 / 81.0, one block for every four tiles 40.7 / 40.8 / 41.6; Rand-k 5 % of 17 /
// 24 / 32 tiles, where every few calls miss the window: 40 / 31 / 37, 46 / 42 / 56, 33 / 29 / 32.)
// (More candidates than the block holds take an eighth or more of the group's elements just below the threshold, as the full margin
// meets them in the calls after a miss: 32 tiles, 22 000 / 47 000 candidates, a rise, a refill and eight such calls 25.8 / 34.1 us each
// with two kernels, 27.8 / 36.9 now.)
// ---------------------------------------------------------------------------
// Candidates per thread: up to two, found by bisection, seven looks at the chunks' starts each; or up to 16, found chunk by chunk,
// which takes longer where a chunk has few.  (Top-k compress, bisection for up to
// 8192 candidates / chunk by chunk beyond 1024 / the rule: 32 tiles, 720 candidates 10.1 / 9.7 / 9.8 us, 1950 11.5 / 12.5 / 11.7, 6300 15.8 /
// 16.0 / 15.9.  Asked for one after the other, each with a wait of its own: 9.9, 12.3, 19.1, and 24.4 instead of 18.0 for 10 900.)
constexpr int kFewRounds = 2, kManyRounds = 16;
constexpr uint32_t kFewCands = (uint32_t)kFewRounds * kSelThreads, kManyCands = (uint32_t)kManyRounds * kSelThreads;
static_assert(kSmallSelTiles * kWavesPerBlock == 128 && kManyCands <= 0xFFFFu, "");

// job: small_sel_blocks() blocks, of which the first one selects and emits.  MOST: tiles that the group may have.
template <int ALGO, bool EF, int MOST>
__device__ __forceinline__ void small_tail(SparseJob job, RngKey rng, uint32_t sync_blocks, int *status, uint32_t *hist /* LDS: kBins1, */,
                                           uint32_t *pfx /* 2 * kRoundTiles (slow routes), */, uint32_t *small /* 64 words */)
{
    __shared__ uint32_t wtot[kSelWaves], verdict[8];
    __shared__ uint32_t from[kSmallSelTiles * kWavesPerBlock + 1];      // candidates of the group before each chunk
    __shared__ uint32_t kept[kSmallSelTiles];    // entries in each tile
    __shared__ uint32_t clears;
    const uint32_t n = job.g.n;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const SparseScratch &sc = job.sc;
    const uint32_t k = (uint32_t)job.k, ntiles = tiles_in(n);
    const uint64_t runs = wave == 0 && lane < ntiles ? sc.tile_runs[lane] : 0ull;
    const uint32_t hint = *sc.hint, hint_shift = sc.hint[kHintShift], hint_hold = sc.hint[kHintHold], hint_cap = sc.hint[kHintCap];
    const uint32_t open = wave == kSelWaves - 1 ? sc.hist[kHistOpen + lane] : 0u;
    const WindowPart part = read_window(sc, open, wtot);
    for (int b = t; b < kBins3; b += kSelThreads) hist[b] = 0u;
    if (t == 0) verdict[0] = 0u;
    if (wave == 0) {
        const uint32_t total = runs_total(runs), incl = wave_scan_incl(total);
        if (lane < (uint32_t)kSmallSelTiles) {
            uint32_t at = incl - total;
#pragma unroll
            for (int q = 0; q < kWavesPerBlock; ++q) { from[kWavesPerBlock * lane + q] = at; at += (uint32_t)(runs >> (16 * q)) & 0xFFFFu; }
            kept[lane] = 0u;
            if (lane == kSmallSelTiles - 1u) from[kWavesPerBlock * kSmallSelTiles] = at;
        }
    }
    __syncthreads();
    // The window is read by all blocks of the group: the last of them clears it.
    uint32_t readers = job.blocks;
    if (t == 0 && job.blocks > 1u) readers = 1u + __hip_atomic_fetch_add(sc.arrive + kArriveWindow, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t N = from[kWavesPerBlock * kSmallSelTiles];
    uint32_t mode = 0, lo = 0, T = 0;
    uint64_t need = 0;
    // The route, behind the candidates' loads; true if it is the usual one and the block holds the candidates.
    auto usual = [&] {
        find_bin(part, k, wtot, verdict);
        if (t == 0) clears = readers == job.blocks ? 1u : 0u;
        __syncthreads();
        if (clears) clear_window(sc);
        record_verdict(job, verdict, hint, hint_shift, hint_hold, hint_cap, mode, lo, need);
        if (N > kManyCands && (mode & kModeLean)) mode = kModeFast | kModeDense;
        return (mode & kModeLean) != 0u;
    };
    auto finish = [&](auto form) {
        constexpr bool MANY = decltype(form)::value;
        constexpr int ROUNDS = MANY ? kManyRounds : kFewRounds;
        // Candidates wave * 64 rounds ... are the wavefront's, 64 a round, all asked for at once.
        const uint32_t rounds = min((N + kSelThreads - 1u) / kSelThreads, (uint32_t)ROUNDS), first = wave * 64u * rounds + lane;
        uint32_t bits[ROUNDS], loc[ROUNDS], chunks[(ROUNDS + 3) / 4];      // (a chunk's number is below 128)
        auto load = [&](int r, uint32_t ch, uint32_t in) {
            const uint32_t slot = ch * (uint32_t)kChunk + in;
            bits[r] = sc.cand_bits[slot];
            loc[r] = sc.cand_loc[slot];          // (added to the chunk's start where it is used: not waited for here)
            chunks[r / 4] = r % 4 ? chunks[r / 4] | ch << (8 * (r % 4)) : ch;
        };
        auto chunk = [&](int r) { return chunks[r / 4] >> (8 * (r % 4)) & 0xFFu; };
        if (job.block == 0 && N - 1u < kManyCands) {
            if (!MANY) {                         // by bisection: seven looks a round, or five
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) {
                    if ((uint32_t)r < rounds) {
                        const uint32_t p = min(first + 64u * r, N - 1u);
                        uint32_t ch = 0;         // the last chunk that starts at or before p
#pragma unroll
                        for (uint32_t step = kWavesPerBlock * MOST / 2; step >= 1; step >>= 1) if (from[ch + step] <= p) ch += step;
                        load(r, ch, p - from[ch]);
                    }
                }
            } else {                             // chunk after chunk: a round has hardly more than one
                const uint32_t start[2] = {from[lane], from[64u + lane]}, end[2] = {from[lane + 1u], from[65u + lane]};
                auto of = [](const uint32_t (&x)[2], uint32_t c) { return (uint32_t)__builtin_amdgcn_readlane((int)(c < 64u ? x[0] : x[1]), (int)(c & 63u)); };
                const uint32_t p0 = min(first - lane, N - 1u);
                uint32_t c = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(start[0] <= p0)) + (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(start[1] <= p0)) - 1u;
                uint32_t beg = of(start, c), lim = of(end, c);
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) {
                    if ((uint32_t)r < rounds) {
                        const uint32_t p = min(first + 64u * r, N - 1u), last = min(first - lane + 64u * r + 63u, N - 1u);
                        uint32_t ch = c, at = beg;
                        while (lim <= last) {    // another chunk's candidates start in this round
                            ++c;
                            beg = lim;
                            lim = of(end, c);
                            ch = p >= beg ? c : ch;
                            at = p >= beg ? beg : at;
                        }
                        load(r, ch, p - at);
                    }
                }
            }
        }
        if (!usual()) return false;
        if (job.block) return true;
        // ---- the threshold key, and the number of keys equal to it to take
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if ((uint32_t)r < rounds) {
                const uint32_t key = bits[r] & 0x7FFFFFFFu;
                if (first + 64u * r < N && key >= lo && key - lo < (uint32_t)kBins3) atomicAdd(&hist[key - lo], 1u);
            }
        }
        __syncthreads();
        uint32_t bin;
        resolve_block<kBins3>(hist, need, bin, need, small, small + 8);
        T = lo + bin;
        // ---- keys above / equal to it before this wavefront's (16 bits each: there are 16384 candidates at most)
        uint32_t both = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if ((uint32_t)r < rounds) {
                const uint32_t key = bits[r] & 0x7FFFFFFFu;
                const bool valid = first + 64u * r < N;
                both += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(valid && key > T)) + ((uint32_t)__popcll(__builtin_amdgcn_ballot_w64(valid && key == T)) << 16);
            }
        }
        if (lane == 0) wtot[wave] = both;
        __syncthreads();
        const uint32_t v = lane < (uint32_t)kSelWaves ? wtot[lane] : 0u, before = (uint32_t)__builtin_amdgcn_readlane((int)(wave_scan_incl(v) - v), (int)wave);
        uint32_t gt0 = before & 0xFFFFu, eq0 = before >> 16;
        uint32_t *idx = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(job.hdr) + kHeaderBytes);
        float *val = reinterpret_cast<float *>(idx + k);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if ((uint32_t)r < rounds &&
                emit_head<ALGO, EF>(bits[r], loc[r], first + 64u * r < N, chunk(r), n, k, job.st, idx, val, T, (uint32_t)need, gt0, eq0))
                atomicAdd(&kept[chunk(r) / (uint32_t)kWavesPerBlock], 1u);
        __syncthreads();
        return true;
    };
    if (!(N <= kFewCands ? finish(std::false_type{}) : finish(std::true_type{}))) {
        const uint32_t blocks = min(job.blocks, sync_blocks);
        if (job.block < blocks)
            slow_routes<ALGO, EF, ALGO == MC_ALGO_DGC || EF, ALGO == MC_ALGO_RANDK>(job, rng, mode, lo, need, blocks, status, hist, pfx, small);
        return;
    }
    if (job.block) return;
    if (wave == 0) {
        const uint32_t own = lane < (uint32_t)kSmallSelTiles ? kept[lane] : 0u, incl = wave_scan_incl(own);
        uint32_t *dir = payload_directory(job.hdr, k);
        if (lane < ntiles) dir[lane] = incl - own;
        if (lane == 0) {
            dir[ntiles] = k;                     // (the selection keeps exactly k)
            put_sparse_header(job.hdr, ALGO, n, k);
            publish_hint(sc, T);
            record_sent_key<ALGO, EF>(job.st, T);
        }
    }
}

template <int ALGO, bool EF, class SRC>
__global__ __launch_bounds__(kSelThreads) void lean_small_k(SRC src, RngKey rng, uint32_t sync_blocks, int *status)
{
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins1];
    __shared__ uint32_t pfx[2 * kRoundTiles], small[64];
    const SparseJob job = src.small_job();
    if (job.block >= job.blocks) return;
    small_tail<ALGO, EF, kSmallSelTiles>(job, rng, sync_blocks, status, hist, pfx, small);
}

template <int ALGO, bool EF, class SRC>
static void sparse_compress_t(const LaunchCtx &lc, const SRC &src, const SparseBlocks &nb, const SparseCall &call)
{
    const RngKey rng{call.seed, call.worker, call.iter_lo};
    // the slow routes run on blocks that the device holds at once: one per compute unit
    const uint32_t sync = std::max(1u, std::min(call.sync_blocks, (uint32_t)(kRoundTiles / kSelWaves)));
    if (nb.same) {
        MC_LAUNCH((sparse_accum_k<ALGO, EF, SRC, kSpreadSteps, true>), dim3(nb.tiles), dim3(kSpread), lc, src, call.momentum, rng, call.status);      // (the profiler is off)
        return;
    }
    prof_begin(lc, K_SPARSE_ACCUM);
    if (nb.tiles <= kSpreadTiles) MC_LAUNCH((sparse_accum_k<ALGO, EF, SRC, kSpreadSteps>), dim3(nb.tiles), dim3(kSpread), lc, src, call.momentum, rng, (SampleRule{0u, 0u, 0u}));
    else MC_LAUNCH((sparse_accum_k<ALGO, EF, SRC>), dim3(nb.tiles), dim3(kBlock), lc, src, call.momentum, rng, (SampleRule{0u, 0u, 0u}));
    prof_end(lc, K_SPARSE_ACCUM);
    if (nb.small) {
        MC_LAUNCH((lean_small_k<ALGO, EF, SRC>), dim3(nb.small), dim3(kSelThreads), lc, src, rng, sync, call.status);      // (the profiler is off)
        return;
    }
    // the two-kernel tail
    prof_begin(lc, K_LEAN_SELECT);
    MC_LAUNCH((lean_select_k<ALGO, EF, SRC>), dim3(nb.select), dim3(kSelThreads), lc, src, rng, sync, call.status);
    prof_end(lc, K_LEAN_SELECT);
    prof_begin(lc, K_LEAN_EMIT);
    MC_LAUNCH((lean_emit_k<ALGO, EF, SRC>), dim3(nb.emit), dim3(kEmitThreads), lc, src);
    prof_end(lc, K_LEAN_EMIT);
}

// DGC with a sampled threshold, one group: src.k is the payload's capacity, the threshold the sample_need-th largest key of the
// sample, which starts at sample_first
static void sampled_dgc(const LaunchCtx &lc, const OneSparse &src, const SparseCall &call)
{
    const GroupView &g = src.g;
    const SparseScratch &sc = src.sc;
    const RngKey rng{call.seed, call.worker, call.iter_lo};
    const uint32_t stride = call.sample_stride;
    const SampleRule smp{stride, call.sample_first, stride > 1 ? (uint32_t)((1ull << 32) / stride) : 0u};
    const uint32_t nt = tiles_in(g.n), nch = chunks_of(g.n);
    const uint32_t sblocks = (nch + 15) / 16 < 256 ? (nch + 15) / 16 : 256;      // enough to stream the group in a refill
    dim3 block(kBlock), cgrid((nt + kWavesPerBlock - 1) / kWavesPerBlock);
    prof_begin(lc, K_SPARSE_ACCUM);
    MC_LAUNCH((sparse_accum_k<MC_ALGO_DGC, true, OneSparse>), dim3(nt), block, lc, src, call.momentum, rng, smp);
    prof_end(lc, K_SPARSE_ACCUM);
    prof_begin(lc, K_SPARSE_SEED);
    MC_LAUNCH(sparse_seed_k, dim3(sblocks), dim3(kSeedThreads), lc, g.n, src.st, call.sample_need, sc, smp);
    prof_end(lc, K_SPARSE_SEED);
    prof_begin(lc, K_CAND_HIST2);
    MC_LAUNCH(cand_hist_k<2>, cgrid, block, lc, g.n, nt, sc, smp);
    prof_end(lc, K_CAND_HIST2);
    prof_begin(lc, K_CAND_HIST3);
    MC_LAUNCH(cand_hist_k<3>, cgrid, block, lc, g.n, nt, sc, smp);
    prof_end(lc, K_CAND_HIST3);
    prof_begin(lc, K_CAND_COUNT);
    MC_LAUNCH(cand_count_k, cgrid, block, lc, g.n, nt, sc);
    prof_end(lc, K_CAND_COUNT);
    prof_begin(lc, K_CAND_EMIT);
    MC_LAUNCH(cand_emit_k, cgrid, block, lc, g.n, nt, src.st, src.hdr, src.k, sc);
    prof_end(lc, K_CAND_EMIT);
}

template <class SRC>
void launch_sparse_compress(const LaunchCtx &lc, int algo, const SRC &src, const SparseBlocks &nb, bool ef, const SparseCall &call)
{
    if (nb.tiles == 0) return;
    // (the sampled threshold is taken group by group: compress_all never asks for it)
    if constexpr (std::is_same_v<SRC, OneSparse>) if (algo == MC_ALGO_DGC && call.sample_stride) { sampled_dgc(lc, src, call); return; }
    if (algo == MC_ALGO_DGC) sparse_compress_t<MC_ALGO_DGC, true>(lc, src, nb, call);
    else if (algo == MC_ALGO_RANDK) sparse_compress_t<MC_ALGO_RANDK, true>(lc, src, nb, call);
    else if (ef) sparse_compress_t<MC_ALGO_TOPK, true>(lc, src, nb, call);
    else sparse_compress_t<MC_ALGO_TOPK, false>(lc, src, nb, call);
}
template void launch_sparse_compress<OneSparse>(const LaunchCtx &, int, const OneSparse &, const SparseBlocks &, bool, const SparseCall &);
template void launch_sparse_compress<AllSparse>(const LaunchCtx &, int, const AllSparse &, const SparseBlocks &, bool, const SparseCall &);

// ---------------------------------------------------------------------------
// Sparse decompress-and-sum.  Every worker's indices ascend, so a 4096-element output tile owns one contiguous run of
// each list, and the directory that ends a payload says where that run starts and ends.  A wavefront accumulates its
// chunk of the tile in LDS of its own, one worker after the other in ascending worker order -- the same order of fp32
// additions as a dense sum, since adding the +0 of an absent entry changes nothing -- and writes it once.  No atomics in
// memory, no pre-zeroed output, no block barrier, bit-reproducible.
// The LDS operations of one wavefront are carried out in the order issued, so a worker's additions see the ones before.
// (A directory replaced a kernel that recorded the runs of all payloads in per-call tables before this one could start: 5 of
// 38 us.  Before, the block's wavefronts shared a tile's entries of a worker where one had more than 64, with a read, an
// addition, a write and a block barrier per worker: 25.6 M elements, 8 workers, Top-k 1 % 26.0 us, now 22.9 (21.7 if nothing
// was sent at all), 5 % 59 / 37, 16 workers 34 / 25.9; 44.5 M heavy-tailed in four calls 59 / 52.6.  With LDS additions that
// return nothing instead of a read, an addition and a write: 40, exact too, but about a lane per clock.)
// ---------------------------------------------------------------------------
constexpr int kSparseBatch = 8;    // workers whose entries are in flight together
constexpr int kFewWorkers = 6;
constexpr uint32_t kNear = 768u;   // longest run of which add_entries<.., true> looks for the chunk's part where it ought to be
constexpr int kSparseRounds = 4;   // rounds of 64 entries of a chunk's run, of half as many workers, where a run has more than 128

// Entries from[b] .. from[b] + len[b] - 1 of workers b0 .. b0 + NB - 1 of a batch, ROUNDS of 64 of each asked for at once; of
// these, those in the chunk at `base` are added to its sums.  No load and no addition is under a condition: a lane without an
// entry reads the run's last one (of an empty run what lies in the payload where it would start) and adds it to a word
// that nobody reads.  (With conditions every load waited for the one before, the registers of one path being taken for those
// of another.)
// NEAR: of a run longer than that, the ROUNDS of 64 around the place where the chunk's part lies if the run is spread evenly
// over the tile.  Whether they hold all of it, their first and last entry say; false, and nothing added, if not.
template <int NB, int ROUNDS, bool NEAR = false>
__device__ __forceinline__ bool add_entries(const uint8_t *const (&pl)[kSparseBatch], int b0, uint32_t k, const uint32_t (&from)[kSparseBatch],
                                            const uint32_t (&len)[kSparseBatch], uint32_t base, float *sums /* LDS, kChunk and a word that nobody reads */)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t ix[NB][ROUNDS];
    float vv[NB][ROUNDS];
    // (Ordinary loads: the tile's four wavefronts read the same lines, and neighbouring tiles share theirs.  As non-temporal
    // loads each went to memory, behind the stores: 25.6 M elements, 8 workers, Top-k 1 % 31.3 us, then 27.3; thinly spread
    // payloads (Rand-k) 34.3, then 26.1; 44.5 M heavy-tailed ones 50.1, then 39.3.)
    constexpr uint32_t kMost = 64u * ROUNDS;
    const uint32_t eighth = 2u * (base / (uint32_t)kChunk % (uint32_t)kWavesPerBlock) + 1u;      // the chunk's middle, in eighths of the tile
    auto skipped = [&](int b) {                  // entries of the run before those that are looked at
        const uint32_t n = len[b0 + b], middle = n * eighth >> 3;
        return n <= kMost || middle <= kMost / 2 ? 0u : min(middle - kMost / 2, n - kMost);
    };
    auto fetch = [&](int b, uint32_t at) {
        const uint32_t n = len[b0 + b];
        const global_ptr<const uint8_t> idx = in_global(pl[b0 + b] + kHeaderBytes) + 4u * (uint64_t)from[b0 + b], val = idx + 4u * (uint64_t)k;
        if (NEAR) at = skipped(b);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t o = at + 64u * r + lane, e = 4u * (o < n ? o : n ? n - 1u : 0u);      // in bytes: 16 KiB at most
            ix[b][r] = *(global_ptr<const uint32_t>)(idx + e);
            vv[b][r] = *(global_ptr<const float>)(val + e);
        }
    };
    auto add = [&](int b, uint32_t at) {
        uint32_t to[ROUNDS];
        float old[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t local = ix[b][r] - base;
            to[r] = local < (uint32_t)kChunk && (NEAR ? skipped(b) : at) + 64u * r + lane < len[b0 + b] ? local : (uint32_t)kChunk;
            old[r] = sums[to[r]];
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) sums[to[r]] = old[r] + vv[b][r];        // (a worker's entries are different elements)
        __builtin_amdgcn_wave_barrier();
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) fetch(b, 0u);
    if (NEAR) {
        bool missed = false;
#pragma unroll
        for (int b = 0; b < NB; ++b) {           // (the entries ascend)
            const uint32_t n = len[b0 + b], at = skipped(b);
            missed = missed || (at && (uint32_t)__builtin_amdgcn_readlane((int)ix[b][0], 0) > base) ||
                     (at + kMost < n && (uint32_t)__builtin_amdgcn_readlane((int)ix[b][ROUNDS - 1], 63) < base + (uint32_t)kChunk - 1u);
        }
        if (missed) return false;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        add(b, 0u);
        if (!NEAR && ROUNDS >= kSparseRounds)
            for (uint32_t at = kMost; at < len[b0 + b]; at += kMost) { fetch(b, at); add(b, at); }
    }
    return true;
}

// k64: entries a payload has room for (the exact k, or the capacity when DGC takes its threshold from a sample: the
// header then says how many are in use and repeats the capacity)
// FEW: up to kFewWorkers workers.  Two kernels, because every form of add_entries is a copy of its own and every copy costs both
// registers and spilled scalars: 106 of those leave 7 wavefronts per SIMD (8 when asked for, with 154 spilled instead of 81: up to 9 %
// slower), and with the forms for few workers in the same kernel the sum of eight took 0.5 to 2 % longer.
template <class SRC, bool FEW>
__global__ __launch_bounds__(kBlock) void sparse_decompress_k(int algo, SRC src, int W, float alpha, int *status, int capped)
{
    __shared__ float acc[kWavesPerBlock][kChunk + 32];
    if (blockIdx.x < SRC::kCheckers) { src.check({(uint32_t)algo, true, capped != 0}, W, status); return; }
    const auto job = src.template job<BLK_TILE>();
    const GroupView &out = job.out;
    const uint64_t k64 = job.k;
    const uint32_t k = (uint32_t)k64;
    const uint32_t tile = job.block;
    const Chunk c = my_chunk(out.n, tile);
    if (c.base >= out.n) return;
    const uintptr_t entry = chunk_entry(out, c);        // needed last, asked for first: overlaps with the table loads
    const uint32_t rot = chunk_rotation(entry);
    float *sums = acc[(c.base / (uint32_t)kChunk) % (uint32_t)kWavesPerBlock];
    bool touched = false;
#pragma unroll 1
    for (int w0 = 0; w0 < (FEW ? 1 : W); w0 += kSparseBatch) {
        // the tile's run in the list of every worker of the batch, as the directories have it; of absent workers none
        const uint8_t *pl[kSparseBatch];
        uint32_t lo[kSparseBatch], hi[kSparseBatch];
        job.template payloads<kSparseBatch>(w0, W, pl);
#pragma unroll
        for (int b = 0; b < kSparseBatch; ++b) {
            // block-uniform addresses, kept on the scalar path whatever the compiler makes of the rest
            const uint32_t *dir = reinterpret_cast<const uint32_t *>(pl[b] + kHeaderBytes + 8u * k64) + tile;
            lo[b] = hi[b] = 0u;
            if (w0 + b < W) { lo[b] = ld_uniform(dir); hi[b] = ld_uniform(dir + 1); }
        }
        hold(lo);
        hold(hi);
        uint32_t len[kSparseBatch], most = 0;
#pragma unroll
        for (int b = 0; b < kSparseBatch; ++b) {
            lo[b] = lo[b] < k ? lo[b] : k;
            hi[b] = hi[b] < k ? hi[b] : k;
            // inconsistent payload (a directory that does not ascend): a tile holds at most 4096 entries
            len[b] = hi[b] < lo[b] || hi[b] - lo[b] > (uint32_t)kTile ? 0u : hi[b] - lo[b];
            most = len[b] > most ? len[b] : most;
        }
        if (most == 0) continue;
        if (!touched) {
#pragma unroll
            for (int j = 0; j < kSteps; ++j) sums[64 * j + c.lane] = 0.0f;
            __builtin_amdgcn_wave_barrier();
            touched = true;
        }
        // Runs of at most 64 entries, of up to six workers 256, are read whole by each of the tile's wavefronts.  (Finding the
        // chunk's part first is one more wait for memory.  5 % of 25 M elements, spread evenly, 2 / 3 / 5 workers: 23.9 / 25.8 / 28.1 ->
        // 20.5 / 22.5 / 26.4 us, 4.4 M 7.8 / 7.8 / 9.7 -> 7.0 / 7.4 / 8.4.)
        const int there = W - w0;
        if (FEW) {
            if (there == 1 && most <= kNear && add_entries<1, kSparseRounds, true>(pl, 0, k, lo, len, c.base, sums)) continue;
            if (there <= kSparseBatch / 2 && most <= 64u) { add_entries<kSparseBatch / 2, 1>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there > kSparseBatch / 2 && most <= 64u) { add_entries<kFewWorkers, 1>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there == 2 && most <= kNear && add_entries<2, kSparseRounds, true>(pl, 0, k, lo, len, c.base, sums)) continue;
            if (there > 2 && most <= 64u * kSparseRounds) {
                add_entries<kSparseBatch / 2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums);
                if (there > kSparseBatch / 2) add_entries<2, kSparseRounds>(pl, kSparseBatch / 2, k, lo, len, c.base, sums);
                continue;
            }
            // Longer runs are read where the chunk's part ought to be, 256 entries (five and six workers: 192 while that surely
            // holds it), which needs no such wait where the run is spread evenly over the tile, as it is but where tensors of
            // different scales meet.  (4.4 M elements, 1 / 2 / 3 / 4 / 5 / 6 workers, found first -> so: 7 %, 6.4 / 6.8 / 8.3 / 8.2 / 8.6 / 8.6 ->
            // 6.4 / 6.5 / 7.2 / 7.0 / 7.8 / 7.9 us, 12 % 7.3 / 7.0 / 8.2 / 8.2 / 10.0 / 10.0 -> 6.1 / 6.1 / 6.9 / 7.0 / 8.2 / 8.4; 25 M, 15 %, 1 / 3 / 6 workers
            // 21.0 / 30.2 / 46.5 -> 20.0 / 30.7 / 43.5.  Read whole up to 512, three and four workers: 7 % 7.6 / 7.7, but of 25 M elements
            // 10 % 31.4 instead of 29.2.)
            if (there > 2 && there <= kSparseBatch / 2 && most <= kNear && add_entries<kSparseBatch / 2, kSparseRounds, true>(pl, 0, k, lo, len, c.base, sums)) continue;
            if (there > kSparseBatch / 2) {
                if (most <= 512u && add_entries<kFewWorkers, kSparseRounds - 1, true>(pl, 0, k, lo, len, c.base, sums)) continue;
                if (most <= kNear && add_entries<kSparseBatch / 2, kSparseRounds, true>(pl, 0, k, lo, len, c.base, sums)) {
                    if (add_entries<2, kSparseRounds, true>(pl, kSparseBatch / 2, k, lo, len, c.base, sums)) continue;
#pragma unroll
                    for (int b = 0; b < kSparseBatch / 2; ++b) len[b] = 0u;      // (added already)
                }
            }
        } else {
            if (there == 1 && most <= 64u * kSparseRounds) { add_entries<1, kSparseRounds>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there > kSparseBatch / 2 && most <= 64u) { add_entries<kSparseBatch, 1>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there <= kSparseBatch / 2 && most <= 64u) { add_entries<kSparseBatch / 2, 1>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there == 1 && most <= 128u * kSparseRounds) { add_entries<1, 2 * kSparseRounds>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there == 2 && most <= 128u * kSparseRounds) { add_entries<2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there <= kSparseBatch / 2 && most <= 64u * kSparseRounds) { add_entries<kSparseBatch / 2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums); continue; }
            if (there <= 6 && most <= 64u * kSparseRounds) {
                add_entries<kSparseBatch / 2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums);
                add_entries<2, kSparseRounds>(pl, kSparseBatch / 2, k, lo, len, c.base, sums);
                continue;
            }
        }
        // Else the run's part that lies in the chunk is found first, to a 64th of the run: every 64th entry of it (at most: the
        // runs are that short) in a lane, of all workers at once.
        uint32_t at[kSparseBatch] = {};
        auto sample = [&](int b) { at[b] = *(global_ptr<const uint32_t>)(in_global(pl[b] + kHeaderBytes) + 4u * (uint64_t)lo[b] + 4u * (len[b] * c.lane >> 6)); };
#pragma unroll
        for (int b = 0; b < kSparseBatch / 2; ++b) sample(b);
        if (there > kSparseBatch / 2)
#pragma unroll
            for (int b = kSparseBatch / 2; b < kSparseBatch; ++b) sample(b);
        most = 0;
#pragma unroll
        for (int b = 0; b < kSparseBatch; ++b) {
            const uint32_t below = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(at[b] < c.base));                        // samples before the chunk
            const uint32_t up_to = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(at[b] < c.base || at[b] - c.base < (uint32_t)kChunk));      // ... or in it
            const uint32_t from = below ? (len[b] * (below - 1u) >> 6) + 1u : 0u, to = up_to < 64u ? len[b] * up_to >> 6 : len[b];
            lo[b] += from;
            len[b] = to > from ? to - from : 0u;             // (none between two samples)
            most = len[b] > most ? len[b] : most;
        }
        if (there == 1) add_entries<1, 2 * kSparseRounds>(pl, 0, k, lo, len, c.base, sums);
        else if (there == 2) add_entries<2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums);
        else if (most <= 128u && there > kSparseBatch / 2) add_entries<FEW ? kFewWorkers : kSparseBatch, 2>(pl, 0, k, lo, len, c.base, sums);
        else {
            add_entries<kSparseBatch / 2, kSparseRounds>(pl, 0, k, lo, len, c.base, sums);
            if (there > kSparseBatch / 2) add_entries<FEW ? kFewWorkers - kSparseBatch / 2 : kSparseBatch / 2, kSparseRounds>(pl, kSparseBatch / 2, k, lo, len, c.base, sums);
        }
    }
    // Stored in the mapping rotated onto the output's 128-byte lines (payloads spread thinly over all tiles: 37.2 -> 36.3 us;
    // clustered ones: 32.3 -> 32.1; where no entry lies, 0.5 us).  Most tiles hold no kept entry at all: they are just zero-filled.
    float v[kSteps];
    if (touched) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < kSteps; ++j) v[j] = alpha * sums[rotated(j, c.lane, rot)];
    } else {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) v[j] = alpha * 0.0f;
    }
    store_seg_rot(out, c, v, entry, rot);
}

template <class SRC>
static void sparse_decompress_t(const LaunchCtx &lc, int algo, const SRC &src, uint32_t tiles, int W, float alpha, int *status, bool capped)
{
    prof_begin(lc, K_SPARSE_DECOMPRESS);
    const dim3 grid(tiles + SRC::kCheckers), block(kBlock);         // (the first blocks check the headers)
    if (W <= kFewWorkers) MC_LAUNCH((sparse_decompress_k<SRC, true>), grid, block, lc, algo, src, W, alpha, status, capped ? 1 : 0);
    else MC_LAUNCH((sparse_decompress_k<SRC, false>), grid, block, lc, algo, src, W, alpha, status, capped ? 1 : 0);
    prof_end(lc, K_SPARSE_DECOMPRESS);
}
template <class SRC>
void launch_sparse_decompress(const LaunchCtx &lc, int algo, const SRC &src, uint32_t tiles, int W, float alpha, int *status, bool capped)
{
    if (tiles == 0) return;
    if constexpr (std::is_same_v<SRC, OneDecompress>) if (W <= kFewRoom) { sparse_decompress_t(lc, algo, with_few(src), tiles, W, alpha, status, capped); return; }
    sparse_decompress_t(lc, algo, src, tiles, W, alpha, status, capped);
}
template void launch_sparse_decompress<OneDecompress>(const LaunchCtx &, int, const OneDecompress &, uint32_t, int, float, int *, bool);
template void launch_sparse_decompress<AllDecompress>(const LaunchCtx &, int, const AllDecompress &, uint32_t, int, float, int *, bool);

}  // namespace mc

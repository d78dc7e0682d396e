// Host side of the C ABI declared in include/mergecomp.h: partition policies,
// the context (segment tables, scratch, pointer-table cache), argument checks
// and the per-algorithm launch sequences.  Nothing here computes on gradient
// values; every step of the path runs in the kernels.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <limits>
#include <vector>

#include "mc_internal.h"

using namespace mc;

namespace {

constexpr uint64_t kMaxGroupElems = (1ull << 32) - (1ull << 24);
constexpr uint32_t kBarrierSpinLimit = 1u << 21;     // polls (about a microsecond each) before a block of the slow selection routes gives up waiting
// Cached device copies of per-call tensor address lists: kPtrSlots that any group takes, and with more than one group
// kGroupSlots of each group's own.  (With the first alone a layer-wise training step -- 161 groups, two gradients and an
// output each -- replaced every list before it came round again, two launches more in every call; with the second
// alone so did a caller with more than 32 buffers in rotation for one of many groups.)
constexpr int kPtrSlots = 256, kGroupSlots = 32;
constexpr int kAllSlots = 256;           // ... and of the address lists of calls over all groups (64 simulated workers use 65)

struct Group {
    int32_t t0 = 0, t1 = 0;              // tensor range [t0, t1) of the model's list
    std::vector<int32_t> live;           // tensors of the group that hold at least one element
    uint32_t n = 0;
    uint64_t goff = 0;
    uint64_t k = 0;
    uint32_t *d_seg_off = nullptr;       // live.size() + 1 flat offsets
    uint32_t *d_chunk_seg = nullptr;     // per 1024-element chunk: tensor holding its first element
};

struct PtrSlot {
    uint64_t stamp = 0;                  // 0: never used
    int32_t group = -1;
    std::vector<uintptr_t> host;
    uintptr_t *dev = nullptr;            // tensor addresses
    uintptr_t *dev_chunk = nullptr;      // per-chunk direct addresses derived from them
};

// The address list of a call over all groups.  W = 0: compress (tensors, a state and a payload per group), else
// decompress-and-sum (tensors, W payloads per group).
struct AllSlot {
    int32_t W = -1;
    uint64_t stamp = 0;
    bool apart = false;                  // no buffer that the call writes overlaps another of its buffers
    std::vector<uintptr_t> host;
    uintptr_t *dev = nullptr, *dev_chunk = nullptr;
};
struct Span { uintptr_t from, to; bool written; };

// ---- scratch of the allocation-free entry point (mc_compress_static) ------------------------------------
// The per-tile reduction partials of the dense compressors (three arrays of one double per 4096-element tile:
// OneBit reduces two sums and a count) for groups of up to kStaticMaxElems elements, in a file-scope device
// array that every GPU the library runs on holds from the moment the code object is loaded.  The array's name
// is only a host-side handle: its device address is looked up once per device (static_scratch_for) and it is
// that pointer which the kernels receive.
constexpr uint64_t kStaticMaxElems = 1ull << 26;
constexpr size_t kStaticMaxTiles = (size_t)(kStaticMaxElems / kTile);
constexpr size_t kStaticScratchBytes = 3 * kStaticMaxTiles * sizeof(double);        // 384 KiB
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_static_mutex;
static void *g_static_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device`, which must be the current device (each GPU holds its own copy of the
// array at its own address).  Looked up on the first call for a device, then served from the table.
static void *static_scratch_for(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[device]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        g_static_ptr[device] = ptr;
    }
    return g_static_ptr[device];
}

struct ProfEvent { int id; hipEvent_t a, b; };

struct Profiler {
    bool on = false;
    uint64_t mask = ~0ull;            // kernel slots that are timed while `on`
    std::vector<ProfEvent> pending;
    std::vector<hipEvent_t> pool;
    int64_t launches[K_COUNT] = {};
    double ms[K_COUNT] = {};
};

}  // namespace

struct mc_ctx {
    mc_config cfg{};
    int device = 0;
    std::vector<Group> groups;
    uint32_t max_tiles = 0;
    size_t max_live = 0;
    double *d_partial = nullptr;
    double *d_slots = nullptr;          // a double per tile, empty between calls (fill_slot)
    size_t slot_bytes = 0;
    uint64_t *d_arrive = nullptr;       // per group: blocks of small groups that have put their partial, over all calls
    uint32_t *d_large = nullptr;        // groups of more than kSmallTiles tiles, the last ones first
    uint32_t large_groups = 0;
    uint32_t wait_looks = kWaitLooks;   // of the small quantizer groups' blocks (mc_set_barrier_spin_limit)
    uint32_t collect_looks = kCollectLooks;      // of the collectors (the same)
    SparseScratch sparse{};
    uint32_t *d_hints = nullptr;        // candidate-filter hints: kHintWorkers per group (worker id modulo that)
    const uint32_t *last_hint = nullptr; // the record the most recent sparse mc_compress used (mc_select_stats)
    int *d_status = nullptr;
    void *static_scratch = nullptr;     // this device's copy of the file-scope scratch array (mc_compress_static)
    std::vector<PtrSlot> slots;         // group_slots per group, one group after the other, then those that any group takes
    size_t group_slots = 0;
    std::vector<uintptr_t> want;        // the address list of the call in progress (reserved at creation)
    // calls over all groups (contexts of more than one)
    bool own_scratch = false;           // sparsifiers: every group has a part of the scratch of its own
    GroupConst *d_groups = nullptr;
    uint32_t *d_block_group[BLK_KINDS] = {};
    uint32_t all_blocks[BLK_KINDS] = {};
    uint32_t last_group = 0;            // the last group that holds elements
    bool all_select_small = true;       // sparsifiers: every group's selection is one block's
    size_t all_live = 0;
    uint32_t all_subs = 0;              // sublists of keys of all groups' scratch
    std::vector<int64_t> tensor_numel;  // elements of every tensor of the model
    std::vector<uint32_t> first_tile, first_sub;       // per group, of its part of the sparsifiers' scratch
    std::vector<AllSlot> all_slots;
    std::vector<uintptr_t> want_all;
    std::vector<Span> spans;
    const SelectState *last_sel = nullptr;             // what the most recent sparse mc_compress recorded of its selection
    std::vector<void *> held;           // the context's device memory
    uint64_t clock = 0;
    uint32_t sync_blocks = 1;           // blocks of 1024 threads the device holds at once for sure: one per compute unit
    Profiler prof;
};

namespace mc {
static hipEvent_t prof_event(Profiler *p)
{
    hipEvent_t e = nullptr;
    if (!p->pool.empty()) { e = p->pool.back(); p->pool.pop_back(); }
    else if (hipEventCreate(&e) != hipSuccess) e = nullptr;
    return e;
}
void prof_begin(const LaunchCtx &lc, int id)
{
    Profiler *p = static_cast<Profiler *>(lc.prof);
    lc.ev_a = lc.ev_b = nullptr;
    if (!p || !p->on || !((p->mask >> id) & 1ull)) return;
    hipEvent_t a = prof_event(p), b = prof_event(p);
    if (!a || !b) {
        if (a) p->pool.push_back(a);
        if (b) p->pool.push_back(b);
        return;
    }
    lc.ev_a = a;
    lc.ev_b = b;
}
void prof_end(const LaunchCtx &lc, int id)
{
    Profiler *p = static_cast<Profiler *>(lc.prof);
    if (!p || !lc.ev_a) return;
    p->pending.push_back({id, lc.ev_a, lc.ev_b});
    lc.ev_a = lc.ev_b = nullptr;
}
}  // namespace mc

static const char *kKernelNames[K_COUNT] = {
    "upload_ptrs", "efsign_compress", "scalar_finalize", "accum_reduce", "qsgd_encode", "tern_encode",
    "fp16_compress", "dense_decompress", "sparse_accum", "sparse_seed", "cand_hist2", "cand_hist3", "cand_count",
    "cand_emit", "sparse_decompress", "state_convert", "lean_select", "lean_emit"};

static void prof_drain(Profiler &p)
{
    for (ProfEvent &e : p.pending) {
        float ms = 0.0f;
        if (hipEventSynchronize(e.b) == hipSuccess && hipEventElapsedTime(&ms, e.a, e.b) == hipSuccess) {
            p.launches[e.id] += 1;
            p.ms[e.id] += ms;
        }
        p.pool.push_back(e.a);
        p.pool.push_back(e.b);
    }
    p.pending.clear();
}

static uint64_t topk_count(uint64_t n, uint32_t ppm)
{
    if (n == 0) return 0;
    unsigned __int128 prod = (unsigned __int128)n * ppm;
    uint64_t k = (uint64_t)(prod / 1000000u);
    if (k < 1) k = 1;
    if (k > n) k = n;
    return k;
}

// Philox-4x32-10 on the host: the sampled-threshold DGC draws where its sample starts from the word of the
// group's first element (counter = (J lo, J hi, worker, iteration), J = model-global index / 4, key = seed).
static uint32_t philox_word(uint64_t seed, uint32_t worker, uint32_t iter_lo, uint64_t global_index)
{
    const uint64_t J = global_index >> 2;
    uint32_t c[4] = {(uint32_t)J, (uint32_t)(J >> 32), worker, iter_lo};
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = 0xD2511F53ull * c[0], p1 = 0xCD9E8D57ull * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1; c[3] = (uint32_t)p0; c[0] = n0; c[2] = n2;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return c[global_index & 3u];
}

// makes the context's device current for the duration of a call that synchronises or copies
struct DeviceGuard {
    int prev = -1;
    bool switched = false;
    explicit DeviceGuard(int device)
    {
        if (hipGetDevice(&prev) == hipSuccess && prev != device) switched = hipSetDevice(device) == hipSuccess;
    }
    ~DeviceGuard() { if (switched) (void)hipSetDevice(prev); }
};

static size_t lines(size_t addresses) { return (addresses + 31) / 32 * 32; }      // a table's size in addresses, so that the next one starts on a line
static bool is_sparse(int algo) { return algo == MC_ALGO_TOPK || algo == MC_ALGO_DGC || algo == MC_ALGO_RANDK; }
// n-element vectors of a group's state: the residual (DGC: v and u; SigNUM: the momentum; SignSGD: nothing)
static uint32_t state_vectors(int algo) { return algo == MC_ALGO_DGC ? 2u : algo == MC_ALGO_SIGNSGD ? 0u : 1u; }
static bool always_state(int algo) { return algo == MC_ALGO_DGC || algo == MC_ALGO_SIGNUM || algo == MC_ALGO_RANDK; }

// ---- device memory of a context
template <class T>
static bool grab(mc_ctx *ctx, T **p, size_t bytes)
{
    void *q = nullptr;
    if (hipMalloc(&q, bytes) != hipSuccess) { (void)hipGetLastError(); return false; }
    ctx->held.push_back(q);              // (reserved)
    *p = static_cast<T *>(q);
    return true;
}
template <class T>
static int grab_zeroed(mc_ctx *ctx, T **p, size_t bytes)
{
    if (!grab(ctx, p, bytes)) return MC_ERR_ALLOC;
    return hipMemset(*p, 0, bytes) == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}
template <class T>
static int grab_copy(mc_ctx *ctx, T **p, const std::vector<T> &host)
{
    if (host.empty()) return MC_OK;
    if (!grab(ctx, p, host.size() * sizeof(T))) return MC_ERR_ALLOC;
    return hipMemcpy(*p, host.data(), host.size() * sizeof(T), hipMemcpyHostToDevice) == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}
// all that was allocated after the first `keep` pieces
static void give_back(mc_ctx *ctx, size_t keep)
{
    for (; ctx->held.size() > keep; ctx->held.pop_back()) (void)hipFree(ctx->held.back());
}

// A part of the scratch for every group lets the sparsifiers' calls over all groups run as one launch per step; a
// model for which that is more than 2 GiB of candidates (350 M elements) or a quarter of that in histograms or key
// lists is large enough per group to be taken one group at a time, in scratch of the size of the largest.
static bool own_scratch_fits(const mc_ctx *ctx)
{
    return is_sparse(ctx->cfg.algo) && !ctx->cfg.dgc_sample_ppm && (size_t)ctx->all_blocks[BLK_TILE] * (6u * (size_t)kTile) <= (size_t(2) << 30) &&
           ctx->groups.size() * kHistWords * sizeof(uint32_t) <= (size_t(512) << 20) && (size_t)ctx->all_subs * kUCap * sizeof(UEntry) <= (size_t(512) << 20);
}

// Tables and scratch of a context whose groups are known.  all: also what a launch over all groups needs; own: the
// sparsifiers' scratch for every group instead of for the largest.  After MC_ERR_ALLOC the caller gives back what there is.
static int set_up(mc_ctx *ctx, bool all, bool own)
{
    const mc_config *cfg = &ctx->cfg;
    const size_t y = ctx->groups.size(), tiles = std::max<size_t>(ctx->max_tiles, 1), all_tiles = ctx->all_blocks[BLK_TILE];
    int rc = MC_OK;
    ctx->own_scratch = own;
    ctx->all_slots.clear();
    if (all) {
        std::vector<GroupConst> table(y);
        std::vector<uint32_t> block_group[BLK_KINDS];
        uint32_t ptrs = 0;
        for (size_t j = 0; j < y; ++j) {
            const Group &g = ctx->groups[j];
            const uint32_t blocks[BLK_KINDS] = {tiles_in(g.n), plane_blocks(g.n), sparse_blocks(g.n).select, sparse_blocks(g.n).emit};
            GroupConst &c = table[j];
            c.seg_off = g.d_seg_off; c.chunk_seg = g.d_chunk_seg;
            c.goff = g.goff; c.k = g.k; c.n = g.n; c.nseg = (uint32_t)g.live.size();
            c.first_ptr = ptrs; c.first_sub = ctx->first_sub[j];
            for (int b = 0; b < BLK_KINDS; ++b) {
                c.first[b] = (uint32_t)block_group[b].size();
                block_group[b].insert(block_group[b].end(), blocks[b], (uint32_t)j);
            }
            ptrs += c.nseg;
        }
        if ((rc = grab_copy(ctx, &ctx->d_groups, table)) != MC_OK) return rc;
        for (int b = 0; b < BLK_KINDS; ++b) if ((rc = grab_copy(ctx, &ctx->d_block_group[b], block_group[b])) != MC_OK) return rc;
        std::vector<uint32_t> large;
        for (size_t j = y; j-- > 0 && !is_sparse(cfg->algo);) if (tiles_in(ctx->groups[j].n) > kSmallTiles) large.push_back((uint32_t)j);
        ctx->large_groups = (uint32_t)large.size();
        if ((rc = grab_copy(ctx, &ctx->d_large, large)) != MC_OK) return rc;
    }
    if (!grab(ctx, &ctx->d_partial, 3 * std::max(tiles, all ? all_tiles : 0) * sizeof(double))) return MC_ERR_ALLOC;
    if (!is_sparse(cfg->algo)) {
        ctx->slot_bytes = std::max(tiles, all ? all_tiles : 0) * sizeof(double);
        if (!grab(ctx, &ctx->d_slots, ctx->slot_bytes)) return MC_ERR_ALLOC;
        if (hipMemset(ctx->d_slots, 0xFF, ctx->slot_bytes) != hipSuccess) return MC_ERR_DEVICE;
    }
    if ((rc = grab_zeroed(ctx, &ctx->d_arrive, y * kArriveStride * sizeof(uint64_t))) != MC_OK) return rc;
    if ((rc = grab_zeroed(ctx, &ctx->d_status, sizeof(int))) != MC_OK) return rc;
    if (is_sparse(cfg->algo)) {
        SparseScratch &sp = ctx->sparse;
        const size_t parts = own ? y : 1, stiles = own ? all_tiles : tiles;
        const size_t lists = own ? ctx->all_subs + kUSub : (size_t)kUSub;      // (the emit kernel looks at kUSub sublists of any group)
        const size_t slots = stiles * kTile + kCandPad;
        if ((rc = grab_zeroed(ctx, &sp.hist, parts * kHistWords * sizeof(uint32_t))) != MC_OK) return rc;
        if ((rc = grab_zeroed(ctx, &sp.sel, parts * 4 * sizeof(SelectState))) != MC_OK) return rc;
        if ((rc = grab_zeroed(ctx, &ctx->d_hints, y * kHintWorkers * kHintWords * sizeof(uint32_t))) != MC_OK) return rc;
        if (!grab(ctx, &sp.cand_bits, slots * sizeof(uint32_t)) || !grab(ctx, &sp.cand_loc, slots * sizeof(uint16_t)) ||
            !grab(ctx, &sp.tile_cnt, stiles * sizeof(uint32_t)) || !grab(ctx, &sp.blk_cnt, stiles * sizeof(uint32_t)) ||
            !grab(ctx, &sp.ulist, lists * kUCap * sizeof(UEntry))) return MC_ERR_ALLOC;
        if ((rc = grab_zeroed(ctx, &sp.tile_runs, stiles * sizeof(uint64_t))) != MC_OK) return rc;
        if ((rc = grab_zeroed(ctx, &sp.ucount, parts * kUSub * kUCountStride * sizeof(uint32_t))) != MC_OK) return rc;
        if ((rc = grab_zeroed(ctx, &sp.arrive, parts * kUCountStride * sizeof(uint32_t))) != MC_OK) return rc;
        if ((rc = grab_zeroed(ctx, &sp.sync, 64 * sizeof(uint32_t))) != MC_OK) return rc;
        ctx->last_sel = sp.sel;
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus < 1) return MC_ERR_DEVICE;
        ctx->sync_blocks = (uint32_t)cus;
        sp.spin_limit = kBarrierSpinLimit;
    }
    {
        // slots that hold the list of any group: 256 MiB in all (or four), and every group's own: the same (or four each)
        const size_t live = lines(ctx->max_live), chunks = lines(tiles * kWavesPerBlock);
        size_t words = 0;                    // of one slot of every group
        for (const Group &g : ctx->groups) words += lines(g.live.size()) + lines((size_t)tiles_in(g.n) * kWavesPerBlock);
        auto fit = [](size_t most, size_t each) { return std::min(most, std::max<size_t>(4, (size_t(256) << 20) / (std::max<size_t>(each, 1) * sizeof(uintptr_t)))); };
        const size_t common = fit(kPtrSlots, live + chunks);
        uintptr_t *at = nullptr, *own_at = nullptr;
        if (!grab(ctx, &at, common * (live + chunks) * sizeof(uintptr_t))) return MC_ERR_ALLOC;
        ctx->group_slots = y > 1 ? fit(kGroupSlots, words) : 0;
        const size_t own_bytes = ctx->group_slots * words * sizeof(uintptr_t);
        if (own_bytes == 0 || !grab(ctx, &own_at, own_bytes)) ctx->group_slots = 0;      // (no need, or no room)
        ctx->slots.assign(ctx->group_slots * y + common, PtrSlot());
        for (size_t i = 0; i < ctx->slots.size(); ++i) {
            PtrSlot &s = ctx->slots[i];
            const bool own_slot = i < ctx->group_slots * y;
            const Group *g = own_slot ? &ctx->groups[i / ctx->group_slots] : nullptr;
            uintptr_t *&from = own_slot ? own_at : at;
            s.dev = from;
            from += g ? lines(g->live.size()) : live;
            s.dev_chunk = from;
            from += g ? lines((size_t)tiles_in(g->n) * kWavesPerBlock) : chunks;
            s.host.reserve(g ? g->live.size() : ctx->max_live);
        }
        ctx->want.reserve(ctx->max_live);
        ctx->prof.pending.reserve(1024);
        ctx->prof.pool.reserve(2048);
    }
    if (all) {
        // lists of calls over all groups: a decompress-and-sum of the most workers needs the longest; 256 MiB in all
        const size_t most = lines(ctx->all_live + (size_t)kMaxWorkers * y), chunks = lines(all_tiles * kWavesPerBlock);
        const size_t count = std::min<size_t>(kAllSlots, std::max<size_t>(2, (size_t(256) << 20) / ((most + chunks) * sizeof(uintptr_t))));
        uintptr_t *at = nullptr;
        if (!grab(ctx, &at, count * (most + chunks) * sizeof(uintptr_t))) return MC_ERR_ALLOC;
        ctx->all_slots.resize(count);
        for (AllSlot &s : ctx->all_slots) {
            s.dev = at; s.dev_chunk = at + most;
            at += most + chunks;
            s.host.reserve(most);
        }
        ctx->want_all.reserve(most);
        ctx->spans.reserve(most);
    }
    return MC_OK;
}

extern "C" {

const char *mc_version(void) { return "mergecomp-gfx950 0.1"; }

const char *mc_strerror(int status)
{
    switch (status) {
    case MC_OK: return "ok";
    case MC_ERR_INVALID_ARG: return "invalid argument";
    case MC_ERR_RANGE: return "value out of range";
    case MC_ERR_ALLOC: return "allocation failed";
    case MC_ERR_DEVICE: return "HIP runtime error";
    case MC_ERR_PAYLOAD: return "payload header does not match the context";
    default: return "unknown status";
    }
}

int mc_partition(const int64_t *numel, int32_t n_tensors, int32_t y, int32_t policy, const int32_t *user_bounds,
                 int32_t *bounds_out)
{
    if (!numel || !bounds_out || n_tensors < 1 || y < 1) return MC_ERR_INVALID_ARG;
    for (int32_t t = 0; t < n_tensors; ++t) if (numel[t] < 0) return MC_ERR_INVALID_ARG;
    if (policy != MC_PART_EVEN_COUNT && policy != MC_PART_EVEN_ELEMS && policy != MC_PART_USER) return MC_ERR_INVALID_ARG;
    if (policy == MC_PART_USER && !user_bounds) return MC_ERR_INVALID_ARG;
    if (y > n_tensors) return MC_ERR_RANGE;
    const int32_t N = n_tensors;
    if (policy == MC_PART_EVEN_COUNT) {
        for (int32_t j = 0; j <= y; ++j) bounds_out[j] = (int32_t)(((int64_t)j * N) / y);
        return MC_OK;
    }
    if (policy == MC_PART_USER) {
        if (user_bounds[0] != 0 || user_bounds[y] != N) return MC_ERR_RANGE;
        for (int32_t j = 0; j < y; ++j) if (user_bounds[j + 1] <= user_bounds[j]) return MC_ERR_RANGE;
        std::copy(user_bounds, user_bounds + y + 1, bounds_out);
        return MC_OK;
    }
    // even by elements: one sweep over the prefix sums; boundary j is the first tensor
    // count whose prefix reaches j/y of the model, kept inside [previous + 1, N - (y - j)]
    unsigned __int128 D = 0;
    for (int32_t t = 0; t < N; ++t) D += (uint64_t)numel[t];
    bounds_out[0] = 0;
    bounds_out[y] = N;
    unsigned __int128 prefix = 0;
    int32_t t = 0;
    for (int32_t j = 1; j < y; ++j) {
        while (t < N && prefix * (unsigned)y < D * (unsigned)j) prefix += (uint64_t)numel[t++];
        int32_t b = std::min(std::max(t, bounds_out[j - 1] + 1), N - (y - j));
        bounds_out[j] = b;
    }
    return MC_OK;
}

static bool valid_model(const mc_time_model *m)
{
    return m && m->fwd_time >= 0 && m->B_h >= 0 && m->gamma_h >= 0 && m->B_g >= 0 && m->gamma_g >= 0;
}

int mc_partition_cost(const int64_t *numel, const double *bwd_time, int32_t n_tensors, const mc_time_model *model,
                      const int32_t *bounds, int32_t y, double *F_out)
{
    if (!numel || !bwd_time || !bounds || !F_out || !valid_model(model) || n_tensors < 1 || y < 1) return MC_ERR_INVALID_ARG;
    if (y > n_tensors || bounds[0] != 0 || bounds[y] != n_tensors) return MC_ERR_RANGE;
    for (int32_t j = 0; j < y; ++j) if (bounds[j + 1] <= bounds[j]) return MC_ERR_RANGE;
    double gpu = model->fwd_time, net = 0.0;
    for (int32_t j = 0; j < y; ++j) {
        double x = 0.0;
        for (int32_t t = bounds[j]; t < bounds[j + 1]; ++t) {
            if (numel[t] < 0 || bwd_time[t] < 0) return MC_ERR_INVALID_ARG;
            gpu += bwd_time[t];
            x += (double)numel[t];
        }
        gpu += model->B_h + model->gamma_h * x;
        net = std::max(gpu, net) + (model->B_g + model->gamma_g * x);
    }
    *F_out = net;
    return MC_OK;
}

int mc_partition_search(const int64_t *numel, const double *bwd_time, int32_t n_tensors, const mc_time_model *model,
                        int32_t Y, double alpha, int32_t *bounds_out, int32_t *y_out, double *F_out)
{
    if (!numel || !bwd_time || !bounds_out || !y_out || !valid_model(model) || n_tensors < 1 || Y < 1) return MC_ERR_INVALID_ARG;
    if (!(alpha >= 0.0 && alpha < 1.0)) return MC_ERR_INVALID_ARG;
    const int32_t N = n_tensors;
    if (Y > N) Y = N;
    try {
        // prefix sums over tensors: elements and back-propagation time
        std::vector<double> elems(N + 1, 0.0), bwd(N + 1, 0.0);
        for (int32_t t = 0; t < N; ++t) {
            if (numel[t] < 0 || bwd_time[t] < 0) return MC_ERR_INVALID_ARG;
            elems[t + 1] = elems[t] + (double)numel[t];
            bwd[t + 1] = bwd[t] + bwd_time[t];
        }
        // when the GPU has compressed the i-th group if that group ends before tensor e
        auto gpu_done = [&](int32_t e, int32_t i) { return model->fwd_time + bwd[e] + i * model->B_h + model->gamma_h * elems[e]; };
        auto send = [&](int32_t from, int32_t to) { return model->B_g + model->gamma_g * (elems[to] - elems[from]); };
        // net[e]: earliest time the network is free after i groups that cover tensors [0, e); from[i][e]: where the
        // last of them starts.  The time the network is free only ever delays what follows, so the earliest is best.
        const double inf = std::numeric_limits<double>::infinity();
        std::vector<double> net(N + 1, inf), next(N + 1, inf);
        std::vector<std::vector<int32_t>> from(Y + 1, std::vector<int32_t>(N + 1, 0));
        std::vector<int32_t> best_bounds, cur_bounds;
        double F_prev = 0.0;
        int32_t y_best = 1;
        for (int32_t i = 1; i <= Y; ++i) {
            std::fill(next.begin(), next.end(), inf);
            for (int32_t e = i; e <= N - 0; ++e) {
                if (i == 1) { next[e] = gpu_done(e, 1) + send(0, e); from[1][e] = 0; continue; }
                for (int32_t s0 = i - 1; s0 < e; ++s0) {
                    if (net[s0] == inf) continue;
                    const double f = std::max(gpu_done(e, i), net[s0]) + send(s0, e);
                    if (f < next[e]) { next[e] = f; from[i][e] = s0; }
                }
            }
            net.swap(next);
            const double F_now = net[N];
            cur_bounds.assign(i + 1, 0);
            cur_bounds[i] = N;
            for (int32_t j = i, e = N; j >= 1; --j) { e = from[j][e]; cur_bounds[j - 1] = e; }
            if (i == 1) { F_prev = F_now; best_bounds = cur_bounds; continue; }
            if (F_prev < F_now) break;                               // more groups made it worse: keep y - 1
            const bool stop = F_prev - F_now < alpha * F_prev;       // marginal benefit too small: keep y and stop
            F_prev = F_now; best_bounds = cur_bounds; y_best = i;
            if (stop) break;
        }
        for (int32_t j = 0; j <= y_best; ++j) bounds_out[j] = best_bounds[j];
        *y_out = y_best;
        if (F_out) *F_out = F_prev;
    } catch (const std::bad_alloc &) {
        return MC_ERR_ALLOC;
    }
    return MC_OK;
}

int mc_ctx_destroy(mc_ctx *ctx)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    int prev = 0;
    bool switched = hipGetDevice(&prev) == hipSuccess && prev != ctx->device && hipSetDevice(ctx->device) == hipSuccess;
    (void)hipDeviceSynchronize();
    prof_drain(ctx->prof);
    for (hipEvent_t e : ctx->prof.pool) (void)hipEventDestroy(e);
    give_back(ctx, 0);
    if (switched) (void)hipSetDevice(prev);
    delete ctx;
    return MC_OK;
}

int mc_ctx_create(mc_ctx **out, const mc_config *cfg, const int64_t *numel, int32_t n_tensors, const int32_t *bounds,
                  int32_t y)
{
    if (!out) return MC_ERR_INVALID_ARG;
    *out = nullptr;
    if (!cfg || !numel || !bounds || n_tensors < 1 || y < 1) return MC_ERR_INVALID_ARG;
    if (cfg->algo < MC_ALGO_EFSIGN || cfg->algo > MC_ALGO_RANDK) return MC_ERR_INVALID_ARG;
    if (cfg->dgc_sample_ppm > 1000000u || (cfg->dgc_sample_ppm != 0 && cfg->algo != MC_ALGO_DGC)) return MC_ERR_INVALID_ARG;
    if (cfg->use_ef != 0 && cfg->use_ef != 1) return MC_ERR_INVALID_ARG;
    if (always_state(cfg->algo) && cfg->use_ef != 1) return MC_ERR_INVALID_ARG;
    if (cfg->algo == MC_ALGO_SIGNSGD && cfg->use_ef != 0) return MC_ERR_INVALID_ARG;
    if (cfg->algo == MC_ALGO_QSGD && (cfg->qsgd_bits < 2 || cfg->qsgd_bits > 8)) return MC_ERR_INVALID_ARG;
    if (is_sparse(cfg->algo) && (cfg->ratio_ppm < 1 || cfg->ratio_ppm > 1000000u)) return MC_ERR_INVALID_ARG;
    if (y > n_tensors) return MC_ERR_RANGE;
    if (bounds[0] != 0 || bounds[y] != n_tensors) return MC_ERR_RANGE;
    for (int32_t j = 0; j < y; ++j) if (bounds[j + 1] <= bounds[j]) return MC_ERR_RANGE;
    for (int32_t t = 0; t < n_tensors; ++t) if (numel[t] < 0) return MC_ERR_INVALID_ARG;
    for (int32_t j = 0; j < y; ++j) {      // flat indices of a group are 32-bit
        uint64_t n = 0;
        for (int32_t t = bounds[j]; t < bounds[j + 1]; ++t) {
            if ((uint64_t)numel[t] >= kMaxGroupElems) return MC_ERR_RANGE;
            n += (uint64_t)numel[t];
            if (n >= kMaxGroupElems) return MC_ERR_RANGE;
        }
    }

    mc_ctx *ctx = new (std::nothrow) mc_ctx();
    if (!ctx) return MC_ERR_ALLOC;
    ctx->cfg = *cfg;
    if (hipGetDevice(&ctx->device) != hipSuccess) { delete ctx; return MC_ERR_DEVICE; }
    int rc = MC_OK;
    try {
        ctx->groups.resize(y);
        ctx->held.reserve(2 * (size_t)y + 32);           // (the groups' tables, and what set_up allocates)
        ctx->tensor_numel.assign(numel, numel + n_tensors);
        uint64_t goff = 0;
        for (int32_t j = 0; j < y && rc == MC_OK; ++j) {
            Group &g = ctx->groups[j];
            g.t0 = bounds[j]; g.t1 = bounds[j + 1]; g.goff = goff;
            std::vector<uint32_t> off;
            uint64_t n = 0;
            for (int32_t t = g.t0; t < g.t1; ++t) {
                if (numel[t] == 0) continue;
                g.live.push_back(t - g.t0);
                off.push_back((uint32_t)n);
                n += (uint64_t)numel[t];
            }
            off.push_back((uint32_t)n);
            g.n = (uint32_t)n;
            g.k = is_sparse(cfg->algo) ? topk_count(n, cfg->ratio_ppm) : 0;
            if (cfg->dgc_sample_ppm) g.k = std::min<uint64_t>(2 * g.k, n);     // sampled threshold: the payload's capacity
            goff += n;
            if (!grab(ctx, &g.d_seg_off, off.size() * sizeof(uint32_t))) { rc = MC_ERR_ALLOC; break; }
            if (hipMemcpy(g.d_seg_off, off.data(), off.size() * sizeof(uint32_t), hipMemcpyHostToDevice) != hipSuccess) { rc = MC_ERR_DEVICE; break; }
            std::vector<uint32_t> cseg((size_t)((n + kChunk - 1) / kChunk) + 1, 0u);
            for (size_t c = 0, sidx = 0; c * kChunk < n; ++c) {
                while (off[sidx + 1] <= c * kChunk) ++sidx;
                cseg[c] = (uint32_t)sidx;
            }
            if (!grab(ctx, &g.d_chunk_seg, cseg.size() * sizeof(uint32_t))) { rc = MC_ERR_ALLOC; break; }
            if (hipMemcpy(g.d_chunk_seg, cseg.data(), cseg.size() * sizeof(uint32_t), hipMemcpyHostToDevice) != hipSuccess) { rc = MC_ERR_DEVICE; break; }
            ctx->max_tiles = std::max<uint32_t>(ctx->max_tiles, (uint32_t)((n + kTile - 1) / kTile));
            ctx->max_live = std::max(ctx->max_live, g.live.size());
        }
        for (const Group &g : ctx->groups) {
            const uint32_t blocks[BLK_KINDS] = {tiles_in(g.n), plane_blocks(g.n), sparse_blocks(g.n).select, sparse_blocks(g.n).emit};
            ctx->first_tile.push_back(ctx->all_blocks[BLK_TILE]);
            ctx->first_sub.push_back(ctx->all_subs);
            for (int b = 0; b < BLK_KINDS; ++b) ctx->all_blocks[b] += blocks[b];
            ctx->all_subs += std::min<uint32_t>(blocks[BLK_TILE], kUSub);
            ctx->all_live += g.live.size();
            ctx->all_select_small = ctx->all_select_small && selects_small(g.n, g.k);
            if (g.n) ctx->last_group = (uint32_t)(&g - ctx->groups.data());
        }
        if (rc == MC_OK) {
            // What only the calls over all groups need, foremost a scratch for every group, a context can do without: where the
            // device has no room for it, it takes these calls one group at a time, in a scratch of the size of the largest.
            const size_t tables = ctx->held.size();
            const bool all = y > 1 && ctx->all_blocks[BLK_TILE] > 0, own = all && own_scratch_fits(ctx);
            rc = set_up(ctx, all, own);
            if (rc == MC_ERR_ALLOC && own) { give_back(ctx, tables); rc = set_up(ctx, all, false); }
            if (rc == MC_ERR_ALLOC && all) { give_back(ctx, tables); rc = set_up(ctx, false, false); }
        }
        // the device address of the static scratch array, looked up here with the context's device current
        if (rc == MC_OK && !(ctx->static_scratch = static_scratch_for(ctx->device))) rc = MC_ERR_DEVICE;
        if (rc == MC_OK && hipDeviceSynchronize() != hipSuccess) rc = MC_ERR_DEVICE;
    } catch (const std::bad_alloc &) {
        rc = MC_ERR_ALLOC;
    }
    if (rc != MC_OK) { mc_ctx_destroy(ctx); return rc; }
    *out = ctx;
    return MC_OK;
}

static const Group *group_of(const mc_ctx *ctx, int32_t group)
{
    if (!ctx || group < 0 || (size_t)group >= ctx->groups.size()) return nullptr;
    return &ctx->groups[group];
}

int64_t mc_group_numel(const mc_ctx *ctx, int32_t group) { const Group *g = group_of(ctx, group); return g ? (int64_t)g->n : -1; }
int64_t mc_group_k(const mc_ctx *ctx, int32_t group) { const Group *g = group_of(ctx, group); return g ? (int64_t)g->k : -1; }
int32_t mc_group_tensors(const mc_ctx *ctx, int32_t group) { const Group *g = group_of(ctx, group); return g ? g->t1 - g->t0 : -1; }

size_t mc_payload_bytes(const mc_ctx *ctx, int32_t group)
{
    const Group *g = group_of(ctx, group);
    if (!g) return 0;
    const uint64_t n = g->n, words = (n + 31) / 32;
    switch (ctx->cfg.algo) {
    case MC_ALGO_EFSIGN:
    case MC_ALGO_ONEBIT:
    case MC_ALGO_SIGNSGD:
    case MC_ALGO_SIGNUM: return kHeaderBytes + 4 * words;
    case MC_ALGO_TERNGRAD: return kHeaderBytes + 8 * words;
    case MC_ALGO_QSGD: return kHeaderBytes + (n + 3) / 4 * 4;
    case MC_ALGO_FP16: return kHeaderBytes + (2 * n + 3) / 4 * 4;
    default: return kHeaderBytes + 8 * g->k + (n ? 4 * ((n + kTile - 1) / kTile + 1) : 0);      // index and value lists, directory
    }
}

size_t mc_state_bytes(const mc_ctx *ctx, int32_t group)
{
    const Group *g = group_of(ctx, group);
    if (!g) return 0;
    if (ctx->cfg.algo == MC_ALGO_DGC) return kHeaderBytes + sizeof(float) * (dgc_u_offset(g->n) + (size_t)g->n);
    return kHeaderBytes + sizeof(float) * (size_t)g->n * state_vectors(ctx->cfg.algo);
}

// Device view of a group over a per-call tensor address list (only tensors that hold
// elements).  Lists seen before are served from the cache; a new list replaces the
// least recently used slot: it is uploaded through a kernel's argument buffer and
// expanded into the per-chunk address table, in stream order with the kernels that
// will read it.
static GroupView group_view(mc_ctx *ctx, const LaunchCtx &lc, int32_t group, const Group &g, const void *const *ptrs)
{
    std::vector<uintptr_t> &want = ctx->want;     // capacity max_live: no allocation here
    want.clear();
    for (int32_t rel : g.live) want.push_back(reinterpret_cast<uintptr_t>(ptrs[rel]));
    GroupView gv{g.d_seg_off, g.d_chunk_seg, nullptr, nullptr, (uint32_t)g.live.size(), g.n, g.goff};
    PtrSlot *victim = nullptr;                    // the one used longest ago among those that this group may take
    auto look = [&](size_t from, size_t to) -> PtrSlot * {
        for (PtrSlot *s = ctx->slots.data() + from; s != ctx->slots.data() + to; ++s) {
            if (s->group == group && std::memcmp(s->host.data(), want.data(), want.size() * sizeof(uintptr_t)) == 0) return s;      // (a group's lists have one length)
            if (!victim || s->stamp < victim->stamp) victim = s;
        }
        return nullptr;
    };
    PtrSlot *hit = look((size_t)group * ctx->group_slots, ((size_t)group + 1) * ctx->group_slots);
    if (!hit) hit = look(ctx->groups.size() * ctx->group_slots, ctx->slots.size());
    if (hit) {
        hit->stamp = ++ctx->clock;
        gv.ptrs = hit->dev;
        gv.chunk_addr = hit->dev_chunk;
        return gv;
    }
    victim->group = group;
    victim->stamp = ++ctx->clock;
    victim->host = want;
    gv.ptrs = victim->dev;
    gv.chunk_addr = victim->dev_chunk;
    if (!want.empty()) {
        launch_upload_ptrs(lc, want.data(), victim->dev, (uint32_t)want.size());
        launch_expand_ptrs(lc, gv, victim->dev_chunk);
    }
    return gv;
}

static GroupTable all_table(const mc_ctx *ctx, const AllSlot &slot)
{
    GroupTable tb{ctx->d_groups, {}, slot.dev, slot.dev_chunk, (uint32_t)ctx->all_live, (uint32_t)ctx->groups.size()};
    for (int b = 0; b < BLK_KINDS; ++b) tb.block_group[b] = ctx->d_block_group[b];
    return tb;
}

// The slot of the list in ctx->want_all (its buffers in ctx->spans), uploaded if it has not been seen before.
static const AllSlot &all_slot(mc_ctx *ctx, const LaunchCtx &lc, int32_t W)
{
    const std::vector<uintptr_t> &want = ctx->want_all;
    AllSlot *victim = &ctx->all_slots[0];
    for (AllSlot &s : ctx->all_slots) {
        if (s.W == W && s.host.size() == want.size() && std::memcmp(s.host.data(), want.data(), want.size() * sizeof(uintptr_t)) == 0) {
            s.stamp = ++ctx->clock;
            return s;
        }
        if (s.stamp < victim->stamp) victim = &s;
    }
    victim->W = W;
    victim->stamp = ++ctx->clock;
    victim->host = want;
    // One group after the other, a call may use a buffer that an earlier group wrote; all at once it may not.
    std::vector<Span> &spans = ctx->spans;
    std::sort(spans.begin(), spans.end(), [](const Span &a, const Span &b) { return a.from < b.from; });
    uintptr_t any = 0, written = 0;                  // how far the buffers so far reach, and those of them that are written
    victim->apart = true;
    for (const Span &s : spans) {
        if (s.from == s.to) continue;
        if (s.from < (s.written ? any : written)) { victim->apart = false; break; }
        any = std::max(any, s.to);
        if (s.written) written = std::max(written, s.to);
    }
    if (victim->apart) {
        launch_upload_ptrs(lc, want.data(), victim->dev, (uint32_t)want.size());
        launch_expand_all(lc, all_table(ctx, *victim), ctx->all_blocks[BLK_TILE], victim->dev_chunk);
    }
    return *victim;
}
static int check_launch() { return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE; }

}  // extern "C"

static uint32_t qsgd_levels(const mc_config &cfg) { return cfg.algo == MC_ALGO_QSGD ? (1u << (cfg.qsgd_bits - 1)) - 1u : 0u; }

template <class SRC>
static void decompress_launch(mc_ctx *ctx, const LaunchCtx &lc, const SRC &src, uint32_t tiles, uint32_t planes, int32_t W, float alpha)
{
    const mc_config &cfg = ctx->cfg;
    if (is_sparse(cfg.algo)) { launch_sparse_decompress(lc, cfg.algo, src, tiles, W, alpha, ctx->d_status, cfg.dgc_sample_ppm != 0); return; }
    const bool by_word = cfg.algo != MC_ALGO_QSGD && cfg.algo != MC_ALGO_FP16;       // bit planes: 8192 elements per block
    launch_dense_decompress(lc, cfg.algo, src, by_word ? planes : tiles, W, alpha, qsgd_levels(cfg), ctx->d_status);
}

// The kernels of a dense compressor over one group or all: `tiles` blocks of 4096 elements, `groups` groups.
template <class SRC>
static void dense_compress(const mc_config &cfg, const LaunchCtx &lc, SRC src, uint32_t tiles, uint32_t groups, uint32_t most_tiles, uint32_t worker,
                           uint32_t iter_lo, uint32_t looks)
{
    // most_tiles: of any of the groups.  Small ones combine their partial sums in the kernel that makes them.
    // (While the profiler is on every step is a kernel of its own, so that its time can be read.)
    const Profiler *prof = static_cast<const Profiler *>(lc.prof);
    const bool apart = !src.arrive || (prof && prof->on), small = !apart && most_tiles <= kSmallTiles;
    // (OneBit's three sums take a collector more registers than its streaming pass has.)
    const bool after = apart || (!small && (cfg.algo == MC_ALGO_ONEBIT || most_tiles > kCollectTiles));
    if (after) src.slots = nullptr;
    const bool ef = cfg.use_ef != 0;
    const uint32_t levels = qsgd_levels(cfg), algo = (uint32_t)cfg.algo;
    switch (cfg.algo) {
    case MC_ALGO_EFSIGN:
    case MC_ALGO_ONEBIT:
    {
        const bool means = cfg.algo == MC_ALGO_ONEBIT;
        launch_sign_compress(lc, means ? SIGN_MEANS : SIGN_EF, src, tiles, ef, 0.0f, algo, small);
        if (after) launch_scalar_finalize(lc, src, groups, means ? RED_MEANS : RED_MEAN_ABS, algo, 0, ef);
    }
        break;
    case MC_ALGO_SIGNSGD:
    case MC_ALGO_SIGNUM:
        launch_sign_compress(lc, cfg.algo == MC_ALGO_SIGNSGD ? SIGN_PLAIN : SIGN_MOMENTUM, src, tiles, ef, cfg.dgc_momentum, algo, false);
        break;
    case MC_ALGO_QSGD:
        if (small) { launch_quantize_small(lc, RED_L2, src, tiles, ef, levels, cfg.seed, worker, iter_lo, looks); break; }
        launch_accum_reduce(lc, src, tiles, ef, RED_L2, levels, cfg.seed);
        if (after) launch_scalar_finalize(lc, src, groups, RED_L2, algo, levels, false);
        launch_qsgd_encode(lc, src, tiles, ef, levels, cfg.seed, worker, iter_lo);
        break;
    case MC_ALGO_TERNGRAD:
        if (small) { launch_quantize_small(lc, RED_MAX_ABS, src, tiles, ef, 0, cfg.seed, worker, iter_lo, looks); break; }
        launch_accum_reduce(lc, src, tiles, ef, RED_MAX_ABS, 0, cfg.seed);
        if (after) launch_scalar_finalize(lc, src, groups, RED_MAX_ABS, algo, 0, false);
        launch_tern_encode(lc, src, tiles, ef, cfg.seed, worker, iter_lo);
        break;
    default:
        launch_fp16_compress(lc, src, tiles, ef);
        break;
    }
}
// the payload of an empty group: its header
static void empty_compress(const mc_config &cfg, const LaunchCtx &lc, PayloadHeader *hdr)
{
    const bool votes = cfg.algo == MC_ALGO_SIGNSGD || cfg.algo == MC_ALGO_SIGNUM;
    launch_scalar_finalize(lc, OneCompress{GroupView{}, nullptr, hdr, nullptr, nullptr, nullptr, nullptr, 0u}, 1, votes ? RED_ONE : -1, (uint32_t)cfg.algo, qsgd_levels(cfg), false);
}
static SparseCall sparse_call(const mc_ctx *ctx, uint32_t worker, uint64_t iter)
{
    SparseCall c{ctx->cfg.dgc_momentum, ctx->cfg.seed, worker, (uint32_t)iter, ctx->sync_blocks, ctx->d_status};
    return c;
}

// partial: the per-tile reduction partials (three arrays of one double per tile of the group); prof: the context's
// profiler, or null for a call that must not create events
static int compress_impl(mc_ctx *ctx, int32_t group, uint32_t worker, uint64_t iter, const float *const *grad_ptrs, void *state,
                         void *payload_out, void *stream, double *partial, Profiler *prof)
{
    const Group *gp = group_of(ctx, group);
    if (!gp || !payload_out) return MC_ERR_INVALID_ARG;
    const Group &G = *gp;
    const mc_config &cfg = ctx->cfg;
    const bool ef = cfg.use_ef != 0;
    if (ef && !state) return MC_ERR_INVALID_ARG;
    if (G.t1 > G.t0 && !grad_ptrs) return MC_ERR_INVALID_ARG;
    for (int32_t rel : G.live) if (!grad_ptrs[rel] || (reinterpret_cast<uintptr_t>(grad_ptrs[rel]) & 3u)) return MC_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(payload_out) & 15u) || (reinterpret_cast<uintptr_t>(state) & 15u)) return MC_ERR_INVALID_ARG;

    LaunchCtx lc{static_cast<hipStream_t>(stream), prof, nullptr, nullptr};
    (void)hipGetLastError();
    PayloadHeader *hdr = static_cast<PayloadHeader *>(payload_out);
    float *sf = state ? reinterpret_cast<float *>(static_cast<uint8_t *>(state) + kHeaderBytes) : nullptr;
    const uint32_t n = G.n;

    if (n == 0) {   // nothing to encode: the payload is its header
        empty_compress(cfg, lc, hdr);
        return check_launch();
    }
    GroupView gv = group_view(ctx, lc, group, G, reinterpret_cast<const void *const *>(grad_ptrs));
    if (!is_sparse(cfg.algo)) {
        // (the static entry point may not rely on what an earlier call left in its array: no count of arrivals)
        uint64_t *arrive = partial == ctx->d_partial ? ctx->d_arrive + (size_t)group * kArriveStride : nullptr;
        dense_compress(cfg, lc, OneCompress{gv, sf, hdr, partial, arrive, ctx->d_slots, ctx->d_status, ctx->collect_looks}, tiles_in(n), 1, tiles_in(n), worker, (uint32_t)iter, ctx->wait_looks);
        return check_launch();
    }
    SparseScratch sp = ctx->sparse;
    // a context may compress for several simulated workers whose thresholds differ: each keeps its own hint
    sp.hint = ctx->d_hints + (worker % kHintWorkers) * kHintWords;
    if (ctx->own_scratch) sp = scratch_of(sp, (uint32_t)group, ctx->first_tile[group], ctx->first_sub[group]);
    else sp.hint += (size_t)group * kHintWorkers * kHintWords;
    ctx->last_hint = sp.hint;
    ctx->last_sel = sp.sel;
    SparseCall call = sparse_call(ctx, worker, iter);
    if (cfg.dgc_sample_ppm) {       // sample: every stride-th element from `first`; threshold = its need-th largest key
        const uint32_t stride = std::max<uint32_t>(1u, 1000000u / cfg.dgc_sample_ppm);
        const uint32_t first = philox_word(cfg.seed, worker, (uint32_t)iter, G.goff) % stride;
        const uint64_t m = n > first ? ((uint64_t)n - first + stride - 1) / stride : 0;
        call.sample_stride = stride;
        call.sample_first = first;
        call.sample_need = m ? std::max<uint64_t>(1, (uint64_t)(((unsigned __int128)m * cfg.ratio_ppm) / 1000000u)) : 0;
    }
    SparseBlocks nb = sparse_blocks(n);
    if (selects_small(n, G.k) && !(prof && prof->on)) { nb.small = small_sel_blocks(nb.tiles); nb.same = nb.small == 1u; }
    launch_sparse_compress(lc, cfg.algo, OneSparse{gv, sf, hdr, G.k, sp}, nb, ef, call);
    return check_launch();
}

// All groups of one worker with one launch per step.  Returns 1 if the call has to be taken group by group instead: where
// the context keeps no scratch for that, where an argument is not in order (the loop stops at the first such group), or
// where buffers overlap so that the order of the groups matters.
static int compress_all(mc_ctx *ctx, uint32_t worker, uint64_t iter, const float *const *grads, void *const *states, void *const *payloads,
                        void *stream)
{
    const mc_config &cfg = ctx->cfg;
    const size_t y = ctx->groups.size();
    const bool ef = cfg.use_ef != 0, sparse = is_sparse(cfg.algo);
    if (ctx->all_slots.empty() || (sparse && !ctx->own_scratch) || !grads) return 1;
    std::vector<uintptr_t> &want = ctx->want_all;        // (both reserved at creation: no allocation here)
    std::vector<Span> &spans = ctx->spans;
    want.clear();
    spans.clear();
    bool plain = true;
    auto add = [&](const void *p, size_t bytes, uintptr_t align, bool written) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p);
        plain = plain && a != 0 && (a & (align - 1u)) == 0;
        want.push_back(a);
        spans.push_back({a, a + bytes, written});
    };
    for (const Group &G : ctx->groups) for (int32_t rel : G.live) add(grads[G.t0 + rel], sizeof(float) * (size_t)ctx->tensor_numel[G.t0 + rel], 4, false);
    for (size_t j = 0; j < y; ++j) {
        if (ef) add(states[j], mc_state_bytes(ctx, (int32_t)j), 16, true);
        else {                                   // not used, but refused if it could not be one
            plain = plain && !(states && (reinterpret_cast<uintptr_t>(states[j]) & 15u));
            want.push_back(0);
        }
    }
    for (size_t j = 0; j < y; ++j) add(payloads[j], mc_payload_bytes(ctx, (int32_t)j), 16, true);
    if (!plain) return 1;
    LaunchCtx lc{static_cast<hipStream_t>(stream), &ctx->prof, nullptr, nullptr};
    (void)hipGetLastError();
    const AllSlot &slot = all_slot(ctx, lc, 0);
    if (!slot.apart) return 1;
    const GroupTable tb = all_table(ctx, slot);
    if (sparse) {
        SparseScratch sp = ctx->sparse;
        sp.hint = ctx->d_hints + (worker % kHintWorkers) * kHintWords;
        const SparseScratch last = scratch_of(sp, ctx->last_group, ctx->first_tile[ctx->last_group], ctx->first_sub[ctx->last_group]);
        ctx->last_hint = last.hint;
        ctx->last_sel = last.sel;
        const bool one_each = small_sel_blocks(ctx->max_tiles) <= 1u;
        SparseBlocks nb{ctx->all_blocks[BLK_TILE], ctx->all_blocks[BLK_SELECT], ctx->all_blocks[BLK_EMIT]};
        if (ctx->all_select_small && !ctx->prof.on) {
            nb.small = one_each ? (uint32_t)y : nb.emit;
            nb.same = one_each && nb.tiles <= kSameTiles;
        }
        launch_sparse_compress(lc, cfg.algo, AllSparse{tb, sp, ctx->last_group, one_each}, nb, ef, sparse_call(ctx, worker, iter));
    } else dense_compress(cfg, lc, AllCompress{tb, ctx->d_partial, ctx->d_arrive, ctx->d_slots, ctx->d_status, ctx->collect_looks, ctx->all_blocks[BLK_TILE],
                                                  ctx->large_groups, ctx->d_large}, ctx->all_blocks[BLK_TILE], (uint32_t)y, ctx->max_tiles, worker,
                        (uint32_t)iter, ctx->wait_looks);
    for (size_t j = 0; j < y; ++j) if (ctx->groups[j].n == 0) empty_compress(cfg, lc, static_cast<PayloadHeader *>(payloads[j]));
    return check_launch();
}

extern "C" {

int mc_compress(mc_ctx *ctx, int32_t group, uint32_t worker, uint64_t iter, const float *const *grad_ptrs, void *state,
                void *payload_out, void *stream)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    return compress_impl(ctx, group, worker, iter, grad_ptrs, state, payload_out, stream, ctx->d_partial, &ctx->prof);
}

int mc_compress_static(mc_ctx *ctx, int32_t group, uint32_t worker, uint64_t iter, const float *const *grad_ptrs, void *state,
                       void *payload_out, void *stream)
{
    const Group *gp = group_of(ctx, group);
    if (!gp) return MC_ERR_INVALID_ARG;
    // the sparsifiers' scratch (candidate slots, 6 bytes per element) is not what the static array holds
    if (is_sparse(ctx->cfg.algo)) return MC_ERR_INVALID_ARG;
    if ((uint64_t)gp->n > kStaticMaxElems) return MC_ERR_RANGE;
    if (!ctx->static_scratch) return MC_ERR_DEVICE;
    // every tile's partial is written by the compress kernel before the one-block combine reads it: nothing in the
    // array has to start at zero, whatever an earlier call left there
    return compress_impl(ctx, group, worker, iter, grad_ptrs, state, payload_out, stream,
                         static_cast<double *>(ctx->static_scratch), nullptr);
}

size_t mc_static_scratch_bytes(void) { return kStaticScratchBytes; }
int64_t mc_static_max_elems(void) { return (int64_t)kStaticMaxElems; }

int mc_decompress_sum(mc_ctx *ctx, int32_t group, const void *const *payloads, int32_t W, float alpha,
                      float *const *out_ptrs, void *stream)
{
    const Group *gp = group_of(ctx, group);
    if (!gp || !payloads || W < 1) return MC_ERR_INVALID_ARG;
    if (W > kMaxWorkers) return MC_ERR_RANGE;
    const Group &G = *gp;
    if (G.t1 > G.t0 && !out_ptrs) return MC_ERR_INVALID_ARG;
    for (int32_t rel : G.live) if (!out_ptrs[rel] || (reinterpret_cast<uintptr_t>(out_ptrs[rel]) & 3u)) return MC_ERR_INVALID_ARG;
    for (int32_t w = 0; w < W; ++w) if (!payloads[w] || (reinterpret_cast<uintptr_t>(payloads[w]) & 15u)) return MC_ERR_INVALID_ARG;
    if (G.n == 0) return MC_OK;
    LaunchCtx lc{static_cast<hipStream_t>(stream), &ctx->prof, nullptr, nullptr};
    (void)hipGetLastError();
    GroupView gv = group_view(ctx, lc, group, G, reinterpret_cast<const void *const *>(out_ptrs));
    OneDecompress src;
    src.out = gv;
    src.k = G.k;
    for (int32_t w = 0; w < (W <= kFewRoom ? kFewRoom : kMaxWorkers); ++w)
        src.pl[w] = static_cast<const uint8_t *>(payloads[w < W ? w : 0]);      // (kernels read the addresses of several workers at once)
    decompress_launch(ctx, lc, src, tiles_in(G.n), plane_blocks(G.n), W, alpha);
    return check_launch();
}

// All groups with one launch; 1 if the call has to be taken group by group (see compress_all).
static int decompress_all(mc_ctx *ctx, const void *const *payloads, int32_t W, float alpha, float *const *outs, void *stream)
{
    const size_t y = ctx->groups.size();
    if (ctx->all_slots.empty() || !outs) return 1;
    std::vector<uintptr_t> &want = ctx->want_all;
    std::vector<Span> &spans = ctx->spans;
    want.clear();
    spans.clear();
    bool plain = true;
    auto add = [&](const void *p, size_t bytes, uintptr_t align, bool written) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p);
        plain = plain && a != 0 && (a & (align - 1u)) == 0;
        want.push_back(a);
        spans.push_back({a, a + bytes, written});
    };
    for (const Group &G : ctx->groups) for (int32_t rel : G.live) add(outs[G.t0 + rel], sizeof(float) * (size_t)ctx->tensor_numel[G.t0 + rel], 4, true);
    for (size_t j = 0; j < y; ++j)
        for (int32_t w = 0; w < W; ++w) add(payloads[(size_t)w * y + j], mc_payload_bytes(ctx, (int32_t)j), 16, false);
    if (!plain) return 1;
    LaunchCtx lc{static_cast<hipStream_t>(stream), &ctx->prof, nullptr, nullptr};
    (void)hipGetLastError();
    const AllSlot &slot = all_slot(ctx, lc, W);
    if (!slot.apart) return 1;
    decompress_launch(ctx, lc, AllDecompress{all_table(ctx, slot), W}, ctx->all_blocks[BLK_TILE], ctx->all_blocks[BLK_PLANE], W, alpha);
    return check_launch();
}

int mc_compress_groups(mc_ctx *ctx, uint32_t worker, uint64_t iter, const float *const *grad_ptrs_all, void *const *states,
                       void *const *payloads_out, void *stream)
{
    if (!ctx || !payloads_out || (ctx->cfg.use_ef && !states)) return MC_ERR_INVALID_ARG;
    const int done = compress_all(ctx, worker, iter, grad_ptrs_all, states, payloads_out, stream);
    if (done != 1) return done;
    for (size_t j = 0; j < ctx->groups.size(); ++j) {
        const Group &G = ctx->groups[j];
        const int rc = compress_impl(ctx, (int32_t)j, worker, iter, grad_ptrs_all ? grad_ptrs_all + G.t0 : nullptr, states ? states[j] : nullptr,
                                     payloads_out[j], stream, ctx->d_partial, &ctx->prof);
        if (rc != MC_OK) return rc;
    }
    return MC_OK;
}

int mc_decompress_sum_groups(mc_ctx *ctx, const void *const *payloads, int32_t W, float alpha, float *const *out_ptrs_all, void *stream)
{
    if (!ctx || !payloads || W < 1) return MC_ERR_INVALID_ARG;
    if (W > kMaxWorkers) return MC_ERR_RANGE;
    const int done = decompress_all(ctx, payloads, W, alpha, out_ptrs_all, stream);
    if (done != 1) return done;
    const size_t y = ctx->groups.size();
    const void *one[kMaxWorkers];
    for (size_t j = 0; j < y; ++j) {
        for (int32_t w = 0; w < W; ++w) one[w] = payloads[(size_t)w * y + j];
        const int rc = mc_decompress_sum(ctx, (int32_t)j, one, W, alpha, out_ptrs_all ? out_ptrs_all + ctx->groups[j].t0 : nullptr, stream);
        if (rc != MC_OK) return rc;
    }
    return MC_OK;
}

static int state_convert(mc_ctx *ctx, int32_t group, const void *src, void *dst, bool to_residual, void *stream)
{
    const Group *g = group_of(ctx, group);
    if (!g) return MC_ERR_INVALID_ARG;
    const size_t nf = (size_t)g->n * state_vectors(ctx->cfg.algo);
    // an empty group has no residual: the plain side may be null, the opaque side never
    if (!(to_residual ? src : dst) || (nf > 0 && !(to_residual ? dst : src))) return MC_ERR_INVALID_ARG;
    // Nothing to convert (an empty group, or SignSGD, which keeps no state vector): neither side is touched.  The
    // kernel below indexes by the group's n, so it must never run for an algorithm without state vectors.
    if (nf == 0) return MC_OK;
    LaunchCtx lc{static_cast<hipStream_t>(stream), &ctx->prof, nullptr, nullptr};
    (void)hipGetLastError();
    launch_state_convert(lc, ctx->cfg.algo, to_residual, g->n, src, dst, qsgd_levels(ctx->cfg), ctx->cfg.seed, g->goff);
    return check_launch();
}

int mc_state_export_residual(mc_ctx *ctx, int32_t group, const void *state, float *e_out, void *stream)
{
    return state_convert(ctx, group, state, e_out, true, stream);
}

int mc_state_import_residual(mc_ctx *ctx, int32_t group, const float *e_in, void *state, void *stream)
{
    return state_convert(ctx, group, e_in, state, false, stream);
}

int mc_last_device_status(mc_ctx *ctx)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    int flag = 0;
    DeviceGuard on(ctx->device);
    if (hipDeviceSynchronize() != hipSuccess) return MC_ERR_DEVICE;
    if (hipMemcpy(&flag, ctx->d_status, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return MC_ERR_DEVICE;
    if (flag) {
        // (partial sums that came after their call had given up; nothing of the context runs)
        if (flag == FLAG_GAVE_UP && ctx->d_slots && hipMemset(ctx->d_slots, 0xFF, ctx->slot_bytes) != hipSuccess) return MC_ERR_DEVICE;
        if (hipMemset(ctx->d_status, 0, sizeof(int)) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return MC_ERR_DEVICE;
    }
    return flag == FLAG_GAVE_UP ? MC_ERR_DEVICE : flag ? MC_ERR_PAYLOAD : MC_OK;
}

int mc_last_select_route(mc_ctx *ctx)
{
    if (!ctx || !is_sparse(ctx->cfg.algo) || !ctx->sparse.sel) return MC_ERR_INVALID_ARG;
    SelectState s;
    DeviceGuard on(ctx->device);
    if (hipDeviceSynchronize() != hipSuccess) return MC_ERR_DEVICE;
    if (hipMemcpy(&s, ctx->last_sel, sizeof(s), hipMemcpyDeviceToHost) != hipSuccess) return MC_ERR_DEVICE;
    return (s.mode & 8u) ? MC_SELECT_DENSE : (s.mode & 1u) ? MC_SELECT_FAST : (s.mode & 2u) && !(s.mode & 16u) ? MC_SELECT_REFILL : MC_SELECT_ABOVE;
}

int mc_select_stats(mc_ctx *ctx, mc_select_counts *out, int32_t reset)
{
    if (!ctx || !out || !is_sparse(ctx->cfg.algo) || !ctx->sparse.sync) return MC_ERR_INVALID_ARG;
    uint32_t w[16] = {};
    DeviceGuard on(ctx->device);
    if (hipDeviceSynchronize() != hipSuccess) return MC_ERR_DEVICE;
    if (hipMemcpy(w, ctx->sparse.sync + 32, sizeof(w), hipMemcpyDeviceToHost) != hipSuccess) return MC_ERR_DEVICE;
    for (int r = 0; r < 4; ++r) out->calls[r] = w[r];
    out->last_bin_keys = w[8];
    out->last_candidates = w[9];
    out->margin_halvings = out->margin_cap = -1;
    if (ctx->last_hint) {
        uint32_t h[kHintWords] = {};
        if (hipMemcpy(h, ctx->last_hint, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess) return MC_ERR_DEVICE;
        out->margin_halvings = h[1];
        out->margin_cap = 4 - (int64_t)std::min<uint32_t>(h[3] & 0xFFu, 4u);
    }
    if (reset && hipMemset(ctx->sparse.sync + 32, 0, 4 * sizeof(uint32_t)) != hipSuccess) return MC_ERR_DEVICE;
    return MC_OK;
}

int mc_set_barrier_spin_limit(mc_ctx *ctx, uint32_t polls)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    const int algo = ctx->cfg.algo;
    // polls = 1: give up after the first look
    if (is_sparse(algo)) { ctx->sparse.spin_limit = polls ? polls - 1u : kBarrierSpinLimit; return MC_OK; }
    const bool quantizer = algo == MC_ALGO_QSGD || algo == MC_ALGO_TERNGRAD;
    if (!quantizer && !(algo == MC_ALGO_EFSIGN && ctx->max_tiles > kSmallTiles)) return MC_ERR_INVALID_ARG;
    ctx->wait_looks = polls ? polls - 1u : kWaitLooks;
    ctx->collect_looks = polls ? polls - 1u : kCollectLooks;
    return MC_OK;
}

int mc_profile_enable(mc_ctx *ctx, int32_t on)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    ctx->prof.on = on != 0;
    return MC_OK;
}

int mc_profile_select(mc_ctx *ctx, uint64_t kernel_mask)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    ctx->prof.mask = kernel_mask;
    return MC_OK;
}

int mc_profile_reset(mc_ctx *ctx)
{
    if (!ctx) return MC_ERR_INVALID_ARG;
    prof_drain(ctx->prof);
    for (int i = 0; i < K_COUNT; ++i) { ctx->prof.launches[i] = 0; ctx->prof.ms[i] = 0.0; }
    return MC_OK;
}

int32_t mc_profile_kernels(void) { return K_COUNT; }

int mc_profile_read(mc_ctx *ctx, int32_t id, const char **name, int64_t *launches, double *total_ms)
{
    if (!ctx || id < 0 || id >= K_COUNT) return MC_ERR_INVALID_ARG;
    prof_drain(ctx->prof);
    if (name) *name = kKernelNames[id];
    if (launches) *launches = ctx->prof.launches[id];
    if (total_ms) *total_ms = ctx->prof.ms[id];
    return MC_OK;
}

}  // extern "C"

// The HIP runtime and the kernel launchers as the library's host code sees them, without a device: allocations are
// addresses that nobody reads, copies and fills do nothing, a launcher counts that it was called.  Linked with
// mc_api.hip in place of the runtime and the kernels, so that what the host code does -- what it allocates, what it does
// when that fails, which launches a call consists of -- can be tested on any machine.
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "../../paper_2103_15195_amd/csrc/mc_internal.h"

static std::map<uintptr_t, size_t> g_live;             // allocations by address
static std::multiset<size_t> g_ever;                   // sizes of all allocations that succeeded since the last reset
static size_t g_limit = ~(size_t)0, g_held = 0;
static long g_denied = 0, g_bad_free = 0;
static uintptr_t g_next = 0x100000000ull;
static std::map<std::string, long> g_launches;

extern "C" {
// ---- for the test
void nd_reset(size_t limit) { g_limit = limit; g_denied = g_bad_free = 0; g_ever.clear(); g_launches.clear(); }
size_t nd_held(void) { return g_held; }
long nd_denied(void) { return g_denied; }
long nd_bad_free(void) { return g_bad_free; }
long nd_allocated(size_t bytes) { return (long)g_ever.count(bytes); }
long nd_launches(const char *what) { auto i = g_launches.find(what); return i == g_launches.end() ? 0 : i->second; }

// ---- the runtime
hipError_t hipMalloc(void **p, size_t bytes)
{
    if (bytes > g_limit || g_held > g_limit - bytes) { *p = nullptr; ++g_denied; return hipErrorOutOfMemory; }
    *p = reinterpret_cast<void *>(g_next);
    g_next += (bytes + 0xFFFFu) & ~(size_t)0xFFFFu;
    g_live[reinterpret_cast<uintptr_t>(*p)] = bytes;
    g_ever.insert(bytes);
    g_held += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    auto i = g_live.find(reinterpret_cast<uintptr_t>(p));
    if (i == g_live.end()) { ++g_bad_free; return hipErrorInvalidValue; }
    g_held -= i->second;
    g_live.erase(i);
    return hipSuccess;
}
// a copy or a fill has to lie in an allocation
static hipError_t inside(const void *p, size_t bytes)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    auto i = g_live.upper_bound(a);
    return i != g_live.begin() && (--i, a + bytes <= i->first + i->second) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipMemset(void *p, int, size_t bytes) { return inside(p, bytes); }
hipError_t hipMemcpy(void *dst, const void *src, size_t bytes, hipMemcpyKind kind)
{
    if (kind == hipMemcpyDeviceToHost) { std::memset(dst, 0, bytes); return inside(src, bytes); }
    return inside(dst, bytes);
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = reinterpret_cast<void *>(0x1000); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}

namespace mc {
#define COUNT(what) (void)++g_launches[what]
void launch_upload_ptrs(const LaunchCtx &, const uintptr_t *, uintptr_t *, uint32_t) { COUNT("upload"); }
void launch_expand_ptrs(const LaunchCtx &, const GroupView &, uintptr_t *) { COUNT("expand"); }
void launch_expand_all(const LaunchCtx &, const GroupTable &, uint32_t, uintptr_t *) { COUNT("expand_all"); }
void launch_state_convert(const LaunchCtx &, int, bool, uint32_t, const void *, void *, uint32_t, uint64_t, uint64_t) { COUNT("state_convert"); }
template <class SRC> void launch_sign_compress(const LaunchCtx &, int, const SRC &, uint32_t, bool, float, uint32_t, bool) { COUNT("compress"); }
template <class SRC> void launch_quantize_small(const LaunchCtx &, int, const SRC &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t, uint32_t) { COUNT("compress"); }
template <class SRC> void launch_scalar_finalize(const LaunchCtx &, const SRC &, uint32_t, int, uint32_t, uint32_t, bool) { COUNT("finalize"); }
template <class SRC> void launch_accum_reduce(const LaunchCtx &, const SRC &, uint32_t, bool, int, uint32_t, uint64_t) { COUNT("accum_reduce"); }
template <class SRC> void launch_qsgd_encode(const LaunchCtx &, const SRC &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t) { COUNT("compress"); }
template <class SRC> void launch_tern_encode(const LaunchCtx &, const SRC &, uint32_t, bool, uint64_t, uint32_t, uint32_t) { COUNT("compress"); }
template <class SRC> void launch_fp16_compress(const LaunchCtx &, const SRC &, uint32_t, bool) { COUNT("compress"); }
template <class SRC> void launch_dense_decompress(const LaunchCtx &, int, const SRC &, uint32_t, int, float, uint32_t, int *) { COUNT("decompress"); }
template <class SRC> void launch_sparse_compress(const LaunchCtx &, int, const SRC &, const SparseBlocks &, bool, const SparseCall &) { COUNT("compress"); }
template <class SRC> void launch_sparse_decompress(const LaunchCtx &, int, const SRC &, uint32_t, int, float, int *, bool) { COUNT("decompress"); }
#define BOTH_FORMS(S)                                                                                                                  \
    template void launch_sign_compress<S>(const LaunchCtx &, int, const S &, uint32_t, bool, float, uint32_t, bool);                   \
    template void launch_quantize_small<S>(const LaunchCtx &, int, const S &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t, uint32_t); \
    template void launch_scalar_finalize<S>(const LaunchCtx &, const S &, uint32_t, int, uint32_t, uint32_t, bool);                    \
    template void launch_accum_reduce<S>(const LaunchCtx &, const S &, uint32_t, bool, int, uint32_t, uint64_t);                       \
    template void launch_qsgd_encode<S>(const LaunchCtx &, const S &, uint32_t, bool, uint32_t, uint64_t, uint32_t, uint32_t);         \
    template void launch_tern_encode<S>(const LaunchCtx &, const S &, uint32_t, bool, uint64_t, uint32_t, uint32_t);                   \
    template void launch_fp16_compress<S>(const LaunchCtx &, const S &, uint32_t, bool);
BOTH_FORMS(OneCompress)
BOTH_FORMS(AllCompress)
template void launch_dense_decompress<OneDecompress>(const LaunchCtx &, int, const OneDecompress &, uint32_t, int, float, uint32_t, int *);
template void launch_dense_decompress<AllDecompress>(const LaunchCtx &, int, const AllDecompress &, uint32_t, int, float, uint32_t, int *);
template void launch_sparse_compress<OneSparse>(const LaunchCtx &, int, const OneSparse &, const SparseBlocks &, bool, const SparseCall &);
template void launch_sparse_compress<AllSparse>(const LaunchCtx &, int, const AllSparse &, const SparseBlocks &, bool, const SparseCall &);
template void launch_sparse_decompress<OneDecompress>(const LaunchCtx &, int, const OneDecompress &, uint32_t, int, float, int *, bool);
template void launch_sparse_decompress<AllDecompress>(const LaunchCtx &, int, const AllDecompress &, uint32_t, int, float, int *, bool);
}  // namespace mc

"""The library's host code without a device: mc_api.hip linked with tests/host/no_device.hip, whose allocator counts (and
refuses beyond a limit) and whose launchers count what a call consists of.  No kernel runs here."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2103_15195_amd import binding as B
from paper_2103_15195_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))
TILE = 4096
NO_LIMIT = 2 ** 64 - 1


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host"))
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-shared", "-O3")]
    objects, jobs = [], []
    for src in (os.path.join(hip_build.CSRC, "mc_api.hip"), os.path.join(HERE, "host", "no_device.hip")):
        objects.append(os.path.join(out, os.path.basename(src) + ".o"))
        jobs.append(subprocess.Popen([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "-c", *flags, "-o", objects[-1], src],
                                     stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    for job in jobs:
        text, _ = job.communicate()
        assert job.returncode == 0, text
    path = os.path.join(out, "libhostonly.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", path, *objects, "-lpthread"], check=True)
    return path


class Buffer:
    """Stands for a tensor: an address."""
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


@pytest.fixture
def host(built, monkeypatch):
    """The counters; while it is in use the binding drives the library without a device."""
    monkeypatch.setattr(B, "LIB_PATH", built)
    monkeypatch.setattr(B, "_lib", None)
    made = []

    class Context(B.Context):
        def __init__(self, *a, **k):
            made.append(self)
            super().__init__(*a, **k)
    monkeypatch.setattr(B, "Context", Context)
    L = B.lib()
    L.nd_reset.argtypes = [C.c_size_t]
    L.nd_held.restype = C.c_size_t
    L.nd_denied.restype = L.nd_bad_free.restype = L.nd_launches.restype = L.nd_allocated.restype = C.c_long
    L.nd_launches.argtypes = [C.c_char_p]
    L.nd_allocated.argtypes = [C.c_size_t]
    L.nd_reset(NO_LIMIT)
    held = L.nd_held()
    yield L
    for ctx in made:                             # by the library that made them, also after a test that failed
        ctx.close()
    assert L.nd_held() == held and L.nd_bad_free() == 0          # everything a test allocated is given back


def launches(L, *what):
    return [L.nd_launches(w.encode()) for w in what]


@pytest.mark.parametrize("algo", ["topk", "dgc", "randk"])
@pytest.mark.parametrize("numel,bounds", [([4 * TILE], [0, 1]), ([3 * TILE, 5 * TILE], [0, 1, 2]), ([100, 2 * TILE - 1], [0, 1, 2])])
def test_candidate_arrays_cover_what_the_kernels_read(host, algo, numel, bounds):
    """The select and emit kernels read a chunk of 1024 candidate slots as a head of 64 and units of 256, masking what lies
    beyond the chunk's candidates after the load: a chunk with more than 64 + 3 x 256 reads 64 + 4 x 256 slots, the
    scratch's last one past its own 1024."""
    furthest = 0
    for cnt in range(1025):
        units = max(0, -(-(cnt - 64) // 256))
        furthest = max(furthest, 64 + 256 * units)               # slots that the loads of this chunk cover
    assert furthest == 1088
    tiles = sum(-(-n // TILE) for n in numel)                    # of all groups: every group has its part of the scratch
    read = (tiles * TILE - 1024) + furthest
    ctx = B.Context(algo, numel, bounds)
    most = tiles * TILE + 1024                                   # (exact sizes: none but the candidate arrays lie in between)
    assert any(host.nd_allocated(4 * s) for s in range(read, most)), "values"
    assert any(host.nd_allocated(2 * s) for s in range(read, most)), "positions"
    ctx.close()


@pytest.mark.parametrize("algo", list(B.ALGO_IDS))
def test_who_takes_a_limit_on_waits(host, algo):
    """The sparsifiers (their blocks wait on the rare routes) and the quantizers (on small groups); all others refuse it."""
    ctx = B.Context(algo, [100], [0, 1])
    if algo in ("topk", "dgc", "randk", "qsgd", "terngrad"):
        ctx.mc_set_barrier_spin_limit(1)
        ctx.mc_set_barrier_spin_limit(0)
    else:
        with pytest.raises(B.McError) as e:
            ctx.mc_set_barrier_spin_limit(1)
        assert e.value.status == B.MC_ERR_INVALID_ARG
    ctx.close()


@pytest.mark.parametrize("numel,waits", [([64 * TILE], False), ([64 * TILE + 1], True), ([100, 65 * TILE], True), ([100, 64 * TILE], False)])
def test_efsign_takes_a_limit_where_its_blocks_wait(host, numel, waits):
    """... which is where one of them combines the partial sums of a group of more than 64 tiles."""
    ctx = B.Context("efsign", numel, list(range(len(numel) + 1)))
    if waits:
        ctx.mc_set_barrier_spin_limit(1)
        ctx.mc_set_barrier_spin_limit(0)
    else:
        with pytest.raises(B.McError) as e:
            ctx.mc_set_barrier_spin_limit(1)
        assert e.value.status == B.MC_ERR_INVALID_ARG
    ctx.close()


def groups_call(ctx, n):
    """mc_compress_groups and mc_decompress_sum_groups (two workers) with buffers that do not overlap."""
    at = 1 << 40
    grads, states, payloads = [], [], []
    for kind in (grads, states, payloads, payloads):
        for _ in n:
            kind.append(Buffer(at))
            at += 1 << 32
    ctx.mc_compress_groups(0, 0, grads, states, payloads[:len(n)], stream=0)
    ctx.mc_decompress_sum_groups(payloads, 2, 1.0, grads, stream=0)


@pytest.mark.parametrize("algo", ["efsign", "qsgd", "terngrad"])
@pytest.mark.parametrize("tiles,kernels", [(12288, 0), (12289, 1)])
def test_sums_of_very_large_groups_have_a_kernel_of_their_own(host, algo, tiles, kernels):
    """... by itself and beside others in one call: a block of the launch that makes the sums falls behind it there."""
    for numel in ([tiles * TILE], [100, tiles * TILE - 1, 70 * TILE]):
        ctx = B.Context(algo, numel, list(range(len(numel) + 1)))
        host.nd_reset(NO_LIMIT)
        if len(numel) == 1:
            ctx.mc_compress(0, 0, 0, [Buffer(1 << 40)], Buffer(1 << 41), Buffer(1 << 42), stream=0)
        else:
            at = [[Buffer((b << 44) + (j << 36)) for j in range(3)] for b in (1, 2, 3)]
            ctx.mc_compress_groups(0, 0, *at, stream=0)
        assert launches(host, "finalize") == [kernels]
        ctx.close()


@pytest.mark.filterwarnings("ignore:calls go through ctypes")
def test_calls_without_the_extension_module(built, monkeypatch, request):
    """The same calls, and the same refusals, where only the library has been built."""
    import sys

    import paper_2103_15195_amd as package
    monkeypatch.setitem(sys.modules, package.__name__ + "._fastcall", None)
    monkeypatch.delattr(package, "_fastcall", raising=False)
    host = request.getfixturevalue("host")
    assert B.lib().fast.compress() is None
    for algo in B.ALGO_IDS:
        test_who_takes_a_limit_on_waits(host, algo)
    for algo in ("efsign", "qsgd", "topk"):
        host.nd_reset(NO_LIMIT)
        ctx = B.Context(algo, [100, 5000], [0, 1, 2])
        groups_call(ctx, [100, 5000])
        assert launches(host, "compress", "decompress") == [1, 1]
        ctx.mc_compress(1, 0, 0, [Buffer(1 << 40)], Buffer(1 << 41), Buffer(1 << 42), stream=0)
        ctx.mc_decompress_sum(1, [Buffer(1 << 42)], 1.0, [Buffer(1 << 40)], stream=0)
        assert launches(host, "compress", "decompress") == [2, 2]
        with pytest.raises(B.McError):
            ctx.mc_compress(2, 0, 0, [Buffer(1 << 40)], Buffer(1 << 41), Buffer(1 << 42), stream=0)
        ctx.close()


@pytest.mark.parametrize("algo", ["topk", "randk", "dgc", "efsign"])
def test_a_context_does_without_what_there_is_no_room_for(host, algo):
    """A context of many groups allocates more than its calls for one group need.  Where the device has no room for that, it is
    created all the same and takes the calls over all groups one group at a time."""
    numel = [300000, 5] + [300000] * 14
    y = len(numel)
    bounds = list(range(y + 1))
    ctx = B.Context(algo, numel, bounds)
    most = host.nd_held()
    groups_call(ctx, numel)
    assert launches(host, "compress", "decompress") == [1, 1]
    ctx.close()
    ways, least = [], None                       # launches of a compress and a decompress, from the most to the least memory
    for limit in range(most, 0, -most // 200):
        host.nd_reset(limit)
        try:
            ctx = B.Context(algo, numel, bounds)
        except B.McError as e:
            assert e.status == B.MC_ERR_ALLOC and host.nd_held() == 0
            break
        assert host.nd_held() <= limit
        groups_call(ctx, numel)
        way = launches(host, "compress", "decompress")
        if way not in ways:
            ways.append(way)
        least = limit
        ctx.close()
    if algo == "efsign":
        assert ways == [[1, 1], [y, y]]
    else:                                        # the sparsifiers' scratch goes first, and is most of what there is
        assert ways == [[1, 1], [y, 1], [y, y]] and least < most // 2


@pytest.mark.parametrize("algo", ["topk", "qsgd"])
def test_a_context_that_cannot_be_created_gives_everything_back(host, algo):
    for limit in (0, 100, 10000, 1 << 20):
        host.nd_reset(limit)
        with pytest.raises(B.McError) as e:
            B.Context(algo, [4000000, 10], [0, 1, 2])
        assert e.value.status == B.MC_ERR_ALLOC and host.nd_held() == 0 and host.nd_denied() > 0


@pytest.mark.parametrize("y,lists", [(1, 250), (2, 250), (8, 250), (161, 250), (8, 40)])
def test_a_caller_may_rotate_many_buffers(host, y, lists):
    """Address lists seen before are served from the context: as many as the caller's rotation of one group's buffers holds,
    whatever the number of groups, also while every group has a few lists of its own in use."""
    ctx = B.Context("signsgd", [5000] * y, list(range(y + 1)))
    payload = Buffer(1 << 50)

    def step(j, i):
        ctx.mc_compress(j, 0, 0, [Buffer((1 << 40) + (j << 32) + (i << 20))], None, payload, stream=0)
    for turn in range(3):
        host.nd_reset(NO_LIMIT)
        for i in range(lists):
            step(0, i)
        for j in range(1, y):
            for i in range(3):
                step(j, i)
    assert launches(host, "upload", "expand") == [0, 0]
    ctx.close()


@pytest.mark.parametrize("y,lists", [(2, 65), (161, 65), (2, 200)])
def test_calls_over_all_groups_may_rotate_many_buffers(host, y, lists):
    """The same for the lists of whole calls: the most workers that can be decompressed, each with buffers of its own."""
    ctx = B.Context("signsgd", [5000] * y, list(range(y + 1)))

    def tensors(i):
        return [Buffer((1 << 40) + (i << 30) + (j << 20)) for j in range(y)]
    for turn in range(3):
        host.nd_reset(NO_LIMIT)
        for i in range(lists):
            ctx.mc_compress_groups(i, 0, tensors(2 * i), None, tensors(2 * i + 1), stream=0)
    assert launches(host, "upload", "expand_all", "expand", "compress") == [0, 0, 0, lists]
    ctx.close()


@pytest.mark.parametrize("algo,use_ef", [("efsign", 0), ("signsgd", 0), ("qsgd", 0), ("topk", 0), ("topk", 1), ("fp16", 1)])
@pytest.mark.parametrize("bad", ["grad", "state", "payload"])
@pytest.mark.parametrize("off", [None, 1, 2, 8])
def test_the_same_arguments_are_refused_for_all_groups_as_for_one(host, algo, use_ef, bad, off):
    """An address of one group is null or off by some bytes: the call over all groups returns what the group's own does,
    after the groups before it.  (A state that is not used has to be aligned too, if there is one.)"""
    y = 3
    ctx = B.Context(algo, [5000] * y, list(range(y + 1)), use_ef=use_ef)
    at = {kind: [(1 << 40) + (i << 36) + (j << 32) for j in range(y)] for i, kind in enumerate(("grad", "state", "payload"))}
    at[bad][1] = at[bad][1] + off if off else 0
    grads, states, payloads = ((C.c_void_p * y)(*at[kind]) for kind in ("grad", "state", "payload"))

    def one(j):
        return host.mc_compress(ctx._h, j, 0, 0, C.byref(grads, 8 * j), states[j], payloads[j], None)
    alone = [one(j) for j in range(y)]
    assert alone[0] == alone[2] == B.MC_OK
    host.nd_reset(NO_LIMIT)
    assert host.mc_compress_groups(ctx._h, 0, 0, grads, states, payloads, None) == alone[1]
    if alone[1] != B.MC_OK:
        assert alone[1] == B.MC_ERR_INVALID_ARG and launches(host, "compress") == [1]
    ctx.close()

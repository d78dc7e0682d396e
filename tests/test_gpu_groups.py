"""The calls over all groups (one launch per step for every group of the context) against the same groups one call at a
time: payloads, states and sums byte for byte, and the same selection routes."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# groups of one tensor each around the sizes where the blocks of either kind (4096 and 8192 elements, 4 and 16 tiles)
# begin and end, empty ones, one that starts off a multiple of four elements, and two that the slow selection routes
# take with all blocks (more than 64 tiles)
SIZES = [1, 0, 31, 1024, 4095, 4096, 4097, 8191, 8193, 16385, 65537, 0, 270001, 3, 400000, 0]
CASES = [(a, {}) for a in B.ALGO_IDS] + [("topk", {"use_ef": 0}), ("qsgd", {"use_ef": 0, "qsgd_bits": 4}), ("terngrad", {"use_ef": 0}),
                                         ("dgc", {"dgc_sample_ppm": 50000})]


def tensors(rng, scale, ties):
    x = [rng.standard_normal(n).astype(np.float32) * np.float32(scale) for n in SIZES]
    if ties:
        x = [np.round(v * 2).astype(np.float32) for v in x]
    return [torch.from_numpy(v).to(DEV) for v in x]


def buffers(ctx, size, many):
    """One buffer per group, 16-byte aligned parts of one allocation."""
    at, off = [], 0
    for j in range(ctx.y):
        at.append(off)
        off += (size(j) + 15) // 16 * 16
    whole = torch.zeros(many, off, dtype=torch.uint8, device=DEV)
    return whole, [[whole[w, at[j]:at[j] + size(j)] for j in range(ctx.y)] for w in range(many)]


@pytest.mark.parametrize("algo,kw", CASES)
def test_same_as_group_by_group(algo, kw):
    W, bounds = 3, list(range(len(SIZES) + 1))
    a, b = (B.Context(algo, SIZES, bounds, ratio_ppm=20000, seed=5, **kw) for _ in range(2))
    (pa, one_p), (pb, all_p) = buffers(a, a.payload_bytes, W), buffers(b, b.payload_bytes, W)
    (sa, one_s), (sb, all_s) = buffers(a, a.state_bytes, W), buffers(b, b.state_bytes, W)
    out = [[torch.full((n,), 7.0, device=DEV) for n in SIZES] for _ in range(2)]
    ef = a.cfg.use_ef
    rng = np.random.default_rng(11)
    # steady, then a jump up and down in scale (the slow selection routes), then many equal values
    for it, (scale, ties) in enumerate([(1.0, 0), (1.0, 0), (1.05, 0), (8.0, 0), (0.5, 0), (1.0, 1), (1.0, 1)]):
        for w in range(W):
            g = tensors(rng, scale, ties)
            for j in range(a.y):
                a.mc_compress(j, w, it, [g[j]], one_s[w][j] if ef else None, one_p[w][j])
            b.mc_compress_groups(w, it, g, all_s[w] if ef else None, all_p[w])
            torch.cuda.synchronize()
        assert torch.equal(pa, pb) and torch.equal(sa, sb), f"iteration {it}"
        for j in range(a.y):
            a.mc_decompress_sum(j, [one_p[w][j] for w in range(W)], 0.25, [out[0][j]])
        b.mc_decompress_sum_groups([all_p[w][j] for w in range(W) for j in range(b.y)], W, 0.25, out[1])
        assert all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(*out)), f"iteration {it}"
    if algo in ("topk", "dgc", "randk") and not kw.get("dgc_sample_ppm"):
        ra, rb = a.mc_select_stats(), b.mc_select_stats()
        assert ra == rb and ra["fast"] and ra["refill"]
        # Rand-k's keys do not depend on the values; with error feedback equal gradients do not make equal keys
        assert (ra["above"] or algo == "randk") and (ra["dense"] or a.cfg.use_ef)
        assert a.mc_last_select_route() == b.mc_last_select_route()
    assert a.mc_last_device_status() == B.MC_OK and b.mc_last_device_status() == B.MC_OK


def test_buffers_that_overlap_are_taken_in_order():
    """Group 1's gradient is a part of group 0's payload: group 0 has to be done before group 1 begins."""
    numel, bounds = [4096, 64], [0, 1, 2]
    res = []
    for together in (False, True):
        ctx = B.Context("fp16", numel, bounds, use_ef=0)
        x = torch.linspace(-2, 2, 4096, device=DEV)
        pay = [torch.zeros(ctx.payload_bytes(0), dtype=torch.uint8, device=DEV), torch.zeros(ctx.payload_bytes(1), dtype=torch.uint8, device=DEV)]
        inner = pay[0][128:128 + 256].view(torch.float32)
        if together:
            ctx.mc_compress_groups(0, 0, [x, inner], None, pay)
        else:
            ctx.mc_compress(0, 0, 0, [x], None, pay[0])
            ctx.mc_compress(1, 0, 0, [inner], None, pay[1])
        # ... and one output for both groups' sums: the later group's is what stays
        out = torch.zeros(4096, device=DEV)
        if together:
            ctx.mc_decompress_sum_groups([pay[0], pay[1]], 1, 1.0, [out, out[:64]])
        else:
            ctx.mc_decompress_sum(0, [pay[0]], 1.0, [out])
            ctx.mc_decompress_sum(1, [pay[1]], 1.0, [out[:64]])
        res.append((pay[0].clone(), pay[1].clone(), out))
    for p, q in zip(*res):
        assert torch.equal(p.view(torch.uint8), q.view(torch.uint8))


def test_more_lists_than_are_kept():
    """More address lists than the context keeps, so that the oldest are replaced; and again the first ones."""
    numel, bounds = [5000, 3, 9000], [0, 1, 3]
    ctx = B.Context("signsgd", numel, bounds)
    grads = [[torch.randn(n, device=DEV) for n in numel] for _ in range(300)]
    pay = [torch.zeros(ctx.payload_bytes(j), dtype=torch.uint8, device=DEV) for j in range(2)]
    for g in grads + grads[:5]:
        ctx.mc_compress_groups(0, 0, g, None, pay)
        for j, x in enumerate((g[0], torch.cat(g[1:]))):
            bits = np.unpackbits(pay[j].cpu().numpy()[128:], bitorder="little")[:x.numel()]
            assert np.array_equal(bits, (x >= 0).cpu().numpy())


def test_calls_go_to_the_current_stream():
    """Without a stream argument a call goes to torch's current stream, of whichever thread and context it is made in."""
    side = torch.cuda.Stream()
    assert B._current_stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._current_stream() == side.cuda_stream
        # ordered behind work of that stream only: the gradient is written there just before
        ctx = B.Context("fp16", [4096, 1], [0, 1, 2], use_ef=0)
        pay = [torch.zeros(ctx.payload_bytes(j), dtype=torch.uint8, device=DEV) for j in range(2)]
        g = [torch.zeros(n, device=DEV) for n in (4096, 1)]
        torch.cuda._sleep(20_000_000)
        for t in g:
            t.fill_(1.0)
        ctx.mc_compress_groups(0, 0, g, None, pay)
    side.synchronize()
    assert bool((pay[0][128:].view(torch.float16) == 1).all()) and float(pay[1][128:].view(torch.float16)[0]) == 1.0
    assert B._current_stream() == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("W", [5, 9, 17, 64])
@pytest.mark.parametrize("algo", list(B.ALGO_IDS))
def test_sums_of_many_workers(algo, W):
    """More workers than the decode kernels take at a time (four; eight of one bit plane or of a sparsifier)."""
    ctx = B.Context(algo, SIZES, list(range(len(SIZES) + 1)), ratio_ppm=20000, seed=5)
    y, own = ctx.y, 3
    whole, pay = buffers(ctx, ctx.payload_bytes, own)
    _, st = buffers(ctx, ctx.state_bytes, own)
    rng = np.random.default_rng(W)
    for w in range(own):
        ctx.mc_compress_groups(w, 0, tensors(rng, 10.0 ** -w, 0), st[w] if ctx.cfg.use_ef else None, pay[w])
    order = [int(w) for w in rng.integers(0, own, W)]            # the workers' payloads are three in turn
    out = [[torch.full((n,), 7.0, device=DEV) for n in SIZES] for _ in range(2)]
    for j in range(y):
        ctx.mc_decompress_sum(j, [pay[w][j] for w in order], 1.0 / W, [out[0][j]])
    ctx.mc_decompress_sum_groups([pay[w][j] for w in order for j in range(y)], W, 1.0 / W, out[1])
    assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(*out))
    assert ctx.mc_last_device_status() == B.MC_OK


@pytest.mark.parametrize("algo", ["topk", "dgc", "randk"])
def test_groups_that_share_the_scratch(algo):
    """More groups of 64 tiles than a context keeps key lists for (512 MiB): scratch of the size of the largest, which the
    groups of a call use in turn."""
    numel = [64 * 4096 - 1] * 255 + [64 * 4096, 70000, 3]
    y = len(numel)
    a, b = (B.Context(algo, numel, list(range(y + 1)), ratio_ppm=1000, seed=6) for _ in range(2))
    (pa, one_p), (pb, all_p) = buffers(a, a.payload_bytes, 1), buffers(b, b.payload_bytes, 1)
    (sa, one_s), (sb, all_s) = buffers(a, a.state_bytes, 1), buffers(b, b.state_bytes, 1)
    a.profile_enable(True)
    b.profile_enable(True)
    for it in range(3):
        g = list(torch.randn(sum(numel), device=DEV, generator=torch.Generator(DEV).manual_seed(it)).split(numel))
        for j in range(y):
            a.mc_compress(j, 0, it, [g[j]], one_s[0][j], one_p[0][j])
        b.mc_compress_groups(0, it, g, all_s[0], all_p[0])
        assert torch.equal(pa, pb) and torch.equal(sa, sb), it
    assert a.profile_read()["lean_select"]["launches"] == b.profile_read()["lean_select"]["launches"] == 3 * y
    # ... and the last groups against the oracle
    cfg = O.Config(B.ALGO_IDS[algo], ratio_ppm=1000, seed=6)
    for j in (y - 3, y - 2, y - 1):
        held = O.new_state(cfg, numel[j])
        for it in range(3):
            x = torch.randn(sum(numel), device=DEV, generator=torch.Generator(DEV).manual_seed(it)).split(numel)[j].cpu().numpy()
            want, _ = O.compress(cfg, x, held, group_off=sum(numel[:j]), worker=0, it=it)
        assert np.array_equal(one_p[0][j].cpu().numpy()[:want.size], want), j

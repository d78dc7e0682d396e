"""Sparsified groups whose selection is one block's (at most 32 tiles of 4096 elements and 6144 kept entries), around both
limits and where more candidates pass the filter than the block holds: payload, residual and route against the oracle, and
byte for byte against the two-kernel form (which runs while the profiler is on) in calls of every kind."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu
ALGOS = ["topk", "dgc", "randk"]


def levels(rng, n):
    """Few magnitudes, many of each: the threshold is always one of several equal keys, of both signs."""
    return (np.round(rng.standard_normal(n) * 200.0) / 200.0).astype(np.float32)


def pile(rng, n):
    """A sixth of the values within a tenth below the largest 6144: on a call's way through the filter there are more than 16384."""
    g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    g[rng.permutation(n)[:6144]] = rng.uniform(1.0, 1.1, 6144).astype(np.float32)[:n]
    at = rng.permutation(n)[:n // 6]
    g[at] = np.where(np.abs(g[at]) < 0.5, rng.uniform(0.9, 0.999, len(at)), g[at]).astype(np.float32)
    return g


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("n, ppm, draw", [
    (1, 10000, "normal"), (64, 1000000, "normal"), (1025, 10000, "levels"), (4097, 100000, "levels"), (16 * 4096 + 1, 10000, "levels"),
    (6144, 1000000, "normal"), (6145, 1000000, "normal"),                                       # kept: everything, the most and one more
    (32 * 4096, 46875, "normal"), (32 * 4096, 46883, "normal"), (32 * 4096 + 1, 10000, "normal"),      # kept 6144, 6145; tiles 33
    (32 * 4096, 46875, "pile"), (20 * 4096 + 77, 70000, "pile")])
def test_around_the_limits(algo, n, ppm, draw):
    ctx = B.Context(algo, [n], [0, 1], ratio_ppm=ppm, seed=4)
    cfg = O.Config(B.ALGO_IDS[algo], ratio_ppm=ppm, seed=4)
    state = torch.zeros(ctx.state_bytes(0), dtype=torch.uint8, device=H.DEV)
    pay = torch.full((ctx.payload_bytes(0),), 0xAB, dtype=torch.uint8, device=H.DEV)
    held = O.new_state(cfg, n)
    rng = np.random.default_rng([n, ppm])
    passed = []                                  # the filter, on the usual route
    for it in range(5):
        g = {"normal": lambda: rng.standard_normal(n).astype(np.float32), "levels": lambda: levels(rng, n), "pile": lambda: pile(rng, n)}[draw]()
        ctx.mc_compress(0, 0, it, H.device_tensors(g, [n]), state, pay)
        want, _ = O.compress(cfg, g, held, group_off=0, worker=0, it=it)
        assert np.array_equal(pay.cpu().numpy(), want), (it, ctx.mc_select_stats())
        if ctx.mc_last_select_route() == B.MC_SELECT_FAST:
            passed.append(ctx.mc_select_stats()["last_candidates"])
    assert draw != "pile" or algo != "topk" or max(passed) > 16384
    e = torch.empty(O.state_floats(cfg, n), dtype=torch.float32, device=H.DEV)
    ctx.mc_state_export_residual(0, state, e)
    assert H.same_bits(e.cpu().numpy(), held)
    assert ctx.mc_last_device_status() == B.MC_OK
    ctx.close()


@pytest.mark.parametrize("algo", ALGOS)
def test_same_as_the_two_kernels_in_calls_of_every_kind(algo):
    numel, bounds = [30000, 3, 0, 200, 131072, 5], [0, 2, 3, 4, 5, 6]
    a, b = (B.Context(algo, numel, bounds, seed=2, ratio_ppm=20000) for _ in range(2))
    a.profile_enable(True)                       # one kernel per step
    rng = np.random.default_rng(3)
    bufs = [([torch.zeros(c.state_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(5)],
             [torch.zeros(c.payload_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(5)]) for c in (a, b)]
    for it in range(10):
        g = [torch.from_numpy((rng.standard_normal(n) * (4.0 if it == 6 else 1.0)).astype(np.float32)).to(H.DEV) for n in numel]
        b.profile_enable(it in (4, 5))           # (the forms take turns on one context, too)
        for c, (st, pay) in zip((a, b), bufs):
            if it % 2:
                c.mc_compress_groups(0, it, g, st, pay)
            else:
                for j in range(5):
                    c.mc_compress(j, 0, it, g[bounds[j]:bounds[j + 1]], st[j], pay[j])
        for x, y in zip(bufs[0][0] + bufs[0][1], bufs[1][0] + bufs[1][1]):
            assert torch.equal(x, y), it
        ra, rb = a.mc_select_stats(), b.mc_select_stats()
        assert ra == rb and a.mc_last_select_route() == b.mc_last_select_route()
    a.profile_enable(False)
    assert "lean_emit" in a.profile_read()
    a.close()
    b.close()


@pytest.mark.parametrize("tiles", [8, 9, 32])            # on the slow routes: one block, three, eight
@pytest.mark.parametrize("passed", [600, 1023, 1025, 2047, 2048, 2049, 4097, 16383, 16384, 16385, 32000])
def test_as_many_candidates(tiles, passed):
    """So many elements within half a percent of each other and all others far below: they and no others pass the filter,
    spread over the group, and crowded into as few chunks as hold them."""
    n = tiles * 4096 - 5
    ppm = 1000000 * 600 // n
    cfg = O.Config(O.TOPK, use_ef=0, ratio_ppm=ppm, seed=4)
    for crowded in (False, True):
        ctx = B.Context("topk", [n], [0, 1], use_ef=0, ratio_ppm=ppm, seed=4)
        pay = torch.full((ctx.payload_bytes(0),), 0xAB, dtype=torch.uint8, device=H.DEV)
        rng = np.random.default_rng([tiles, passed, crowded])
        for it in range(4):
            g = (rng.standard_normal(n) * 1e-4).astype(np.float32)
            at = n - passed + np.arange(passed) if crowded else rng.permutation(n)[:passed]
            g[at] = rng.uniform(1.0, 1.005, passed).astype(np.float32) * np.where(rng.random(passed) < 0.5, 1.0, -1.0).astype(np.float32)
            ctx.mc_compress(0, 0, it, H.device_tensors(g, [n]), None, pay)
            want, _ = O.compress(cfg, g, None, group_off=0, worker=0, it=it)
            assert np.array_equal(pay.cpu().numpy(), want), (crowded, it)
            if it:                               # (the first call of a context takes no filter)
                assert ctx.mc_last_select_route() == B.MC_SELECT_FAST and ctx.mc_select_stats()["last_candidates"] == passed
        assert ctx.mc_last_device_status() == B.MC_OK
        ctx.close()


@pytest.mark.parametrize("algo", ALGOS)
def test_slow_routes_of_groups_of_every_size(algo):
    """The largest values rise and fall by turns, so that every call misses the window, and then many are equal: groups whose slow
    routes run on one to eight blocks, each by itself and all in one call."""
    numel = [4096 * t - 3 for t in (1, 4, 8, 9, 12, 13, 17, 29, 32)]
    y = len(numel)
    a, b = (B.Context(algo, numel, list(range(y + 1)), ratio_ppm=10000, seed=2) for _ in range(2))
    cfg = O.Config(B.ALGO_IDS[algo], ratio_ppm=10000, seed=2)
    bufs = [([torch.zeros(c.state_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(y)],
             [torch.zeros(c.payload_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(y)]) for c in (a, b)]
    held = [O.new_state(cfg, n) for n in numel]
    off = np.concatenate([[0], np.cumsum(numel)])
    rng = np.random.default_rng(5)
    for it in range(6):
        scale = [1.0, 20.0, 400.0, 0.01, 8000.0, 1.0][it]
        g = [(rng.standard_normal(n) * scale).astype(np.float32) for n in numel]
        if it >= 4:
            g = [(np.sign(v) * scale).astype(np.float32) for v in g]
        dev = [torch.from_numpy(v).to(H.DEV) for v in g]
        for j in range(y):
            a.mc_compress(j, 0, it, [dev[j]], bufs[0][0][j], bufs[0][1][j])
        b.mc_compress_groups(0, it, dev, *bufs[1])
        for j in range(y):
            want, _ = O.compress(cfg, g[j], held[j], group_off=int(off[j]), worker=0, it=it)
            assert np.array_equal(bufs[0][1][j].cpu().numpy(), want), (it, j)
            assert torch.equal(bufs[0][1][j], bufs[1][1][j]) and torch.equal(bufs[0][0][j], bufs[1][0][j]), (it, j)
    ra, rb = a.mc_select_stats(), b.mc_select_stats()
    assert all(ra[r] == rb[r] for r in ("above", "fast", "refill", "dense")) and ra["fast"] < 6 * y
    assert a.mc_last_device_status() == B.MC_OK and b.mc_last_device_status() == B.MC_OK
    a.close()
    b.close()

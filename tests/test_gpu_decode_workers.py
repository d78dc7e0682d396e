"""Decompress-and-sum around the batches of eight in which the workers' payloads are asked for, with scales for which a term
is not a product of two exact factors (an odd subnormal, infinity, NaN): bit for bit against the oracle's sums."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALE, SCALE_LO = 24, 32          # bytes of the header
ODD = {"plain": [0.01], "tiny": [3 * 2.0 ** -149, 2.0 ** -149, 0.01], "inf": [0.01, np.inf, 0.5], "nan": [np.nan, 0.25, 0.0]}


@pytest.mark.parametrize("algo", ["efsign", "onebit", "signsgd", "terngrad", "qsgd", "fp16", "topk"])
@pytest.mark.parametrize("kind", list(ODD))
def test_numbers_of_workers(algo, kind):
    scaled = algo in ("efsign", "onebit", "terngrad")
    if kind != "plain" and not scaled:
        pytest.skip("no scale that the decode multiplies with")
    n, sizes = 12345, [8192, 1, 4000, 152]
    ef = 0 if algo == "signsgd" else 1
    cfg = O.Config(B.ALGO_IDS[algo], use_ef=ef, seed=1)
    ctx = B.Context(algo, sizes, [0, 4], use_ef=ef, seed=1)
    rng = np.random.default_rng(list(ODD).index(kind))
    sent = []
    for w in range(64):
        p, _ = O.compress(cfg, rng.standard_normal(n).astype(np.float32), O.new_state(cfg, n) if ef else None, worker=w)
        if kind != "plain":
            p[SCALE:SCALE + 4] = np.array([ODD[kind][w % len(ODD[kind])]], np.float32).view(np.uint8)
            if algo == "onebit":
                p[SCALE_LO:SCALE_LO + 4] = np.array([ODD[kind][(w + 1) % len(ODD[kind])]], np.float32).view(np.uint8)
        sent.append(p)
    dev = [torch.from_numpy(p).to(DEV) for p in sent]
    for W in (1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 25, 64):
        out = [torch.full((m,), 5.0, device=DEV) for m in sizes]
        ctx.mc_decompress_sum(0, dev[:W], 0.5, out)
        got, want = torch.cat(out).cpu().numpy(), O.decompress_sum(sent[:W], n, 0.5)
        gone = np.isnan(want)
        assert np.array_equal(np.isnan(got), gone), W
        assert np.array_equal(got.view(np.uint32)[~gone], want.view(np.uint32)[~gone]), W
    assert ctx.mc_last_device_status() == B.MC_OK


@pytest.mark.parametrize("algo", list(B.ALGO_IDS))
@pytest.mark.parametrize("byte", [0, 4, 8, 13, 16])
def test_each_field_of_a_header_is_checked(algo, byte):
    """The last worker's header with one byte changed (magic, algorithm, elements, kept entries); 16: only where there are any."""
    if byte == 16 and algo not in ("topk", "dgc", "randk"):
        pytest.skip("k is not used")
    ef = 0 if algo == "signsgd" else 1
    ctx = B.Context(algo, [5000], [0, 1], use_ef=ef, seed=1)
    cfg = O.Config(B.ALGO_IDS[algo], use_ef=ef, seed=1)
    p, _ = O.compress(cfg, np.random.default_rng(0).standard_normal(5000).astype(np.float32), O.new_state(cfg, 5000) if ef else None)
    good, bad = torch.from_numpy(p.copy()).to(DEV), torch.from_numpy(p.copy()).to(DEV)
    bad[byte] ^= 0x40
    out = [torch.zeros(5000, device=DEV)]
    for W in (1, 9, 64):
        ctx.mc_decompress_sum(0, [good] * W, 1.0, out)
        assert ctx.mc_last_device_status() == B.MC_OK
        ctx.mc_decompress_sum(0, [good] * (W - 1) + [bad], 1.0, out)
        assert ctx.mc_last_device_status() == B.MC_ERR_PAYLOAD


RUNS = [0, 1, 63, 64, 65, 127, 128, 129, 256, 257, 511, 1023, 1024, 1025, 2500, 4096]


@pytest.mark.parametrize("W", [1, 2, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("where", ["anywhere", "one chunk", "chunk edges", "first and last"])
def test_runs_of_a_tile(W, where):
    """One tile in the middle with runs of very different lengths from worker to worker, spread or crowded into a part of it."""
    n, tile = 5 * 4096 + 77, 2 * 4096
    k = O.topk_count(n, 220000)
    ctx = B.Context("topk", [9000, n - 9000], [0, 2], ratio_ppm=220000)
    rng = np.random.default_rng([W, len(where)])
    for first in (0, 5, 11):
        sent = []
        for w in range(W):
            run = RUNS[(first + w) % len(RUNS)]
            if where == "one chunk" and run <= 1024:
                inside = tile + 1024 + rng.choice(1024, run, replace=False)
            elif where == "chunk edges" and run <= 1024:
                edge = np.concatenate([1024 * c + np.r_[0:128, 896:1024] for c in range(4)])
                inside = tile + rng.choice(edge, run, replace=False)
            elif where == "first and last" and run <= 2048:
                inside = tile + rng.choice(np.r_[0:1024, 3072:4096], run, replace=False)
            else:
                inside = tile + rng.choice(4096, run, replace=False)
            others = np.r_[0:tile, tile + 4096:n]
            idx = np.sort(np.concatenate([inside, rng.choice(others, k - run, replace=False)])).astype(np.uint32)
            sent.append(O.with_directory(B.ALGO_IDS["topk"], n, idx, rng.standard_normal(k).astype(np.float32)))
        out = [torch.full((m,), 5.0, device=DEV) for m in (9000, n - 9000)]
        ctx.mc_decompress_sum(0, [torch.from_numpy(p).to(DEV) for p in sent], 0.25, out)
        got, want = torch.cat(out).cpu().numpy(), O.decompress_sum(sent, n, 0.25)
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), first
    assert ctx.mc_last_device_status() == B.MC_OK


@pytest.mark.parametrize("W", [3, 6, 10, 11])
def test_runs_of_a_tile_with_other_numbers_of_workers(W):
    for where in ("anywhere", "one chunk", "chunk edges", "first and last"):
        test_runs_of_a_tile(W, where)


@pytest.mark.parametrize("algo", ["qsgd", "efsign", "terngrad", "topk"])
@pytest.mark.parametrize("W", [1, 16, 64])
def test_every_header_of_a_call_over_all_groups_is_checked(algo, W):
    """37 groups, empty ones among them, the first and the last: up to 2368 headers, more than the threads of one block look at.
    One header at a time with a byte changed (at every edge of what 256 threads see, the first and the last of a group)."""
    sizes = [0, 70, 5000, 0, 4096] + [33 + 7 * j for j in range(30)] + [9000, 0]
    y = len(sizes)
    cfg = O.Config(B.ALGO_IDS[algo], seed=1)
    ctx = B.Context(algo, sizes, list(range(y + 1)), seed=1)
    room = [(ctx.payload_bytes(j) + 15) // 16 * 16 for j in range(y)]
    at = np.concatenate([[0], np.cumsum(room)])
    rng = np.random.default_rng(0)
    one = np.full(at[-1], 0xAB, np.uint8)        # (an empty group's payload is not looked at)
    for j, n in enumerate(sizes):
        if n:
            p, _ = O.compress(cfg, rng.standard_normal(n).astype(np.float32), O.new_state(cfg, n))
            one[at[j]:at[j] + p.size] = p
    wire = torch.from_numpy(one).to(DEV).repeat(W, 1)
    pays = B.ptr_array([wire[w, at[j]:at[j + 1]] for w in range(W) for j in range(y)])
    outs = [torch.zeros(n, device=DEV) for n in sizes]
    for _ in range(2):                           # (twice: a list of addresses that is new, and one that is known)
        ctx.mc_decompress_sum_groups(pays, W, 1.0, outs)
        assert ctx.mc_last_device_status() == B.MC_OK
    live = [j for j in range(y) if sizes[j]]
    flat = sorted({j * W + w for j in (live[0], live[1], live[-1]) for w in (0, W - 1)} | {i for b in range(0, y * W, 256) for i in (b - 1, b) if i >= 0})
    for i in flat:                               # (number of the header in the order in which the call lists them)
        j, w = divmod(i, W)
        if not sizes[j]:
            continue
        for byte in (0, 4, 8):
            wire[w, at[j] + byte] ^= 0x40
            ctx.mc_decompress_sum_groups(pays, W, 1.0, outs)
            assert ctx.mc_last_device_status() == B.MC_ERR_PAYLOAD, (j, w, byte)
            wire[w, at[j] + byte] ^= 0x40
    ctx.mc_decompress_sum_groups(pays, W, 1.0, outs)
    assert ctx.mc_last_device_status() == B.MC_OK


def near_window(n, chunk, size):
    """The entries of a run that are looked at for a chunk of its tile: `size` around where they lie if spread evenly."""
    middle = n * (2 * chunk + 1) // 8
    return 0 if n <= size or middle <= size // 2 else min(middle - size // 2, n - size)


@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 9, 12, 14])
@pytest.mark.parametrize("n_run", [256, 257, 300, 511, 512, 513, 640, 768, 769])
def test_long_runs_of_few_workers(W, n_run):
    """Runs that are read where the chunk's part ought to be, of all workers the same length or nearly: spread evenly (the
    part is there), and of one worker crowded so that a chunk's part begins or ends up to one entry beside what is read."""
    n, tile = 5 * 4096 + 77, 2 * 4096
    k = O.topk_count(n, 60000)
    ctx = B.Context("topk", [9000, n - 9000], [0, 2], ratio_ppm=60000)
    rng = np.random.default_rng([W, n_run])
    others = np.r_[0:tile, tile + 4096:n]
    cases = [("even", 0, 0, 0, 256)] + [(side, c, d, w, size) for side in ("begins", "ends") for c in range(4) for d in (-1, 0, 1)
                                        for w, size in {(0, 256), (W - 1, 256), (W - 1, 192)}]
    for side, c, d, astray, size in cases:
        sent = []
        for w in range(W):
            run = n_run - (w % 3 == 1)
            inside = np.sort(rng.choice(4096, run, replace=False))
            if side != "even" and w == astray:
                at = near_window(run, c, size) + (d if side == "begins" else size + d)           # entries before the edge
                edge = 1024 * (c if side == "begins" else c + 1)
                at = min(max(at, run - (4096 - edge)), min(run, edge), run) if 0 <= at <= run else run * edge // 4096
                inside = np.concatenate([rng.choice(edge, at, replace=False), edge + rng.choice(4096 - edge, run - at, replace=False)])
                if d == 0 and edge < 4096 and run > at:      # ... and the first one behind it right there
                    inside[at] = edge if edge not in inside[at:] else inside[at]
            idx = np.sort(np.concatenate([tile + inside, rng.choice(others, k - run, replace=False)])).astype(np.uint32)
            sent.append(O.with_directory(B.ALGO_IDS["topk"], n, idx, rng.standard_normal(k).astype(np.float32)))
        out = [torch.full((m,), 5.0, device=DEV) for m in (9000, n - 9000)]
        ctx.mc_decompress_sum(0, [torch.from_numpy(p).to(DEV) for p in sent], 0.25, out)
        got, want = torch.cat(out).cpu().numpy(), O.decompress_sum(sent, n, 0.25)
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), (side, c, d, astray, size)
    assert ctx.mc_last_device_status() == B.MC_OK


# A launch of so many blocks that a wavefront holds all it can: more than 240 of 8192 elements (bit planes), 256 of 4096 (one code per element)
RAGGED = [1, 37, 1000, 3, 5000, 64, 1023, 1025, 2, 2048, 4095]
LARGE = {"planes": 240 * 8192 + 1, "codes": 256 * 4096 + 1}


def check_large(algo, kind, workers, n, off):
    """One group of many ragged tensors in front of and behind a large one, by itself and in one call with another group."""
    sizes = RAGGED * 3 + [0] + RAGGED[::-1] * 3
    sizes[len(RAGGED) * 3] = n - sum(sizes)
    ef = 0 if algo == "signsgd" else 1
    cfg = O.Config(B.ALGO_IDS[algo], use_ef=ef, seed=1)
    ctx = B.Context(algo, sizes + [70], [0, len(sizes), len(sizes) + 1], use_ef=ef, seed=1)
    rng = np.random.default_rng([n, off, list(ODD).index(kind)])
    sent = []
    for m in (n, 70):
        sent.append([])
        for w in range(min(max(workers), 9)):
            p, _ = O.compress(cfg, rng.standard_normal(m).astype(np.float32), O.new_state(cfg, m) if ef else None, worker=w)
            if kind != "plain":
                p[SCALE:SCALE + 4] = np.array([ODD[kind][w % len(ODD[kind])]], np.float32).view(np.uint8)
                if algo == "onebit":
                    p[SCALE_LO:SCALE_LO + 4] = np.array([ODD[kind][(w + 1) % len(ODD[kind])]], np.float32).view(np.uint8)
            sent[-1].append(p)
    dev = [[torch.from_numpy(p).to(DEV) for p in ps] for ps in sent]
    for W in workers:
        pick = [w % len(sent[0]) for w in range(W)]
        want = np.concatenate([O.decompress_sum([sent[j][w] for w in pick], m, 0.5) for j, m in enumerate((n, 70))])
        for together in (False, True):
            outs = [torch.full((m + 4,), 5.0, device=DEV)[off:off + m] for m in sizes + [70]]
            if together:
                ctx.mc_decompress_sum_groups([dev[j][w] for w in pick for j in range(2)], W, 0.5, outs)
            else:
                ctx.mc_decompress_sum(0, [dev[0][w] for w in pick], 0.5, outs[:-1])
                ctx.mc_decompress_sum(1, [dev[1][w] for w in pick], 0.5, outs[-1:])
            got = torch.cat(outs).cpu().numpy()
            gone = np.isnan(want)
            assert np.array_equal(np.isnan(got), gone), (W, together)
            assert np.array_equal(got.view(np.uint32)[~gone], want.view(np.uint32)[~gone]), (W, together)
    assert ctx.mc_last_device_status() == B.MC_OK
    ctx.close()


@pytest.mark.parametrize("kind,off", [("plain", 0), ("plain", 2), ("tiny", 1), ("inf", 3), ("nan", 0)])
@pytest.mark.parametrize("algo", ["efsign", "onebit", "terngrad", "signsgd", "signum"])
def test_numbers_of_workers_of_many_planes(algo, kind, off):
    if kind != "plain" and algo in ("signsgd", "signum"):
        pytest.skip("no scale that the decode multiplies with")
    check_large(algo, kind, (1, 3, 8, 9, 17, 64), LARGE["planes"], off)


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("algo", ["qsgd", "fp16"])
def test_numbers_of_workers_of_many_codes(algo, off):
    check_large(algo, "plain", (1, 3, 4, 5, 9, 17), LARGE["codes"], off)

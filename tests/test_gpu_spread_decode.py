"""Decompress-and-sum on few tiles, where a wavefront holds a quarter of a chunk and eight workers are one batch, or, of bit planes, a byte per
lane: sizes around what a wavefront and a block hold and around the number of tiles where a wavefront holds more again, outputs at every alignment, in one tensor and
in many, by themselves and in a call over all groups: bit for bit against the oracle's sums."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu


def check(algo, sizes, workers, off):
    n = sum(sizes)
    ef = 0 if algo == "signsgd" else 1
    cfg = O.Config(B.ALGO_IDS[algo], use_ef=ef, seed=3, qsgd_bits=8)
    ctx = B.Context(algo, [7] + sizes, [0, 1, 1 + len(sizes)], use_ef=ef, seed=3, qsgd_bits=8)
    rng = np.random.default_rng([n, len(sizes), off])
    made = [[O.compress(cfg, (rng.standard_normal(m) * (w + 1)).astype(np.float32), O.new_state(cfg, m) if ef else None, worker=w)[0] for w in range(min(max(workers), 9))]
            for m in (7, n)]
    dev = [[torch.from_numpy(p).to(H.DEV) for p in ps] for ps in made]
    for W in workers:
        pick = [w % len(made[0]) for w in range(W)]
        want = [O.decompress_sum([made[j][w] for w in pick], m, 0.25) for j, m in ((0, 7), (1, n))]
        for together in (False, True):
            outs = [torch.full((m + 4,), 5.0, device=H.DEV)[off:off + m] for m in [7] + sizes]
            if together:
                ctx.mc_decompress_sum_groups([dev[j][w] for w in pick for j in range(2)], W, 0.25, outs)
            else:
                for j, (a, b) in enumerate(((0, 1), (1, 1 + len(sizes)))):
                    ctx.mc_decompress_sum(j, [dev[j][w] for w in pick], 0.25, outs[a:b])
            got = torch.cat(outs).cpu().numpy()
            assert np.array_equal(got.view(np.uint32), np.concatenate(want).view(np.uint32)), (W, together)
    assert ctx.mc_last_device_status() == B.MC_OK
    ctx.close()


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("algo", ["qsgd", "fp16"])
def test_sizes(algo, off):
    for n in (1, 63, 255, 256, 257, 769, 1023, 1024, 1025, 4096, 4097, 3 * 4096 + 1026):
        check(algo, [n], (1, 4, 8, 9, 17), off)
        check(algo, [37] * (n // 37) + [n % 37 + 1], (8, 9), off)


@pytest.mark.parametrize("algo", ["qsgd", "fp16"])
@pytest.mark.parametrize("tiles", [254, 255, 256, 257])
def test_number_of_tiles(algo, tiles):
    check(algo, [tiles * 4096 - 1000, 999], (1, 8), 0)


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("algo", ["efsign", "onebit", "signsgd", "signum", "terngrad"])
def test_sizes_of_planes(algo, off):
    for n in (1, 7, 9, 31, 33, 511, 512, 513, 1025, 8191, 8192, 8193, 2 * 8192 + 1537):
        check(algo, [n], (1, 4, 8, 9, 17), off)
        check(algo, [37] * (n // 37) + [n % 37 + 1], (8, 9), off)


@pytest.mark.parametrize("algo", ["efsign", "onebit", "signsgd", "signum", "terngrad"])
@pytest.mark.parametrize("blocks", [238, 239, 240, 241])
def test_number_of_blocks(algo, blocks):
    check(algo, [blocks * 8192 - 1000, 999], (1, 9), 0)

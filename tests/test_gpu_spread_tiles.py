"""Small groups of the two-pass quantizers, four consecutive elements per thread: sizes around four, a wavefront's 256, a
chunk's 1024 and a tile's 4096, in groups that start at every place inside a block of the random stream, in one tensor and
in many."""
import numpy as np
import pytest

from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ef", [1, 0])
@pytest.mark.parametrize("before", [4, 1, 2, 3])
@pytest.mark.parametrize("algo", ["qsgd", "terngrad"])
def test_sizes_and_places(algo, before, ef):
    for n in (1, 2, 3, 4, 5, 31, 33, 255, 256, 257, 1022, 1025, 4095, 4097, 8191, 3 * 4096 + 258):
        rng = np.random.default_rng([before, n])
        for numel in ([before, n], [before] + [7] * (n // 7) + [n % 7]):
            H.run_parity(numel, algo, 2, 2, 2, lambda w, it: rng.standard_normal(sum(numel)).astype(np.float32), policy=B.MC_PART_USER,
                         user_bounds=[0, 1, len(numel)], use_ef=ef, layout="misaligned" if n % 2 else "separate")


@pytest.mark.parametrize("algo", ["efsign", "onebit", "signsgd", "signum", "fp16", "topk", "dgc", "randk"])
def test_quarters_of_a_chunk(algo):
    """The one-pass compressors on few tiles, where a wavefront holds a quarter of a chunk: sizes around its 256 elements, and
    candidates in every quarter."""
    for n in (1, 63, 64, 255, 256, 257, 511, 513, 767, 769, 1023, 1025, 4095, 4097, 3 * 4096 + 258):
        rng = np.random.default_rng(n)
        for numel in ([3, n], [3] + [37] * (n // 37) + [n % 37]):
            H.run_parity(numel, algo, 2, 2, 2, lambda w, it: rng.standard_normal(sum(numel)).astype(np.float32), policy=B.MC_PART_USER,
                         user_bounds=[0, 1, len(numel)], layout="misaligned" if n % 2 else "separate", ratio_ppm=300000)


@pytest.mark.parametrize("tiles", [128, 512])
@pytest.mark.parametrize("algo", ["efsign", "onebit", "signsgd", "signum", "fp16", "topk", "dgc", "randk"])
def test_around_the_number_of_tiles(algo, tiles):
    for n in (tiles * 4096, tiles * 4096 + 1):
        rng = np.random.default_rng(n)
        numel = [n // 3, 5, n - n // 3 - 5]
        H.run_parity(numel, algo, 1, 1, 2, lambda w, it: rng.standard_normal(n).astype(np.float32), check_decompress=False)

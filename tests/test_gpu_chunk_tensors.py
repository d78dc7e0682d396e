"""Chunks of 1024 elements that hold several tensors, at the counts and places where their walk changes form: one, 64 (the
most whose bounds fit a wavefront's lanes), 65 and more tensors in a chunk, tensors that end at, before and behind the
wavefront's steps of 64 elements, and last chunks of one element, of whole steps and of all but one."""
import numpy as np
import pytest

import harness as H

pytestmark = pytest.mark.gpu
LISTS = {
    "exactly 64": [16] * 64,
    "64 and a last one": [16] * 64 + [1],
    "65": [15] * 64 + [64],
    "64 and part of the next": [15] * 63 + [200, 3],
    "single elements": [1] * 1030,
    "around the steps": [63, 1, 64, 65, 127, 128, 1, 1, 62, 512, 1024, 1],
    "after a whole chunk": [1024, 1000, 24, 2048, 5, 64, 959],
    "last chunk of one element": [4095, 1, 1],
    "last chunk all but one": [700, 1347],
    "last chunk of whole steps": [1000, 24 + 64, 64],
}


@pytest.mark.parametrize("name", LISTS)
@pytest.mark.parametrize("algo", ["efsign", "onebit", "signum", "qsgd", "terngrad", "fp16", "topk", "dgc", "randk"])
def test_tensors_of_a_chunk(algo, name):
    numel = LISTS[name]
    rng = np.random.default_rng(len(numel))
    H.run_parity(numel, algo, 1, 3, 3, lambda w, it: rng.standard_normal(sum(numel)).astype(np.float32), layout="misaligned" if len(numel) % 2 else "separate",
                 ratio_ppm=100000)

"""A sparsifier whose scratch ends in a crowded chunk: the last 1024 elements of the last tile hold 832 to 1024 candidates, so
that on the usual route the select and emit kernels read the chunk's fourth unit, of which the last part lies behind the
chunk.  One group, and the last of two (each has its own part of the scratch).  Those two kernels serve groups of more
than 32 tiles; the groups of two and three tiles are selected from by the kernel for small groups, entry by entry."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("large", [832, 833, 1000, 1024])
@pytest.mark.parametrize("numel", [[2 * 4096], [5000, 3 * 4096], [33 * 4096], [5000, 34 * 4096]])
def test_last_chunk_is_crowded(large, numel):
    y, n = len(numel), numel[-1]
    ppm = 1000000 * 600 // n                     # k = 600 of the last group: the large values and no others are candidates
    ctx = B.Context("topk", numel, list(range(y + 1)), use_ef=0, ratio_ppm=ppm, seed=2)
    ocfg = O.Config(O.TOPK, use_ef=0, ratio_ppm=ppm, seed=2)
    pay = torch.full((ctx.payload_bytes(y - 1),), 0xAB, dtype=torch.uint8, device=H.DEV)
    scale = np.full(n, 1e-3, np.float32)
    scale[n - large:] = 1.0
    for it in range(4):
        rng = np.random.default_rng([17, it])
        g = (rng.uniform(1.0, 1.1, n) * np.where(rng.random(n) < 0.5, 1.0, -1.0)).astype(np.float32) * scale
        ctx.mc_compress(y - 1, 0, it, H.device_tensors(g, numel[-1:]), None, pay)
        op, _ = O.compress(ocfg, g, None, group_off=sum(numel[:-1]), worker=0, it=it)
        assert np.array_equal(pay.cpu().numpy(), op), it
        if it:                                   # (the first call of a context takes no filter)
            assert ctx.mc_last_select_route() == B.MC_SELECT_FAST and ctx.mc_select_stats()["last_candidates"] == large
    ctx.close()

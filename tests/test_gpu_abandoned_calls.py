"""What is left behind by a sparsifier's call whose blocks gave up waiting for each other (forced from the host: with a limit
of one look every kernel still ends normally): the status that is reported, and the context's next calls."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu


def test_a_bad_payload_does_not_hide_an_abandoned_call():
    """The abandoned call leaves its payload unwritten; a decompress-and-sum that then meets it reports the payload, but
    what happened first, and says more, is what the caller has to see."""
    n = 200000
    ctx = B.Context("topk", [n], [0, 1], use_ef=0, seed=1)
    g = torch.randn(n, device=H.DEV)
    pay = torch.zeros(ctx.payload_bytes(0), dtype=torch.uint8, device=H.DEV)
    out = torch.empty(n, device=H.DEV)
    ctx.mc_set_barrier_spin_limit(1)
    ctx.mc_compress(0, 0, 0, [g], None, pay)
    ctx.mc_decompress_sum(0, [pay], 1.0, [out])
    assert ctx.mc_last_device_status() == B.MC_ERR_DEVICE
    ctx.mc_decompress_sum(0, [torch.zeros_like(pay)], 1.0, [out])
    assert ctx.mc_last_device_status() == B.MC_ERR_PAYLOAD
    ctx.mc_set_barrier_spin_limit(0)
    ctx.close()

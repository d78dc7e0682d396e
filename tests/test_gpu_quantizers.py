"""QSGD and TernGrad where their encode pass changes form: whole chunks of a group that starts on a Philox block go four
consecutive elements per lane, all others one element per lane and step.  Payloads against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2103_15195_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ALGO = [("qsgd", 8), ("qsgd", 2), ("terngrad", 8)]


def check(algo, bits, ef, numel, bounds, group, worker, iters=2, shift=0):
    """The group's payloads over a few iterations; `shift`: its tensors start that many elements off a 16-byte boundary."""
    ctx = B.Context(algo, numel, bounds, use_ef=ef, qsgd_bits=bits, seed=0x123456789ABCDEF)
    cfg = O.Config(B.ALGO_IDS[algo], seed=0x123456789ABCDEF, use_ef=ef, qsgd_bits=bits)
    sizes = numel[bounds[group]:bounds[group + 1]]
    n, first = sum(sizes), sum(numel[:bounds[group]])
    state = torch.zeros(ctx.state_bytes(group), dtype=torch.uint8, device=DEV)
    payload = torch.full((ctx.payload_bytes(group),), 0xAA, dtype=torch.uint8, device=DEV)
    held = O.new_state(cfg, n)
    rng = np.random.default_rng([n, first & 0xFFFF, ef])
    for it in range(iters):
        flat = (rng.standard_normal(n) * np.exp(rng.standard_normal(n))).astype(np.float32)
        flat[rng.integers(0, n, 5)] = np.array([0.0, -0.0, 1e-40, -3.0, 0.5], dtype=np.float32)
        parts, at = [], 0
        for s in sizes:
            t = torch.zeros(s + shift, device=DEV)[shift:]
            t.copy_(torch.from_numpy(flat[at:at + s]))
            parts.append(t)
            at += s
        ctx.mc_compress(group, worker, it, parts, state if ef else None, payload)
        want, _ = O.compress(cfg, flat, held, group_off=first, worker=worker, it=it)
        got = payload.cpu().numpy()
        assert O.header(got)["scale"] == O.header(want)["scale"]        # sums in fp64 on both sides
        assert np.array_equal(got, want), (algo, it)


@pytest.mark.parametrize("ef", [0, 1])
@pytest.mark.parametrize("algo,bits", ALGO)
@pytest.mark.parametrize("before", [0, 1, 2, 3, 4])
def test_chunk_edges(algo, bits, ef, before):
    for n in (1023, 1024, 1025, 4096, 5119, 8193):
        check(algo, bits, ef, [before, n], [0, 1, 2], 1, 3)


@pytest.mark.parametrize("algo,bits", ALGO)
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_tensors_off_16_bytes(algo, bits, shift):
    """Without error feedback the pass reads the tensors themselves: whole chunks in one tensor, and straddling ones."""
    check(algo, bits, 0, [5000, 1, 3000, 2048], [0, 4], 0, 1, shift=shift)


@pytest.mark.parametrize("algo,bits", ALGO[::2])
@pytest.mark.parametrize("below", [1028, 1024, 1020, 4])
def test_block_number_past_32_bits(algo, bits, below):
    """A group in which the Philox block number (element / 4) passes 2^32: behind 2^34 - below elements of other groups,
    of which nothing exists but their sizes."""
    large = 4278190000
    numel = [large] * 4 + [2 ** 34 - below - 4 * large, 3000]
    check(algo, bits, 1, numel, list(range(7)), 5, 2)

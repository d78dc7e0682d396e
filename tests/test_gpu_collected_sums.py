"""Group scalars that a block of the compressing launch collects (EF-Sign, QSGD and TernGrad, groups of more than 64 tiles of 4096 elements): payload and
state byte for byte those of a kernel that combines the sums (which runs while the profiler is on), call after call, around the numbers of tiles at
which the collector goes round once more, without error feedback too, and with more groups than there are collectors."""
import pytest
import torch

from paper_2103_15195_amd import binding as B

import harness as H

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.mark.parametrize("ef", [0, 1])
@pytest.mark.parametrize("numel", [
    [65 * TILE], [128 * TILE + 1], [1024 * TILE], [1024 * TILE + 1], [2049 * TILE - 3],      # one group: spread tiles and not, rounds of 1024 tiles
    [65 * TILE, 0, 7, 1500 * TILE + 5], [66 * TILE - 1] + [31 + 997 * j for j in range(140)]])      # groups of all sizes, an empty one; more than 64
@pytest.mark.parametrize("algo", ["efsign", "qsgd", "terngrad"])
def test_the_scalars_of_a_kernel_of_its_own(algo, numel, ef):
    y = len(numel)
    gen = torch.Generator(device=H.DEV).manual_seed(sum(numel) + ef)
    got, want = (B.Context(algo, numel, list(range(y + 1)), use_ef=ef, seed=9) for _ in range(2))
    want.profile_enable(True)
    held = [([torch.zeros(c.state_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(y)],
             [torch.zeros(c.payload_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(y)]) for c in (got, want)]
    for it in range(3):
        grads = [torch.empty(n, device=H.DEV).normal_(generator=gen) * 10.0 ** (it - 1) for n in numel]
        for c, (state, payload) in zip((got, want), held):
            if it % 2 == 0:
                c.mc_compress_groups(2, it, grads, state if ef else None, payload)
            else:
                for j in range(y):
                    c.mc_compress(j, 2, it, grads[j:j + 1], state[j] if ef else None, payload[j])
        for a, b in zip(held[0][0] + held[0][1], held[1][0] + held[1][1]):
            assert torch.equal(a, b), it
    assert "scalar_finalize" in want.profile_read()
    assert got.mc_last_device_status() == B.MC_OK
    got.close(); want.close()


@pytest.mark.parametrize("ef", [0, 1])
@pytest.mark.parametrize("numel", [[64 * TILE, 65 * TILE, 1, 64 * TILE + 1, 63 * TILE - 1, TILE, TILE + 1], [257] * 300 + [130 * TILE] + [3 * TILE] * 20,
                                   [64 * TILE + 1 + 59 * j for j in range(70)]])
@pytest.mark.parametrize("algo", ["efsign", "qsgd", "terngrad"])
def test_groups_of_both_kinds_in_one_call(algo, numel, ef):
    """Groups of at most 64 tiles beside larger ones: their last block to arrive combines their sums, in calls of their own and in one call, by turns;
    and more larger groups than there are blocks to collect for them."""
    test_the_scalars_of_a_kernel_of_its_own(algo, numel, ef)

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


@pytest.mark.parametrize("tiles", [17, 18, 19, 20, 33])
def test_an_abandoned_call_leaves_no_counts_behind(tiles):
    """A call that gave up after its blocks had counted the threshold bin's keys one by one (the route of heavy ties), and
    then calls that take the same route: none of those counts may enter theirs.  From 17 tiles on the route waits."""
    n, ppm = tiles * 4096 - 5, 100000
    ctx = B.Context("topk", [n], [0, 1], use_ef=0, ratio_ppm=ppm, seed=1)
    ocfg = O.Config(O.TOPK, use_ef=0, ratio_ppm=ppm, seed=1)
    pay = torch.zeros(ctx.payload_bytes(0), dtype=torch.uint8, device=H.DEV)
    rng = np.random.default_rng(tiles)

    def call(it, tie_key):
        # 30 % of the elements have one magnitude, which is where the threshold of the largest 10 % falls
        g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
        tie = rng.random(n) < 0.3
        g[tie] = np.uint32(tie_key).view(np.float32) * np.where(rng.random(int(tie.sum())) < 0.5, 1, -1).astype(np.float32)
        ctx.mc_compress(0, 0, it, H.device_tensors(g, [n]), None, pay)
        return O.compress(ocfg, g, None, group_off=0, worker=0, it=it)[0]

    one = 0x3F800000
    for it in range(2):
        assert np.array_equal(call(it, one), pay.cpu().numpy())
    assert ctx.mc_last_select_route() == B.MC_SELECT_DENSE
    ctx.mc_set_barrier_spin_limit(1)
    call(2, one + 1900)                          # counted near the top of a bin of 2048 keys
    assert ctx.mc_last_device_status() == B.MC_ERR_DEVICE
    ctx.mc_set_barrier_spin_limit(0)
    for it in (3, 4):
        assert np.array_equal(call(it, one + 100), pay.cpu().numpy()), it
        assert ctx.mc_last_select_route() == B.MC_SELECT_DENSE
    assert ctx.mc_last_device_status() == B.MC_OK
    ctx.close()


@pytest.mark.parametrize("ef", [0, 1])
@pytest.mark.parametrize("numel", [[65 * 4096], [1500 * 4096 + 5], [65 * 4096, 0, 7, 700 * 4096 + 5]])
@pytest.mark.parametrize("algo", ["efsign", "qsgd", "terngrad"])
def test_partial_sums_that_came_too_late_enter_no_later_call(algo, numel, ef):
    """EF-Sign, QSGD and TernGrad on groups of more than 2^18 elements, whose combining block left before the other blocks' sums were there: the
    payloads say so, also of the calls until the status has been read, and from then on calls are those of a context that always waited."""
    y, large = len(numel), [j for j, n in enumerate(numel) if n > 2 ** 18]
    held = []
    for _ in range(2):
        ctx = B.Context(algo, numel, list(range(y + 1)), use_ef=ef, seed=5)
        held.append((ctx, [torch.zeros(ctx.state_bytes(j), dtype=torch.uint8, device=H.DEV) for j in range(y)],
                     [torch.full((ctx.payload_bytes(j),), 0xAB, dtype=torch.uint8, device=H.DEV) for j in range(y)]))
    (got, state, payload), (want, _, _) = held
    gen = torch.Generator(device=H.DEV).manual_seed(len(numel))

    def call(ctxs, it, together):
        grads = [torch.empty(n, device=H.DEV).normal_(generator=gen) * 2.0 ** it for n in numel]
        for c, s, p in ctxs:
            if together:
                c.mc_compress_groups(1, it, grads, s if ef else None, p)
            else:
                for j in range(y):
                    c.mc_compress(j, 1, it, grads[j:j + 1], s[j] if ef else None, p[j])

    for round in range(2):
        together = round == 0
        got.mc_set_barrier_spin_limit(1)
        call(held[:1], 0, together)
        got.mc_set_barrier_spin_limit(0)
        assert all(O.header(payload[j].cpu().numpy())["magic"] == 0 for j in large)
        call(held[:1], 1, not together)          # not read yet
        assert all(O.header(payload[j].cpu().numpy())["magic"] == 0 for j in large)
        assert got.mc_last_device_status() == B.MC_ERR_DEVICE
        assert got.mc_last_device_status() == B.MC_OK
        out = [torch.zeros(numel[large[0]], device=H.DEV)]
        got.mc_decompress_sum(large[0], [payload[large[0]]], 1.0, out)
        assert got.mc_last_device_status() == B.MC_ERR_PAYLOAD
        for c, s, _ in held:                     # "import a residual again"
            for j in range(y if ef else 0):
                if numel[j]:
                    c.mc_state_import_residual(j, torch.linspace(-1.0, 1.0, numel[j], device=H.DEV), s[j])
        for it in range(2, 5):
            call(held, it, it % 2 == 0)
            for a, b in zip(held[0][2] + (held[0][1] if ef else []), held[1][2] + (held[1][1] if ef else [])):
                assert torch.equal(a, b), (round, it)
        assert got.mc_last_device_status() == B.MC_OK
    got.close(); want.close()

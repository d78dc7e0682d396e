"""The work that a data-parallel training program has this library do, as cases that can be timed and checked.

One pass is what one rank does per iteration: it compresses its own gradient, group by group (its error-feedback
memory is updated on the way), and decompresses and sums the payloads that all ranks sent, its own among them.  What
the network does in between is not part of it: the peers' payloads lie in device memory, as an allgather leaves them,
and are made here in the documented wire format without the library.  A few cases take one of the two directions by
itself.  The tensor lists are those of the repository's benchmark configurations, or generic ragged ones.
"""
import math
import random

import numpy as np
import torch

from paper_2103_15195_amd import binding as B
from paper_2103_15195_amd import workloads as WL

DEV = "cuda:0"
MODELS = {"mlp": 0, "resnet20": 1, "resnet50": 2, "resnet101": 3, "maskrcnn": 4}
HEADER = 128                      # bytes in front of a payload's body and of a state's floats
MAGIC = 0x3150434D
TILE = 4096                       # elements per entry of a sparse payload's directory
PLACE = 512                       # bytes: what the caching allocator rounds a tensor's place to
SPARSE = ("topk", "dgc", "randk")
STATELESS = ("signsgd",)
ALWAYS_STATE = ("dgc", "signum", "randk")
GRADIENTS = 2                     # gradients in rotation: an iteration's differs from the one before
SEED = 7                          # of the stochastic compressors: a constant of the training run


def _case(name, model, algo, y, W, direction="step", calls="groups", ppm=10000, ef=1, bits=8, sample=0, tensors=0, elems=0, shape_seed=0):
    c = dict(model=model, algo=algo, groups=y, workers=W, direction=direction, calls=calls, ppm=ppm, ef=ef, bits=bits, sample=sample,
             tensors=tensors, elems=elems, shape_seed=shape_seed)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest: a perceptron in two groups, each compressed as soon as back-propagation has it; nothing but latency
        _case("mlp_efsign", "mlp", "efsign", 2, 4, calls="each"),
        # a small convolutional network in a few groups, sparsified and quantized
        _case("resnet20_topk", "resnet20", "topk", 4, 8),
        _case("resnet20_qsgd", "resnet20", "qsgd", 8, 8),
        # the layer-wise baseline that the paper starts from: one group per tensor, 161 of them, from 64 elements to 2.4 million
        _case("resnet50_layerwise_efsign", "resnet50", "efsign", 161, 8),
        # the headline: the whole model merged into one group
        _case("resnet50_efsign", "resnet50", "efsign", 1, 8, calls="each"),
        # the other headline algorithm, each direction by itself
        _case("resnet50_topk_compress", "resnet50", "topk", 1, 8, direction="compress", calls="each"),
        _case("resnet50_topk_decompress", "resnet50", "topk", 1, 8, direction="decompress", calls="each"),
        # two and three groups, as the partition search returns them, momentum state and a two-pass quantizer
        _case("resnet50_dgc", "resnet50", "dgc", 2, 8, ppm=1000),
        _case("resnet50_qsgd", "resnet50", "qsgd", 3, 8),
        # the largest: sixteen workers
        _case("resnet101_efsign_w16", "resnet101", "efsign", 1, 16, calls="each"),
        # heavy-tailed values, group starts that are no multiple of four elements, overlapped with back-propagation
        _case("maskrcnn_topk", "maskrcnn", "topk", 4, 8, calls="each"),
        # odd tensor sizes throughout and an odd number of workers
        _case("ragged_terngrad", "ragged", "terngrad", 1, 5, tensors=97, elems=10000019, shape_seed=1, calls="each"),
    ]


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        model = rng.choice(list(MODELS) + ["ragged"] * 5)
        algo = rng.choice(["efsign", "topk", "dgc", "qsgd", "terngrad", "fp16", "signsgd", "signum", "onebit", "randk"])
        tensors, elems, shape_seed = 0, 0, 0
        if model == "ragged":
            elems = int(10.0 ** rng.uniform(3.0, 7.6)) | 1
            tensors = max(1, min(int(10.0 ** rng.uniform(0.0, 2.5)), elems // 8))
            shape_seed = rng.randrange(1 << 20)
        c = _case(None, model, algo, 1, rng.choice([1, 2, 3, 4, 5, 8, 8, 12, 16]), tensors=tensors, elems=elems, shape_seed=shape_seed,
                  direction=rng.choice(["step", "step", "step", "compress", "decompress"]), calls=rng.choice(["groups", "each"]))
        count = len(_numel(c))
        c["groups"] = min(count, rng.choice([1, 1, 2, 3, 4, 8, 16, 161]))
        if algo in SPARSE:
            c["ppm"] = rng.choice([1000, 10000, 10000, 50000])
        if algo == "dgc" and rng.random() < 0.25:
            c["sample"] = 10000
        if algo == "qsgd":
            c["bits"] = rng.choice([4, 8, 8])
        if algo in STATELESS or (algo not in ALWAYS_STATE and rng.random() < 0.15):
            c["ef"] = 0
        if work(c)["bytes"] <= most:
            return c


# ---- sizes ---------------------------------------------------------------------------------------------------------
def _numel(case):
    if case["model"] in MODELS:
        return [int(n) for n in WL.workload(MODELS[case["model"]]).numel]
    rng = random.Random(case["shape_seed"])                 # sizes over three decades, odd ones among them
    share = [10.0 ** rng.uniform(0.0, 3.0) for _ in range(case["tensors"])]
    total = sum(share)
    sizes = [max(1, int(case["elems"] * s / total)) for s in share]
    sizes[rng.randrange(len(sizes))] += max(0, case["elems"] - sum(sizes))
    return sizes


def _std(case):
    if case["model"] in MODELS:
        return WL.tensor_std(WL.workload(MODELS[case["model"]]))
    rng = random.Random(case["shape_seed"] + 1)
    return np.array([10.0 ** rng.uniform(-4.0, -1.0) for _ in range(case["tensors"])])


def _even(numel, y):
    """Group boundaries, even by number of elements, every group at least one tensor."""
    N, total, before, bounds, t = len(numel), sum(numel), 0, [0], 0
    for j in range(1, y):
        while t < N and before * y < total * j:
            before += numel[t]
            t += 1
        bounds.append(min(max(t, bounds[-1] + 1), N - (y - j)))
    return bounds + [N]


def _sizes(case):
    """(tensor sizes, boundaries, elements of the groups)"""
    numel = _numel(case)
    bounds = _even(numel, case["groups"])
    return numel, bounds, [sum(numel[bounds[j]:bounds[j + 1]]) for j in range(case["groups"])]


def _kept(case, n):
    return min(n, max(1, n * case["ppm"] // 1000000))


def _room(case, n):
    """Entries that a sparse payload has room for."""
    return min(n, 2 * _kept(case, n)) if case["sample"] else _kept(case, n)


def _payload_bytes(case, n):
    algo, words = case["algo"], (n + 31) // 32
    if algo in ("efsign", "onebit", "signsgd", "signum"):
        return HEADER + 4 * words
    if algo == "terngrad":
        return HEADER + 8 * words
    if algo == "qsgd":
        return HEADER + (n + 3) // 4 * 4
    if algo == "fp16":
        return HEADER + (2 * n + 3) // 4 * 4
    return HEADER + 8 * _room(case, n) + 4 * ((n + TILE - 1) // TILE + 1)


def work(case):
    _, _, sizes = _sizes(case)
    n, W = sum(sizes), case["workers"]
    sent = sum(_payload_bytes(case, m) for m in sizes)
    b = f = 0
    if case["direction"] != "decompress":
        memory = 0 if case["algo"] in STATELESS or not case["ef"] else 16 if case["algo"] == "dgc" else 8      # read and written
        b += n * (4 + memory) + sent
        f += 4 * n
    if case["direction"] != "compress":
        b += W * sent + 4 * n
        f += (W if case["algo"] not in SPARSE else 1) * n
    return {"bytes": b, "flops": f}


def tolerance(case):
    # values, indices, codes and the order of the sums are fixed bit for bit; only the group scalars of these come out of
    # a sum (in 64 bits), whose order may move their last bit, and with it the memory of later passes and a code at the edge
    # (a payload of the smallest group has few words, one of them the scalar)
    if case["algo"] in ("efsign", "onebit", "qsgd"):
        return {"rel": 2.5e-7, "max": 1e-5, "differ": 1e-3}
    return "exact"


# ---- values --------------------------------------------------------------------------------------------------------
def _gradient(case, seed, worker, it):
    """One worker's gradient as one flat fp32 vector, from the seed alone."""
    numel = _numel(case)
    total = sum(numel)
    gen = torch.Generator(device=DEV)
    gen.manual_seed((seed * 1000003 + worker * 1009 + it) & 0x7FFFFFFFFFFF)
    x = torch.empty(total, dtype=torch.float32, device=DEV).normal_(generator=gen)
    if case["model"] == "maskrcnn":                              # Student's t with three degrees of freedom
        c = torch.zeros_like(x)
        for _ in range(3):
            c += torch.empty_like(x).normal_(generator=gen).square_()
        x *= (c / 3.0).rsqrt_()
    std = torch.tensor(_std(case), dtype=torch.float32, device=DEV)
    x *= torch.repeat_interleave(std, torch.tensor(numel, device=DEV), output_size=total)
    return x, gen


def _philox(case, first, n, worker, it):
    """Words of the documented random stream for elements first .. first + n - 1 of the model."""
    J = torch.arange(first >> 2, (first + n + 3) >> 2, dtype=torch.int64, device=DEV)
    low = 0xFFFFFFFF
    c0, c1 = J & low, J >> 32
    c2, c3 = torch.full_like(J, worker), torch.full_like(J, it & low)
    k0, k1 = SEED & low, SEED >> 32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57              # the low 64 bits of the products, whatever their sign
        c0, c1, c2, c3 = ((p1 >> 32) & low) ^ c1 ^ k0, p1 & low, ((p0 >> 32) & low) ^ c3 ^ k1, p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    off = first & 3
    return torch.stack([c0, c1, c2, c3], dim=1).reshape(-1)[off:off + n]


def _largest(key, k):
    """Ascending positions of the k largest entries, equal ones in the order of their positions."""
    T = torch.topk(key, k, sorted=True).values[-1]
    above = key > T
    level = torch.nonzero(key == T).reshape(-1)[:k - int(above.sum())]
    return torch.cat([torch.nonzero(above).reshape(-1), level]).sort().values


def _plane(bit):
    n = bit.numel()
    full = torch.zeros((n + 31) // 32 * 32, dtype=torch.int64, device=DEV)
    full[:n] = bit
    return (full.reshape(-1, 32) << torch.arange(32, device=DEV)).sum(1).to(torch.int32)


def _header(case, n, k=0, scale=0.0, levels=0, scale2=0.0):
    h = np.zeros(HEADER // 4, dtype=np.uint32)
    h[0], h[1], h[7] = MAGIC, B.ALGO_IDS[case["algo"]], levels
    h[2:4] = np.array([n], dtype=np.uint64).view(np.uint32)
    h[4:6] = np.array([k], dtype=np.uint64).view(np.uint32)
    h[6:7] = np.array([scale], dtype=np.float32).view(np.uint32)
    h[8:9] = np.array([scale2], dtype=np.float32).view(np.uint32)
    return torch.from_numpy(h.view(np.uint8)).to(DEV)


def _encode(case, x, gen):
    """What a peer sends of the group x, and what that decodes to in 64 bits: (payload, how to decode)."""
    algo, n = case["algo"], x.numel()
    body, head, value = [], {}, None
    if algo in ("efsign", "onebit", "signsgd", "signum"):
        up = x >= 0
        hi, lo = 1.0, -1.0
        if algo == "efsign":
            hi = float(np.float32(float(x.double().abs().mean())))
            lo = -hi
        elif algo == "onebit":
            hi = float(np.float32(float(x[up].double().mean()))) if bool(up.any()) else 0.0
            lo = float(np.float32(float(x[~up].double().mean()))) if not bool(up.all()) else 0.0
        body = [_plane(up)]
        head = dict(scale=hi, scale2=lo if algo == "onebit" else 0.0)
        value = torch.where(up, hi, lo).double()
    elif algo == "terngrad":
        top = float(x.abs().max())
        nz = torch.empty_like(x).uniform_(generator=gen) * top < x.abs()
        body = [_plane(nz), _plane(nz & (x < 0))]
        head = dict(scale=top)
        value = nz.double() * torch.sign(x).double() * top
    elif algo == "qsgd":
        s = 2 ** (case["bits"] - 1) - 1
        norm = float(np.float32(math.sqrt(float(x.double().square().sum()))))
        a = x.abs().double() * (s / norm if norm else 0.0)
        level = torch.floor(a + torch.empty_like(x).uniform_(generator=gen)).clamp_(max=s)
        code = (torch.sign(x) * level).to(torch.int8)
        body = [torch.nn.functional.pad(code, (0, -n % 4))]
        head = dict(scale=norm, levels=s)
        value = code.double() * (norm / s)
    elif algo == "fp16":
        half = x.half()
        body = [torch.nn.functional.pad(half, (0, n % 2))]
        value = half.double()
    else:
        k, room = _kept(case, n), _room(case, n)
        key = torch.empty_like(x).uniform_(generator=gen) if algo == "randk" else x.abs()
        at = _largest(key, k)
        idx = torch.nn.functional.pad(at, (0, room - k)).to(torch.int32)
        val = torch.nn.functional.pad(x[at], (0, room - k))
        edges = torch.arange((n + TILE - 1) // TILE + 1, device=DEV) * TILE
        body = [idx, val, torch.searchsorted(at, edges).to(torch.int32)]
        head = dict(k=k, levels=room if case["sample"] else 0)
        value = torch.zeros(n, dtype=torch.float64, device=DEV)
        value[at] = x[at].double()
    return torch.cat([_header(case, n, **head)] + [b.contiguous().view(torch.uint8) for b in body]), value


# ---- what a program has in hand ------------------------------------------------------------------------------------
def _places(sizes, grain):
    """Offsets of buffers of these sizes, each on a multiple of `grain`, and the size of the whole."""
    at, off = [], 0
    for s in sizes:
        at.append(off)
        off += (s + grain - 1) // grain * grain
    return at, off


def prepare(case, seed):
    numel, bounds, sizes = _sizes(case)
    y, W = case["groups"], case["workers"]
    ctx = B.Context(case["algo"], numel, bounds, use_ef=case["ef"], ratio_ppm=case["ppm"], qsgd_bits=case["bits"], seed=SEED,
                    dgc_sample_ppm=case["sample"])
    s = {"ctx": ctx, "case": case, "y": y, "W": W, "bounds": bounds, "it": 0, "alpha": 1.0 / W}
    sent = [ctx.payload_bytes(j) for j in range(y)]
    at, whole = _places(sent, PLACE)
    # the payloads of all ranks as an allgather leaves them, this rank's first
    s["wire"] = torch.zeros(W, whole, dtype=torch.uint8, device=DEV)
    s["payloads"] = [[s["wire"][w, at[j]:at[j] + sent[j]] for j in range(y)] for w in range(W)]
    firsts = [sum(sizes[:j]) for j in range(y)]
    first_peer = {"decompress": 0, "step": 1, "compress": W}[case["direction"]]      # whose payloads are here before the pass
    for w in range(first_peer, W):
        x, gen = _gradient(case, seed, w, 0)
        for j in range(y):
            s["payloads"][w][j].copy_(_encode(case, x[firsts[j]:firsts[j] + sizes[j]], gen)[0])
    s["wire_ptrs"] = B.ptr_array([s["payloads"][w][j] for w in range(W) for j in range(y)])
    s["group_ptrs"] = [B.ptr_array([s["payloads"][w][j] for w in range(W)]) for j in range(y)]
    if case["direction"] != "decompress":
        s["grads"] = []
        for it in range(GRADIENTS):
            x, _ = _gradient(case, seed, 0, it)
            s["grads"].append([t.clone() for t in torch.split(x, numel)])          # every tensor an allocation of its own
        s["grad_ptrs"] = [B.ptr_array(g) for g in s["grads"]]
        s["group_grads"] = [[B.ptr_array(g[bounds[j]:bounds[j + 1]]) for j in range(y)] for g in s["grads"]]
        s["states"] = None
        if case["algo"] not in STATELESS and case["ef"]:
            held = [ctx.state_bytes(j) for j in range(y)]
            at, whole = _places(held, PLACE)
            s["memory"] = torch.zeros(whole, dtype=torch.uint8, device=DEV)
            s["states"] = [s["memory"][at[j]:at[j] + held[j]] for j in range(y)]
            s["state_ptrs"] = B.ptr_array(s["states"])
        s["own_ptrs"] = B.ptr_array(s["payloads"][0])
    if case["direction"] != "compress":
        at, whole = _places([4 * n for n in numel], PLACE)
        s["sum"] = torch.zeros(whole // 4, dtype=torch.float32, device=DEV)
        outs = [s["sum"][at[t] // 4:at[t] // 4 + numel[t]] for t in range(len(numel))]
        s["out_ptrs"] = B.ptr_array(outs)
        s["group_outs"] = [B.ptr_array(outs[bounds[j]:bounds[j + 1]]) for j in range(y)]
    return s


def run(s):
    case, ctx, it = s["case"], s["ctx"], s["it"]
    out = {}
    if case["direction"] != "decompress":
        g = it % GRADIENTS
        if case["calls"] == "groups":
            ctx.mc_compress_groups(0, it, s["grad_ptrs"][g], s["state_ptrs"] if s["states"] else None, s["own_ptrs"])
        else:
            for j in range(s["y"]):
                ctx.mc_compress(j, 0, it, s["group_grads"][g][j], s["states"][j] if s["states"] else None, s["payloads"][0][j])
        out["payload"] = s["wire"][0].view(torch.int32)
        if s["states"]:
            # one view per group behind its header; of many groups the whole buffer
            out["state"] = [t[HEADER:].view(torch.float32) for t in s["states"]] if s["y"] <= 16 else s["memory"].view(torch.int32)
    if case["direction"] != "compress":
        if case["calls"] == "groups":
            ctx.mc_decompress_sum_groups(s["wire_ptrs"], s["W"], s["alpha"], s["out_ptrs"])
        else:
            for j in range(s["y"]):
                ctx.mc_decompress_sum(j, s["group_ptrs"][j], s["alpha"], s["group_outs"][j])
        out["sum"] = s["sum"]
    s["it"] = it + 1
    return out


# ---- the same in 64 bits -------------------------------------------------------------------------------------------
def _own(case, x, first):
    """What this rank's first pass sends of the group x decodes to, in 64 bits."""
    algo, n, x = case["algo"], x.numel(), x.double()
    if algo in ("efsign", "signsgd", "signum", "onebit"):
        up = x >= 0
        hi = x.abs().mean() if algo == "efsign" else x[up].mean() if algo == "onebit" and bool(up.any()) else torch.tensor(1.0 if algo != "onebit" else 0.0, device=DEV)
        lo = x[~up].mean() if algo == "onebit" and not bool(up.all()) else -hi
        return torch.where(up, hi, lo).double()
    if algo == "fp16":
        return x.half().double()
    if algo in ("topk", "dgc"):
        if case["sample"]:
            return None                       # which entries reach the sample's threshold is not a question of precision
        at = _largest(x.abs(), _kept(case, n))
    else:
        word = _philox(case, first, n, 0, 0)
        u = (word >> 8).double() * 2.0 ** -24
        if algo == "randk":
            at = _largest(word >> 1, _kept(case, n))
        elif algo == "terngrad":
            top = x.abs().max()
            return (u * top < x.abs()).double() * torch.sign(x) * top
        else:
            s = 2 ** (case["bits"] - 1) - 1
            norm = x.square().sum().sqrt()
            a = (x.abs() * (s / norm)).clamp(max=s)
            level = torch.floor(a) + (u < a - torch.floor(a)).double()
            return torch.sign(x) * level * (norm / s)
    value = torch.zeros(n, dtype=torch.float64, device=DEV)
    value[at] = x[at]
    return value


def exact(case, seed):
    numel, bounds, sizes = _sizes(case)
    y, W, algo = case["groups"], case["workers"], case["algo"]
    firsts = [sum(sizes[:j]) for j in range(y)]
    out = {}
    if case["direction"] == "compress" and (algo in STATELESS or not case["ef"] or y > 16):
        return None                           # nothing but codes
    mine, _ = _gradient(case, seed, 0, 0)
    if case["direction"] != "decompress":
        out["payload"] = None
        if algo not in STATELESS and case["ef"]:
            out["state"] = []
            for j in range(y):
                x = mine[firsts[j]:firsts[j] + sizes[j]].double()
                if algo in ("topk", "dgc"):   # sent entries above the smallest one sent stay for the next pass to drop, those equal to it do not
                    at = _largest(x.abs(), _kept(case, sizes[j]))
                    least = x[at].abs().min()
                    x = x.clone()
                    x[at[x[at].abs() == least]] = 0.0
                if algo == "signum":
                    m = x * (1.0 - float(np.float32(0.9)))
                elif algo == "dgc":           # velocity, a gap up to a line of 32, momentum
                    m = torch.cat([x, torch.zeros(-sizes[j] % 32, dtype=torch.float64, device=DEV), x])
                elif algo == "fp16":
                    m = x - x.half().double()
                else:
                    m = x
                if algo == "randk" or (algo == "dgc" and case["sample"]):
                    m = None                  # what was sent, a matter of the random stream, is zero already
                out["state"].append(m)
            if y > 16:
                out["state"] = None
    if case["direction"] != "compress":
        total = [torch.zeros(n, dtype=torch.float64, device=DEV) for n in sizes]
        for w in range(W):
            x, gen = (mine, None) if w == 0 and case["direction"] == "step" else _gradient(case, seed, w, 0)
            for j in range(y):
                part = x[firsts[j]:firsts[j] + sizes[j]]
                if w == 0 and case["direction"] == "step":
                    # momentum: the sign of (1 - beta) g is that of g
                    d = _own(case, part, firsts[j])
                else:
                    d = _encode(case, part, gen)[1]
                if d is None:
                    total = None
                    break
                total[j] += d
            if total is None:
                break
        if total is None:
            out["sum"] = None
        else:
            flat = torch.cat(total)
            flat = torch.sign(flat) / W if algo in ("signsgd", "signum") else flat / W
            at, whole = _places([4 * n for n in numel], PLACE)
            out["sum"] = torch.zeros(whole // 4, dtype=torch.float64, device=DEV)
            off = 0
            for t, n in enumerate(numel):
                out["sum"][at[t] // 4:at[t] // 4 + n] = flat[off:off + n]
                off += n
    if out.get("sum") is None and not any(m is not None for m in out.get("state") or []):
        return None
    return out

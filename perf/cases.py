"""The layer calls a user of this package makes, as measurable cases.

Every case is one pass through `layer.py`, the package's public interface:

  linear   ExpandedLayer.forward on a prepared layer (per-batch or static activation grid), or
           forward_fused where the case asks for it and the library says it pays
  chain    ConvChain.forward: un-lowered convolutions with codes between the layers
  prepare  ExpandedLayer.prepare_weights: channel selection, halving and quantization of weights
  act_ocs  ExpandedLayer.forward_act_ocs: the channels chosen on the batch itself

Shapes come from the package's five workloads (workloads.py: a small fully connected layer, a 3x3
convolution at 14 x 14, the 1x1 convolutions, the LSTM gates, the 53 convolutions of a ResNet-50-shaped
network); draws spread over the ranges these span.  Values follow the same pictures: post-ReLU
half-normal activations, fully connected inputs with heavy-tailed outliers, [x ; tanh h] for the LSTM;
bell-shaped weights, some with outliers.  Everything is made on the device from the seed.
"""
import math

import numpy as np
import torch

from paper_1901_09504_amd.layer import ConvChain, ExpandedLayer

# ---- the cases -------------------------------------------------------------------------------


def _linear(name, M, C, g, N, r, bits_w, grid, fused=False, bits_x=8, clip_w=1.0, w="he", x="half"):
    return dict(name=name, kind="linear", M=M, C=C, g=g, N=N, r=r, bits_w=bits_w, bits_x=bits_x, grid=grid,
                fused=fused, clip_w=clip_w, w=w, x=x)


def listed():
    return [
        # the smallest workload: one fully connected layer on a batch of 64, grid taken from the batch
        _linear("fc_256_256_b64", 64, 256, 1, 256, 0.05, 8, "batch", w="outliers", x="outliers"),
        # one time step of the LSTM language model at batch 20: what generation runs, step after step
        _linear("lstm_step_b20", 20, 3000, 1, 6000, 0.05, 5, "static", w="tails", x="lstm"),
        # the same gates over the 20 x 35 positions of a training-length window, grid from the batch
        _linear("lstm_gates_b20x35", 700, 3000, 1, 6000, 0.05, 5, "batch", w="tails", x="lstm"),
        # 3x3 convolution at 14 x 14, batch 64, lowered, grid from the batch
        _linear("conv3x3_256_b64", 12544, 256, 9, 256, 0.02, 8, "batch", w="laplace"),
        # 1x1 convolution of a late stage at batch 128, profiled grid
        _linear("conv1x1_1024_256_b128", 25088, 1024, 1, 256, 0.05, 6, "static", w="outliers"),
        # the network's layer with the most arithmetic per byte (512 -> 512 3x3, batch 256)
        _linear("conv3x3_512_b256", 12544, 512, 9, 512, 0.05, 4, "static", clip_w=0.9),
        # the network's largest lowered activation (64 -> 64 3x3, batch 256) as the one-launch layer
        _linear("conv3x3_64_b256", 802816, 64, 9, 64, 0.05, 4, "static", fused=True, clip_w=0.9),
        # few inputs, many outputs (64 -> 256 1x1, batch 256): the output is most of the traffic
        _linear("conv1x1_64_256_b256", 802816, 64, 1, 256, 0.05, 4, "static", clip_w=0.9),
        # the 7x7 stem at batch 32: rows of 147 values, unaligned, grid from the batch
        _linear("stem_7x7_b32", 401408, 3, 49, 64, 0.05, 4, "batch"),
        # a stage-1 bottleneck at batch 32 given un-lowered, codes between its three layers
        dict(name="bottleneck_chain_b32", kind="chain", B=32, H=56, C=256, specs="64/1,64/3,256/1", r=0.05, bits_w=4),
        # off-line: the LSTM gates' weights (150 splits of 3000 channels)
        dict(name="prepare_lstm_gates", kind="prepare", N=6000, C=3000, g=1, r=0.05, bits_w=5, clip_w=1.0, qa=False,
             w="tails"),
        # activation splitting with the channels chosen on each batch (1x1, 7 x 7, batch 128)
        dict(name="act_ocs_2048_512_b128", kind="act_ocs", M=6272, C=2048, g=1, N=512, r=0.05, bits_w=6, x="half",
             w="outliers"),
    ]


# the largest listed case's work, which no drawn case exceeds
MOST_BYTES, MOST_FLOPS = 2.0e9, 6.0e10


def draw(rng):
    """One more case: sizes spread over the workloads' ranges by their logarithm, odd ones among them."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["linear"] * 8 + ["chain"] * 2 + ["prepare", "prepare", "act_ocs"])
        r = rng.choice([0.01, 0.02, 0.05, 0.1])
        bits_w = rng.choice([4, 5, 6, 8])
        if kind == "chain":
            H = rng.choice([7, 14, 28, 56, size(7, 56)])
            width = rng.choice([64, 128, 256, 512, size(32, 512)])
            specs = rng.choice([f"{width}/1,{width}/3,{4 * width}/1", f"{width}/3", f"{width}/3,{width}/3"])
            case = dict(kind=kind, B=size(1, 128), H=H, C=rng.choice([64, 256, 512, size(32, 1024)]), specs=specs, r=r,
                        bits_w=bits_w)
        else:
            g = rng.choice([1, 1, 9])
            C = rng.choice([64, 256, 512, size(32, 3000 if g == 1 else 512), size(32, 3000 if g == 1 else 512)])
            N = rng.choice([64, 256, 1024, size(32, 6000 if g == 1 else 512), size(32, 6000 if g == 1 else 512)])
            w = rng.choice(["he", "outliers", "laplace", "tails"])
            if kind == "prepare":
                case = dict(kind=kind, N=N, C=C, g=g, r=r, bits_w=bits_w, clip_w=rng.choice([1.0, 0.9, 0.8]),
                            qa=rng.random() < 0.3, w=w)
            elif kind == "act_ocs":
                case = dict(kind=kind, M=size(16, 50000), C=C, g=g, N=N, r=r, bits_w=bits_w, x="half", w=w)
            else:
                if rng.random() < 0.15:
                    C, g = 3, 49
                    N = 64
                grid = rng.choice(["batch", "static"])
                case = _linear(None, size(1, 800000), C, g, N, r, bits_w, grid, grid == "static" and rng.random() < 0.5,
                               clip_w=rng.choice([1.0, 0.9, 0.8]), w=w, x=rng.choice(["half", "outliers"]))
                del case["name"]
        c = work(case)
        if c["bytes"] <= MOST_BYTES and c["flops"] <= MOST_FLOPS:
            return case


# ---- inputs ----------------------------------------------------------------------------------


def _specs(case):
    return [(int(n), int(k), 1, int(k) // 2) for n, k in (p.split("/") for p in case["specs"].split(","))]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(190109504 + 7919 * int(seed))


def _weights(kind, N, C, g, gen):
    def normal():
        return torch.randn((N, C * g), device="cuda", generator=gen)

    def uniform():
        return torch.rand((N, C * g), device="cuda", generator=gen)

    if kind == "he":
        return normal().mul_(math.sqrt(2.0 / (C * g)))
    if kind == "laplace":
        u = uniform().sub_(0.5)
        return (-0.02) * u.sign() * (1 - 2 * u.abs()).clamp_min_(1e-7).log_()
    if kind == "outliers":                               # N(0, 0.02), one in a thousand ten times larger
        w = normal().mul_(0.02)
        return torch.where(uniform() < 0.001, w * 10, w)
    w = uniform().sub_(0.5).mul_(0.08)                   # U(-.04, .04), one row in a hundred heavy-tailed
    rows = max(1, N // 100)
    t = torch.randn((rows, C * g), device="cuda", generator=gen)
    chi = torch.randn((3, rows, C * g), device="cuda", generator=gen).square_().mean(0).sqrt_()
    w[torch.randperm(N, device="cuda", generator=gen)[:rows]] = 0.04 * t / chi
    return w


def _acts(kind, M, K, gen):
    x = torch.randn((M, K), device="cuda", generator=gen)
    if kind == "half":
        return x.abs_()
    if kind == "lstm":
        x[:, K // 2:] = x[:, K // 2:].tanh()
        return x
    pick = torch.rand((M, K), device="cuda", generator=gen) < 0.01   # one in a hundred heavy-tailed
    return torch.where(pick, x * 6, x)


def _inputs(case, seed):
    gen = _gen(seed)
    if case["kind"] == "chain":
        C, ws = case["C"], []
        for n, k, _, _ in _specs(case):
            ws.append(_weights("he", n, C, k * k, gen))
            C = n
        A = _acts("half", case["B"] * case["H"] * case["H"], case["C"], gen).view(case["B"], case["H"], case["H"], -1)
        # profiled input ranges: half-normal inputs first; he-scaled layers keep the standard
        # deviation of their outputs near sqrt(2)
        return A, ws, [4.5] + [6.0] * (len(ws) - 1)
    W = _weights(case["w"], case["N"], case["C"], case["g"], gen)
    if case["kind"] == "prepare":
        return (W,)
    return W, _acts(case["x"], case["M"], case["C"] * case["g"], gen)


# a profiled grid's range: what clips the outermost values of either distribution a little
_STATIC = 4.0


def _dev(v):
    return torch.tensor([v], dtype=torch.float32, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "chain":
        A, ws, thr = _inputs(case, seed)
        chain = ConvChain(case["C"], _specs(case), case["r"], case["bits_w"], 8)
        chain.prepare_weights(ws)
        return dict(kind=kind, chain=chain, A=A, thr=[_dev(t) for t in thr])
    L = ExpandedLayer(case["N"], case["C"], case["g"], case["r"], case["bits_w"], case.get("bits_x", 8),
                      clip_ratio_w=case.get("clip_w", 1.0), max_rows=case.get("M"))
    if kind == "prepare":
        return dict(kind=kind, L=L, W=_inputs(case, seed)[0], qa=case["qa"])
    W, X = _inputs(case, seed)
    if kind == "act_ocs":
        return dict(kind=kind, L=L, W=W, X=X)
    L.prepare_weights(W)
    thr = _dev(_STATIC) if case["grid"] == "static" else None
    return dict(kind="fused" if case["fused"] and thr is not None and L.fused_pays(X) else kind, L=L, X=X, thr=thr)


def run(state):
    kind = state["kind"]
    if kind == "chain":
        return state["chain"].forward(state["A"], state["thr"])
    L = state["L"]
    if kind == "linear":
        return L.forward(state["X"], state["thr"])
    if kind == "fused":
        return L.forward_fused(state["X"], state["thr"])
    if kind == "act_ocs":
        Y = L.forward_act_ocs(state["W"], state["X"])
        return [Y, L.chan_src, L.chan_depth, L.split_src[:L.s]]
    L.prepare_weights(state["W"], qa=state["qa"])
    return [L.Wq, L.scale_w, L.chan_src, L.chan_depth, L.split_src[:L.s]]


# ---- what a pass cannot do without -------------------------------------------------------------


def _splits(case, C):
    return math.ceil(case["r"] * C)


def work(case):
    if case["kind"] == "chain":
        P = case["B"] * case["H"] * case["H"]
        C, specs = case["C"], _specs(case)
        nbytes, flops = 4 * P * C + 4 * P * specs[-1][0], 0
        for n, k, _, _ in specs:
            Ke = (C + _splits(case, C)) * k * k
            nbytes += n * Ke
            flops += 2 * P * n * Ke
            C = n
        return dict(bytes=nbytes, flops=flops)
    C, g, N = case["C"], case["g"], case["N"]
    K, Ke = C * g, (C + _splits(case, C)) * g
    if case["kind"] == "prepare":
        return dict(bytes=4 * N * K + N * Ke, flops=2 * N * Ke)
    M = case["M"]
    return dict(bytes=4 * M * K + N * Ke + 4 * M * N, flops=2 * M * N * Ke)


def tolerance(case):
    # Codes, lists and integer sums leave no room; the float output is the exact sum times the two
    # steps, three roundings (int to float, step product, final multiply) and the two of the steps
    # themselves, each at most 2^-24.
    if case["kind"] == "prepare":
        return "exact"
    return dict(rel=4e-7, max=6e-7, differ=0.0)


# ---- the same in plain torch, sums and scale factors in 64 bits ----------------------------------
# The codes are whole numbers decided by the method's stated arithmetic (one 32-bit division, one
# 32-bit multiply, round half to even), so they are decided in 32 bits here as well.


def _codes(x, T, bits, floor=False):
    qmax = np.float32(2 ** (bits - 1) - 1)
    inv = float(min(qmax / np.float32(T), np.finfo(np.float32).max)) if T > 0 else 0.0
    p = (x * inv).clamp_(-float(qmax), float(qmax))
    return (p + 0.5).floor_() if floor else p.round_()


def _select(T, C, g, s):
    """The greedy choice on the channel maxima: split list, sources, depths, largest value left."""
    m = T.abs().amax(0).view(C, g).amax(1).cpu().numpy().astype(np.float32)
    vals = np.full(C + s, -1, np.float32)
    vals[:C] = m
    src, dep, picks = np.arange(C + s), np.zeros(C + s, np.int64), []
    for i in range(s):
        j = int(np.argmax(vals))
        vals[j] *= np.float32(0.5)
        dep[j] += 1
        vals[C + i], src[C + i], dep[C + i] = vals[j], src[j], dep[j]
        picks.append(j)
    return picks, src, dep, np.float32(vals.max())


def _expand(x, src, g):
    cols = (torch.as_tensor(src)[:, None] * g + torch.arange(g)[None, :]).reshape(-1).to(x.device)
    return x[:, cols]


def _lists(src, dep, picks):
    return [torch.tensor(np.asarray(v, np.int32)) for v in (src, dep, picks)]


def _split_weights(W, C, g, s, bits, clip, qa=False):
    picks, src, dep, top = _select(W, C, g, s)
    T = np.float32(clip) * top
    qmax = np.float32(2 ** (bits - 1) - 1)
    if qa:
        half = float(T / qmax * np.float32(0.5))
        parts = list(W.view(-1, C, g).unbind(1))
        for j in picks:
            v = parts[j]
            parts[j] = (v - half) * 0.5
            parts.append((v + half) * 0.5)
        Wx = torch.cat(parts, 1)
    else:
        Wx = _expand(W, src, g)
        d = torch.as_tensor(np.repeat(dep, g)).to(W.device)
        for _ in range(int(dep.max(initial=0))):
            Wx = torch.where(d > 0, Wx * 0.5, Wx)
            d = d - 1
    return _codes(Wx, T, bits, floor=qa), T, np.float32(T / qmax), src, dep, picks


def _product(xq_of, M, wq, rows=32768):
    """Sums of code products, 64 bits, rows of the left side in blocks."""
    wt = wq.double().t().contiguous()
    return torch.cat([xq_of(i, min(i + rows, M)).double() @ wt for i in range(0, M, rows)])


def _step(T, bits):
    return float(T) / (2 ** (bits - 1) - 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "chain":
        return _exact_chain(case, seed)
    C, g, bw, bx = case["C"], case["g"], case["bits_w"], case.get("bits_x", 8)
    s = _splits(case, C)
    if kind == "prepare":
        (W,) = _inputs(case, seed)
        wq, T, step, src, dep, picks = _split_weights(W, C, g, s, bw, case["clip_w"], case["qa"])
        Ke = wq.shape[1]           # code rows end in zeros: up to 16 bytes when short, else up to 128
        pitch = -(-Ke // 16) * 16 if -(-Ke // 64) * 64 <= 320 else -(-Ke // 128) * 128
        q = torch.zeros((case["N"], pitch), dtype=torch.int8)
        q[:, :Ke] = wq.to(torch.int8).cpu()
        return [q, torch.tensor([T, step]), *_lists(src, dep, picks)]
    W, X = _inputs(case, seed)
    if kind == "act_ocs":
        picks, src, dep, T = _select(X, C, g, s)
        Tw = W.abs().max().item()
        wq = _expand(_codes(W, np.float32(Tw), bw), src, g)
        scale = torch.as_tensor(np.repeat(0.5 ** dep.astype(np.float64), g)).float().cuda()

        def block(a, b):
            return _codes(_expand(X[a:b], src, g) * scale, T, bx)

        Y = _product(block, case["M"], wq) * (_step(T, bx) * _step(Tw, bw))
        return [Y, *_lists(src, dep, picks)]
    wq, Tw, _, src, _, _ = _split_weights(W, C, g, s, bw, case["clip_w"])
    T = np.float32(_STATIC) if case["grid"] == "static" else np.float32(X.abs().max().item())
    # (a copy of a column meets the sum of its channel's weight codes: the un-expanded product)
    folded = torch.zeros((case["N"], C, g), device="cuda", dtype=torch.float64)
    folded.index_add_(1, torch.as_tensor(src).cuda(), wq.double().view(case["N"], -1, g))
    Y = _product(lambda a, b: _codes(X[a:b].clone(), T, bx), case["M"], folded.view(case["N"], -1))
    return Y.mul_(_step(T, bx) * _step(Tw, bw))


def _exact_chain(case, seed):
    A, ws, thr = _inputs(case, seed)
    B, H, C = case["B"], case["H"], case["C"]
    x = _codes(A.view(-1, C).clone(), np.float32(thr[0]), 8)
    for i, ((n, k, _, pad), W) in enumerate(zip(_specs(case), ws)):
        g = k * k
        s = _splits(case, C)
        wq, Tw, step_w, src, _, _ = _split_weights(W, C, g, s, case["bits_w"], 1.0)
        folded = torch.zeros((n, C, g), device="cuda", dtype=torch.float64)
        folded.index_add_(1, torch.as_tensor(src).cuda(), wq.double().view(n, -1, g))
        img = x.view(B, H, H, C).permute(0, 3, 1, 2)

        def block(a, b, img=img, k=k, pad=pad):
            cols = torch.nn.functional.unfold(img[a // (H * H):b // (H * H)].double(), k, padding=pad)
            return cols.transpose(1, 2).reshape(b - a, -1)

        per = max(1, 32768 // (H * H)) * H * H
        acc = _product(block, B * H * H, folded.view(n, -1), per)
        if i + 1 == len(ws):
            return acc.mul_(_step(thr[i], 8) * _step(Tw, case["bits_w"]))
        y = acc.float() * float(np.float32(np.float32(thr[i]) / np.float32(127)) * step_w)
        x = _codes(y.clamp_min_(0), np.float32(thr[i + 1]), 8)
        C = n

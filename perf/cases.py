"""The work that programs built on this library have it do, as cases that can be timed and compared.

A case is a dict of plain values; its "kind" says which part of a program it stands for:

  linear       one quantized linear layer called by itself
  decode       one decode step of `layers` transformer layers (q/k/v, o, gate/up, down) for `M` tokens that are
               generated together, captured once into a graph and replayed, as a serving loop does it
  layer        the same four groups of projections for `M` tokens of prompts, called one after the other; the width
               of the activation grid, its zero point and TRIP factors are options
  attn_probs   softmax probabilities x V with log2-quantized probabilities, token pruning on the importance it
               returns, and the two projections that follow on the tokens that are left
  attn_qk      attention from int8 Q, K and V in one call, with the importance of every token
  stack        `blocks` whole transformer blocks with the cascade of token pruning

Sizes are those of the LLaMA-7B and -13B shapes and of the 768-wide layer that the tests and the benchmark of this
repository use; draw() takes others of the same ranges.  Inputs follow paper_2312_05693_amd/synth.py: unit normals with
whole outlier channels times 20, normal weights rounded to four bits per output channel, a start-token stripe on the
attention map."""
from __future__ import annotations

import math

import torch

from paper_2312_05693_amd import binding as agq

DEVICE = "cuda"
ROPE_BASE = 10000.0
RMS_EPS = 1e-5
TRIP_REFINEMENTS = 4


def listed():
    return [
        # the smallest call: one narrow layer for a prompt of 128 tokens; launches and the host's share are what counts
        dict(name="linear_768_128rows", kind="linear", M=128, K=768, N=768, bits=8, zp=0, codes=False),
        # generation for one user: every weight is read once per step
        dict(name="decode_7b_1row", kind="decode", layers=4, M=1, d=4096, F=11008, bits=8),
        # generation for a few users at a time
        dict(name="decode_7b_4rows", kind="decode", layers=4, M=4, d=4096, F=11008, bits=8),
        # generation for the largest batch that the weight-streaming kernels take in one go
        dict(name="decode_13b_16rows", kind="decode", layers=4, M=16, d=5120, F=13824, bits=8),
        # a short prompt, or a large generation batch: between streaming weights and being bound by the matrix cores
        dict(name="layer_7b_100rows", kind="layer", M=100, d=4096, F=11008, bits=8, zp=0, trip=False),
        # a prompt of ordinary length on the unsigned 4-bit grid
        dict(name="layer_13b_333rows_w4a4_zp", kind="layer", M=333, d=5120, F=13824, bits=4, zp=8, trip=False),
        # a full-length prompt: the matrix cores
        dict(name="layer_7b_2048rows", kind="layer", M=2048, d=4096, F=11008, bits=8, zp=0, trip=False),
        # a long prompt whose activations carry TRIP factors for their outlier channels
        dict(name="layer_7b_1000rows_trip", kind="layer", M=1000, d=4096, F=11008, bits=8, zp=0, trip=True),
        # attention on a probability map that the program already has, pruning to half of the tokens, two projections
        dict(name="attn_probs_13b_2048", kind="attn_probs", H=40, S=2048, D=128, causal=True, qmax=15, keep=1024, F=13824),
        # attention from the codes of Q and K at full length
        dict(name="attn_qk_13b_2048", kind="attn_qk", H=40, S=2048, D=128, causal=True, qmax=15),
        # one whole block at full length, half of the tokens pruned after its attention
        dict(name="block_13b_2048_prune", kind="stack", blocks=1, S=2048, H=40, D=128, F=13824, qmax=15, bits_o=4, keep=0.5),
        # a short ragged prompt through several blocks with the pruning cascade
        dict(name="stack_7b_300", kind="stack", blocks=4, S=300, H=32, D=128, F=11008, qmax=15, bits_o=4, keep=0.5),
    ]


def _spread(rng, lo, hi):
    """An integer of lo..hi, spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_once(rng):
    kind = rng.choice(["linear", "linear", "decode", "decode", "layer", "layer", "layer", "attn_probs", "attn_qk", "stack", "stack"])
    d = 128 * _spread(rng, 6, 40)                       # 768 .. 5120
    F = 128 * int(round(d * rng.uniform(2.5, 4.0) / 128))
    D = rng.choice([64, 128])
    if kind == "linear":
        return dict(kind=kind, M=_spread(rng, 1, 2048), K=128 * _spread(rng, 6, 108), N=_spread(rng, 500, 13824), bits=rng.choice([8, 8, 4]),
                    zp=rng.choice([0, 0, 5]), codes=rng.choice([False, False, True]))
    if kind == "decode":
        return dict(kind=kind, layers=rng.randint(3, 6), M=_spread(rng, 1, 16), d=max(d, 1536), F=max(F, 4096), bits=rng.choice([8, 8, 4]))
    if kind == "layer":
        trip = rng.random() < 0.25
        return dict(kind=kind, M=_spread(rng, 17, 2048), d=d, F=F, bits=rng.choice([8, 8, 4]), zp=0 if trip else rng.choice([0, 0, 8]), trip=trip)
    if kind == "attn_probs":
        S = 8 * _spread(rng, 32, 256)                   # 256 .. 2048
        return dict(kind=kind, H=rng.randint(8, 40), S=S, D=D, causal=rng.random() < 0.8, qmax=rng.choice([15, 15, 7]),
                    keep=max(1, int(S * rng.uniform(0.3, 0.9))), F=F)
    if kind == "attn_qk":
        return dict(kind=kind, H=rng.randint(8, 40), S=128 * _spread(rng, 2, 16), D=D, causal=rng.random() < 0.8, qmax=rng.choice([15, 15, 7]))
    blocks = rng.randint(1, 4)
    return dict(kind=kind, blocks=blocks, S=_spread(rng, 40, 2048 // blocks), H=max(6, d // 128) * (128 // D), D=D, F=F, qmax=rng.choice([15, 15, 7]),
                bits_o=rng.choice([4, 8]), keep=rng.choice([1.0, 0.5, 0.6]))


def draw(rng):
    """One more case of these ranges, no dearer than the largest listed one."""
    most = [work(c) for c in listed()]
    bytes_most, flops_most = max(w["bytes"] for w in most), max(w["flops"] for w in most)
    while True:
        case = _draw_once(rng)
        if case["kind"] in ("attn_probs", "stack") and (case["H"] * case["D"]) % 128:
            continue                                    # the projections behind the heads take multiples of 128
        w = work(case)
        if w["bytes"] <= bytes_most and w["flops"] <= flops_most:
            return case


# inputs ----------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _activation(g, M, K, outliers):
    """fp16 [M,K]: unit normals, `outliers` whole channels times 20."""
    x = torch.randn(M, K, generator=g, device=DEVICE)
    x[:, torch.randperm(K, generator=g, device=DEVICE)[:outliers]] *= 20.0
    return x.to(torch.float16)


def _weight(g, N, K, std=0.02):
    """4-bit weights by symmetric rounding per output channel: (int8 codes [N,K], fp16 scales [N])."""
    w = torch.randn(N, K, generator=g, device=DEVICE)
    w *= std
    scale = (w.abs().amax(dim=1) / 7.0).to(torch.float16)
    wq = (w / scale.float()[:, None]).round_().clamp_(-8, 7).to(torch.int8)
    return wq, scale


def _exponent(x, bits):
    return int(agq.calibrate_act_exp(x, bits).item())


def _outliers(K, M):
    """Four outlier channels where tokens are generated, 1 % of the channels where prompts are read."""
    return 4 if M <= 16 else -(-K // 100)


def _groups(d, F):
    """(K, widths of the projections that share one activation) of one layer: q/k/v, o, gate/up, down."""
    return [(d, (d, d, d)), (d, (d,)), (d, (F, F)), (F, (d,))]


def _workspace(M, N, K):
    return torch.empty(max(16, agq.gemm_workspace_bytes(M, N, K)), dtype=torch.uint8, device=DEVICE)


def _prepare_groups(g, case, M, d, F, bits, zp=0, trip=False):
    """The four groups of one layer: activations, packed weights, outputs and workspaces."""
    groups = []
    for i, (K, widths) in enumerate(_groups(d, F)):
        x = _activation(g, M, K, _outliers(K, M))
        e, extra, alpha = _exponent(x, bits), None, None
        if trip and i in (0, 2):                        # the inputs whose outlier channels get factors
            e -= TRIP_REFINEMENTS
            alpha = agq.trip_search(x, bits, e, TRIP_REFINEMENTS).cpu().numpy()
        projs = []
        for N in widths:
            wq, scale = _weight(g, N, K)
            if alpha is None:
                blob = agq.pack_w4(wq)
            else:
                blob, extra = agq.pack_w4_trip(wq, alpha)
            projs.append((blob, scale, N, torch.empty(M, N, dtype=torch.float16, device=DEVICE), None))
        total = sum(widths)
        if extra is None:
            workspace = _workspace(M, total, K)
        else:
            workspace = torch.empty(max(16, agq.lib().agq_gemm_trip_workspace_bytes(M, total, K, extra)), dtype=torch.uint8, device=DEVICE)
        groups.append(dict(x=x, e=e, K=K, projs=projs, bits=bits, zp=zp, extra=extra, workspace=workspace))
    return groups


def _run_groups(groups):
    out = []
    for s in groups:
        if s["extra"] is not None:
            out += agq.gemm_trip_multi(s["x"], s["bits"], s["e"], s["projs"], s["extra"], s["K"], workspace=s["workspace"])
        else:
            multi = agq.gemm_w4a8_multi if s["bits"] == 8 else agq.gemm_w4a4_multi
            out += multi(s["x"], s["e"], s["projs"], s["K"], workspace=s["workspace"], zp=s["zp"])
    return out


def _prepare_linear(g, case):
    M, K, N, bits, zp = (case[k] for k in ("M", "K", "N", "bits", "zp"))
    x = _activation(g, M, K, _outliers(K, M))
    e = _exponent(x, bits)
    wq, scale = _weight(g, N, K)
    if case["codes"]:
        x = agq.quantize_act(x, bits, e, zp)
    return dict(x=x, e=e, blob=agq.pack_w4(wq), scale=scale, y=torch.empty(M, N, dtype=torch.float16, device=DEVICE),
                workspace=_workspace(M, N, K))


def _prepare_decode(g, case):
    layers = [_prepare_groups(g, case, case["M"], case["d"], case["F"], case["bits"]) for _ in range(case["layers"])]
    groups = [s for layer in layers for s in layer]
    _run_groups(groups)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _run_groups(groups)
    return dict(groups=groups, graph=graph, out=[p[3] for s in groups for p in s["projs"]])


def _prepare_attn_probs(g, case):
    H, S, D = case["H"], case["S"], case["D"]
    p = torch.empty(H, S, S, dtype=torch.float16, device=DEVICE)
    above = torch.ones(S, S, dtype=torch.bool, device=DEVICE).triu_(1) if case["causal"] else None
    for h in range(H):
        q, k = torch.randn(S, D, generator=g, device=DEVICE), torch.randn(S, D, generator=g, device=DEVICE)
        logits = torch.mm(q, k.t().contiguous()) / math.sqrt(D)
        logits[:, 0] += 4.0 + 2.0 * torch.randn(S, generator=g, device=DEVICE)
        if above is not None:
            logits.masked_fill_(above, float("-inf"))
        p[h] = torch.softmax(logits, dim=1).to(torch.float16)
    v = torch.randn(H * S, D, generator=g, device=DEVICE).to(torch.float16)
    e_v = _exponent(v, 8)
    vq = agq.quantize_act(v, 8, e_v).view(H, S, D)
    d, F, keep = H * D, case["F"], case["keep"]
    o, _, _ = agq.log2_quant_softmax(p, vq, e_v, qmax=case["qmax"], causal=case["causal"])
    e_o = _exponent(o, 8)
    w_o, s_o = _weight(g, d, d)
    blob_o = agq.pack_w4(w_o)
    e_f = _exponent(agq.gemm_w4a8(o, e_o, blob_o, s_o, d, d), 8)
    w_f, s_f = _weight(g, F, d)
    return dict(p=p, vq=vq, e_v=e_v, d=d, F=F, e_o=e_o, e_f=e_f, blob_o=blob_o, s_o=s_o, blob_f=agq.pack_w4(w_f), s_f=s_f,
                y_o=torch.empty(keep, d, dtype=torch.float16, device=DEVICE), y_f=torch.empty(keep, F, dtype=torch.float16, device=DEVICE),
                ws_o=_workspace(keep, d, d), ws_f=_workspace(keep, F, d))


def _prepare_attn_qk(g, case):
    """int8 codes in steps of 1/32 with a direction shared by every query and the first key."""
    H, S, D = case["H"], case["S"], case["D"]
    q, k, v = (torch.randn(H, S, D, generator=g, device=DEVICE) for _ in range(3))
    u = torch.randn(H, 1, D, generator=g, device=DEVICE) / math.sqrt(D)
    q += u * (4.0 + torch.randn(H, S, 1, generator=g, device=DEVICE))
    k[:, :1] += 8.0 * u
    to8 = lambda t: (t * 32.0).round_().clamp_(-127, 127).to(torch.int8)  # noqa: E731
    return dict(q=to8(q), k=to8(k), v=to8(v))


def _keeps(case):
    """Tokens that each block keeps: every second block prunes (a block by itself does too), in equal ratios."""
    n, left, out = case["blocks"], case["S"], []
    pruning = [l for l in range(n) if l % 2 == 1 or n == 1]
    stages = agq.cascade_keep(case["S"], 1.0 - case["keep"], len(pruning)) if case["keep"] < 1.0 else [left] * len(pruning)
    for l in range(n):
        if l in pruning:
            left = stages[pruning.index(l)]
        out.append(int(left))
    return out


def _prepare_stack(g, case):
    S, H, D, F = case["S"], case["H"], case["D"], case["F"]
    d, keep = H * D, _keeps(case)
    x = _activation(g, S, d, max(1, d // 128))
    pos = torch.arange(S, dtype=torch.int32, device=DEVICE)
    angle = torch.arange(S, dtype=torch.float64)[:, None] * ROPE_BASE ** (-torch.arange(0, D, 2, dtype=torch.float64) / D)[None, :]
    cos, sin = angle.cos().float().to(DEVICE), angle.sin().float().to(DEVICE)
    shapes = dict(q=(d, d), k=(d, d), v=(d, d), o=(d, d), gate=(F, d), up=(F, d), down=(d, F))
    blocks, t, p = [], x, pos
    for l in range(case["blocks"]):
        weights = {n: (1.0 + 0.1 * torch.randn(d, generator=g, device=DEVICE)).to(torch.float16) for n in ("g_attn", "g_mlp")}
        for n, (N, K) in shapes.items():
            wq, weights["s_" + n] = _weight(g, N, K, 1.0 / math.sqrt(K))
            weights["w_" + n] = agq.pack_w4(wq)
        blk = agq.make_block(d, H, F, weights, qmax=case["qmax"], bits_attn_out=case["bits_o"], rms_eps=RMS_EPS)
        t, p, _, _ = agq.block_forward(blk, t, p, cos, sin, n_keep=keep[l], calibrate=True)   # static exponents
        blocks.append(blk)
    state = dict(blocks=blocks, keep=keep, x=x, pos=pos, cos=cos, sin=sin, workspace=None)
    if case["blocks"] == 1:
        state["workspace"] = torch.empty(agq.block_layout(blocks[0], S, keep[0]).total, dtype=torch.uint8, device=DEVICE)
    else:
        state["workspace"] = agq.stack_forward(blocks, keep, x, pos, cos, sin)[2]
    state["out"] = (torch.empty(keep[-1], d, dtype=torch.float16, device=DEVICE), torch.empty(keep[-1], dtype=torch.int32, device=DEVICE))
    return state


_PREPARE = dict(linear=_prepare_linear, decode=_prepare_decode, attn_probs=_prepare_attn_probs, attn_qk=_prepare_attn_qk,
                stack=_prepare_stack,
                layer=lambda g, c: dict(groups=_prepare_groups(g, c, c["M"], c["d"], c["F"], c["bits"], c["zp"], c["trip"])))


def prepare(case, seed):
    state = _PREPARE[case["kind"]](_generator(seed), case)
    state["case"] = case
    return state


# one pass --------------------------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        gemm = agq.gemm_w4a8 if case["bits"] == 8 else agq.gemm_w4a4
        return gemm(state["x"], state["e"], state["blob"], state["scale"], case["N"], case["K"],
                    x_kind=agq.AGQ_X_Q if case["codes"] else agq.AGQ_X_F16, y=state["y"], workspace=state["workspace"], zp=case["zp"])
    if kind == "decode":
        state["graph"].replay()
        return state["out"]
    if kind == "layer":
        return _run_groups(state["groups"])
    if kind == "attn_probs":
        o, _, score = agq.log2_quant_softmax(state["p"], state["vq"], state["e_v"], qmax=case["qmax"], causal=case["causal"])
        idx, kept = agq.prune_tokens(score, case["keep"], o)
        y_o = agq.gemm_w4a8(kept, state["e_o"], state["blob_o"], state["s_o"], state["d"], state["d"], y=state["y_o"], workspace=state["ws_o"])
        y_f = agq.gemm_w4a8(y_o, state["e_f"], state["blob_f"], state["s_f"], state["F"], state["d"], y=state["y_f"], workspace=state["ws_f"])
        return dict(o=o, score=score, idx=idx, y_o=y_o, y_f=y_f)
    if kind == "attn_qk":
        o, _, score = agq.qk_log2_softmax(state["q"], state["k"], state["v"], -5, -5, -5, qmax=case["qmax"], causal=case["causal"])
        return dict(o=o, score=score)
    if case["blocks"] == 1:
        x_out, pos_out, _, _ = agq.block_forward(state["blocks"][0], state["x"], state["pos"], state["cos"], state["sin"], n_keep=state["keep"][0],
                                                 workspace=state["workspace"], out=state["out"])
    else:
        x_out, pos_out, _ = agq.stack_forward(state["blocks"], state["keep"], state["x"], state["pos"], state["cos"], state["sin"],
                                              workspace=state["workspace"], out=state["out"])
    return dict(x=x_out, pos=pos_out)


# what a pass cannot do without -----------------------------------------------------------------------------------

def _gemm_work(M, K, N, x_bytes=2.0):
    return M * K * x_bytes + N * K / 2 + 2 * N + 2 * M * N, 2.0 * M * N * K


def _add(*parts):
    return sum(p[0] for p in parts), sum(p[1] for p in parts)


def _layer_work(M, d, F):
    parts = []
    for K, widths in _groups(d, F):
        b, f = _gemm_work(M, K, sum(widths))
        parts.append((b, f))
    return _add(*parts)


def _pairs(S, causal):
    return S * (S + 1) / 2 if causal else float(S * S)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _gemm_work(case["M"], case["K"], case["N"], (case["bits"] / 8 if case["codes"] else 2.0))
    elif kind == "decode":
        b, f = _layer_work(case["M"], case["d"], case["F"])
        b, f = b * case["layers"], f * case["layers"]
    elif kind == "layer":
        b, f = _layer_work(case["M"], case["d"], case["F"])
    elif kind == "attn_probs":
        H, S, D, keep = case["H"], case["S"], case["D"], case["keep"]
        d, pairs = H * D, _pairs(S, case["causal"])
        attn = (2 * H * pairs + H * S * D + 2 * S * d + 4 * S, 2.0 * H * pairs * D)
        prune = (2.0 * 2 * keep * d + 4 * keep, 0.0)
        b, f = _add(attn, prune, _gemm_work(keep, d, d), _gemm_work(keep, d, case["F"]))
    elif kind == "attn_qk":
        H, S, D = case["H"], case["S"], case["D"]
        b, f = 3.0 * H * S * D + 2 * S * H * D + 4 * S, 4.0 * H * _pairs(S, case["causal"]) * D
    else:
        d, F, parts, S = case["H"] * case["D"], case["F"], [], case["S"]
        parts.append((2.0 * S * d + 4 * S, 0.0))
        for keep in _keeps(case):
            weights = (4 * d * d + 3 * d * F) / 2 + 2 * (5 * d + 2 * F) + 4 * d
            flops = 2.0 * S * 3 * d * d + 4.0 * _pairs(S, True) * d + 2.0 * keep * (d * d + 3 * d * F)
            parts.append((weights, flops))
            S = keep
        parts.append((2.0 * S * d + 4 * S, 0.0))
        b, f = _add(*parts)
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """What another correct evaluation may differ by.  The products are exact integers and their dequantization is one
    product in fp32 rounded to fp16: against a float64 evaluation 3.6e-7 of the values were off, by one fp16 ulp
    (2-norm 1.6e-6).  Attention from codes evaluates -log2 p in fp32, and a code that lies on a rounding boundary
    (about one in 1e5) halves or doubles one weight: 2-norm 1.5e-4, largest difference 0.08 of the mean square root;
    the importance sums one code per head.  Through a block these differences mostly vanish in the next quantizer."""
    if case["kind"] == "attn_qk":
        return {"rel": 6e-4, "max": 0.3, "differ": 0.002}
    if case["kind"] == "stack":
        return {"rel": 5e-4, "max": 0.3, "differ": 0.002}
    return {"rel": 1e-5, "max": 2e-3}


# the same in 64 bits ---------------------------------------------------------------------------------------------

def _exponent64(x, bits):
    """The smallest e with max |x| <= (2^(bits-1) - 1) 2^e."""
    top, qmax, e = float(x.abs().max()), 2 ** (bits - 1) - 1, -64
    while top > qmax * 2.0 ** e:
        e += 1
    return e


def _linear64(x, e, bits, zp, wq, scale):
    """2^e scale[n] sum_k (q - zp) w with Eq.2's codes q of fp16 x."""
    lo, hi = (0, 2 ** bits - 1) if zp else (-2 ** (bits - 1), 2 ** (bits - 1) - 1)
    q = (x.double() * 2.0 ** -e).round_().add_(zp).clamp_(lo, hi).sub_(zp)
    return torch.mm(q, wq.double().t().contiguous()) * (scale.double() * 2.0 ** e)


def _exact_groups(g, M, d, F, bits, zp):
    out = []
    for K, widths in _groups(d, F):
        x = _activation(g, M, K, _outliers(K, M))
        e = _exponent64(x, bits)
        for N in widths:
            out.append(_linear64(x, e, bits, zp, *_weight(g, N, K)))
    return out


def _log2_weights(t, qmax, above):
    """2^(qmax - c) of Eq.3's codes c = clip(round(t)), t = -log2 p; 0 above the diagonal."""
    w = torch.exp2(qmax - t.round_().clamp_(0, qmax))
    return w if above is None else w.masked_fill_(above, 0.0)


def _exact_attn_probs(g, case):
    H, S, D, qmax = case["H"], case["S"], case["D"], case["qmax"]
    above = torch.ones(S, S, dtype=torch.bool, device=DEVICE).triu_(1) if case["causal"] else None
    weights, score = [], torch.zeros(S, dtype=torch.float64, device=DEVICE)
    for h in range(H):
        q, k = torch.randn(S, D, generator=g, device=DEVICE), torch.randn(S, D, generator=g, device=DEVICE)
        logits = torch.mm(q, k.t().contiguous()) / math.sqrt(D)
        logits[:, 0] += 4.0 + 2.0 * torch.randn(S, generator=g, device=DEVICE)
        if above is not None:
            logits.masked_fill_(above, float("-inf"))
        p = torch.softmax(logits, dim=1).to(torch.float16)
        score += p[:, 0].double() * 2.0 ** 24
        weights.append(_log2_weights(-torch.log2(p.double()), qmax, above).half())     # powers of two: exact
    v = torch.randn(H * S, D, generator=g, device=DEVICE).to(torch.float16)
    e_v = _exponent64(v, 8)
    vq = (v.double() * 2.0 ** -e_v).round_().clamp_(-128, 127).view(H, S, D)
    o = torch.cat([torch.mm(w.double(), vq[h]) for h, w in enumerate(weights)], dim=1) * 2.0 ** (e_v - qmax)
    d, F = H * D, case["F"]
    o16 = o.to(torch.float16)                          # the entry points hand fp16 tensors on
    w_o, s_o = _weight(g, d, d)
    e_o = _exponent64(o16, 8)
    all_o = _linear64(o16, e_o, 8, 0, w_o, s_o).to(torch.float16)
    idx = torch.sort(torch.sort(score, descending=True, stable=True)[1][:case["keep"]])[0]
    y_o = _linear64(o16[idx], e_o, 8, 0, w_o, s_o)
    y_f = _linear64(y_o.to(torch.float16), _exponent64(all_o, 8), 8, 0, *_weight(g, F, d))
    return dict(o=o, score=None, idx=None, y_o=y_o, y_f=y_f)


def _exact_attn_qk(g, case):
    state, H, S, D, qmax = _prepare_attn_qk(g, case), case["H"], case["S"], case["D"], case["qmax"]
    above = torch.ones(S, S, dtype=torch.bool, device=DEVICE).triu_(1) if case["causal"] else None
    parts = []
    for h in range(H):
        logits = torch.mm(state["q"][h].double(), state["k"][h].double().t().contiguous()) * (2.0 ** -10 / math.sqrt(D))
        if above is not None:
            logits.masked_fill_(above, float("-inf"))
        t = torch.log_softmax(logits, dim=1) / -math.log(2.0)
        parts.append(torch.mm(_log2_weights(t, qmax, above), state["v"][h].double()))
    return dict(o=torch.cat(parts, dim=1) * 2.0 ** (-5 - qmax), score=None)


def exact(case, seed):
    """run()'s floating outputs in 64 bits.  None where the way there has no such value: factors that a search picks, and
    blocks, in which a rounding to fp16 decides codes and the tokens that are kept."""
    g, kind = _generator(seed), case["kind"]
    if kind == "linear":
        x = _activation(g, case["M"], case["K"], _outliers(case["K"], case["M"]))
        return _linear64(x, _exponent64(x, case["bits"]), case["bits"], case["zp"], *_weight(g, case["N"], case["K"]))
    if kind == "decode":
        return [y for _ in range(case["layers"]) for y in _exact_groups(g, case["M"], case["d"], case["F"], case["bits"], 0)]
    if kind == "layer":
        return None if case["trip"] else _exact_groups(g, case["M"], case["d"], case["F"], case["bits"], case["zp"])
    if kind == "attn_probs":
        return _exact_attn_probs(g, case)
    return _exact_attn_qk(g, case) if kind == "attn_qk" else None

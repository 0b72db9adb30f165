"""The workloads that the library's speed is measured on.

Three kinds of case, each through the public entry points of ``paper_2502_11880_amd``:

* ``stack``  -- the linears of the given number of transformer layers in layer order: per layer the four activation
  groups (q/k/v share one input, then o, gate/up, down), one ``bitnet_mpgemm_fused`` call per group with the outputs
  [M, N] of every linear in buffers of its own.  Decode cases capture the calls once in a HIP graph and a pass is one
  replay, as a serving loop does it; they take enough layers that the packed weights (over 512 MB) come from HBM and
  not from the 256 MB last-level cache.  Prefill cases (tens of tokens per layer and up) make the calls directly.
* ``linear`` -- one linear layer called directly: fused, as quantiser + product, or with the no-allocation product.
* ``pack``   -- the offline direction: every fp32 weight of one layer ternarised and packed.

Outputs are all that the calls write: the fp32 products, int8 codes, scales and code sums; packed bytes and betas.
"""
import math

import torch

import paper_2502_11880_amd as B
from paper_2502_11880_amd import inputs

DEV = "cuda"
INT_CARD = {"c4g2": 4, "c5g2": 5, "c3g5": 3}
LOSSY = ("tl2_0", "tl1_0")
INT_BETA = 0.02                       # the caller's scale of integer weights (as in the benchmark)


def listed():
    return [
        # the smallest call: one linear layer, one token, called directly; latency and the host path
        dict(name="linear-1536x4096-i2s-m1", kind="linear", api="fused", layout="i2s", K=1536, N=4096, tokens=1),
        # single-user decode of the 3B-class model: odd hidden size (3200 = 12.5 blocks), short launches
        dict(name="decode-3b-i2s-m1", kind="stack", layout="i2s", hidden=3200, kv=3200, ffn=8640, tokens=1, layers=17,
             graph=True),
        # single-user decode of the 8B-class model in the smallest lossless layout
        dict(name="decode-8b-tl2-m1", kind="stack", layout="tl2", hidden=4096, kv=1024, ffn=14336, tokens=1, layers=12,
             graph=True),
        # single-user decode of the 100B-class model: the bandwidth-bound headline workload
        dict(name="decode-100b-i2s-m1", kind="stack", layout="i2s", hidden=12288, kv=12288, ffn=33024, tokens=1,
             layers=2, graph=True),
        # batched decode: eight concurrent users of the 8B-class model
        dict(name="decode-8b-i2s-m8", kind="stack", layout="i2s", hidden=4096, kv=1024, ffn=14336, tokens=8, layers=10,
             graph=True),
        # small-batch serving (between decode and prefill), an odd number of tokens, the pair-code layout
        dict(name="decode-8b-tl1-m45", kind="stack", layout="tl1", hidden=4096, kv=1024, ffn=14336, tokens=45,
             layers=10, graph=True),
        # a short prompt through one 8B-class layer
        dict(name="prefill-8b-i2s-m512", kind="stack", layout="i2s", hidden=4096, kv=1024, ffn=14336, tokens=512,
             layers=1, graph=False),
        # a long prompt through one 8B-class layer
        dict(name="prefill-8b-i2s-m2048", kind="stack", layout="i2s", hidden=4096, kv=1024, ffn=14336, tokens=2048,
             layers=1, graph=False),
        # a ragged prompt through one 3B-class layer, weights kept in TL2
        dict(name="prefill-3b-tl2-m777", kind="stack", layout="tl2", hidden=3200, kv=3200, ffn=8640, tokens=777,
             layers=1, graph=False),
        # batched decode with 2-bit integer weights (table lookups)
        dict(name="decode-3b-c4g2-m8", kind="stack", layout="c4g2", hidden=3200, kv=3200, ffn=8640, tokens=8,
             layers=17, graph=True),
        # batched decode with the lossy int8 tables
        dict(name="decode-8b-tl2_0-m8", kind="stack", layout="tl2_0", hidden=4096, kv=1024, ffn=14336, tokens=8,
             layers=10, graph=True),
        # loading a model: one 8B-class layer's fp32 weights into the default layout
        dict(name="pack-8b-i2s", kind="pack", layout="i2s", hidden=4096, kv=1024, ffn=14336),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(v, m, lo):
    return max(lo, int(round(v / m)) * m)


def draw(rng):
    """One more case of the same ranges: any layout, hidden sizes 1024..12288 in steps of 64 (320 for c3g5, whose rows
    are whole runs of five-weight groups), one token to a 2048-token prompt, odd token counts included."""
    kind = rng.choice(["decode", "decode", "batch", "batch", "small", "prefill", "prefill", "linear", "pack"])
    layout = rng.choice(["i2s", "i2s", "i2s", "tl2", "tl2", "tl1"] if kind in ("small", "prefill", "pack") else
                        ["i2s", "i2s", "i2s", "tl2", "tl2", "tl1", "c4g2", "c5g2", "c3g5", "tl2_0", "tl1_0"])
    step = 320 if layout == "c3g5" else 64
    if kind == "linear":
        K, N = _multiple(_log(rng, 640, 12288), step, step), _multiple(_log(rng, 1024, 12288), 16, 16)
        M = 1 if rng.random() < 0.5 else int(round(_log(rng, 2, 64)))
        M = M if layout not in INT_CARD and layout not in LOSSY else min(M, 8)
        apis = ["fused", "separate"]
        if B.bitnet_mpgemm_workspace_bytes(layout, M, N, K) <= B.NOALLOC_SCRATCH_BYTES:
            apis.append("noalloc")
        return dict(kind="linear", api=rng.choice(apis), layout=layout, K=K, N=N, tokens=M)
    table = layout in INT_CARD or layout in LOSSY
    hidden = _multiple(_log(rng, 1024, 3840 if table or kind in ("small", "prefill", "pack") else 12288), step, step)
    ffn = _multiple(hidden * rng.uniform(2.5, 3.5), step, step)
    kv = rng.choice([hidden, _multiple(hidden / 4, step, step)])
    case = dict(kind="stack", layout=layout, hidden=hidden, kv=kv, ffn=ffn)
    if kind == "pack":
        case["kind"] = "pack"
        return case
    if kind == "prefill":
        case.update(tokens=int(round(_log(rng, 113, 2048))), layers=1, graph=False)
        return case
    case["tokens"] = {"decode": 1, "batch": rng.randint(2, 8 if table else 16), "small": rng.randint(17, 112)}[kind]
    per_layer = sum(B.bitnet_packed_bytes(layout, N, K) for _, K, N in _linears(case))
    case.update(layers=min(17, max(1, math.ceil((512 << 20) / per_layer))), graph=True)
    return case


# ------------------------------------------------------------------------------------------------------------------
# The linears of a case and their inputs
# ------------------------------------------------------------------------------------------------------------------
GROUPS = (("q", "k", "v"), ("o",), ("gate", "up"), ("down",))


def _linears(case):
    """(name, K, N) of one layer, in call order."""
    if case["kind"] == "linear":
        return [("proj", case["K"], case["N"])]
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [("q", h, h), ("k", h, kv), ("v", h, kv), ("o", h, h), ("gate", h, f), ("up", h, f), ("down", f, h)]


def _groups(case):
    """The activation groups of one layer: lists of (index, name, K, N)."""
    lin = [(i, *l) for i, l in enumerate(_linears(case))]
    if case["kind"] == "linear":
        return [lin]
    return [[l for l in lin if l[1] in g] for g in GROUPS]


def _seed(seed, layer, index):
    return (int(seed) * 1_000_003 + layer * 101 + index) & 0x7FFFFFFF


def _weight(case, seed, layer, index, K, N):
    if case["layout"] in INT_CARD:
        return inputs.int_weights(N, K, INT_CARD[case["layout"]], _seed(seed, layer, index), DEV)
    return inputs.weight_f32(N, K, _seed(seed, layer, index), DEV)


def _activation(case, seed, layer, group, K):
    return inputs.activation_f32(case["tokens"], K, _seed(seed, layer, 50 + group), DEV)


def _pack(layout, W):
    N, K = W.shape
    packed = torch.empty(B.bitnet_packed_bytes(layout, N, K), dtype=torch.uint8, device=DEV)
    beta = torch.full((1,), INT_BETA, dtype=torch.float32, device=DEV)
    if layout in INT_CARD:
        B.bitnet_pack_int_weights(layout, W, packed)
    else:
        ws = torch.empty(B.bitnet_pack_workspace_bytes(N, K), dtype=torch.uint8, device=DEV)
        B.bitnet_pack_weights(layout, W, packed, beta, ws)
    return packed, beta


# ------------------------------------------------------------------------------------------------------------------
# prepare / run
# ------------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    layout = case["layout"]
    if case["kind"] == "pack":
        state = dict(case=case, W=[], packed=[], beta=[], ws=[])
        for i, (_, K, N) in enumerate(_linears(case)):
            state["W"].append(_weight(case, seed, 0, i, K, N))
            state["packed"].append(torch.empty(B.bitnet_packed_bytes(layout, N, K), dtype=torch.uint8, device=DEV))
            state["beta"].append(torch.empty(1, dtype=torch.float32, device=DEV))
            state["ws"].append(torch.empty(B.bitnet_pack_workspace_bytes(N, K), dtype=torch.uint8, device=DEV))
        return state

    M, layers = case["tokens"], case.get("layers", 1)
    out = {}                                                   # one tensor per linear / group, its layers stacked
    calls, ws_bytes = [], 16
    for g, group in enumerate(_groups(case)):
        K = group[0][2]
        out["xq%d" % g] = torch.empty((layers, M, K), dtype=torch.int8, device=DEV)
        out["s%d" % g] = torch.empty((layers, M), dtype=torch.float32, device=DEV)
        out["rs%d" % g] = torch.empty((layers, M), dtype=torch.int32, device=DEV)
        for _, name, _, N in group:
            # rows of scales and sums are 4-byte aligned whatever M is; M * N is a multiple of 16
            out["y_" + name] = torch.empty((layers, M, N), dtype=torch.float32, device=DEV)
        Ns = [l[3] for l in group]
        ws_bytes = max(ws_bytes, B.bitnet_mpgemm_fused_workspace_bytes(layout, Ns, K, M))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)  # calls on one stream share it
    for layer in range(layers):
        for g, group in enumerate(_groups(case)):
            K = group[0][2]
            x = _activation(case, seed, layer, g, K)
            packed, betas = zip(*[_pack(layout, _weight(case, seed, layer, i, K, N)) for i, _, _, N in group])
            ys = [out["y_" + name][layer] for _, name, _, _ in group]
            calls.append(dict(packed=packed, betas=betas, x=x, K=K, N=group[0][3], xq=out["xq%d" % g][layer],
                              s=out["s%d" % g][layer], rs=out["rs%d" % g][layer], ys=ys,
                              args=B.FusedArgs(packed, betas, ys)))
    state = dict(case=case, calls=calls, ws=ws, out=out, graph=None)
    if case.get("graph"):
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            _calls(state)                                      # first launches outside the capture
        torch.cuda.current_stream().wait_stream(stream)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _calls(state)
    return state


def _calls(state):
    layout, api = state["case"]["layout"], state["case"].get("api", "fused")
    for c in state["calls"]:
        if api == "fused":
            B.bitnet_mpgemm_fused(layout, c["packed"], c["betas"], c["x"], c["xq"], c["s"], c["rs"], c["ys"],
                                  ws=state["ws"], args=c["args"])
            continue
        B.bitnet_quantize_act(c["x"], c["xq"], c["s"], c["rs"])
        if api == "separate":
            B.bitnet_mpgemm(layout, c["packed"][0], c["betas"][0], c["N"], c["K"], c["xq"], c["s"], c["ys"][0],
                            ws=state["ws"], x_rowsum=c["rs"])
        else:
            B.bitnet_mpgemm_noalloc(layout, c["packed"][0], c["betas"][0], c["N"], c["K"], c["xq"], c["s"],
                                    c["ys"][0], x_rowsum=c["rs"])


def run(state):
    case = state["case"]
    if case["kind"] == "pack":
        for W, packed, beta, ws in zip(state["W"], state["packed"], state["beta"], state["ws"]):
            B.bitnet_pack_weights(case["layout"], W, packed, beta, ws)
        return dict(packed=state["packed"], beta=state["beta"])
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _calls(state)
    return state["out"]


# ------------------------------------------------------------------------------------------------------------------
# What the path cannot do without, and what its results are held to
# ------------------------------------------------------------------------------------------------------------------
def work(case):
    bytes_, flops = 0, 0
    if case["kind"] == "pack":
        for _, K, N in _linears(case):
            bytes_ += 4 * N * K + B.bitnet_packed_bytes(case["layout"], N, K) + 4
            flops += 4 * N * K                                 # |w|, its sum, the division, the rounding
        return {"bytes": bytes_, "flops": flops}
    M = case["tokens"]
    for group in _groups(case):
        K = group[0][2]
        bytes_ += 5 * M * K + 8 * M                            # x in; codes, scales and code sums out
        for _, _, _, N in group:
            bytes_ += B.bitnet_packed_bytes(case["layout"], N, K) + 4 + 4 * M * N
            flops += 2 * M * N * K
    layers = case.get("layers", 1)
    return {"bytes": bytes_ * layers, "flops": flops * layers}


def tolerance(case):
    # Codes, code sums, packed bytes are whole numbers defined exactly and may not differ.  The sums behind y are
    # exact integers; y then takes two to three fp32 roundings (the scale quotient, the product, the activation
    # scale), at most 1.8e-7 of the value: 6e-8 measured against 64 bits.
    return {"rel": 2.4e-7, "max": 4e-7, "differ": 0.0}


def _shift(mx):
    """The smallest s >= 0 with mx <= 127 * 2^s (mx: int64 tensor)."""
    s = torch.zeros_like(mx)
    for _ in range(4):                                         # entries are sums of at most three codes
        s = torch.where(mx > 127 * (1 << s), s + 1, s)
    return s


def _lossy_part(xq, t, g, per_block):
    """sum over groups of g weights of 2^s rint((t . xq) / 2^s), s per token and block of per_block groups; f64 [M, N].
    The block's largest |entry| is that of the full ternary table: the largest sum of |xq| over a group."""
    M, K = xq.shape
    N, G = t.shape[0], K // g
    tg = t.reshape(N, G, g)
    acc = torch.zeros((M, N), dtype=torch.float64, device=xq.device)
    for m in range(M):
        xg = xq[m].double().reshape(G, g)
        mx = xg.abs().sum(1).to(torch.int64).reshape(G // per_block, per_block).amax(1)
        scale = (2.0 ** _shift(mx).double()).repeat_interleave(per_block)
        for n0 in range(0, N, 4096):
            dots = (tg[n0:n0 + 4096] * xg).sum(2)
            acc[m, n0:n0 + 4096] = (torch.round(dots / scale) * scale).sum(1)
    return acc


def exact(case, seed):
    layout = case["layout"]

    def ternary(layer, i, K, N):
        W = _weight(case, seed, layer, i, K, N)
        if layout in INT_CARD:
            return W.double(), float(torch.tensor(INT_BETA, dtype=torch.float32))
        beta = (W.abs().sum(dtype=torch.float64) / W.numel()).float()
        t = torch.clamp(torch.round(W / beta), -1, 1) if float(beta) > 0 else torch.zeros_like(W)
        return t.double(), float(beta)

    if case["kind"] == "pack":
        beta = [_weight(case, seed, 0, i, K, N).abs().mean(dtype=torch.float64).reshape(1)
                for i, (_, K, N) in enumerate(_linears(case))]
        return dict(packed=[None] * len(beta), beta=beta)

    layers, M = case.get("layers", 1), case["tokens"]
    out = {}
    for layer in range(layers):
        for g, group in enumerate(_groups(case)):
            K = group[0][2]
            x = _activation(case, seed, layer, g, K)
            # the quantiser is defined in fp32 (a tensor dividend: a number's division is a product by the reciprocal)
            s = torch.full((M,), 127.0, device=x.device) / torch.clamp(x.abs().amax(1), min=1e-5)
            xq = torch.clamp(torch.round(x * s[:, None]), -128, 127)
            s64 = 127.0 / torch.clamp(x.abs().amax(1).double(), min=1e-5)
            out.setdefault("xq%d" % g, []).append(xq.to(torch.int8))
            out.setdefault("s%d" % g, []).append(s64)
            out.setdefault("rs%d" % g, []).append(xq.double().sum(1).to(torch.int32))
            for i, name, _, N in group:
                t, beta = ternary(layer, i, K, N)
                if layout == "tl1_0":
                    acc = _lossy_part(xq, t, 2, 32)
                elif layout == "tl2_0":
                    three = K // 384 * 384
                    acc = torch.zeros((M, N), dtype=torch.float64, device=x.device)
                    if three:
                        acc += _lossy_part(xq[:, :three], t[:, :three], 3, 128)
                    if K > three:
                        acc += _lossy_part(xq[:, three:], t[:, three:], 2, 32)
                else:
                    acc = xq.double() @ t.t().contiguous()
                out.setdefault("y_" + name, []).append(acc * beta / s64[:, None])
    return {k: torch.stack(v) for k, v in out.items()}

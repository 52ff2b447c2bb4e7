"""The work that users of the HLQ GEMV / GEMM library have it do, as a list of measurable cases.

A case is a dict of plain values; `prepare` makes what a program holds before the call (packed weights, activations,
outputs, workspace, captured graph), `run` is one pass through the public entry points, `exact` the same result in
64-bit arithmetic by plain torch.  Four kinds:

  linear    one weight matrix, one hlq_lut_gemv / hlq_lut_gemm call
  group     the seven projections of a decoder layer as one grouped launch, for `layers` layers in a row
  token     the projections of `layers` decoder layers in stream order (q|k|v, o, gate|up, down: four dependent
            launches a layer), captured in a graph once and replayed per token
  quantize  real-valued weights to codes, scales and zeros (Alg. 1), with `pack` also to the packed blob

Value distributions are those of the repository's generators: codes uniform, scales |N(0, 0.02)| descending over the
planes, zeros N(0, 0.005), activations N(0, 1) with 1 % of the channels times 20 where `outliers` is set, real-valued
weights N(0, 0.02)."""
import math
import zlib

import torch

from paper_2510_19482_amd import binding as hlq

LAYER_8B = dict(hidden=4096, kv=1024, ffn=14336)
HEAD_70B = (8192, 128256)

# the largest listed cases, which bound what draw() may give
MOST_WEIGHTS = HEAD_70B[0] * HEAD_70B[1]
MOST_PRODUCTS = 2048 * 218103808


def listed():
    layer = dict(LAYER_8B, layers=1, outliers=True)
    return [
        # one narrow projection of one token: what a call costs when there is next to nothing to stream
        dict(name="gemv_kv", kind="linear", K=4096, N=1024, q=2, G=128, M=1, f32=False, outliers=False),
        # sizes that fill no tile and no split evenly, narrow quant groups, fp32 results
        dict(name="gemv_ragged", kind="linear", K=11008, N=5000, q=3, G=64, M=1, f32=True, outliers=True),
        # one decoded token of an 8B-shaped model: 32 layers of dependent launches replayed from a graph
        dict(name="token_8b", kind="token", q=2, G=128, M=1, f32=False, **dict(layer, layers=32)),
        # four layers with the projections of a layer in one launch: the headline workload of the benchmark
        dict(name="layers_8b", kind="group", q=2, G=128, M=1, f32=False, **dict(layer, layers=4)),
        # the widest matrix in use, the LM head of a 70B-shaped model with narrow groups
        dict(name="head_70b", kind="linear", K=HEAD_70B[0], N=HEAD_70B[1], q=2, G=64, M=1, f32=False, outliers=False),
        # small-batch decode, a few sequences and a full batch, at four planes
        dict(name="layer_8b_m4", kind="group", q=4, G=128, M=4, f32=False, **layer),
        dict(name="layer_8b_m16", kind="group", q=4, G=128, M=16, f32=False, **layer),
        # a batch or a short prompt that is no power of two, three planes, narrow groups, one call
        dict(name="proj_m24", kind="linear", K=4096, N=14336, q=3, G=64, M=24, f32=False, outliers=True),
        # prefill of a prompt of 512 and of 2048 tokens
        dict(name="layer_8b_m512", kind="group", q=2, G=128, M=512, f32=False, **layer),
        dict(name="layer_8b_m2048", kind="group", q=2, G=128, M=2048, f32=False, **layer),
        # offline preparation of a matrix: Alg. 1 alone, and Alg. 1 and packing at four planes with narrow groups
        dict(name="quantize_q2", kind="quantize", K=4096, N=4096, q=2, G=128, t_max=10, pack=False),
        dict(name="quantize_pack_q4", kind="quantize", K=4096, N=1024, q=4, G=64, t_max=10, pack=True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi, step):
    return max(lo, min(hi, int(round(_log(rng, lo, hi) / step)) * step))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "group", "group", "token", "quantize"])
    q, G = rng.randint(1, 4), rng.choice([32, 64, 128, 128, 256])
    step = max(128, G)
    if kind == "quantize":
        return dict(kind=kind, K=_size(rng, 512, 8192, step), N=_size(rng, 512, 4096, 8), q=q, G=G, t_max=rng.choice([5, 10]), pack=rng.random() < 0.5)
    f32, outliers = rng.random() < 0.3, rng.random() < 0.5
    M = rng.choice([1, 1, rng.randint(2, 16), rng.randint(17, 100), int(_log(rng, 100, 2048))])
    if kind == "linear":
        K, N = _size(rng, 512, 28672, step), _size(rng, 512, 128256, 8)
        while K * N > MOST_WEIGHTS or M * K * N > MOST_PRODUCTS // 2:
            N = max(512, N // 16 * 8)
        return dict(kind=kind, K=K, N=N, q=q, G=G, M=M, f32=f32, outliers=outliers)
    hidden = _size(rng, 1024, 4096, 256)
    shape = dict(hidden=hidden, kv=rng.choice([256, 512, 1024]), ffn=_size(rng, 2 * hidden, 14336, 256))
    if kind == "token":
        return dict(kind=kind, q=q, G=G, M=1, f32=f32, layers=rng.randint(4, 24), outliers=outliers, **shape)
    return dict(kind=kind, q=q, G=G, M=M, f32=f32, layers=4 if M == 1 else 1, outliers=outliers, **shape)


# ---- what a case consists of ---------------------------------------------------------------------------------------

def _inputs(case):
    """[(name of the activation, K)] of one layer, or of the one matrix."""
    if case["kind"] == "linear":
        return [("x", case["K"])]
    h, f = case["hidden"], case["ffn"]
    return [("attn", h), ("o", h), ("ffn", h), ("down", f)]


def _matrices(case):
    """[(K, N, name of the activation)] of one layer, or the one matrix."""
    if case["kind"] == "linear":
        return [(case["K"], case["N"], "x")]
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    if case["kind"] == "token":   # projections that read the same activation are stored as one matrix
        return [(h, h + 2 * kv, "attn"), (h, h, "o"), (h, 2 * f, "ffn"), (f, h, "down")]
    return [(h, h, "attn"), (h, kv, "attn"), (h, kv, "attn"), (h, h, "o"), (h, f, "ffn"), (h, f, "ffn"), (f, h, "down")]


def _generator(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) % (1 << 30) << 32) ^ zlib.crc32(repr(key).encode()))
    return g


def _weight(case, seed, layer, i, K, N):
    g = _generator(seed, "weight", layer, i)
    q, G = case["q"], case["G"]
    codes = torch.randint(0, 1 << q, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    scales = torch.randn((q, K // G, N), device="cuda", generator=g).mul_(0.02).abs_().sort(dim=0, descending=True).values.half()
    zeros = torch.randn((K // G, N), device="cuda", generator=g).mul_(0.005).half()
    return codes, scales.contiguous(), zeros


def _activation(case, seed, layer, name, K):
    g = _generator(seed, "x", layer, name)
    x = torch.randn((case["M"], K), device="cuda", generator=g)
    if case["outliers"]:
        x[:, torch.randperm(K, device="cuda", generator=g)[:max(1, round(0.01 * K))]] *= 20.0
    return x.half()


def _dense(case, seed):
    return torch.randn((case["K"], case["N"]), device="cuda", generator=_generator(seed, "dense")).mul_(0.02)


def _blob(desc, weight):
    return hlq.hlq_pack(desc, *weight)


# ---- state, pass ---------------------------------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "quantize":
        return dict(case=case, desc=hlq.make_desc(case["K"], case["N"], case["q"], case["G"]), W=_dense(case, seed))
    M, odt = case["M"], torch.float32 if case["f32"] else torch.float16
    mats = _matrices(case)
    descs = [hlq.make_desc(K, N, case["q"], case["G"]) for K, N, _ in mats]
    if case["kind"] == "linear":
        K, N, _ = mats[0]
        x = _activation(case, seed, 0, "x", K)
        return dict(case=case, desc=descs[0], packed=_blob(descs[0], _weight(case, seed, 0, 0, K, N)), x=x[0] if M == 1 else x,
                    y=torch.empty(N if M == 1 else (M, N), dtype=odt, device="cuda"), ws=hlq.alloc_workspace(descs[0], M))
    layers = []
    if case["kind"] == "token":
        ws = max((hlq.alloc_workspace(d, 1) for d in descs), key=lambda t: t.numel())   # calls follow each other on one stream
        total = sum(N for _, N, _ in mats)
        out = torch.empty((case["layers"], total), dtype=odt, device="cuda")
        for l in range(case["layers"]):
            xs = {n: _activation(case, seed, l, n, K)[0] for n, K in _inputs(case)}
            at = 0
            for i, (K, N, n) in enumerate(mats):
                layers.append((descs[i], _blob(descs[i], _weight(case, seed, l, i, K, N)), xs[n], out[l, at:at + N]))
                at += N

        def token():
            for desc, packed, x, y in layers:
                hlq.hlq_lut_gemv(desc, packed, x, y, out_f32=case["f32"], ws=ws)

        token()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            token()
        return dict(case=case, graph=graph, out=out, keep=(layers, ws))
    ws = None
    for l in range(case["layers"]):
        xs = {n: _activation(case, seed, l, n, K) for n, K in _inputs(case)}
        packed = [_blob(descs[i], _weight(case, seed, l, i, K, N)) for i, (K, N, _) in enumerate(mats)]
        ys = [torch.empty((M, N), dtype=odt, device="cuda") for _, N, _ in mats]
        if M == 1:
            launch = hlq.GemvBatch(descs, packed, [xs[n][0] for _, _, n in mats], [y[0] for y in ys], out_f32=case["f32"], ws=ws)
        else:
            launch = hlq.GemmBatch(descs, packed, [xs[n] for _, _, n in mats], ys, out_f32=case["f32"], ws=ws)
        ws = launch.ws   # the layers follow each other on one stream
        layers.append((launch, ys))
    return dict(case=case, layers=layers)


def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        codes, scales, zeros = hlq.hlq_quantize(state["desc"], state["W"], case["t_max"])
        if case["pack"]:
            return codes, scales, zeros, hlq.hlq_pack(state["desc"], codes, scales, zeros)
        return codes, scales, zeros
    if case["kind"] == "token":
        state["graph"].replay()
        return state["out"]
    if case["kind"] == "linear":
        call = hlq.hlq_lut_gemv if case["M"] == 1 else hlq.hlq_lut_gemm
        return call(state["desc"], state["packed"], state["x"], state["y"], out_f32=case["f32"], ws=state["ws"])
    for launch, _ in state["layers"]:
        launch.launch()
    return [ys for _, ys in state["layers"]]


def work(case):
    q, G = case["q"], case["G"]
    if case["kind"] == "quantize":
        K, N = case["K"], case["N"]
        params = 2 * (q + 1) * K * N // G
        blob = K * N * q // 8 + params if case["pack"] else 0
        # 2^q candidate distances (subtract, magnitude, compare) and the distinct sums of the normal equations per
        # weight and round
        return dict(bytes=4 * K * N + K * N + params + blob, flops=case["t_max"] * K * N * (3 * 2 ** q + (q + 1) * (q + 2) // 2))
    layers, M = case.get("layers", 1), case["M"]
    weights = sum(K * N for K, N, _ in _matrices(case))
    out = sum(N for _, N, _ in _matrices(case))
    packed = weights * q // 8 + 2 * (q + 1) * weights // G
    return dict(bytes=layers * (packed + 2 * M * sum(K for _, K in _inputs(case)) + (4 if case["f32"] else 2) * M * out),
                flops=layers * 2 * M * weights)


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    # about four times the error against exact() seen over the listed and forty drawn cases.  One row: products are
    # exact and summed in fp32 (the matrix core adds runs of eight in fixed point), so an fp16 result carries its own
    # rounding only.  More rows: from a few rows on the weights are rounded to fp16 when they are rebuilt.
    if case["M"] == 1:
        return dict(rel=8e-5, max=1.5e-3) if case["f32"] else dict(rel=9e-4, max=2.2e-3)
    return dict(rel=1.6e-3, max=1e-2)


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

def _product(case, weight, x, block=8192):
    codes, scales, zeros = weight
    x, G, out = x.double(), case["G"], []
    for n in range(0, codes.shape[1], block):
        c, s = codes[:, n:n + block], scales[:, :, n:n + block].double()
        w = zeros[:, n:n + block].double().repeat_interleave(G, 0)
        for j in range(case["q"]):
            w += s[j].repeat_interleave(G, 0) * ((c >> j) & 1)
        out.append(x @ w)
    return torch.cat(out, 1)


def exact(case, seed):
    if case["kind"] == "quantize":
        got = _alternating(case, _dense(case, seed))
        return got + (None,) if case["pack"] else got
    answer = []
    for l in range(case.get("layers", 1)):
        xs = {n: _activation(case, seed, l, n, K) for n, K in _inputs(case)}
        answer.append([_product(case, _weight(case, seed, l, i, K, N), xs[n]) for i, (K, N, n) in enumerate(_matrices(case))])
    if case["kind"] == "linear":
        return answer[0][0][0] if case["M"] == 1 else answer[0][0]
    if case["kind"] == "token":
        return torch.stack([torch.cat([y[0] for y in ys]) for ys in answer])
    return answer


def _alternating(case, W):
    """Alg. 1: codes by nearest candidate (the smallest code of equally near ones), parameters by least squares; a
    column of [1 b_0 b_1 ..] that depends on the earlier ones keeps its parameter."""
    K, N, q, G = case["K"], case["N"], case["q"], case["G"]
    P, ng = q + 1, K // G
    w = W.double().reshape(ng, G, N).permute(0, 2, 1).reshape(ng * N, G)
    bits = torch.tensor([[1.0] + [float((c >> j) & 1) for j in range(q)] for c in range(1 << q)], dtype=torch.float64, device=W.device)
    lo, hi = w.amin(1), w.amax(1)
    theta = torch.stack([lo] + [(hi - lo) / (2 ** q - 1) * 2 ** j for j in range(q)], 1)
    codes = None
    for _ in range(case["t_max"]):
        what, best, code = w - theta[:, :1], None, None
        for c in range(1 << q):
            v = torch.zeros_like(theta[:, 0])
            for j in range(q):
                v = v + theta[:, 1 + j] * bits[c, 1 + j]
            d = (what - v[:, None]).abs()
            if best is None:
                best, code = d, torch.zeros_like(d, dtype=torch.uint8)
            else:
                code = torch.where(d < best, torch.full_like(code, c), code)
                best = torch.minimum(best, d)
        codes = code
        count = torch.stack([(code == c).sum(1) for c in range(1 << q)], 1).double()
        total = torch.stack([torch.where(code == c, w, 0.0).sum(1) for c in range(1 << q)], 1)
        rows = (bits[:, :, None] * bits[:, None, :]).reshape(1 << q, P * P)
        A = (count @ rows).reshape(-1, P, P)
        r = total @ bits
        # columns that depend on the earlier ones, from the Gram matrix of the distinct rows present (small integers)
        gram = ((count > 0).double() @ rows).reshape(-1, P, P)
        active, prev = [], torch.ones_like(lo)
        for k in range(P):
            pv = gram[:, k, k].clone()
            on = pv != 0
            active.append(on)
            new = (gram * pv[:, None, None] - gram[:, :, k:k + 1] * gram[:, k:k + 1, :]) / prev[:, None, None]
            gram = torch.where(on[:, None, None], new, gram)
            prev = torch.where(on, pv, prev)
        act = torch.stack(active, 1)
        r = r - torch.where(act[:, None, :], 0.0, A * theta[:, None, :]).sum(2)
        r = torch.where(act, r, theta)
        eye = torch.eye(P, dtype=torch.float64, device=W.device)
        A = torch.where(act[:, :, None] & act[:, None, :], A, eye)
        theta = torch.linalg.solve(A, r)
    theta = theta.reshape(ng, N, P)
    return (codes.reshape(ng, N, G).permute(0, 2, 1).reshape(K, N), theta[..., 1:].permute(2, 0, 1), theta[..., 0])

"""The workloads this library is timed on: what a program that serves a model
with SBVR weights asks of it, through the package's public calls.

A case names an operation and its sizes:

  op      "gemv", "batch", "prefill", "decompress" or "quantise"
  shapes  the weight matrices of one layer as OxI (out_features x
          in_features), in call order; matrices joined by "+" read the same
          activations (q+k+v, gate+up)
  layers  how many layers, each with weights and activations of its own
  k       bitvector planes per 128-weight group

and the options of the operation.  ``listed()`` holds the Llama-3-8B and -70B
projection shapes that the benchmark and the tests use, ``draw()`` gives
further shapes of the same ranges: any out_features, any multiple of 128
in_features, k = 1..4, every batch size, prompts of 1 to 2048 tokens.
"""
import math

import torch

import paper_2509_18172_amd as sb

GROUP = 128
SIGMA = 0.02  # standard deviation of the weights
LAYER_8B = "4096x4096+1024x4096+1024x4096,4096x4096,14336x4096+14336x4096,4096x14336"
LAYER_70B = "8192x8192+1024x8192+1024x8192,8192x8192,28672x8192+28672x8192,8192x28672"


def _case(op, shapes, k, layers=1, name=None, **options):
    c = {"op": op, "shapes": shapes, "k": k, "layers": layers, **options}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # one small projection called on its own: launch and call latency
        _case("gemv", "1024x1024", 4, name="gemv_1024", launch="separate", graph=False, a8=False, indexed=False),
        # the decode step of a 32-layer 8B model: 224 projections, batch 1,
        # replayed as one captured graph
        _case("gemv", LAYER_8B, 4, 32, name="decode_8b", launch="separate", graph=True, a8=False, indexed=False),
        # the same step as a serving loop issues it, with 8-bit activations
        # (W4A8) and the projections that share an input in one launch
        _case("gemv", LAYER_8B, 4, 32, name="decode_8b_w4a8", launch="grouped", graph=True, a8=True, indexed=False),
        # four layers of a 70B model's decode step
        _case("gemv", LAYER_70B, 4, 4, name="decode_70b", launch="separate", graph=True, a8=False, indexed=False),
        # decode on the coefficient-cache storage format
        _case("gemv", LAYER_8B, 4, 8, name="decode_8b_indexed", launch="separate", graph=True, a8=False, indexed=True),
        # decode of eight concurrent sequences
        _case("batch", LAYER_8B, 4, 8, name="batch8_8b", batch=8, graph=True),
        # three sequences on a 3-bit model
        _case("batch", LAYER_8B, 3, 8, name="batch3_8b_k3", batch=3, graph=True),
        # a 512-token prompt (or prefill chunk) through one layer's projections
        _case("prefill", LAYER_8B, 4, name="prefill_8b_512", tokens=512),
        # a short prompt of an odd length
        _case("prefill", LAYER_8B, 4, name="prefill_8b_37", tokens=37),
        # a layer's weights expanded to binary16 for a dense GEMM
        _case("decompress", LAYER_8B, 4, name="decompress_8b", indexed=False),
        # a 4096 x 4096 weight matrix quantised and packed for serving
        _case("quantise", "4096x4096", 4, name="quantise_4096", cache=0),
        # the same with the encoder cache, at 3 bits
        _case("quantise", "4096x4096", 3, name="quantise_4096_cached_k3", cache=64),
    ]


# No drawn case reads more weights, computes more or encodes more than the
# listed ones.
MAX_GEMV_BYTES = 3.5e9
MAX_PREFILL_FLOPS = 2.0e11
MAX_DECOMPRESS = 2.0e8
MAX_ENCODE = 1.6e7


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("gemv", "gemv", "gemv", "batch", "batch", "prefill", "prefill", "decompress", "quantise"))
    k = rng.choice((1, 2, 3, 4, 4, 4))
    out, inn = _log_int(rng, 64, 28672), GROUP * _log_int(rng, 2, 224)
    if op in ("gemv", "batch"):
        # one to four matrices on one input
        outs = [out] + [_log_int(rng, 64, 28672) for _ in range(rng.randrange(4))]
        shapes = "+".join("%dx%d" % (o, inn) for o in outs)
        per_layer = sum(outs) * inn * k * 0.140625
        graph = rng.random() < 0.8
        layers = int(min(rng.randint(1, 32), max(1, MAX_GEMV_BYTES // per_layer))) if graph else 1
        if op == "batch":
            return _case(op, shapes, k, layers, batch=rng.randint(2, 8), graph=graph)
        indexed = rng.random() < 0.25
        launch = "separate" if indexed or rng.random() < 0.5 else "grouped"
        return _case(op, shapes, k, layers, launch=launch, graph=graph, a8=rng.random() < 0.4, indexed=indexed)
    if op == "prefill":
        tokens = _log_int(rng, 1, 2048)
        while 2.0 * out * inn * tokens > MAX_PREFILL_FLOPS:
            out = max(64, out // 2)
        return _case(op, "%dx%d" % (out, inn), k, tokens=tokens)
    limit = MAX_DECOMPRESS if op == "decompress" else MAX_ENCODE
    while out * inn > limit:
        out = max(1, out // 2)
    if op == "decompress":
        return _case(op, "%dx%d" % (out, inn), k, indexed=rng.random() < 0.25)
    return _case(op, "%dx%d" % (out, inn), k, cache=rng.choice((0, 0, 16, 64)))


def _layout(case):
    """The layer's matrices: groups of (O, I) that share activations."""
    return [[tuple(int(v) for v in m.split("x")) for m in g.split("+")] for g in case["shapes"].split(",")]


def _sets(O, I):
    """Coefficient sets of an indexed matrix: one per ten groups."""
    return max(1, min(65536, O * (I // GROUP) // 10))


def _coefficients(gen, shape, k):
    """Coefficient sets as the encoder makes them: a geometric series of
    negative ratio scaled to the group's width, plus a small bias."""
    r = -(0.5 + 1.5 * torch.rand(*shape, 1, generator=gen, device="cuda"))
    pw = r ** torch.arange(k, device="cuda")
    s = SIGMA * (4 + 3 * torch.rand(*shape, 1, generator=gen, device="cuda"))
    b = SIGMA * 0.2 * (torch.rand(*shape, 1, generator=gen, device="cuda") - 0.5)
    return (s * pw / pw.abs().sum(-1, keepdim=True) + b).half().view(torch.int16)


def _matrices(case, gen):
    """The canonical tensors of every matrix, in order: (O, I, planes, coeffs)
    or, indexed, (O, I, planes, index, table)."""
    k = case["k"]
    for _ in range(case["layers"]):
        for group in _layout(case):
            for O, I in group:
                G = I // GROUP
                planes = torch.randint(-2**31, 2**31, (O, G, k, 4), dtype=torch.int32, generator=gen, device="cuda")
                if case.get("indexed"):
                    n = _sets(O, I)
                    index = torch.randint(0, n, (O, G), dtype=torch.int32, generator=gen, device="cuda")
                    yield O, I, planes, index.to(torch.int16), _coefficients(gen, (n,), k)
                else:
                    yield O, I, planes, _coefficients(gen, (O, G), k)


def _activations(gen, *shape):
    """Normal activations, one in a thousand ten times as large."""
    x = torch.randn(*shape, generator=gen, device="cuda")
    return torch.where(torch.rand(*shape, generator=gen, device="cuda") < 0.001, 10 * x, x).half()


def _generators(seed):
    return (torch.Generator("cuda").manual_seed(2 * seed), torch.Generator("cuda").manual_seed(2 * seed + 1))


def _rows(case):
    """Leading dimensions of a layer's activations and outputs."""
    return {"batch": (case.get("batch"),), "prefill": (case.get("tokens"),)}.get(case["op"], ())


def _float_weights(case, gen):
    """float32 weights with one in a thousand at +-8 sigma."""
    (O, I), = _layout(case)[0]
    W = SIGMA * torch.randn(O, I, generator=gen, device="cuda")
    far = torch.rand(O, I, generator=gen, device="cuda") < 0.001
    return torch.where(far, 8 * SIGMA * W.sign(), W)


def prepare(case, seed):
    gw, gx = _generators(seed)
    op = case["op"]
    if op == "quantise":
        return {"case": case, "W": _float_weights(case, gw)}
    if case.get("indexed"):
        weights = (sb.pack_indexed(*m[2:]) for m in _matrices(case, gw))
    else:
        weights = (sb.pack(*m[2:]) for m in _matrices(case, gw))
    layout, rows = _layout(case), _rows(case)
    if op == "decompress":
        Ws = list(weights)
        return {"case": case, "Ws": Ws, "out": [torch.empty(W.O, W.I, dtype=torch.float16, device="cuda") for W in Ws]}
    # the outputs of one matrix over all layers lie in one tensor
    out = [torch.empty(case["layers"], *rows, O, dtype=torch.float16, device="cuda") for g in layout for O, _ in g]
    calls = []
    for layer in range(case["layers"]):
        n = 0
        for group in layout:
            x = _activations(gx, *rows, group[0][1])
            Ws = [next(weights) for _ in group]
            calls.append((Ws, x, [out[n + i][layer] for i in range(len(group))]))
            n += len(group)
    state = {"case": case, "calls": calls, "out": out}
    if case.get("graph"):
        _step(state)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _step(state)
    return state


def _step(state):
    c = state["case"]
    op = c["op"]
    for Ws, x, outs in state["calls"]:
        if op == "gemv" and c["launch"] == "grouped":
            sb.gemv_grouped(Ws, [x] * len(Ws), outs, a8=c["a8"])
            continue
        for W, y in zip(Ws, outs):
            if op == "prefill":
                sb.gemm_prefill(W, x, out=y)
            elif op == "batch":
                sb.gemm_small_batch(W, x, out=y)
            elif c["indexed"]:
                sb.gemv_indexed(W, x, out=y, a8=c["a8"])
            elif c["a8"]:
                sb.gemv_a8(W, x, out=y)
            else:
                sb.gemv(W, x, out=y)


def run(state):
    case = state["case"]
    if case["op"] == "quantise":
        if case["cache"]:
            planes, coeffs, mse, hits = sb.encode_cached(state["W"], case["k"], cache_slots=case["cache"])
        else:
            planes, coeffs, mse = sb.encode(state["W"], case["k"], want_mse=True)
            hits = None
        P = sb.pack(planes, coeffs)
        return {"mse": mse, "planes": planes, "coeffs": coeffs, "hits": hits, "packed": P.planes, "packed_c": P.coeffs}
    if case["op"] == "decompress":
        for W, M in zip(state["Ws"], state["out"]):
            sb.decompress(W, out=M)
    elif case.get("graph"):
        state["graph"].replay()
    else:
        _step(state)
    return state["out"]


def work(case):
    k, op, nbytes, flops = case["k"], case["op"], 0.0, 0.0
    for group in _layout(case):
        vectors = (_rows(case) or (1,))[0]
        if op in ("gemv", "batch", "prefill"):
            nbytes += 2.0 * vectors * group[0][1]
        for O, I in group:
            groups = O * (I // GROUP)
            stored = 16.0 * k * groups  # planes, then coefficients or indices and their sets
            stored += 2.0 * groups + 2.0 * k * _sets(O, I) if case.get("indexed") else 2.0 * k * groups
            if op == "quantise":
                # float32 weights read; planes, coefficients and the error of
                # each group written, canonical and packed; every entry of the
                # 1024-entry grid needs the squared errors of its 2^k cells
                nbytes += 4.0 * O * I + 2 * stored + 8.0 * groups + (groups if case["cache"] else 0.0)
                flops += 1024.0 * 6.0 * 2**k * groups
            elif op == "decompress":
                nbytes += stored + 2.0 * O * I
            else:
                nbytes += stored + 2.0 * vectors * O
                flops += 2.0 * vectors * O * I
    return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    # Decoded weights and encodings are defined to the bit.
    if case["op"] in ("decompress", "quantise"):
        return "exact"
    # Outputs are binary16 of binary32 sums: against 64 bits the rounding alone
    # measured 2.1e-4 (2-norm) and 4.9e-4 (largest, half a unit in the last
    # place); four times that.
    return {"rel": 1e-3, "max": 2e-3}


def _dense(planes, coeffs):
    """The decoded weights [O][I] in binary64."""
    O, G, k, _ = planes.shape
    c = coeffs.view(torch.float16).double()
    shift = torch.arange(32, device="cuda", dtype=torch.int32)
    w = torch.zeros(O, G, 4, 32, dtype=torch.float64, device="cuda")
    for i in range(k):
        w += c[:, :, i, None, None] * ((planes[:, :, i, :, None] >> shift) & 1)
    return w.view(O, G * GROUP)


def _codes(x):
    """The values of 8-bit activations: per group q * absmax / 127 with q the
    nearest integer of x over that scale, both in binary32."""
    g = x.float().view(-1, GROUP)
    s = g.abs().amax(1, keepdim=True) / 127
    q = torch.where(s > 0, (g / s).round().clamp(-127, 127), torch.zeros_like(g))
    return (s.double() * q.double()).view(x.shape)


def _encode_error(W, k):
    """Each group's smallest mean squared error over the search grid."""
    D = W.view(-1, GROUP).double()
    mn, mx, avg = D.amin(1), D.amax(1), D.mean(1)
    s_min, s_max = 2 * torch.quantile(D, 0.95, dim=1), 1.1 * (mx - mn)
    b_max = 2 * avg.abs() / k
    bit = (torch.arange(2**k, device="cuda")[:, None] >> torch.arange(k, device="cuda")) & 1
    best = torch.full_like(avg, math.inf)
    for r in [-1 + (i + 1) * 0.0625 for i in range(8)] + [-2 + i * 0.125 for i in range(8)]:
        pw = torch.tensor([r**i for i in range(k)], dtype=torch.float64, device="cuda")
        for j in range(16):
            s = s_min + (j + 1) * ((s_max - s_min) / 16)
            for n in range(4):
                b = -b_max + n * (2 * b_max / 4)
                c = (s[:, None] * pw / pw.abs().sum() + b[:, None]).half().double()
                sums = c @ bit.double().T
                m = (D - sums[:, :1]).abs()
                for p in range(1, 2**k):
                    m = torch.minimum(m, (D - sums[:, p:p + 1]).abs())
                best = torch.where(s > 0, torch.minimum(best, m.square().mean(1)), best)
    return best.view(W.shape[0], -1)


def exact(case, seed):
    gw, gx = _generators(seed)
    op = case["op"]
    if op == "quantise":
        if case["cache"]:
            return None  # which groups hit depends on every earlier one
        mse = _encode_error(_float_weights(case, gw), case["k"])
        return {"mse": mse, "planes": None, "coeffs": None, "hits": None, "packed": None, "packed_c": None}
    mats, layout, rows = _matrices(case, gw), _layout(case), _rows(case)
    out = [[] for g in layout for _ in g]
    for _ in range(case["layers"]):
        n = 0
        for group in layout:
            if op != "decompress":
                x = _activations(gx, *rows, group[0][1])
                x = _codes(x) if case.get("a8") else x.double()
            for _ in group:
                O, I, planes, *c = next(mats)
                step = max(1, 2**24 // I)
                parts = []
                for o in range(0, O, step):
                    cf = c[0][o:o + step]
                    if case.get("indexed"):
                        cf = c[1][cf.long() & 0xffff]
                    w = _dense(planes[o:o + step], cf)
                    if op == "prefill":
                        w = w.half().double()  # the path multiplies the rounded weights
                    parts.append(w if op == "decompress" else x @ w.T)
                out[n].append(torch.cat(parts, 0 if op == "decompress" else -1))
                n += 1
    return [o[0] for o in out] if op == "decompress" else [torch.stack(o) for o in out]

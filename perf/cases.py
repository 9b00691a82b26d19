"""The work whose speed is looked after: whole communication rounds of the algorithms this library serves, called the
way a training loop calls them, from one cache-resident bucket up to BERT-large-sized gradients of 16 workers.

A case is one round of one algorithm ("kind"):

  round     C_LP_S on one bucket per worker: compress on every worker, server step, decode fused into the optimizer step.
            codec "minmax" = QSGD-style gradients + momentum SGD, codec "sign" = compression stage of 1-bit Adam.
  buckets   C_LP_S over many separate buckets through the batched, prepared calls; optionally with the flatten in front.
  gather    C_LP_S with the gather from the layer tensors fused into the compression, and the decode fused into the scatter.
  hier      hierarchical C_LP_S: intra-node average + leader's compression per node, server step, decode.
  topk      C_LP_S with per-chunk top-K, ending in the optimizer step.
  ring_fp   D_FP_S on the ring: every peer's replica averaged with its two neighbours.
  ring_lp   D_LP_S on the ring (compressed differences), all peers at once.
  peers     averaging with one randomly chosen peer per worker, low precision (D_LP_S) or full precision (D_FP_S).
  share     one peer's share of D_LP_S: encode its own difference, apply the neighbours' codes, mix.

All results are defined bit for bit (one rounding per operation in a fixed order), so every case is compared exactly.
"""
import math
import random

import torch

import paper_2107_01499_amd as bg

MINMAX, SIGN = bg.CODEC_MINMAX_U8, bg.CODEC_SIGN1
BUCKET = 6553600            # fp32 elements of a 25 MiB bucket
LARGEST = 75e9              # bytes: no drawn case needs more than the largest listed one


def listed():
    return [
        # the smallest round: one instance of a 4 MiB bucket on four workers; launches and host calls count
        dict(name="qsgd_bucket_1m", kind="round", codec="minmax", k=4, n=1048576, chunk=4096),
        # one 25 MiB bucket per worker in the compression stage of 1-bit Adam
        dict(name="onebit_adam_25mib", kind="round", codec="sign", k=8, n=BUCKET, chunk=2048),
        # ResNet-50-sized gradients, eight workers, five separate buckets each, flatten in front
        dict(name="qsgd_resnet50_buckets", kind="buckets", codec="minmax", k=8, n=25557032, buckets=5, chunk=4096, flatten=True, odd=False),
        # a large model's gradients in 57 separate 25 MiB buckets per worker, sign codec
        dict(name="onebit_57_buckets", kind="buckets", codec="sign", k=8, n=57 * BUCKET, buckets=57, chunk=2048, flatten=False, odd=False),
        # BERT-large-sized gradients of 16 workers, gathered straight from the layer tensors; the largest case
        dict(name="qsgd_bert_large_gather", kind="gather", codec="minmax", k=16, n=335141888, chunk=8192, odd=False),
        # two nodes of four workers each, ResNet-50-sized, last chunk cut short
        dict(name="hier_sign_resnet50", kind="hier", codec="sign", k=2, local=4, n=25557032, chunk=2048),
        # aggressive compression of ResNet-50-sized gradients: 1 entry in 32
        dict(name="topk_resnet50", kind="topk", k=8, n=25657344, chunk=4096, keep=128, opt="sgd"),
        # eight peers on a ring with BERT-base-sized replicas, full and low precision
        dict(name="ring_fp_bert_base", kind="ring_fp", k=8, n=109482240),
        dict(name="ring_lp_bert_base", kind="ring_lp", k=8, n=109482240, chunk=4096),
        # more peers and longer chunks than the ring above, odd length
        dict(name="ring_lp_16_peers", kind="ring_lp", k=16, n=25557031, chunk=8192),
        # random gossip with an odd number of workers: three pairs and one that sits the round out
        dict(name="peers_lp_7_workers", kind="peers", k=7, n=25557032, chunk=4096, lp=True),
        # what one GPU does per bucket when every peer has a GPU of its own; odd length
        dict(name="ring_share_25mib", kind="share", n=BUCKET - 1, chunk=4096),
    ]


def draw(rng):
    """One more case of the same ranges: any kind, sizes spread over their logarithm, odd ones among them."""
    while True:
        kind = rng.choice(["round", "buckets", "gather", "hier", "topk", "ring_fp", "ring_lp", "peers", "share"])
        n = int(2.0 ** rng.uniform(16.0, 27.0))
        n = rng.choice([n, n | 1, n // 256 * 256])
        chunk = rng.choice([1024, 2048, 2048, 4096, 4096, 4096, 8192, 8192, 16384, 1536, 3072])
        codec = rng.choice(["minmax", "sign"])
        k = rng.choice([2, 3, 4, 5, 7, 8, 8, 12, 16])
        case = dict(kind=kind, k=k, n=n, chunk=chunk)
        if kind == "round":
            case.update(codec=codec)
        elif kind == "buckets":
            case.update(codec=codec, buckets=min(64, max(2, n // rng.choice([BUCKET, BUCKET // 4, BUCKET // 16]))),
                        flatten=rng.random() < 0.5, odd=rng.random() < 0.3)
        elif kind == "gather":
            case.update(codec=codec, odd=rng.random() < 0.3)
        elif kind == "hier":
            case.update(codec=codec, k=rng.choice([1, 2, 4]), local=rng.choice([2, 4, 8]))
        elif kind == "topk":
            case.update(keep=max(1, chunk // rng.choice([8, 16, 32, 32, 64, 100, 128])), opt=rng.choice(["sgd", "adam"]))
        elif kind == "ring_fp":
            del case["chunk"]
        elif kind == "peers":
            case.update(lp=rng.random() < 0.6)
        elif kind == "share":
            del case["k"]
        if work(case)["bytes"] <= LARGEST:
            return case


# ---------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(n, g, sigma):
    return torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=g)


def _zeros(n, dtype=torch.float32):
    return torch.zeros(n, dtype=dtype, device="cuda")


def _tensor_sizes(n, seed, odd):
    """Sizes of a model's layer tensors that sum to n: matrices of very different sizes, each with two short vectors."""
    rng, sizes, left = random.Random(seed), [], n
    while left > 0:
        big = int(2.0 ** rng.uniform(11.0, 22.0))
        for s in (big if odd else big // 64 * 64, *(2 * [rng.choice([64, 128, 256, 512, 768, 1024, 2048]) + (rng.choice([0, 1, 3]) if odd else 0)])):
            if left > 0:
                sizes.append(min(s, left))
                left -= sizes[-1]
    return sizes


def _layers(sizes, g, sigmas):
    """Gradient tensors of those sizes, each starting at its own 512-byte boundary as the allocator places them; with
    the storage behind them."""
    starts, at = [], 0
    for s in sizes:
        starts.append(at)
        at += (s + 127) // 128 * 128
    flat = _normal(at, g, 1.0)
    layers = [flat[a:a + s] for a, s in zip(starts, sizes)]
    for t, sigma in zip(layers, sigmas):
        t.mul_(sigma)
    return layers, flat


def _sigmas(count, seed):
    rng = random.Random(seed)
    return [10.0 ** rng.uniform(-5.0, -2.0) for _ in range(count)]


def _code_words(codec, n):
    return (n, torch.uint8) if codec == MINMAX else ((n + 31) // 32, torch.int32)


def _coded(codec, n, chunk):
    """Room for one compressed bucket: codes and per-chunk metadata."""
    words, dtype = _code_words(codec, n)
    return _zeros(words, dtype), _zeros((2 if codec == MINMAX else 1) * bg.num_chunks(n, chunk))


def _offsets(sizes):
    offs, at = [], 0
    for s in sizes:
        offs.append(at)
        at += s
    return offs


def _plan(layers, offs, n_pad):
    ws = torch.empty(bg.bagua_flatten_workspace_bytes(len(layers), n_pad), dtype=torch.uint8, device="cuda")
    bg.bagua_flatten_plan(layers, offs, n_pad, ws)
    return ws


def _pad(n, quantum):
    return (n + quantum - 1) // quantum * quantum


def _codec(case):
    return MINMAX if case["codec"] == "minmax" else SIGN


class _Arena:
    """Buckets that lie apart in one worker's storage (64 elements between them), with the storage as the output."""

    def __init__(self, sizes, dtype=torch.float32):
        starts, at = [], 0
        for s in sizes:
            starts.append(at)
            at += (s + 127) // 64 * 64
        self.flat = _zeros(at, dtype)
        self.parts = [self.flat[a:a + s] for a, s in zip(starts, sizes)]


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, _gen(seed), seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


# ---------------------------------------------------------------------------------------------- round
def _prepare_round(case, g, seed):
    k, n, C, codec = case["k"], case["n"], case["chunk"], _codec(case)
    s = dict(kind="round", codec=codec, n=n, C=C, x=[_normal(n, g, 1e-3) for _ in range(k)],
             res=[_normal(n, g, 1e-5) for _ in range(k)], eps=_normal(n, g, 1e-6),
             wire=[_coded(codec, n, C) for _ in range(k)], back=_coded(codec, n, C),
             param=_normal(n, g, 0.02), m=_normal(n, g, 1e-3))
    if codec == SIGN:
        s["v"] = _normal(n, g, 1e-3).square_().add_(1e-8)
    return s


def _run_round(s):
    codec, n, C = s["codec"], s["n"], s["C"]
    for x, r, (codes, meta) in zip(s["x"], s["res"], s["wire"]):
        if codec == MINMAX:
            bg.bagua_compress_minmax_u8(x, r, C, codes, meta)
        else:
            bg.bagua_momentum_sign_compress_ef(x, s["m"], 0.9, r, C, codes, meta)
    codes, meta = s["back"]
    bg.bagua_decompress_reduce_recompress(codec, [w[0] for w in s["wire"]], [w[1] for w in s["wire"]], s["eps"], n, C, codes, meta)
    if codec == MINMAX:
        bg.bagua_decompress_sgd_step(codec, codes, meta, n, C, s["param"], s["m"], 1e-3, momentum=0.9, weight_decay=1e-4)
    else:
        bg.bagua_decompress_adam_step(codec, codes, meta, n, C, s["param"], s["m"], s["v"], 1e-4, variance_frozen=True)
    return s["res"], s["wire"], s["back"], s["eps"], s["param"], s["m"]


# ---------------------------------------------------------------------------------------------- buckets
def _bucket_sizes(case):
    """Payload and padded length of each bucket: nearly equal shares of n; a flattened bucket is padded to whole
    chunks on every server partition, an unpadded one ends in a short chunk."""
    n, B, quantum = case["n"], case["buckets"], case["k"] * case["chunk"]
    pay = [n // B + (1 if b < n % B else 0) for b in range(B)]
    return pay, [_pad(p, quantum) if case["flatten"] else p for p in pay]


def _prepare_buckets(case, g, seed):
    k, C, B, codec = case["k"], case["chunk"], case["buckets"], _codec(case)
    pay, ns = _bucket_sizes(case)
    words, dtype = [_code_words(codec, n)[0] for n in ns], _code_words(codec, 1)[1]
    metas = [(2 if codec == MINMAX else 1) * bg.num_chunks(n, C) for n in ns]
    s = dict(kind="buckets", keep=[], calls=[], x=[], res=[], codes=[], meta=[], flat=case["flatten"])

    def workspace(workers=0):
        return torch.empty(bg.bagua_batch_workspace_bytes(B, workers), dtype=torch.uint8, device="cuda")

    compress = bg.bagua_compress_minmax_u8_batched if codec == MINMAX else bg.bagua_sign_compress_ef_batched
    for j in range(k):
        x, res, codes, meta = _Arena(ns), _Arena(ns), _Arena(words, dtype), _Arena(metas)
        res.flat.normal_(0.0, 1e-5, generator=g)
        if case["flatten"]:
            plans, Ts = [], []
            for b in range(B):
                sizes = _tensor_sizes(pay[b], b, case["odd"])
                layers, storage = _layers(sizes, g, _sigmas(len(sizes), b))
                plans.append(_plan(layers, _offsets(sizes), ns[b]))
                Ts.append(len(sizes))
                s["keep"].append(storage)
            s["calls"].append(bg.bagua_bucket_flatten_batched_run(plans, Ts, x.parts, workspace(), prepare=True))
        else:
            x.flat.normal_(0.0, 1e-3, generator=g)
        s["calls"].append(compress(x.parts, res.parts, C, codes.parts, meta.parts, workspace(), prepare=True))
        for name, a in (("x", x), ("res", res), ("codes", codes), ("meta", meta)):
            s[name].append(a)
    s["eps"], s["out"], s["back"], s["back_meta"] = _Arena(ns), _Arena(ns), _Arena(words, dtype), _Arena(metas)
    s["eps"].flat.normal_(0.0, 1e-6, generator=g)
    s["calls"].append(bg.bagua_decompress_reduce_recompress_batched(
        codec, [[a.parts[b] for a in s["codes"]] for b in range(B)], [[a.parts[b] for a in s["meta"]] for b in range(B)],
        s["eps"].parts, ns, C, s["back"].parts, s["back_meta"].parts, s["out"].parts, workspace(k), prepare=True))
    return s


def _run_buckets(s):
    for call in s["calls"]:
        call()
    flat = [a.flat for a in s["x"]] if s["flat"] and len(s["x"]) <= 14 else None      # at most 64 outputs
    return (flat, *([a.flat for a in s[name]] for name in ("res", "codes", "meta")),
            *(s[name].flat for name in ("back", "back_meta", "eps", "out")))


# ---------------------------------------------------------------------------------------------- gather
def _prepare_gather(case, g, seed):
    k, C, codec = case["k"], case["chunk"], _codec(case)
    n = _pad(case["n"], k * C)
    sizes = _tensor_sizes(case["n"], 1, case["odd"])
    sigmas, offs = _sigmas(len(sizes), 1), _offsets(sizes)
    s = dict(kind="gather", codec=codec, n=n, C=C, T=len(sizes), keep=[], plans=[],
             res=[_normal(n, g, 1e-5) for _ in range(k)], eps=_normal(n, g, 1e-6),
             wire=[_coded(codec, n, C) for _ in range(k)], back=_coded(codec, n, C))
    for _ in range(k):
        layers, storage = _layers(sizes, g, sigmas)
        s["plans"].append(_plan(layers, offs, n))
        s["keep"].append(storage)
    layers, s["grads"] = _layers(sizes, g, sigmas)       # the tensors the averaged gradient is scattered to
    s["scatter"] = _plan(layers, offs, n)
    return s


def _run_gather(s):
    codec, n, C, T = s["codec"], s["n"], s["C"], s["T"]
    compress = bg.bagua_flatten_compress_minmax_u8 if codec == MINMAX else bg.bagua_flatten_sign_compress_ef
    for plan, r, (codes, meta) in zip(s["plans"], s["res"], s["wire"]):
        compress(plan, T, r, n, C, codes, meta)
    codes, meta = s["back"]
    bg.bagua_decompress_reduce_recompress(codec, [w[0] for w in s["wire"]], [w[1] for w in s["wire"]], s["eps"], n, C, codes, meta)
    bg.bagua_decompress_unflatten(codec, codes, meta, n, C, s["scatter"], T)
    return s["res"], s["wire"], s["back"], s["eps"], s["grads"]


# ---------------------------------------------------------------------------------------------- hier
def _prepare_hier(case, g, seed):
    k, n, C, codec = case["k"], case["n"], case["chunk"], _codec(case)
    return dict(kind="hier", codec=codec, n=n, C=C, x=[[_normal(n, g, 1e-3) for _ in range(case["local"])] for _ in range(k)],
                res=[_normal(n, g, 1e-5) for _ in range(k)], eps=_normal(n, g, 1e-6),
                wire=[_coded(codec, n, C) for _ in range(k)], back=_coded(codec, n, C), out=_zeros(n))


def _run_hier(s):
    codec, n, C = s["codec"], s["n"], s["C"]
    compress = bg.bagua_reduce_compress_minmax_u8 if codec == MINMAX else bg.bagua_reduce_compress_sign_ef
    for xs, r, (codes, meta) in zip(s["x"], s["res"], s["wire"]):
        compress(xs, r, C, codes, meta)
    codes, meta = s["back"]
    bg.bagua_decompress_reduce_recompress(codec, [w[0] for w in s["wire"]], [w[1] for w in s["wire"]], s["eps"], n, C, codes, meta)
    bg.bagua_decompress(codec, codes, meta, n, C, s["out"])
    return s["res"], s["wire"], s["back"], s["eps"], s["out"]


# ---------------------------------------------------------------------------------------------- topk
def _prepare_topk(case, g, seed):
    k, n, C, keep = case["k"], case["n"], case["chunk"], case["keep"]
    slots = bg.num_chunks(n, C) * keep

    def entries():
        return _zeros(slots, torch.int16), _zeros(slots)

    s = dict(kind="topk", n=n, C=C, K=keep, opt=case["opt"], x=[_normal(n, g, 1e-3) for _ in range(k)],
             res=[_normal(n, g, 1e-3) for _ in range(k)], eps=_normal(n, g, 1e-4), wire=[entries() for _ in range(k)],
             back=entries(), param=_normal(n, g, 0.02), m=_normal(n, g, 1e-3))
    if case["opt"] == "adam":
        s["v"] = _normal(n, g, 1e-3).square_().add_(1e-8)
    return s


def _run_topk(s):
    n, C, K = s["n"], s["C"], s["K"]
    for x, r, (idx, val) in zip(s["x"], s["res"], s["wire"]):
        bg.bagua_compress_topk_ef(x, r, C, K, idx, val)
    idx, val = s["back"]
    bg.bagua_decompress_reduce_recompress_topk([w[0] for w in s["wire"]], [w[1] for w in s["wire"]], K, s["eps"], n, C, idx, val)
    if s["opt"] == "sgd":
        bg.bagua_decompress_sgd_step_topk(idx, val, n, C, K, s["param"], s["m"], 1e-3, momentum=0.9)
    else:
        bg.bagua_decompress_adam_step_topk(idx, val, n, C, K, s["param"], s["m"], s["v"], 1e-4)
    return s["res"], s["wire"], s["back"], s["eps"], s["param"], s["m"], s.get("v")


# ---------------------------------------------------------------------------------------------- decentralised
def _replicas(k, n, g):
    base = _normal(n, g, 0.02)
    return [base + _normal(n, g, 1e-3) for _ in range(k)]


def _prepare_ring_fp(case, g, seed):
    return dict(kind="ring_fp", x=_replicas(case["k"], case["n"], g), out=[_zeros(case["n"]) for _ in range(case["k"])])


def _run_ring_fp(s):
    bg.bagua_decentralized_avg(bg.AVG_FP, s["x"], s["out"])
    return s["out"]


def _prepare_ring_lp(case, g, seed):
    # The replicas of two consecutive iterations, taken in turn: between two rounds every replica has moved by its own
    # gradient step, so there is always a difference to publish.
    k, n, C = case["k"], case["n"], case["chunk"]
    x = _replicas(k, n, g)
    return dict(kind="ring_lp", C=C, x=[x, [t + _normal(n, g, 1e-3) for t in x]], turn=0, hat=[t + _normal(n, g, 1e-4) for t in x],
                out=[_zeros(n) for _ in range(k)], wire=[_coded(MINMAX, n, C) for _ in range(k)])


def _run_ring_lp(s):
    x, s["turn"] = s["x"][s["turn"]], 1 - s["turn"]
    bg.bagua_decentralized_avg(bg.AVG_LP_MINMAX_U8, x, s["out"], s["hat"], [w[0] for w in s["wire"]], [w[1] for w in s["wire"]], s["C"])
    return s["out"], s["hat"], s["wire"]


def _prepare_peers(case, g, seed):
    k = case["k"]
    order = list(range(k))
    random.Random(k).shuffle(order)
    peer = list(range(k))                                  # the last one of an odd number keeps its replica
    for a, b in zip(order[0::2], order[1::2]):
        peer[a], peer[b] = b, a
    s = _prepare_ring_lp(case, g, seed) if case["lp"] else _prepare_ring_fp(case, g, seed)
    return dict(s, kind="peers", peer=peer)


def _run_peers(s):
    if "hat" not in s:
        bg.bagua_decentralized_avg_peers(s["x"], s["out"], s["peer"])
        return s["out"]
    x, s["turn"] = s["x"][s["turn"]], 1 - s["turn"]
    bg.bagua_decentralized_avg_peers_lp(x, s["out"], s["hat"], [w[0] for w in s["wire"]], [w[1] for w in s["wire"]], s["peer"], s["C"])
    return s["out"], s["hat"], s["wire"]


def _prepare_share(case, g, seed):
    n, C = case["n"], case["chunk"]
    s = _prepare_ring_lp(dict(k=3, n=n, chunk=C), g, seed)
    own, left, right = s["hat"]
    for j in (0, 2):                                       # what the two neighbours sent this round
        bg.bagua_lp_encode(s["x"][1][j], s["hat"][j].clone(), C, *s["wire"][j])
    return dict(kind="share", C=C, x=[s["x"][0][1], s["x"][1][1]], turn=0, own=own, left=left, right=right, out=s["out"][0],
                wire=s["wire"][1], from_left=s["wire"][0], from_right=s["wire"][2])


def _run_share(s):
    x, s["turn"] = s["x"][s["turn"]], 1 - s["turn"]
    codes, meta = s["wire"]
    bg.bagua_lp_encode(x, s["own"], s["C"], codes, meta)
    bg.bagua_lp_apply_mix(x, s["own"], s["left"], s["right"], *s["from_left"], *s["from_right"], s["C"], s["out"])
    return s["out"], s["own"], s["left"], s["right"], s["wire"]


# ---------------------------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes: every call's inputs read once and its outputs written once.  Operations: the arithmetic of the codec per
    element (statistics, quantisation, error state) and the sums."""
    kind, n, k, C = case["kind"], case["n"], case.get("k", 1), case.get("chunk", 4096)
    nc = math.ceil(n / C)
    minmax = case.get("codec", "minmax") == "minmax"
    wire = n + 8 * nc if minmax else n / 8 + 4 * nc
    if kind == "round":
        b = k * ((12 if minmax else 16) * n + wire) + (k + 1) * wire + 8 * n + wire + (16 if minmax else 16) * n
        f = n * (k * 14 + 8)
    elif kind == "buckets":
        pads = sum(_bucket_sizes(case)[1])
        wire = wire * pads / n
        b = k * ((4 * (n + pads) if case["flatten"] else 0) + 12 * pads + wire) + (k + 1) * wire + 12 * pads
        f = pads * k * 14
    elif kind == "gather":
        pad = _pad(n, k * C)
        wire = wire * pad / n
        b = k * (4 * n + 8 * pad + wire) + (k + 1) * wire + 8 * pad + wire + 4 * n
        f = pad * k * 14
    elif kind == "hier":
        b = k * (4 * n * case["local"] + 8 * n + wire) + (k + 1) * wire + 8 * n + wire + 4 * n
        f = n * k * (case["local"] + 14)
    elif kind == "topk":
        wire = 6 * nc * case["keep"]
        b = k * (12 * n + wire) + (k + 1) * wire + 8 * n + wire + (16 if case["opt"] == "sgd" else 24) * n
        f = n * (k * 4 + 8)
    elif kind in ("ring_fp", "peers") and not case.get("lp"):
        b, f = 8 * n * k, 3 * n * k
    elif kind in ("ring_lp", "peers"):
        b, f = k * (16 * n + wire), 16 * n * k
    else:                                                  # share: encode (x, own copy in and out), then apply and mix
        b, f = 12 * n + wire + 28 * n + 2 * wire, 28 * n
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """Results are defined bit for bit: one rounding per operation in a fixed order."""
    return "exact"

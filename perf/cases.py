"""Timed cases of the top-k library: the calls its users make, over the sizes, key types and
orders they make them with.  Each case goes through the package's public entry points with
device-resident keys, as a program that ranks scores does.

A case is a dict:
  op       "topk" (sorted values and positions), "kth" (k-th value alone), "payload" (top-k with
           the payload of each selected key) or "batch" (many independent problems in one call)
  n, k     problem size (batch: lo, hi bound the log-uniform lengths, k <= kmax, count problems)
  dtype    key type; dist: "uniform" over the type's range, "normal", "ties" (uniform over 16
           values) or "sorted" (ascending normal)
  largest  False: the k smallest;  offset: elements skipped at the head of the keys' buffer
"""
import math
import random

import torch

import paper_2109_08219_amd as drt

_TORCH = {"u32": torch.int32, "i32": torch.int32, "f32": torch.float32,
          "u64": torch.int64, "i64": torch.int64, "f64": torch.float64}
_BYTES = {"u32": 4, "i32": 4, "f32": 4, "u64": 8, "i64": 8, "f64": 8}


def _case(name, op, n, k, dtype, dist, largest=True, offset=0):
    return {"name": name, "op": op, "n": n, "k": k, "dtype": dtype, "dist": dist, "largest": largest, "offset": offset}


def listed():
    return [
        # the ten best of a short candidate list: the smallest call, launch and host latency
        _case("rerank_1k", "topk", 1000, 10, "f32", "normal"),
        # best scores of one row of logits or of one shard's candidates
        _case("row_50k", "topk", 50_000, 64, "f32", "normal"),
        # the single-call latency configuration
        _case("u32_2p20", "topk", 1 << 20, 1024, "u32", "uniform"),
        # nearest neighbours: the smallest distances of a few million, an odd count
        _case("knn_3m", "topk", 3_000_001, 100, "f32", "normal", largest=False),
        # records ranked by score: keys with an 8-byte payload each
        _case("payload_2p25", "payload", (1 << 25) + 7, 10_000, "f32", "normal"),
        # keep the top eighth (sparsified updates): k a fixed share of n
        _case("top_eighth_2p24", "topk", 1 << 24, 1 << 21, "f32", "normal"),
        # the median of an odd count of integers
        _case("median_2p24", "kth", (1 << 24) + 3, (1 << 23) + 2, "i32", "uniform"),
        # 64-bit keys with a large k
        _case("f64_2p28", "topk", 1 << 28, 131_072, "f64", "normal"),
        # degrees or small counts: nearly every key tied
        _case("ties_2p29", "topk", 1 << 29, 16_384, "u32", "ties"),
        # the headline size, at its middle and its largest k
        _case("u32_2p30", "topk", 1 << 30, 1024, "u32", "uniform"),
        _case("f32_2p30_k128k", "topk", 1 << 30, 131_072, "f32", "normal"),
        # thousands of queries' candidate lists of uneven lengths, ranked in one call
        {"name": "batch_4096", "op": "batch", "count": 4096, "lo": 1 << 10, "hi": 1 << 20, "kmax": 2048,
         "largest": True, "layout": 1},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choices(["topk", "kth", "payload", "share", "wide", "batch"], [8, 2, 2, 2, 3, 3])[0]
    largest = rng.random() < 0.7
    if kind == "batch":
        count = _log_int(rng, 2, 4096)
        lo = _log_int(rng, 64, 1 << 12)
        hi = _log_int(rng, lo * 4, 1 << 20)
        return {"op": "batch", "count": count, "lo": lo, "hi": hi, "kmax": _log_int(rng, 8, 2048), "largest": largest,
                "layout": rng.randrange(1 << 20)}
    dtype = rng.choice(["f64", "i64", "u64"] if kind == "wide" else ["u32", "f32", "f32", "i32"])
    dists = ["uniform", "uniform", "normal", "ties"] if dtype[0] != "f" else ["normal", "normal", "normal", "sorted"]
    dist = rng.choice(dists)
    if kind == "share":  # k a fixed share of n
        n = _log_int(rng, 1 << 14, 1 << 24)
        k = max(1, int(n * rng.uniform(0.07, 0.13)))
        return {k_: v for k_, v in _case("", "topk", n, k, dtype, rng.choice(dists[:3]), largest).items() if k_ != "name"}
    hi = (1 << 27) if dtype in ("f64", "i64", "u64") else (1 << 28) if dist in ("ties", "sorted") else (1 << 29)
    if kind == "payload":
        hi = 1 << 27
    n = _log_int(rng, 256, hi)
    k = _log_int(rng, 1, max(1, min(n // 16, 131_072)))
    if kind == "kth" and rng.random() < 0.4:  # a quantile
        n = min(n, 1 << 24)
        k = max(1, int(n * rng.uniform(0.25, 0.75)))
    op = kind if kind in ("kth", "payload") else "topk"
    offset = rng.choice([0, 0, 0, 1, 2]) if dtype in ("u32", "f32", "i32") else 0
    return {k_: v for k_, v in _case("", op, n, k, dtype, dist, largest, offset).items() if k_ != "name"}


def _keys(n, dtype, dist, gen):
    t = _TORCH[dtype]
    if dist == "ties":
        return torch.randint(0, 16, (n,), dtype=t, device="cuda", generator=gen)
    if t.is_floating_point:
        x = torch.randn(n, dtype=t, device="cuda", generator=gen)
        return x.sort().values if dist == "sorted" else x
    if dist == "normal":  # integer scores around a large mean
        return (torch.randn(n, device="cuda", generator=gen) * 1e5 + 1e8).to(t)
    if t == torch.int32:
        return torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=t, device="cuda", generator=gen)
    return torch.randint(-2 ** 63, 2 ** 63 - 1, (n,), dtype=t, device="cuda", generator=gen)


def _lists(case):
    """(kind, n, k) of each problem of a batch, from the case alone."""
    rng = random.Random(case["layout"])
    out = []
    for _ in range(case["count"]):
        n = _log_int(rng, case["lo"], case["hi"])
        out.append((rng.choice(["u32", "f32"]), n, 1 + int(rng.random() * min(n, case["kmax"]))))
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "batch":
        lists = _lists(case)
        flat, at = {}, {"u32": 0, "f32": 0}
        for kind in at:  # every list starts at a 256-byte boundary of its type's buffer
            flat[kind] = _keys(sum(-(-n // 64) * 64 for t, n, _ in lists if t == kind) + 64, kind,
                               "uniform" if kind == "u32" else "normal", gen)
        problems = []
        for kind, n, k in lists:
            problems.append((flat[kind][at[kind]:at[kind] + n], k, kind, case["largest"]))
            at[kind] += -(-n // 64) * 64
        return {"case": case, "batch": drt.Batch(problems)}
    off = case["offset"]
    state = {"case": case, "keys": _keys(case["n"] + off, case["dtype"], case["dist"], gen)[off:]}
    if case["op"] == "payload":
        state["payload"] = torch.randint(0, 2 ** 62, (case["n"],), dtype=torch.int64, device="cuda", generator=gen)
    return state


def run(state):
    case = state["case"]
    if case["op"] == "batch":
        b = state["batch"]
        b.run()
        return b.vals, b.idx, b.kth[::2]
    args = {"dtype": case["dtype"], "largest": case["largest"]}
    if case["op"] == "kth":
        return drt.kth_select(state["keys"], case["k"], **args)
    if case["op"] == "payload":
        return drt.topk_select_payload(state["keys"], state["payload"], case["k"], **args)
    return drt.topk_select(state["keys"], case["k"], **args)


def work(case):
    """Every key read once, every output written once; one comparison a key."""
    if case["op"] == "batch":
        lists = _lists(case)
        n, k = sum(n for _, n, _ in lists), sum(k for _, _, k in lists)
        return {"bytes": 4 * n + 8 * k + 4 * len(lists), "flops": n}
    n, k, w = case["n"], case["k"], _BYTES[case["dtype"]]
    out = {"topk": (w + 4) * k, "kth": w, "payload": (w + 4 + 16) * k}[case["op"]]  # a payload is read and written
    return {"bytes": w * n + out, "flops": n}


def exact(case, seed):
    if case["op"] == "batch":
        return None  # bit patterns and positions only
    state = prepare(case, seed)
    x, k, dtype = state["keys"], case["k"], case["dtype"]
    if dtype == "u32":
        key = x.long() & 0xFFFFFFFF
    elif dtype == "u64":
        key = x ^ (-2 ** 63)
    else:
        key = x.double() if x.is_floating_point() else x.long()
    if not case["largest"]:
        key = -key if x.is_floating_point() else ~key
    if k * 64 > case["n"]:  # in position order, a stable sort ranks ties by position
        pos = torch.arange(case["n"], device=x.device)
    else:
        pos = (key >= torch.topk(key, k).values[-1]).nonzero().flatten()
    order = key[pos].sort(descending=True, stable=True).indices[:k]
    idx = pos[order]
    vals = x[idx].double() if x.is_floating_point() else x[idx].long()
    if case["op"] == "kth":
        return vals[-1:]
    if case["op"] == "payload":
        return vals, idx, state["payload"][idx]
    return vals, idx

"""Workloads of the EmbeddingBag step for performance measurement.

A case is a dict of plain values:
  op       "step" (forward, then backward + SGD), "forward" or "backward"
  storage  "fp32", "split" (BF16 high and 16-bit low halves, FP32 activations)
           or "split_act" (the same with BF16 pooled outputs and gradients)
  pooling  "sum", "weighted" (a weight per look-up) or "mean"; the latter two
           with FP32 tables
  call     how the backward is called: "fused" (one call with a workspace),
           "phases" (prepare, then apply) or "noalloc"
  tables, rows_lo, rows_hi   table t of T has the middle of the t-th of T equal
           steps from rows_lo to rows_hi on a logarithmic scale as its rows
  dim, batch                 row width, bags per table
  bag, ragged                look-ups per bag; ragged bags have 1 .. 2*bag - 1,
           and a tenth of them none
  zipf     exponent of the look-ups' distribution over the rows (0: uniform);
           the ranks are spread over the rows by an affine bijection

All tables of a state lie in one buffer, table after table.
"""
import math
import random

import torch

import paper_2005_04680_amd as pk

LR = 0.1
_DEV = "cuda"
_PIECE = 1 << 20  # look-ups or rows that exact() and the fills take at a time


def _case(name, op, storage, pooling, call, tables, rows_lo, rows_hi, dim, batch, bag, ragged,
          zipf):
    return {"name": name, "op": op, "storage": storage, "pooling": pooling, "call": call,
            "tables": tables, "rows_lo": rows_lo, "rows_hi": rows_hi, "dim": dim, "batch": batch,
            "bag": bag, "ragged": ragged, "zipf": zipf}


def listed():
    return [
        # The smallest training step: launches and host calls are all there is to it.
        _case("tiny_step", "step", "fp32", "sum", "fused", 4, 1000, 1000, 16, 32, 4, False, 0.0),
        # Serving: the forward of a few requests on the Small tables, lists of any length.
        _case("serve_forward", "forward", "fp32", "sum", "fused", 8, 1_000_000, 1_000_000, 64, 64,
              32, True, 1.05),
        # The Small workload's training step.
        _case("small_step", "step", "fp32", "sum", "fused", 8, 1_000_000, 1_000_000, 64, 2048, 32,
              False, 1.05),
        # The paper's own Small shape: 50 uniform look-ups, hardly a row named twice.
        _case("small_p50_uniform", "step", "fp32", "sum", "phases", 8, 1_000_000, 1_000_000, 64,
              2048, 50, False, 0.0),
        # Split-SGD-BF16 training with BF16 activations on the Small tables.
        _case("small_split_act", "step", "split_act", "sum", "fused", 8, 1_000_000, 1_000_000, 64,
              2048, 32, False, 1.05),
        # A captured or allocation-free training loop at a small batch.
        _case("noalloc_step", "step", "fp32", "sum", "noalloc", 8, 1_000_000, 1_000_000, 64, 256,
              32, True, 1.05),
        # Criteo-like tables (one look-up each, any size) at an ordinary minibatch, split storage.
        _case("mlperf_b2048_split", "step", "split", "sum", "fused", 26, 10, 20_000_000, 128, 2048,
              1, False, 1.2),
        # The same tables at the large batch of the MLPerf configuration, FP32.
        _case("mlperf_step", "step", "fp32", "sum", "phases", 26, 10, 20_000_000, 128, 65536, 1,
              False, 1.2),
        # Weighted lists of any length (scores per look-up), a row width that is no power of two.
        _case("weighted_ragged", "step", "fp32", "weighted", "fused", 5, 30_000, 3_000_000, 100,
              3001, 40, True, 1.05),
        # Mean pooling of wide rows (text-like features), ragged lists.
        _case("mean_wide", "step", "fp32", "mean", "fused", 3, 100_000, 400_000, 512, 1500, 20,
              True, 1.05),
        # The Large workload with tables a quarter as long: the bandwidth-bound training step.
        _case("large_step", "step", "fp32", "sum", "phases", 16, 1_500_000, 1_500_000, 256, 8192,
              100, False, 1.05),
        # The same in Split-SGD-BF16 storage with FP32 activations.
        _case("large_split", "step", "split", "sum", "phases", 16, 1_500_000, 1_500_000, 256, 8192,
              100, False, 1.05),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    while True:
        op = rng.choice(["step"] * 6 + ["forward"] * 2 + ["backward"])
        storage = rng.choice(["fp32"] * 3 + ["split", "split_act"])
        pooling = rng.choice(["sum"] * 3 + ["weighted", "mean"]) if storage == "fp32" else "sum"
        call = rng.choice(["fused", "phases"])
        if storage == "fp32" and pooling == "sum" and rng.random() < 0.15:
            call = "noalloc"
        T = _log_int(rng, 1, 64)
        lo = _log_int(rng, 10, 1_000_000)
        hi = max(lo, _log_int(rng, 1000, 20_000_000))
        E = 4 * _log_int(rng, 1, 128) if rng.random() < 0.5 else rng.choice([16, 32, 64, 128, 256])
        B = _log_int(rng, 16, 65536)
        P = _log_int(rng, 1, 100)
        c = _case("", op, storage, pooling, call, T, lo, hi, E, B, P, rng.random() < 0.5,
                  rng.choice([0.0, 0.8, 1.05, 1.05, 1.2]))
        del c["name"]
        ns = T * B * P
        if not 512 <= ns <= 8_000_000 or (call == "noalloc" and ns > 400_000):
            continue
        if ns * E > 1_500_000_000 or T * B * E * 4 > 900_000_000 or sum(_rows(c)) * E * 4 > 16e9:
            continue
        return c


def _rows(c):
    lo, hi, T = c["rows_lo"], c["rows_hi"], c["tables"]
    return [max(1, int(lo * (hi / lo) ** ((t + 0.5) / T))) for t in range(T)]


def _pmf(m, s):
    """Probability of the ranks 1 .. m (64 bits)."""
    p = torch.arange(1, m + 1, dtype=torch.float64, device=_DEV).pow_(-s)
    return p.div_(p.sum())


class State:
    pass


def _inputs(c, seed):
    """Tables (one FP32 buffer), look-ups, offsets, weights and gradients."""
    s = State()
    g = torch.Generator(device=_DEV)
    g.manual_seed(seed)
    s.c, s.rows = c, _rows(c)
    T, B, E, P = c["tables"], c["batch"], c["dim"], c["bag"]
    s.base = [sum(s.rows[:t]) for t in range(T + 1)]
    if c["ragged"]:
        n = torch.randint(1, 2 * P, (T * B,), device=_DEV, generator=g)
        n.masked_fill_(torch.rand(T * B, device=_DEV, generator=g) < 0.1, 0)
    else:
        n = torch.full((T * B,), P, device=_DEV)
    offsets = torch.zeros(T * B + 1, dtype=torch.int64, device=_DEV)
    torch.cumsum(n, 0, out=offsets[1:])
    s.sizes = n
    s.offsets = offsets.to(torch.int32)
    ends = offsets[::B].tolist()
    s.ends = ends
    s.indices = torch.empty(ends[-1], dtype=torch.int32, device=_DEV)
    r = random.Random(12345)  # the rows that are hot are the same for every batch
    cdf = {}
    for t, m in enumerate(s.rows):
        k = ends[t + 1] - ends[t]
        u = torch.rand(k, dtype=torch.float64, device=_DEV, generator=g)
        if c["zipf"] > 0:
            if m not in cdf:
                cdf = {m: torch.cumsum(_pmf(m, c["zipf"]), 0)}
            rank = torch.searchsorted(cdf[m], u, right=True).clamp_(max=m - 1)
        else:
            rank = (u * m).long().clamp_(max=m - 1)
        a = next(x for x in iter(lambda: r.randrange(1, m + 1), None) if math.gcd(x, m) == 1)
        s.indices[ends[t]:ends[t + 1]] = (rank * a + r.randrange(m)) % m
    s.weights = None
    if c["pooling"] == "weighted":
        s.weights = torch.rand(ends[-1], device=_DEV, generator=g) + 0.5
    s.grad = None
    if c["op"] != "forward":
        s.grad = torch.randn(T, B, E, device=_DEV, generator=g)
        if c["storage"] == "split_act":
            s.grad = s.grad.to(torch.bfloat16)
    s.w = torch.empty(s.base[-1], E, device=_DEV)
    s.w.uniform_(-1.0, 1.0, generator=g)
    for t, m in enumerate(s.rows):
        s.w[s.base[t]:s.base[t + 1]].mul_(1.0 / math.sqrt(m))
    return s


def prepare(c, seed):
    s = _inputs(c, seed)
    T, B, E = c["tables"], c["batch"], c["dim"]

    def parts(x):
        return [x[s.base[t]:s.base[t + 1]] for t in range(T)]

    if c["storage"] == "fp32":
        s.tables = pk.Tables(parts(s.w))
    else:
        s.hi = torch.empty(s.w.shape, dtype=torch.bfloat16, device=_DEV)
        s.lo = torch.empty(s.w.shape, dtype=torch.int16, device=_DEV)
        for r0 in range(0, s.base[-1], _PIECE):
            b = s.w[r0:r0 + _PIECE].view(torch.int32)
            s.hi.view(torch.int16)[r0:r0 + _PIECE] = (b >> 16).to(torch.int16)
            s.lo[r0:r0 + _PIECE] = ((b << 16) >> 16).to(torch.int16)
        s.w = None
        s.tables = pk.SplitTables(parts(s.hi), parts(s.lo))
    s.status = torch.zeros(1, dtype=torch.int32, device=_DEV)
    s.out = None
    if c["op"] != "backward":
        s.out = torch.empty(T, B, E, device=_DEV,
                            dtype=torch.bfloat16 if c["storage"] == "split_act" else torch.float32)
    s.ws = None
    if c["op"] != "forward" and c["call"] != "noalloc":
        s.ws = torch.empty(pk.embbag_backward_workspace_bytes(T, B, s.ends[-1], E),
                           dtype=torch.uint8, device=_DEV)
    return s


def _forward(s):
    c, tb, B = s.c, s.tables, s.c["batch"]
    if c["storage"] == "split":
        return pk.embbag_forward_split_bf16(tb, B, s.indices, s.offsets, s.out, s.status)
    if c["storage"] == "split_act":
        return pk.embbag_forward_split_bf16_act(tb, B, s.indices, s.offsets, s.out, s.status)
    if c["pooling"] == "sum":
        return pk.embbag_forward(tb, B, s.indices, s.offsets, s.out, s.status)
    mode = pk.EMBBAG_POOL_MEAN if c["pooling"] == "mean" else pk.EMBBAG_POOL_SUM
    return pk.embbag_forward_pooled(tb, B, s.indices, s.offsets, s.out, s.weights, mode, s.status)


def _backward(s):
    c, tb, B = s.c, s.tables, s.c["batch"]
    if c["storage"] == "split":
        return pk.embbag_backward_sgd_split_bf16(s.grad, B, s.indices, s.offsets, LR, tb, None,
                                                 s.ws, s.status)
    if c["storage"] == "split_act":
        return pk.embbag_backward_sgd_split_bf16_act(s.grad, B, s.indices, s.offsets, LR, tb, None,
                                                     s.ws, s.status)
    if c["call"] == "noalloc":
        return pk.embbag_backward_sgd_noalloc(s.grad, B, s.indices, s.offsets, LR, tb, s.status)
    if c["pooling"] == "sum":
        return pk.embbag_backward_sgd(s.grad, B, s.indices, s.offsets, LR, tb, s.ws, s.status)
    mode = pk.EMBBAG_POOL_MEAN if c["pooling"] == "mean" else pk.EMBBAG_POOL_SUM
    return pk.embbag_backward_sgd_pooled(s.grad, B, s.indices, s.offsets, LR, tb, s.ws, s.weights,
                                         mode, s.status)


def _phases(s):
    c, tb, B, ns = s.c, s.tables, s.c["batch"], s.indices.numel()
    if c["pooling"] != "sum":
        mode = pk.EMBBAG_POOL_MEAN if c["pooling"] == "mean" else pk.EMBBAG_POOL_SUM
        pk.check(pk.embbag_backward_prepare_pooled(tb, c["dim"], B, s.indices, s.offsets, s.ws,
                                                   s.weights, mode, s.status))
        return pk.embbag_backward_apply_sgd_pooled(s.grad, B, s.offsets, ns, LR, tb, s.ws,
                                                   s.weights, mode)
    pk.check(pk.embbag_backward_prepare(tb, c["dim"], B, s.indices, s.offsets, s.ws, s.status))
    if c["storage"] == "split":
        return pk.embbag_backward_apply_sgd_split_bf16(s.grad, B, ns, LR, tb, None, s.ws)
    if c["storage"] == "split_act":
        return pk.embbag_backward_apply_sgd_split_bf16_act(s.grad, B, ns, LR, tb, None, s.ws)
    return pk.embbag_backward_apply_sgd(s.grad, B, ns, LR, tb, s.ws)


def run(s):
    c = s.c
    res = {"status": s.status}
    if c["op"] != "backward":
        pk.check(_forward(s))
        res["pooled"] = s.out
    if c["op"] != "forward":
        pk.check(_phases(s) if c["call"] == "phases" else _backward(s))
        if c["storage"] == "fp32":
            res["tables"] = s.w
        else:
            res["hi"], res["lo"] = s.hi, s.lo
    return res


def _touched(c):
    """Expected number of distinct rows that a batch names."""
    total, seen = 0.0, {}
    n = c["batch"] * c["bag"] * (0.9 if c["ragged"] else 1.0)
    for m in _rows(c):
        if m not in seen:
            if c["zipf"] > 0:
                miss = torch.log1p(_pmf(m, c["zipf"]).neg_().clamp_(min=-1.0 + 1e-15)).mul_(n)
                seen[m] = float(-torch.expm1(miss).sum())
            else:
                seen[m] = m * -math.expm1(n * math.log1p(-1.0 / m)) if m > 1 else 1.0
        total += seen[m]
    return total


def work(c):
    """The touched rows, the bags and their gradients, each once per call; an
    addition per element and look-up (and a product for weights)."""
    T, B, E = c["tables"], c["batch"], c["dim"]
    ns = T * B * c["bag"] * (0.9 if c["ragged"] else 1.0)
    u = _touched(c)
    lists = 4 * ns + 4 * (T * B + 1) + (4 * ns if c["pooling"] == "weighted" else 0)
    act = T * B * E * (2 if c["storage"] == "split_act" else 4)
    add = ns * E * (2 if c["pooling"] == "weighted" else 1)
    byts = flops = 0.0
    if c["op"] != "backward":
        byts += lists + act + u * E * (4 if c["storage"] == "fp32" else 2)
        flops += add
    if c["op"] != "forward":
        byts += lists + act + 2 * u * E * 4
        flops += add + 2 * u * E
    return {"bytes": byts, "flops": flops}


def tolerance(c):
    # Sums are held in 64 bits and rounded once to FP32 (3e-8 from the 64-bit
    # result); another order of them changes the last bit of a few values in
    # 1e8, and where it does, that bit may carry into a BF16 half (2^-8 of the
    # value).
    if c["storage"] == "fp32":
        return {"rel": 2e-7, "max": 2e-6}
    return {"rel": 1e-4, "max": 1e-2, "differ": 1e-4}


def exact(c, seed):
    s = _inputs(c, seed)
    T, B, E = c["tables"], c["batch"], c["dim"]
    coef = s.weights.double() if s.weights is not None else None
    if c["pooling"] == "mean":
        coef = (1.0 / s.sizes.double().clamp(min=1)).repeat_interleave(s.sizes)
    bag = torch.arange(T * B, device=_DEV).repeat_interleave(s.sizes)
    table = torch.repeat_interleave(torch.tensor(s.base[:-1], device=_DEV), torch.tensor(
        [s.ends[t + 1] - s.ends[t] for t in range(T)], device=_DEV))
    row = s.indices.long() + table
    del table
    # (status: whole numbers; lo: the low 16 bits of a weight say nothing alone)
    res = {"status": None}
    step = max(1, _PIECE * 256 // E)
    pieces = [slice(i, i + step) for i in range(0, s.ends[-1], step)]
    if c["op"] != "backward":
        read = s.w if c["storage"] == "fp32" else (s.w.view(torch.int32) & -65536).view(torch.float32)
        y = torch.zeros(T * B, E, dtype=torch.float64, device=_DEV)
        for p in pieces:
            v = read[row[p]].double()
            y.index_add_(0, bag[p], v if coef is None else v * coef[p, None])
            del v
        del read
        res["pooled"] = y.view(T, B, E)
    if c["op"] != "forward":
        w = s.w.double()
        s.w = None
        grad = s.grad.view(T * B, E)
        for p in pieces:
            v = grad[bag[p]].double().mul_(-float(torch.tensor(LR, dtype=torch.float32)))
            w.index_add_(0, row[p], v if coef is None else v * coef[p, None])
            del v
        if c["storage"] == "fp32":
            res["tables"] = w
        else:
            res["hi"], res["lo"] = w, None
    return res

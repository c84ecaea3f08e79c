"""Timed work of the hashed shared-memory embedding layer.

Every case is one thing a program does with the layer through its public
binding: a training step (forward, then backward and optimizer update), an
inference lookup, or the sparse gradient of a batch for the program's own
optimizer.  A case is a dict of plain values:

  op      "train", "lookup" or "sparse_grad"
  T, B    tables and samples of the batch (T * B bags)
  d, Z, M embedding width, chunk size, weights in the shared array
  weight  storage of the array, "f32" or "bf16"
  opt     "sgd" or "adagrad" (training)
  bag     mean bag length (Poisson, empty bags among them when `empty`,
          else clipped to 1..64); 0 = exactly one index per bag
  rows    table rows: the cardinality of every table, or with `spread` the
          largest of cardinalities spread over their logarithm from 3 up
  zipf    exponent of the index distribution, 0 = uniform
  i32, rows_bf16, mean, sign, prepare
          the layer's options (int32 indices, bfloat16 pooled rows, mean
          pooling, chunk signs 0/1/2, the backward's grouping begun by the
          forward)
"""
import math
import random

import torch

from paper_2207_10731_amd import pss

P = 2**31 - 1
LR = {"sgd": 0.1, "adagrad": 0.01}
EPS = 1e-10


def _case(name, op, T, B, d, Z, M, *, weight="f32", opt="sgd", bag=0.0, empty=False, rows=40_000_000,
          spread=False, zipf=1.1, i32=False, rows_bf16=False, mean=False, sign=0, prepare=False):
    c = dict(op=op, T=T, B=B, d=d, Z=Z, M=M, weight=weight, opt=opt, bag=bag, empty=empty, rows=rows,
             spread=spread, zipf=zipf, i32=i32, rows_bf16=rows_bf16, mean=mean, sign=sign,
             prepare=prepare)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest training step: 4 tables of 1000 rows, 256 samples
        _case("tiny_train", "train", 4, 256, 16, 4, 4096, rows=1000, zipf=0.0),
        # online inference: one small request batch against the 10 MB array
        _case("serve_128", "lookup", 26, 128, 128, 32, 2_500_000, spread=True, i32=True),
        # offline inference at batch 16384
        _case("infer_16k", "lookup", 26, 16384, 128, 32, 2_500_000, spread=True),
        # recommendation training at batch 2048
        _case("train_2k", "train", 26, 2048, 128, 32, 2_500_000, spread=True, prepare=True),
        # one table, batch 10240, uniform tokens (1000x compression), Adagrad
        _case("single_table_adagrad", "train", 1, 10240, 128, 32, 1_280_000, opt="adagrad",
              rows=10_000_000, zipf=0.0),
        # ragged multi-hot features with empty bags, mean pooling, bfloat16
        # array and rows, int32 indices: an odd batch of a mixed-precision model
        _case("ragged_mean_bf16", "train", 13, 1777, 96, 8, 3_000_000, weight="bf16", opt="adagrad",
              bag=9.0, empty=True, rows=1_000_000, zipf=1.05, i32=True, rows_bf16=True, mean=True),
        # a small batch against an array much larger than what it reads
        # (low compression), Adagrad: the sparse branch
        _case("low_compression", "train", 8, 1024, 64, 16, 16_000_000, opt="adagrad",
              rows=1_000_000, zipf=1.05),
        # the sparse gradient (locations and values) of a signed batch
        _case("sparse_gradient", "sparse_grad", 26, 4096, 64, 16, 4_000_000, spread=True, sign=1),
        # the benchmark's default: criteo-tb-shaped one-hot batch of 65536
        _case("one_hot_64k", "train", 26, 65536, 128, 32, 2_500_000, spread=True, prepare=True),
        # multi-hot (Poisson 20), Adagrad on a 64 MB array
        _case("multi_hot", "train", 26, 32768, 64, 16, 16_000_000, opt="adagrad", bag=20.0,
              rows=10_000_000, zipf=1.05, prepare=True),
        # per-element hashing trick on a 4 GB array
        _case("hashing_trick", "train", 26, 65536, 128, 1, 1_000_000_000, zipf=0.0),
        # row hash on a bfloat16 array, Adagrad, batch 262144
        _case("row_hash_bf16", "train", 26, 262144, 128, 128, 64_000_000, weight="bf16",
              opt="adagrad", zipf=1.2, prepare=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(["train"] * 6 + ["lookup"] * 3 + ["sparse_grad"])
    T = rng.choice([1, 2, 5, 8, 13, 26])
    B = _log(rng, 96, 100_000)
    Z = rng.choice([1, 4, 8, 16, 16, 32, 32, 32, 64, 128])
    d = Z * rng.choice([c for c in (1, 2, 3, 4, 6, 8, 16, 32, 64, 128) if 16 <= c * Z <= 256])
    bag = 0.0 if rng.random() < 0.6 else round(rng.uniform(1.5, 30.0), 1)
    # contributions of one pass stay below the largest listed batches'
    cap = 250_000_000 if op != "sparse_grad" and Z > 1 else 40_000_000
    B = max(16, min(B, int(cap / (T * d * max(1.0, bag)))))
    M = _log(rng, 20_000, 50_000_000)
    opt = rng.choice(["sgd", "sgd", "adagrad"])
    weight = "bf16" if rng.random() < 0.25 else "f32"
    c = _case(None, op, T, B, d, Z, max(M, d), weight=weight, opt=opt, bag=bag,
              empty=rng.random() < 0.5, rows=_log(rng, 1000, 40_000_000),
              spread=rng.random() < 0.5, zipf=rng.choice([0.0, 1.05, 1.1, 1.2]),
              i32=rng.random() < 0.3, rows_bf16=rng.random() < 0.2,
              mean=bag > 0 and rng.random() < 0.4, sign=rng.choice([0, 0, 0, 1, 2]),
              prepare=op == "train" and rng.random() < 0.5)
    return c


def _hash(seed):
    r = random.Random(seed * 7919 + 17)
    return dict(a=r.randint(1, P - 1), b=r.randint(0, P - 1), sign_a=r.randint(1, P - 1),
                sign_b=r.randint(0, P - 1))


def _batch(case, seed, dev):
    """indices [N], offsets [T*B + 1] (int64) and the random generator."""
    T, B = case["T"], case["B"]
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 1_000_003 + 12345)
    bags = T * B
    if case["bag"]:
        lens = torch.poisson(torch.full((bags,), float(case["bag"]), device=dev), generator=gen).long()
        lens = lens.clamp(0 if case["empty"] else 1, 64)
    else:
        lens = torch.ones(bags, dtype=torch.int64, device=dev)
    offsets = torch.zeros(bags + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=offsets[1:])
    N = int(offsets[-1].item())
    card = torch.full((T,), float(case["rows"]), dtype=torch.float64, device=dev)
    if case["spread"]:
        u = torch.rand(T, dtype=torch.float64, device=dev, generator=gen)
        card = torch.exp(math.log(3.0) + u * (math.log(case["rows"]) - math.log(3.0))).round()
    table = torch.repeat_interleave(torch.arange(T, device=dev).repeat_interleave(B), lens)
    n = card[table]
    u = torch.rand(N, dtype=torch.float64, device=dev, generator=gen)
    if case["zipf"]:
        # continuous bounded Zipf by inversion: rank in [1, n + 1)
        e = 1.0 - case["zipf"]
        rank = (1.0 - u * (1.0 - (n + 1.0) ** e)) ** (1.0 / e)
        idx = rank.floor().sub_(1.0)
    else:
        idx = (u * n).floor()
    idx = torch.minimum(idx.clamp_(min=0.0), n - 1.0).long()
    return idx, offsets, N, gen


def _flags(case):
    f = pss.PSS_BWD_AUTO
    if case["i32"]:
        f |= pss.PSS_INDEX_I32
    if case["rows_bf16"]:
        f |= pss.PSS_ROWS_BF16
    if case["mean"]:
        f |= pss.PSS_POOL_MEAN
    if case["prepare"]:
        f |= pss.PSS_PREPARE_BACKWARD
    return f | (0, pss.PSS_SIGN_PM1, pss.PSS_SIGN_SPARSE)[case["sign"]]


def _tensors(case, seed, dev):
    idx, off, N, gen = _batch(case, seed, dev)
    T, B, d, M = case["T"], case["B"], case["d"], case["M"]
    t = {"N": N, "idx": idx, "off": off}
    if case["op"] != "sparse_grad":
        w = torch.rand(M, device=dev, generator=gen).mul_(0.02).sub_(0.01)
        t["w"] = w.to(torch.bfloat16) if case["weight"] == "bf16" else w
    if case["op"] != "lookup":
        g = torch.randn((B, T * d), device=dev, generator=gen)
        t["grad"] = g.to(torch.bfloat16) if case["rows_bf16"] else g
    # Adagrad's sums of squares as a run in progress has them
    t["state"] = (torch.rand(M, device=dev, generator=gen)
                  if case["op"] == "train" and case["opt"] == "adagrad" else None)
    return t


def prepare(case, seed):
    dev = torch.device("cuda")
    s = _tensors(case, seed, dev)
    T, B, d, M = case["T"], case["B"], case["d"], case["M"]
    if case["i32"]:
        s["idx"], s["off"] = s["idx"].int(), s["off"].int()
    s["hp"] = pss.make_hash_params(
        num_tables=T, batch=B, num_indices=s["N"], eps=EPS, flags=_flags(case),
        weight_dtype=pss.PSS_BF16 if case["weight"] == "bf16" else pss.PSS_F32, **_hash(seed))
    s["case"], s["lr"] = case, LR[case["opt"]]
    if case["op"] == "sparse_grad":
        cap = min(M, s["N"] * d)
        s["loc"] = torch.zeros(cap, dtype=torch.int32, device=dev)
        s["val"] = torch.zeros(cap, dtype=torch.float32, device=dev)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=dev)
    else:
        s["out"] = torch.empty((B, T * d), device=dev,
                               dtype=torch.bfloat16 if case["rows_bf16"] else torch.float32)
    return s


def run(s):
    c = s["case"]
    M, Z, d, hp = c["M"], c["Z"], c["d"], s["hp"]
    if c["op"] == "sparse_grad":
        pss.pss_gradient_sparse(M, Z, d, hp, s["idx"], s["off"], s["grad"], s["loc"], s["val"],
                                s["count"])
        return {"locations": s["loc"], "values": s["val"], "count": s["count"]}
    pss.pss_forward(s["w"], M, Z, d, hp, s["idx"], s["off"], s["out"])
    if c["op"] == "lookup":
        return s["out"]
    pss.pss_backward_update(s["w"], s["state"], M, Z, d, hp, s["idx"], s["off"], s["grad"], s["lr"])
    if s["state"] is None:
        return {"out": s["out"], "weights": s["w"]}
    return {"out": s["out"], "weights": s["w"], "state": s["state"]}


def work(case):
    """Each index, offset and gradient row read once, each pooled row written
    once, each element of the array that the batch can reach read by the
    forward and read and written (with its optimizer state) by the update."""
    bags = case["T"] * case["B"]
    N = bags * (case["bag"] if case["bag"] else 1)
    reads = N * case["d"]
    ib = 4 if case["i32"] else 8
    rb = 2 if case["rows_bf16"] else 4
    wb = 2 if case["weight"] == "bf16" else 4
    reach = min(case["M"], reads)
    stream = N * ib + (bags + 1) * ib
    rows = bags * case["d"] * rb
    if case["op"] == "lookup":
        return {"bytes": stream + rows + reach * wb, "flops": reads}
    if case["op"] == "sparse_grad":
        return {"bytes": stream + rows + reach * 8, "flops": reads}
    state = 8 if case["opt"] == "adagrad" else 0
    return {"bytes": 2 * stream + 2 * rows + reach * (3 * wb + state), "flops": 2 * reads}


def tolerance(case):
    # bfloat16 results: a sum in another order rounds a few values the other
    # way, one unit in the last place (2^-8 of the value, 2^-7 at most) each
    if case["rows_bf16"] or (case["weight"] == "bf16" and case["op"] == "train"):
        return {"rel": 4e-3, "max": 2e-2}
    # float32 sums: about four times the distance from the 64-bit results
    # (5e-7 at most) and between two runs (7e-5 at a single element, where
    # thousands of terms nearly cancel); locations and counts stay the same
    return {"rel": 2e-6, "max": 3e-4, "differ": 0.0}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
_BLOCK = 16_000_000  # (lookup, dim) contributions handled at a time


def _pieces(case, seed, t):
    """Blocks of lookups: (bag [n], address [n, d], factor [n, d] or None)."""
    T, B, d, Z, M = case["T"], case["B"], case["d"], case["Z"], case["M"]
    C, h = d // Z, _hash(seed)
    dev = t["idx"].device
    lens = t["off"][1:] - t["off"][:-1]
    bag = torch.repeat_interleave(torch.arange(T * B, device=dev), lens)
    dims = torch.arange(d, device=dev)
    j, k = dims // Z, dims % Z
    n = max(1, _BLOCK // d)
    for e in range(0, t["N"], n):
        g = bag[e:e + n]
        key = ((t["idx"][e:e + n] * T + torch.div(g, B, rounding_mode="floor")) * C) % P
        key = (key[:, None] + j[None, :]) % P
        addr = ((key * h["a"] + h["b"]) % P % M + k[None, :]) % M
        f = None
        if case["sign"]:
            h2 = (key * h["sign_a"] + h["sign_b"]) % P
            if case["sign"] == 1:
                f = torch.where(h2 >= 2**30, -1.0, 1.0).double()
            else:
                q = P // 6
                f = (h2 < q).double() - ((h2 >= q) & (h2 < 2 * q)).double()
        yield g, addr, f


def exact(case, seed):
    dev = torch.device("cuda")
    t = _tensors(case, seed, dev)
    T, B, d, M = case["T"], case["B"], case["d"], case["M"]
    lens = (t["off"][1:] - t["off"][:-1]).double()
    weigh = 1.0 / lens.clamp(min=1.0) if case["mean"] else None
    out = torch.zeros((T * B, d), dtype=torch.float64, device=dev) if "w" in t else None
    G = torch.zeros(M, dtype=torch.float64, device=dev) if "grad" in t else None
    seen = torch.zeros(M, dtype=torch.bool, device=dev) if case["op"] == "sparse_grad" else None
    # gradient rows by bag (bag t*B + b is row b, columns t*d ..)
    grad = t["grad"].view(B, T, d) if "grad" in t else None
    for g, addr, f in _pieces(case, seed, t):
        if out is not None:
            x = t["w"][addr].double()
            out.index_add_(0, g, x if f is None else x * f)
        if G is not None:
            v = grad[g % B, torch.div(g, B, rounding_mode="floor")].double()
            if weigh is not None:
                v = v * weigh[g][:, None]
            if f is not None:
                v = v * f
            G.index_add_(0, addr.reshape(-1), v.reshape(-1))
        if seen is not None:
            seen[addr.reshape(-1) if f is None else addr[f != 0]] = True
    if case["op"] == "sparse_grad":
        loc = seen.nonzero().reshape(-1)
        n, cap = loc.numel(), min(M, t["N"] * d)
        locations = torch.zeros(cap, dtype=torch.int32, device=dev)
        values = torch.zeros(cap, dtype=torch.float64, device=dev)
        locations[:n] = loc.int()
        values[:n] = G[loc]
        return {"locations": locations, "values": values, "count": torch.tensor([n], device=dev)}
    if weigh is not None:
        out *= weigh[:, None]
    rows = out.view(T, B, d).transpose(0, 1).reshape(B, T * d)
    if case["op"] == "lookup":
        return rows
    w = t["w"].double()
    if t["state"] is None:
        return {"out": rows, "weights": w - LR["sgd"] * G}
    s = t["state"].double() + G * G
    step = LR["adagrad"] * G / (s.sqrt() + EPS)
    return {"out": rows, "weights": w - torch.where(G != 0, step, torch.zeros_like(step)), "state": s}

"""GPU parity of the small batches' deposit (Alg. 1: gradients summed per
token, then scattered), one kernel over pieces of their order by token, against the oracle:
lane groups of 16, 32 and 64 lanes, slabs, chunk entries in LDS (at most 16
chunks) and hashed per lane, pieces of 64 and 128 lookups with ragged ends, their
cuts in the order by token, runs over several lane groups, as many items as bags
but not one each, and the keygen made ahead by the forward or by
pss_prepare_backward; and the batches just past its limits (grouped).
"""
import numpy as np
import pytest
import torch

import synth
import parity
from paper_2207_10731_amd import pss
from parity import Layer

pytestmark = pytest.mark.gpu

C2 = synth.get("c2")
PREP = pss.PSS_PREPARE_BACKWARD


def _step(L, flags=0, explicit=False):
    wl = L.wl
    g = synth.make_grad(wl, B=L.B)
    if explicit:
        pss.pss_prepare_backward(wl.M, wl.Z, wl.d, L.hp, L.indices, L.offsets)
    got = L.forward()
    ref, s_abs = L.ref_forward()
    parity.check_forward(got, ref, s_abs, parity.RTOL[wl.weight_dtype], rows_bf16=L.rows_bf16)
    L.backward(g)
    w_ref, s_ref, G, A, _ = L.ref_backward(g)
    s_gpu = None if L.state is None else L.state.cpu().numpy()
    parity.check_update(L, L.weights(), s_gpu, w_ref, s_ref, G, A, wl.lr)


@pytest.mark.parametrize("bag", ["one", "poisson:5:0:30"])
@pytest.mark.parametrize("d,Z", [(1, 1), (5, 1), (16, 4), (17, 17), (32, 2), (40, 8), (64, 1),
                                 (70, 7), (128, 32), (200, 50), (260, 52), (600, 24)])
def test_piece_widths(d, Z, bag):
    for B, kw in ((43, {}), (21, dict(sign="pm1", mean=True, idx32=True)),
                  (1, dict(sign="sparse", mean=True, rows_bf16=True, flags=PREP))):
        wl = C2.scaled(T=3, B=B, d=d, Z=Z, M=20 * max(d, 40) + 1, cardinality="fixed:30", bag=bag)
        print(f"d={d} Z={Z} B={B} bag={bag} {kw}", flush=True)
        _step(Layer(wl, **kw))


# (T, B): ends of the pieces of 64, and larger batches that are grouped
@pytest.mark.parametrize("T,B", [(1, 63), (1, 64), (1, 65), (4, 8192), (3, 10923), (7, 5000),
                                 (1, 12000), (1, 12001)])
@pytest.mark.parametrize("prep", ["none", "forward", "explicit"])
def test_piece_sizes(T, B, prep):
    # 3 rows: every piece is a few long runs over all lane groups
    for card in ("fixed:3", "fixed:100000"):
        wl = C2.scaled(T=T, B=B, d=16, Z=16, M=50_000, cardinality=card, optimizer="adagrad")
        print(f"T={T} B={B} prep={prep} {card}", flush=True)
        _step(Layer(wl, flags=PREP if prep == "forward" else 0, s0=0.1), explicit=prep == "explicit")


def _with_bags(lengths, T, **kw):
    """A layer whose bags have the given lengths."""
    lengths = np.asarray(lengths, dtype=np.int64)
    wl = C2.scaled(T=T, B=len(lengths) // T, d=64, Z=16, M=30_000, cardinality="fixed:200")
    L = Layer(wl, **kw)
    offsets = np.zeros(len(lengths) + 1, dtype=np.int64)
    np.cumsum(lengths, out=offsets[1:])
    idx = np.random.default_rng(5).integers(0, 200, int(offsets[-1]), dtype=np.int64)
    L.x = synth.gen.Inputs(indices=idx, offsets=offsets, B=L.B)
    L.indices = torch.from_numpy(idx).to(L.dev).to(L.indices.dtype)
    L.offsets = torch.from_numpy(offsets).to(L.dev).to(L.offsets.dtype)
    L.hp.num_indices = len(idx)
    return L


@pytest.mark.parametrize("kw", [{}, dict(mean=True, flags=PREP), dict(mean=True, idx32=True)],
                         ids=["sum", "mean-prepared", "mean-i32"])
@pytest.mark.parametrize("case", ["one-long", "empties", "swap", "big-pieces"])
def test_piece_bags(case, kw):
    if case == "one-long":      # one bag spans many pieces
        lengths = [0, 0, 5000, 1, 0, 3]
    elif case == "empties":     # more empty bags between two items than a piece has lookups
        lengths = ([1] * 40 + [0] * 900) * 4 + [2] * 200 + [0] * 600
    elif case == "swap":        # as many items as bags, not one each
        lengths = [1] * 100 + [0, 2] * 60 + [1] * 30
    else:                       # bags of 0 .. 7 items
        lengths = list(np.random.default_rng(3).integers(0, 8, 12_000))
    print(f"bags {case} {kw}", flush=True)
    _step(_with_bags(lengths, 4 if case == "big-pieces" else 2, **kw))


# (T, B, rows): one piece and its ends, several tables to a region of 1024 lookups with
# a shorter last region, the longest regions of pieces of 64 and of 128 lookups
# and one more each (the last grouped); rows 1 and 2 divide every bin between
# pieces, 40 some, 100000 none
@pytest.mark.parametrize("T,B", [(1, 55), (1, 56), (1, 57), (5, 300), (7, 150), (2, 1024), (1, 2048),
                                 (1, 1536),
                                 (1, 1537), (3, 2049), (2, 4097), (16, 4096), (1, 8192), (1, 8193)])
@pytest.mark.parametrize("kw", [{}, dict(sign="pm1", mean=True, idx32=True, flags=PREP)],
                         ids=["plain", "signed-prepared"])
def test_piece_cuts(T, B, kw):
    for rows in (1, 2, 40, 100_000):
        wl = C2.scaled(T=T, B=B, d=16, Z=8, M=70_001, cardinality=f"fixed:{rows}")
        print(f"cuts T={T} B={B} rows={rows} {kw}", flush=True)
        L = Layer(wl, **kw)
        assert L.route() == (pss.PSS_ROUTE_GROUPED if B > 8192 else pss.PSS_ROUTE_PIECES)
        _step(L)


def _one_hot(T, B, tokens, **kw):
    """A one-hot layer of the given tokens."""
    wl = C2.scaled(T=T, B=B, cardinality="fixed:1000", **kw)
    L = Layer(wl)
    L.x = synth.gen.Inputs(indices=tokens, offsets=L.x.offsets, B=B)
    L.indices = torch.from_numpy(tokens).to(L.dev)
    return L


@pytest.mark.parametrize("T,B", [(1, 1024), (4, 256), (1, 2048), (1, 8192), (13, 4096)])
def test_piece_rounding(T, B):
    """A token's lookups are summed before they are added to its weights, however they
    are spread over the batch: every token is read by 16 lookups, B / 16 apart, and each
    gradient of 2^-26 alone is lost in a weight of 1 (half a unit in the last place
    is 2^-25), their sum of 2^-22 is not.  A token may be divided between two
    pieces, each part rounded by at most 2^-25: at most 2^-24 per token at an
    element, where adding them one by one would lose 2^-22."""
    n = B // 16
    tokens = np.tile(np.tile(np.arange(n, dtype=np.int64), 16), T)
    L = _one_hot(T, B, tokens, d=16, Z=16, M=2_000_003)
    assert L.route() == pss.PSS_ROUTE_PIECES
    L.shared.fill_(1.0)
    w = np.ones(L.wl.M, dtype=np.float32)
    g = np.full((B, T * 16), 2.0**-26, dtype=np.float32)
    print(f"rounding T={T} B={B}", flush=True)
    L.w_host = w
    L.backward(g, lr=1.0)
    _, _, G, _, _ = L.ref_backward(g, lr=1.0)
    err = np.abs(L.weights().astype(np.float64) - (1.0 - G))
    assert (err <= G / 2.0**-22 * 2.0**-24).all(), err.max()


# The grouped deposit (radix sort, then the reduce kernel, which large batches take):
# widths of one to two slabs, more chunks than the LDS table holds (d / Z > 16),
# the options, and the keygen made ahead.
@pytest.mark.parametrize("d,Z", [(16, 4), (64, 16), (64, 2), (128, 32), (256, 64), (512, 128), (260, 52)])
@pytest.mark.parametrize("kw", [dict(sign="pm1"), dict(sign="sparse", mean=True, idx32=True),
                                dict(rows_bf16=True, mean=True), dict(idx32=True, flags=PREP),
                                dict(sign="sparse", rows_bf16=True, flags=PREP)],
                         ids=["pm1", "sparse-mean-i32", "bf16rows-mean", "i32-prep", "sparse-bf16rows-prep"])
def test_grouped_options(d, Z, kw):
    for B, card, bag in ((8300, "fixed:700", "one"), (1300, "fixed:40000", "poisson:4:0:30")):
        wl = C2.scaled(T=1, B=B, d=d, Z=Z, M=50_000, cardinality=card, bag=bag, optimizer="adagrad")
        print(f"grouped d={d} Z={Z} B={B} {bag} {kw}", flush=True)
        L = Layer(wl, s0=0.1, **kw)
        assert L.route() == pss.PSS_ROUTE_GROUPED
        _step(L)


@pytest.mark.parametrize("kw", [dict(mean=True), dict(mean=True, flags=PREP),
                                dict(sign="pm1", mean=True, idx32=True, flags=PREP)],
                         ids=["plain", "prepared", "signed-i32-prepared"])
@pytest.mark.parametrize("T,B", [(1, 8704), (2, 150_000)])
def test_grouped_irregular_one_hot(T, B, kw):
    """As many items as bags, not one each: the keygen's bag search."""
    lengths = np.ones(T * B, dtype=np.int64)
    at = np.random.default_rng(6).permutation(T * B)[:T * B // 8]
    lengths[at[::2]], lengths[at[1::2]] = 0, 2
    lengths[0] += T * B - lengths.sum()
    print(f"grouped irregular T={T} B={B} {kw}", flush=True)
    L = _with_bags(lengths, T, **kw)
    assert L.route() == pss.PSS_ROUTE_GROUPED
    _step(L)

"""GPU parity of the small batches' deposit (Alg. 1: gradients summed per
token, then scattered), one kernel over pieces of consecutive lookups, against the oracle:
lane groups of 16, 32 and 64 lanes, slabs, chunk entries in LDS (at most 16
chunks) and hashed per lane, pieces of 64 and 256 lookups with ragged ends,
runs over several lane groups, bags of many lengths and long runs of empty
bags, and the keygen made ahead by the forward or by pss_prepare_backward.
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


# (T, B): ends of the pieces of 64, the change to pieces of 256, their ends,
# the most lookups per table and one more (grouped)
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
    else:                       # pieces of 256, bags of 0 .. 7 items
        lengths = list(np.random.default_rng(3).integers(0, 8, 12_000))
    print(f"bags {case} {kw}", flush=True)
    _step(_with_bags(lengths, 4 if case == "big-pieces" else 2, **kw))

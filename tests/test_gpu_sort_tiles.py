"""GPU parity of the grouping sort around the sizes where its digit counts
change form: sort tiles of 2048 pairs, whose scatter sums the counts itself up
to 128 tiles, against the oracle (Alg. 1: lookups grouped by token), with the
first pass's counts made by the one-hot keygen or by the histogram kernel.
"""
import pytest

import synth
import parity
from paper_2207_10731_amd import pss
from parity import Layer

pytestmark = pytest.mark.gpu

C2 = synth.get("c2")


@pytest.mark.parametrize("flags", [0, pss.PSS_PREPARE_BACKWARD], ids=["plain", "prepared"])
@pytest.mark.parametrize("T,B", [(2, 65_600), (1, 128 * 2048 - 1), (1, 128 * 2048),
                                 (1, 128 * 2048 + 1), (3, 150_000)])
def test_sort_tiles(T, B, flags):
    wl = C2.scaled(T=T, B=B, d=4, Z=4, M=300_000, cardinality="fixed:50000")
    print(f"sort tiles T={T} B={B} flags={flags}", flush=True)
    L = Layer(wl, flags=flags)
    g = synth.make_grad(wl, B=B)
    L.forward()
    L.backward(g)
    w_ref, s_ref, G, A, _ = L.ref_backward(g)
    parity.check_update(L, L.weights(), None, w_ref, s_ref, G, A, wl.lr)


@pytest.mark.parametrize("B", [9_000, 40_000])
def test_sort_tiles_multi_hot(B):
    """Bags of 12 items on average: two counted passes or one."""
    wl = C2.scaled(T=5, B=B, d=4, Z=4, M=100_000, cardinality="fixed:9000", bag="poisson:12:0:40",
                   optimizer="adagrad")
    print(f"sort tiles multi-hot B={B}", flush=True)
    L = Layer(wl, s0=0.1, mean=True)
    g = synth.make_grad(wl, B=B)
    L.backward(g)
    w_ref, s_ref, G, A, _ = L.ref_backward(g)
    parity.check_update(L, L.weights(), L.state.cpu().numpy(), w_ref, s_ref, G, A, wl.lr)

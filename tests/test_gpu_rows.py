"""GPU parity of the forward kernels at the edges of their lane groups and
slabs (Sec. 2.4 forward, Sec. 2.5 mapping) against the oracle.

A lane group of 4, 8, ... 64 lanes holds one row, 4 elements per lane when the
chunk size is a multiple of 4 and one otherwise; wider rows are cut into
slabs.  Batches with as many items as bags and other batches take different
kernels, and one-hot batches of 2^20 bags on an array beyond 32 MiB a third.
"""
import numpy as np
import pytest

import synth
import parity
from parity import Layer

pytestmark = pytest.mark.gpu

C2 = synth.get("c2")

# d, Z: lane groups of 4 .. 64 lanes (full and ragged), slabs with and without
# a chunk crossing their boundary, single-element lanes
WIDTHS = [(4, 4), (16, 4), (20, 20), (32, 8), (48, 16), (64, 4), (96, 12), (100, 20), (128, 128),
          (252, 36), (256, 4), (260, 52), (512, 128), (516, 12), (4096, 4096),
          (1, 1), (3, 3), (5, 1), (9, 3), (33, 11), (64, 1), (65, 1), (70, 7), (130, 2), (200, 50)]


def _check(L):
    got = L.forward()
    ref, s_abs = L.ref_forward()
    parity.check_forward(got, ref, s_abs, 1e-5, rows_bf16=L.rows_bf16)


@pytest.mark.parametrize("bag", ["one", "poisson:6:0:40"])
@pytest.mark.parametrize("d,Z", WIDTHS)
def test_row_widths(d, Z, bag):
    # an array of a few chunks: many pieces run past its end; odd T and B
    for M in (Z + 3, 40 * max(d, 50) + 1):
        wl = C2.scaled(T=3, B=53 if d < 1000 else 7, d=d, Z=Z, M=M, cardinality="fixed:500", bag=bag)
        print(f"d={d} Z={Z} M={M} bag={bag}", flush=True)
        _check(Layer(wl))
        _check(Layer(wl.scaled(weight_dtype="bf16"), sign="sparse", mean=True, idx32=True,
                     rows_bf16=True))


@pytest.mark.parametrize("M", [40_000, 10_000_001])
@pytest.mark.parametrize("bag", ["one", "poisson:1:0:4"])
def test_many_bags(M, bag):
    """2^18 bags and more (the batch's index arrays are read ahead), and 2^20
    one-hot bags on a 40 MB array (the tiled kernel), with a ragged end."""
    wl = C2.scaled(T=7, B=150_001, d=8, Z=4, M=M, cardinality="fixed:100000", bag=bag)
    print(f"many bags M={M} bag={bag}", flush=True)
    L = Layer(wl, sign="pm1")
    got = L.forward()
    ref, s_abs = L.ref_forward()
    if bag == "one":
        assert np.array_equal(got.astype(np.float64), ref)
    else:
        parity.check_forward(got, ref, s_abs, 1e-5)

"""GPU parity of the dense optimizer pass (Alg. 1, dense branch) against the
oracle: arrays of 1 to a few more elements than whole 4-element pieces, arrays
that start at any element (pieces aligned to one element only), SGD and
Adagrad, both storage types.  Elements that no lookup reads keep their exact
bits, NaNs included.
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


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 7, 1021, 4098, 40_003])
@pytest.mark.parametrize("dtype,opt", [("f32", "adagrad"), ("bf16", "adagrad"), ("bf16", "sgd")])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_optimizer_pieces(M, dtype, opt, shift):
    wl = C2.scaled(T=2, B=33, d=4, Z=1, M=M, cardinality="fixed:50", weight_dtype=dtype, optimizer=opt)
    L = Layer(wl, flags=pss.PSS_BWD_SORTED, s0=0.1)
    g = synth.make_grad(wl, B=L.B)
    # the same array and state at another offset of a larger allocation
    buf = torch.zeros(M + 8, dtype=L.shared.dtype, device=L.dev)
    buf[shift:shift + M] = L.shared
    L.shared = buf[shift:shift + M]
    if L.state is not None:
        sbuf = torch.zeros(M + 8, dtype=torch.float32, device=L.dev)
        sbuf[shift:shift + M] = L.state
        L.state = sbuf[shift:shift + M]
    L.backward(g)
    w_ref, s_ref, G, A, _ = L.ref_backward(g)
    s_gpu = None if L.state is None else L.state.cpu().numpy()
    parity.check_update(L, L.weights(), s_gpu, w_ref, s_ref, G, A, wl.lr)
    assert not buf[:shift].any() and not buf[shift + M:].any()


def test_untouched_elements_keep_their_bits():
    """A NaN with a payload, an infinity and a negative zero in every element
    that the one lookup does not read."""
    wl = C2.scaled(T=1, B=1, d=1, Z=1, M=1003, cardinality="fixed:5", optimizer="adagrad")
    odd = np.array([0x7fc12345, 0xff800000, 0x80000000, 0x7fa00001], dtype=np.uint32)
    w = np.resize(odd, 1003).view(np.float32).copy()
    base = int(pss.pss_hash_bases_host(wl.M, 1, 1, Layer(wl).hp, synth.make_inputs(wl).indices,
                                       np.array([0, 1]))[0, 0])
    w[base] = 1.0
    L = Layer(wl, flags=pss.PSS_BWD_SORTED, s0=0.1, w=w)
    L.backward(np.full((1, 1), 2.0, dtype=np.float32))
    keep = np.arange(1003) != base
    assert np.array_equal(L.weights().view(np.uint32)[keep], w.view(np.uint32)[keep])
    assert L.weights()[base] != 1.0

"""Which form of the backward's kernels a batch takes, on the host: the ends of
every rule's range (the GPU tests of each form assert its route again)."""
import pytest

from paper_2207_10731_amd import pss

PIECES, GROUPED = pss.PSS_ROUTE_PIECES, pss.PSS_ROUTE_GROUPED


def _route(T, B, N, M, Z, d, flags=0, **kw):
    hp = pss.make_hash_params(1, num_tables=T, batch=B, num_indices=N, flags=flags)
    return pss.pss_debug_backward_route(M, Z, d, hp, **kw)


@pytest.mark.parametrize("T,B,N,Z,d,want", [
    (1, 1, 1, 4, 16, PIECES),
    (1, 8192, 8192, 4, 16, PIECES),
    (1, 8193, 8193, 4, 16, GROUPED),          # a table of more lookups than a region
    (4, 8192, 32768, 16, 16, PIECES),
    (5, 8192, 40960, 16, 16, GROUPED),        # more scanned
    (64, 1024, 65536, 16, 16, PIECES),
    (64, 1025, 65600, 16, 16, GROUPED),       # more lookups
    (26, 2048, 53248, 32, 128, PIECES),
    (1, 100, 101, 4, 16, GROUPED),            # several items per bag
    (4, 4096, 16384, 4, 384, PIECES),         # 1.5 M chunk lines
    (4, 4096, 16384, 4, 388, GROUPED),        # more
])
def test_small_batch_deposit(T, B, N, Z, d, want):
    assert _route(T, B, N, 10**6, Z, d) == want
    assert _route(T, B, N, 10**6, Z, d, pss.PSS_BWD_SORTED, adagrad=True) == want


def test_other_variants():
    small = (2, 100, 200, 10**6, 4, 16)
    assert _route(2, 100, 0, 10**6, 4, 16) == pss.PSS_ROUTE_NONE
    assert _route(*small, pss.PSS_BWD_ATOMIC) == pss.PSS_ROUTE_ATOMIC
    assert _route(*small, pss.PSS_DEPOSIT_BY_ADDRESS) == pss.PSS_ROUTE_ADDRESS
    assert _route(2, 100, 200, 10**6, 64, 64, pss.PSS_DEPOSIT_BY_ADDRESS) == pss.PSS_ROUTE_RUNS
    assert _route(*small, pss.PSS_BWD_SPARSE) == pss.PSS_ROUTE_TILES
    assert _route(2, 100, 200, 8191, 4, 16, pss.PSS_BWD_SPARSE) == pss.PSS_ROUTE_SPARSE
    assert _route(*small, adagrad=True) == pss.PSS_ROUTE_TILES  # low compression: AUTO's sparse branch


@pytest.mark.parametrize("tiles,update,listed", [(2, True, True), (4096, True, True),
                                                 (4097, True, False), (16384, True, False),
                                                 (16385, False, False)])
def test_tiles_of_the_sparse_branch(tiles, update, listed):
    want = {True: pss.PSS_ROUTE_TILES, False: pss.PSS_ROUTE_SPARSE}
    M = 4096 * tiles
    assert _route(1, 500, 500, M, 16, 16, pss.PSS_BWD_SPARSE) == want[update]
    assert _route(1, 500, 500, M, 16, 16, sparse_list=True) == want[listed]


def test_arguments():
    with pytest.raises(Exception):
        _route(1, 1, 1, 10**6, 5, 16)

"""The shapes of the GPU tests reach the tiles they are there for (host only)."""

import pytest

import small_tiles as T

ALL = [(t, M, N, 0, K, False) for t, M, N, K in T.ONE_PACKED] + [(t, M, N, 0, K, True) for t, M, N, K in T.ONE_PREPACKED] + \
      [(t, M, Na, Nb, K, False) for t, M, Na, Nb, K in T.TWO_PACKED] + [(t, M, N, N, K, True) for t, M, N, K in T.TWO_PREPACKED]


@pytest.mark.parametrize("tile,M,N_a,N_b,K,prepacked", ALL)
def test_shape_takes_its_tile(tile, M, N_a, N_b, K, prepacked):
    import paper_2410_05265_amd.binding as b
    assert b.pq_gemm_small_tile(M, N_a, N_b, K, prepacked) == tile


def test_every_tile_is_reached():
    assert {c[0] for c in T.ONE_PACKED} == {c[0] for c in T.TWO_PACKED} | {0} == {0, 11, 12, 22, 23, 32}
    assert {c[0] for c in T.ONE_PREPACKED} == {c[0] for c in T.TWO_PREPACKED} == {11, 12, 22, 23, 24, 32, 42}

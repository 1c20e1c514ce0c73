"""Which tiles a product takes (host only): the shapes of the GPU tests, and shapes at which both sides of a rule were measured."""

import pytest

import tile_plans as T


@pytest.fixture(scope="module")
def b():
    import paper_2410_05265_amd.binding as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("M,N,K", T.SQUARE)
def test_shape_takes_square_tiles(b, M, N, K):
    assert b.pq_gemm_square_tiles(M, N, K)


# tokens, channels out, channels in; measured us of the other kernel and of the square tiles
@pytest.mark.parametrize("M,N,K,other_us,square_us", [
    (4096, 4096, 14336, 114, 110), (2048, 8192, 8192, 69.4, 66.4), (512, 28672, 8192, 83.6, 68.7), (2048, 28672, 8192, 273, 248),
    (4445, 2816, 28416, 236, 192), (256, 49152, 4096, 41.8, 44.7), (256, 49152, 6144, 59.1, 57.9),                    # one round
    (450, 128256, 2048, 121, 98), (900, 49152, 4096, 131, 114), (2048, 128256, 4096, 723, 579), (450, 400000, 512, 151, 169),
    (4096, 65536, 3072, 543, 581), (4096, 65552, 3072, 646, 511), (1024, 65536, 3072, 153, 124),                     # rows 128 KiB apart
    (2048, 14336, 4096, 66.5, 72.6), (30000, 16384, 6144, 1655, 1493), (7000, 28000, 5120, 623, 539)])
def test_square_tiles_where_they_were_measured_faster(b, M, N, K, other_us, square_us):
    assert b.pq_gemm_square_tiles(M, N, K) == (square_us < other_us)


def test_square_tiles_are_for_one_matrix_and_whole_pairs(b):
    assert not b.pq_gemm_square_tiles(2048, 8192, 22144)           # an odd count of 128-channel blocks
    assert b.pq_set_gemm_f6_tile(4) == -1
    try:
        assert not b.pq_gemm_square_tiles(2048, 8192, 22272)
    finally:
        assert b.pq_set_gemm_f6_tile(-1) == 4

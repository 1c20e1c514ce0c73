"""Which tiles a product takes (host only): the shapes of the GPU tests, and shapes at which both sides of a rule were measured."""

import math
import random

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


def test_square_tiles_are_for_whole_pairs(b):
    assert not b.pq_gemm_square_tiles(2048, 8192, 22144)           # an odd count of 128-channel blocks
    assert b.pq_set_gemm_f6_tile(4) == -1
    try:
        assert not b.pq_gemm_square_tiles(2048, 8192, 22272)
    finally:
        assert b.pq_set_gemm_f6_tile(-1) == 4


@pytest.mark.parametrize("tile,M,N,K,planes", T.BYTES)
def test_int8_shape_takes_its_tile(b, tile, M, N, K, planes):
    assert b.pq_gemm_w4a8_tile(M, N, K, planes * M * N * 4) == tile


def test_every_int8_tile_is_reached():
    assert {(c[0] > 200, c[0] % 100) for c in T.BYTES} == {(s, h) for s in (False, True) for h in (2, 3, 4, 5, 6)} | {(False, 0), (False, 1)}


def test_int8_workspace_query_asks_for_what_the_call_takes(b):
    """With the bytes that the query asks for, a call takes the tile and the runs that it would take with any amount; without
    runs it asks for none."""
    rng = random.Random(8)
    split = 0
    for _ in range(3000):
        M, N, K = round(math.exp(rng.uniform(0, 8.3))), 16 * rng.randint(1, 1800), 128 * rng.randint(1, 224)
        asked, tile = b.pq_gemm_workspace_bytes(M, N, K, 8), b.pq_gemm_w4a8_tile(M, N, K, 1 << 40)
        assert asked == (tile // 100 * M * N * 4 if tile >= 200 else 0), (M, N, K)
        assert b.pq_gemm_w4a8_tile(M, N, K, asked) == tile, (M, N, K)
        split += asked > 0
    assert split > 300


# tokens, channels out, channels in, with planes; measured us of two streaming launches and of the tiles, weights from HBM
@pytest.mark.parametrize("M,N,K,planes,stream_us,tiles_us", [
    (17, 4096, 1024, False, 8.9, 5.4), (24, 8192, 2048, False, 10.1, 8.4), (17, 512, 2048, False, 8.8, 7.7), (17, 14336, 4096, False, 16.5, 13.4),
    (32, 14336, 8192, False, 28.3, 25.1), (17, 4096, 4096, False, 10.0, 12.7), (17, 8192, 4096, False, 12.2, 12.9), (32, 8192, 8192, False, 20.5, 23.7),
    (24, 4096, 14336, False, 28.4, 37.6), (17, 1024, 8192, True, 12.0, 8.7), (17, 512, 14336, True, 22.4, 8.6), (32, 2048, 4096, True, 10.1, 8.6)])
def test_few_tokens_of_int8_stream_where_it_was_measured_faster(b, M, N, K, planes, stream_us, tiles_us):
    asked = b.pq_gemm_workspace_bytes(M, N, K, 8)
    assert (b.pq_gemm_w4a8_tile(M, N, K, asked if planes else 0) > 0) == (tiles_us < stream_us)


# tokens, channels out, channels in; measured us of the best tile of 16 x 16 results and of 128 x 128 of 32 x 32
@pytest.mark.parametrize("M,N,K,small_us,pairs_us", [(1363, 11024, 1280, 32.4, 29.8), (1900, 27696, 1280, 93.4, 84.7), (539, 11680, 3840, 35.6, 33.1),
                                                     (1029, 7072, 512, 10.1, 9.1), (502, 5776, 6272, 23.8, 26.8)])
def test_int8_tiles_of_32_where_they_were_measured_faster(b, M, N, K, small_us, pairs_us):
    assert (b.pq_gemm_w4a8_tile(M, N, K, 0) == 1) == (pairs_us < small_us)


# tokens, channels; measured us of the prepacked layer with 16 output channels, all rows in fours and the last `singly` single
@pytest.mark.parametrize("M,K,fours_us,single_us,singly", [
    (512, 4096, 12.1, 8.9, 512), (1120, 4096, 15.1, 14.4, 96), (1280, 4096, 15.3, 14.1, 256), (1408, 4096, 15.5, 16.9, 384),
    (320, 8192, 15.3, 14.7, 320), (448, 8192, 15.9, 17.3, 448), (512, 8192, 16.4, 18.2, 512), (640, 8192, 18.6, 17.6, 128),
    (1280, 8192, 24.0, 24.6, 256), (384, 12288, 21.6, 20.6, 64), (1280, 12288, 31.9, 35.5, 256), (192, 16384, 22.0, 21.6, 192),
    (512, 16384, 27.2, 30.2, 512), (320, 16384, 25.1, 23.9, 64), (1280, 16384, 40.0, 44.3, 256), (160, 28672, 34.1, 33.3, 32),
    (512, 28672, 43.8, 53.5, 512)])
def test_rows_are_rotated_singly_where_it_was_measured_faster(b, M, K, fours_us, single_us, singly):
    assert b.pq_rotate4096_single_rows(M, K) == (singly if single_us < fours_us else 0)

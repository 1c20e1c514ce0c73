"""Shapes of the GPU tests beside the tile that they are there for, which the library's own rules are asked for without a GPU
(test_tile_plans.py), so that a change of a rule cannot leave a kernel untested or compare it with itself."""

# prepacked products on tiles of 256 x 256: tokens, channels out, channels in.  Rows and channels end inside a tile and inside a
# 32-row image; odd counts of 256-channel pairs; one to four rounds of tiles; 19 row tiles x 39 panels (no multiples of 8 and 4)
SQUARE = [(2017, 8112, 22016), (2048, 8192, 22272), (500, 65040, 8192), (2048, 8176, 6144), (4439, 2800, 28672), (4850, 9968, 6144),
          (512, 131056, 2048)]

# products of int8 activations: tile (100 * runs of K + blocks of 32 tokens; 1: 128 x 128 of 32 x 32 results), tokens, channels out,
# channels in, planes of scratch memory
BYTES = [(102, 33, 16, 128, 0), (102, 65, 144, 256, 0), (102, 129, 272, 1152, 0), (103, 1441, 2032, 384, 0), (104, 897, 4016, 128, 0),
         (104, 1000, 4080, 256, 0), (105, 2081, 2064, 384, 0), (106, 1345, 4016, 640, 0), (106, 1475, 4080, 128, 0), (1, 1595, 4624, 128, 0),
         (0, 1177, 4640, 128, 0), (802, 70, 272, 4096, 16), (403, 135, 3600, 6400, 16), (304, 390, 2576, 12288, 16), (705, 134, 4208, 14720, 16),
         (506, 2078, 416, 14720, 16)]

"""Shapes of the GPU tests beside the tile that they are there for, which the library's own rules are asked for without a GPU
(test_tile_plans.py), so that a change of a rule cannot leave a kernel untested or compare it with itself."""

# prepacked products on tiles of 256 x 256: tokens, channels out, channels in.  Rows and channels end inside a tile and inside a
# 32-row image; odd counts of 256-channel pairs; one to four rounds of tiles; 19 row tiles x 39 panels (no multiples of 8 and 4)
SQUARE = [(2017, 8112, 22016), (2048, 8192, 22272), (500, 65040, 8192), (2048, 8176, 6144), (4439, 2800, 28672), (4850, 9968, 6144),
          (512, 131056, 2048)]

"""Shapes at which a product takes each tile of the small-tile kernels (10 * blocks of 32 tokens + blocks of 32 channels),
with ragged last tiles in both directions, fewer stages than wavefronts, stage counts the wavefronts do not share evenly
and rows that end in the middle of a stage.  The tiles are checked against the library's own rule without a GPU, so a
change of its estimates cannot leave one untested; 0: shapes that an earlier rule sent here, now on the other kernels."""

# tile, tokens, channels out, channels in
ONE_PREPACKED = [(11, 1, 16, 128), (11, 17, 48, 640), (11, 31, 1040, 1152), (11, 33, 304, 2176), (11, 64, 512, 3200), (11, 5, 80, 4224),
                 (11, 33, 4112, 128), (12, 40, 4240, 2304), (12, 100, 8208, 128), (22, 100, 12304, 256), (22, 500, 4080, 1024),
                 (23, 100, 8208, 1152), (32, 190, 6032, 1280), (32, 333, 4096, 1152), (24, 131, 8208, 2304), (42, 100, 12304, 2304)]
# (from 17 tokens on; fewer take a weight-streaming kernel)
ONE_PACKED = [(11, 17, 16, 128), (11, 17, 48, 640), (11, 31, 1040, 1152), (11, 33, 304, 2176), (11, 64, 512, 3200), (11, 20, 80, 4224),
              (12, 33, 4112, 128), (12, 40, 4240, 2304), (22, 33, 8208, 384), (22, 100, 4176, 1152), (23, 190, 6032, 1280),
              (23, 131, 6032, 2176), (32, 70, 8208, 2176), (0, 100, 8208, 384), (0, 70, 12304, 384), (0, 333, 4080, 1152)]
# tile, tokens, channels out of both matrices, channels in
TWO_PACKED = [(11, 17, 16, 48, 384), (12, 33, 2064, 2064, 384), (12, 33, 4112, 48, 384), (22, 33, 6160, 2064, 384), (23, 131, 4112, 2064, 384),
              (23, 17, 8208, 8208, 384), (32, 70, 6160, 2064, 384), (32, 70, 4112, 4112, 384)]
# one height; tile, tokens, channels out, channels in
TWO_PREPACKED = [(11, 17, 16, 384), (12, 33, 2064, 1152), (22, 33, 12304, 384), (23, 33, 8208, 1152), (24, 33, 12304, 2304), (32, 70, 6032, 1152),
                 (42, 100, 6160, 2304)]

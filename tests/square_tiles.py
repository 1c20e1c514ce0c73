"""Shapes at which the prepacked product takes each near-square tile and each way of storing its output (test_launches.py asks the
library which kernel they launch, test_gpu_square_tiles.py runs them): tile (10 * operands of 16 tokens + of 16 channels per
wavefront), tokens, channels out, channels in, and whether the output goes past the memory-side cache where it starts on a line."""

# ordinary stores: output rows that start anywhere on 32 bytes, few channels in
ONE = [(44, 129, 12208, 1024), (46, 294, 11408, 1024), (48, 1543, 9872, 1024), (58, 1358, 12368, 1024), (64, 270, 11152, 1280),
       (66, 1797, 8752, 1024), (68, 2738, 7248, 1024), (78, 2349, 10032, 1024), (87, 1948, 12304, 1024), (88, 2468, 12816, 1024)]
TWO = [(44, 68, 8368, 1024), (46, 259, 6096, 1024), (48, 2858, 2576, 1024), (58, 591, 13168, 1024), (64, 132, 9040, 1024),
       (66, 651, 11280, 1024), (68, 1471, 6576, 1024), (78, 1538, 7312, 1024), (87, 1156, 9872, 1024), (88, 2922, 4720, 1024)]
# past the cache: rows of whole lines, of whole halves, and of 32-byte pieces with many channels in
STREAM_ONE = [(44, 130, 11072, 1024), (46, 260, 11072, 1024), (48, 1543, 9792, 1024), (58, 1541, 10816, 1024), (64, 261, 11200, 1024),
              (66, 1283, 11840, 1024), (68, 2898, 6720, 1024), (78, 2319, 10048, 1024), (87, 2703, 8896, 1024), (88, 2440, 12864, 1024),
              (44, 132, 10912, 1024), (46, 257, 10912, 1024), (58, 1553, 10784, 1024), (87, 2694, 8864, 1024), (88, 2437, 12832, 1024),
              (44, 131, 11216, 6144), (66, 1281, 11792, 6144), (48, 1539, 9744, 6144), (88, 2312, 11792, 6144)]
STREAM_TWO = [(44, 72, 8384, 1024), (46, 259, 5696, 1024), (48, 1542, 4672, 1024), (58, 772, 9920, 1024), (64, 129, 8512, 1024),
              (66, 643, 10816, 1024), (68, 1284, 7232, 1024), (78, 1033, 10816, 1024), (87, 1168, 9664, 1024), (88, 1800, 7360, 1024),
              (46, 260, 5536, 1024), (87, 1153, 9760, 1024), (46, 258, 5552, 6144)]
# ordinary again: operands that fill the cache, and its half
LARGE = [(88, 2048, 128256, 4096), (87, 2048, 28672, 8192)]

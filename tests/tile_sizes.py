"""Sizes that take each tile shape: the launch-plan tests assert that they do, the GPU tests run them."""

# Dense linears.  (rows, channels, work-groups to a CU): [(rows, K, channels)]; rows one past whole tiles (one tile and one row,
# one row short), the last channel tile partly past the last channel, K-steps: the fewest with which the
# shape is taken (one, where that is so), as many as the ring has stages, one fewer and one more, the last one partial or whole
DENSE_TILES = {
    (128, 128, 2): [(385, 16, 8144), (129, 192, 5616), (383, 256, 8080), (129, 304, 5488), (257, 400, 5616)],
    (128, 128, 3): [(257, 16, 4112), (257, 128, 3472), (257, 208, 10960), (257, 256, 11184), (257, 272, 11040)],
    (128, 256, 2): [(513, 16, 20144), (513, 144, 19744), (513, 208, 20240), (513, 272, 19952)],
    (192, 128, 1): [(257, 528, 14176), (257, 640, 12064), (191, 1040, 16560), (129, 784, 16592)],
    (192, 256, 1): [(513, 336, 21712), (513, 400, 19760), (513, 1040, 15280)],
    (256, 128, 1): [(129, 16, 16400), (255, 256, 16720), (769, 304, 5520), (257, 336, 15504), (513, 400, 8272)],
    (256, 256, 1): [(641, 16, 16480), (641, 208, 16496), (641, 256, 16432), (641, 272, 16432), (641, 336, 16496), (385, 656, 21680)],
}

# Row tiles of the streaming kernel.  Row blocks of 16 to a tile: [(rows, K, channels)]
STREAM_ROWS = {4: [(129, 1040, 528), (257, 592, 16), (1030, 1104, 272)], 6: [(333, 1040, 4096), (257, 608, 3376), (129, 688, 5488)],
               8: [(500, 2112, 4080), (193, 1168, 5456), (385, 2064, 4080)]}

# Expert groups whose down projection takes 192 x 256 tiles.  (H, I, rows of the groups of the tokens' first experts, of their
# second ones): whole 192-row tiles, one row more and one fewer, H no multiple of 256
TALL_GROUPS = [(2112, 1024, (193, 191, 385, 192, 383, 216), (577, 1, 192, 193, 575, 22)),
               (2112, 1024, (384, 385, 577, 454), (768, 193, 191, 648))]

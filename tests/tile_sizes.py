"""Dense linears that take each tile shape: the launch-plan test asserts that they do, the GPU tests run them."""

# (rows, channels, work-groups to a CU): [(rows, K, channels)]; rows one short of, at and one past whole tiles, the last channel
# tile partly past the last channel, one K-step, as many as the ring has stages, one fewer and one more, a last partial one
DENSE_TILES = {
    (128, 128, 3): [(257, 16, 4112), (257, 128, 3472), (257, 208, 10960), (257, 256, 11184), (257, 272, 11040)],
    (256, 128, 1): [(129, 16, 16400), (255, 256, 16720), (769, 304, 5520), (257, 336, 15504), (513, 400, 8272)],
}

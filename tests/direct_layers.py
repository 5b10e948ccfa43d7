"""Passes whose halo boxes and weights other waves of a workgroup stage (csrc/direct_beside_impl.h): what the host's search takes them in is checked on the CPU,
their results on the GPU."""

# f, fo, n, k, s, backward, then 16-map tiles of a workgroup, groups of maps, shares, chunks of a share and halo voxels
BESIDE = [
    (1, 3, (1, 20, 18), (1, 3, 6), 1, 1, (1, 1, 1, 1, 21)),         # the fewest of everything
    (22, 5, (24, 32, 23), (5, 5, 2), 1, 0, (1, 1, 1, 3, 264)),      # two voxels a thread that stages
    (3, 10, (30, 6, 13), (5, 5, 5), 1, 0, (1, 1, 1, 1, 540)),       # four of them
    (25, 2, (13, 32, 34), (4, 5, 3), 2, 1, (2, 1, 1, 1, 550)),      # the same with two map tiles, sublattices
    (6, 41, (31, 15, 9), (1, 5, 5), 2, 0, (1, 3, 1, 1, 640)),       # three groups of maps
    (48, 30, (28, 32, 6), (2, 4, 4), 1, 1, (1, 3, 1, 4, 275)),      # and four chunks
    (56, 28, (16, 33, 13), (5, 1, 5), 2, 1, (2, 2, 1, 4, 495)),     # an even number of chunks
    (85, 17, (11, 9, 22), (5, 2, 2), 1, 1, (2, 3, 1, 3, 120)),      # six map tiles
    (2, 43, (17, 20, 31), (2, 5, 2), 1, 1, (1, 1, 2, 3, 162)),      # two shares of three chunks
    (17, 41, (8, 32, 24), (1, 5, 3), 2, 1, (2, 1, 2, 3, 96)),       # the same with two map tiles
]

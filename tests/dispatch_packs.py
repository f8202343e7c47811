"""Packs that the scheduler's rules send to whole items or to persistent workgroups, with the form of each pass.

Small packs run half items in most passes, so the kernels that large packs run are only met by packs that are chosen for it.
`test_dispatch.py` holds every pack here to its form on the CPU; `test_gpu_whole_items.py` compares its outputs with the oracle."""
WHOLE, HALVES, PERSISTENT = 0, 1, 2

# lengths on both sides of the tile edges, up to ten key tiles: every loop of the kernels' tile walk runs
RAGGED = [600, 577, 513, 512, 449, 385, 257, 256, 193, 192, 129, 128, 65, 64, 1, 600, 590, 640]

# (lengths, q heads, kv heads, head_dim, form of the forward and dQ passes, form of the dK/dV pass)
PACKED = [(RAGGED, 8, 8, d, WHOLE, WHOLE) for d in (64, 40, 72, 80, 88, 96, 104, 112, 128)]
# groups: with few chains of long dK/dV items that pass takes halves, with more it does not
PACKED += [(RAGGED, 8, 2, d, WHOLE, HALVES) for d in (64, 80, 128)] + [(RAGGED, 24, 12, d, WHOLE, WHOLE) for d in (64, 96, 128)]
# more than a thousand dK/dV items of ten tiles and less: persistent workgroups, long enough for the loop that spreads its copies
PERSISTENT_PACKS = [([640, 577, 449, 300, 600, 512, 64, 400] * 3, 12, 12, d, WHOLE, PERSISTENT) for d in (72, 96, 104, 128)]

# (q lengths, k lengths, q positions, k positions): diagonals inside the block with either sign, blocks in the past and in the
# future, empty chunks, ragged tails
GEOMETRY = ([300, 600, 129, 64, 512, 0, 77, 1, 450, 577, 330, 256],
            [512, 600, 257, 130, 300, 90, 0, 300, 450, 385, 640, 256],
            [412, 0, 100, 700, 130, 5, 9, 299, 450, 192, 64, 0],
            [0, 0, 64, 0, 0, 0, 0, 0, 450, 0, 0, 300])
# (q heads, kv heads, head_dim, form of the forward and dQ passes, form of the dK/dV pass)
BLOCKS = [(12, 12, 128, WHOLE, WHOLE), (8, 4, 128, WHOLE, HALVES), (24, 12, 128, WHOLE, WHOLE),
          (32, 16, 64, WHOLE, WHOLE), (12, 12, 104, WHOLE, WHOLE),
          (24, 12, 96, WHOLE, WHOLE),
          (12, 12, 80, WHOLE, WHOLE)]

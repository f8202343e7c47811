"""Packs that the scheduler's rules send to whole items or to persistent workgroups, with the form of each pass.

Small packs run half items in most passes, so the kernels that large packs run are only met by packs that are chosen for it.
`test_dispatch.py` holds every pack here to its form on the CPU; `test_gpu_whole_items.py` and `test_gpu_list_kinds.py` compare its
outputs with the oracle; `test_launched_kernels.py` asks the library which kernels all of them launch together."""
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

# ---- the two kinds of list: in the kernels' arguments (up to 240 slots, 120 of a block plan) or in device memory ----
# lengths on both sides of the tile edges; with one or two heads half items, their lists in the arguments
EDGES = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257, 449]
# one long sequence and many short ones: half items whose lists are too long for the arguments, and more of them than the forward
# has workgroups (544 halves on 512), so that it draws some
HALF_LONG = [2500] + EDGES + [1 + (i * 53) % 128 for i in range(25)]
HALF_LONG_PACKS = [(HALF_LONG, 4, 4, d) for d in (40, 64, 80, 96, 104, 128)] + [(HALF_LONG, 6, 2, d) for d in (64, 128)]
HALF_GEOMETRY = tuple(first + rest for first, rest in zip(([900, 1], [2400, 700], [1700, 300], [0, 0]), GEOMETRY))
HALF_LONG_BLOCKS = [(HALF_GEOMETRY, 6, 2, d) for d in (64, 80, 96, 104, 128)]
# short lists: whole items (one tile each) and half items at the widths that have kernels of their own
ONE_TILE = [1 + (i * 53) % 128 for i in range(29)]
SHORT_PACKS = [(ONE_TILE, 8, 8, d) for d in (64, 80, 96, 104, 128)] + [(EDGES, 2, 2, d) for d in (64, 80, 96, 104, 128)]
ONE_TILE_GEOMETRY = ([min(130 - 7 * i, 128) for i in range(14)], [min(5 + 9 * i, 128) for i in range(14)], [40 + i for i in range(14)],
                     [3 * i for i in range(14)])
# (one step per item: with two the dQ pass of so few items would take halves)
ONE_STEP_GEOMETRY = (ONE_TILE_GEOMETRY[0], [min(n, 64) for n in ONE_TILE_GEOMETRY[1]], *ONE_TILE_GEOMETRY[2:])
SHORT_BLOCKS = [(g, hq, hkv, d) for d in (64, 80, 96, 104, 128)
                for g, hq, hkv in ((ONE_TILE_GEOMETRY, 8, 8), (ONE_STEP_GEOMETRY, 8, 4), (HALF_GEOMETRY, 2, 1))]

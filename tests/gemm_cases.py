"""One product per compiled GEMM kernel, at sizes that are no multiple of its tile.
A CPU test states that the dispatch takes that kernel; a GPU test runs each with
every format set."""

CASES = [  # kernel (as gemm_routes.kernel names it), M, N, split
    ("direct 1 tiles 16 rows", 13, 3001, (544, 160, 320)),
    ("direct 1 tiles 32 rows", 16, 8201, (96, 160, 96)),
    ("direct 2 tiles 16 rows", 23, 3001, (544, 160, 320)),
    ("direct 2 tiles 24 rows", 17, 6001, (544, 160, 320)),
    ("direct 2 tiles 56 rows", 32, 13000, (0, 0, 4096)),
    ("direct 2 tiles 40 rows", 20, 20001, (6144, 1536, 512)),  # two workgroups per CU, 84 MB of weight
    ("direct 4 tiles 16 rows", 37, 3001, (544, 160, 320)),
    ("direct 4 tiles 24 rows", 33, 6001, (96, 64, 2400)),
    ("direct 4 tiles 56 rows", 50, 13000, (0, 0, 4096)),
    ("direct 4 tiles 40 rows", 40, 20001, (0, 0, 2048)),  # two workgroups per CU
    ("split 32x32", 100, 1003, (320, 256, 128)),
    ("split 64x32", 129, 2050, (320, 256, 128)),
    ("split 64x32", 30, 26001, (1536, 384, 128)),
    ("split 64x64", 150, 4100, (544, 160, 320)),
    ("split 64x96", 200, 5400, (1056, 352, 128)),
    ("split 64x128", 500, 4090, (1056, 352, 128)),
    ("tiled 256x128", 1990, 4050, (96, 160, 96)),  # five stages, fewer than the ring's slots
    ("tiled 256x128", 2040, 4090, (640, 96, 160)),
    ("tiled 256x256", 3841, 4001, (640, 224, 96)),
    ("tiled 256x256", 500, 27001, (288, 96, 160)),  # fewer tiles than CUs
]

# the LDS-tiled kernel with few stages: 256 x 128 tiles, in the last two 256 x 256
FEW_STAGES = [(1990, 4050, (32, 0, 0)), (2000, 4040, (0, 0, 96)), (1921, 3841, (160, 32, 64)),
              (2040, 4090, (640, 96, 160)), (1985, 4089, (1152, 0, 0)),
              (4000, 4090, (32, 0, 32)), (3841, 4001, (640, 224, 96))]

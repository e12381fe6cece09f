"""One product per compiled GEMM kernel, at sizes that are no multiple of its tile.
A CPU test states that the dispatch takes that kernel; a GPU test runs each with
every format set."""

CASES = [  # kernel (as gemm_routes.kernel names it), M, N, split
    ("direct 4 tiles 16 rows", 37, 3001, (544, 160, 320)),
    ("direct 4 tiles 24 rows", 33, 6001, (96, 64, 2400)),
    ("direct 4 tiles 56 rows", 50, 13000, (0, 0, 4096)),
    ("direct 4 tiles 40 rows", 40, 20001, (0, 0, 2048)),  # two workgroups per CU
]

"""Products that reach every block shape between the GEMV and the large tiles
(64 MiB workspace): rows, features, K, LoRA columns, and the launch planned for
them: kernel, block, K elements per stage, K ranges launched, K tiles (of 64)
per range of the sum.  The CPU test holds the plans, the GPU test the results."""

WORKSPACE = 64 << 20

CASES = [
    # streaming kernel, 32-row blocks: split, one block over even and odd ranges, 512-byte rows
    (17, 768, 8192, 64, "stream 32 32 128 8 16"),
    (9, 6144, 4096, 64, "stream 32 32 128 1 13"),
    (9, 2304, 5120, 64, "stream 32 64 128 8 10"),
    (17, 20480, 2048, 0, "stream 32 64 128 1 11"),
    (17, 12288, 4096, 192, "stream 32 64 256 1 13"),
    # 64- and 128-row blocks
    (61, 2304, 2048, 64, "stream 64 64 128 4 8"),
    (250, 4096, 2048, 0, "stream 64 64 128 1 11"),
    (400, 1536, 1024, 128, "stream 64 64 128 1 8"),
    (77, 2304, 2048, 64, "stream 128 64 128 4 8"),
    (129, 6144, 1024, 64, "stream 128 64 128 1 8"),
    (256, 4608, 2048, 64, "stream 128 64 128 1 11"),
    # ring tiles
    (700, 6144, 640, 64, "ring 192 128 64 1 10"),
    (150, 20480, 320, 0, "ring 192 128 64 1 5"),
    (200, 12288, 4096, 64, "ring 256 256 64 5 13"),
    (230, 12288, 4096, 0, "ring 256 256 64 4 16"),
    (512, 3072, 16384, 64, "ring 256 256 64 8 32"),
    (129, 6144, 4096, 64, "ring 256 256 64 7 10"),
    # ping-pong tiles, odd and even K tiles with base and LoRA
    (200, 20480, 1024, 0, "pingpong 128 256 64 1 16"),
    (400, 12288, 1088, 64, "pingpong 128 256 64 1 17"),
    (700, 3072, 5120, 64, "pingpong 192 256 64 5 16"),
    (700, 3072, 5184, 192, "pingpong 192 256 64 5 17"),
    (700, 12288, 640, 128, "pingpong 192 256 64 1 10"),
    (1000, 20480, 320, 0, "pingpong 192 256 64 1 5"),
    # the square ping-pong tile, split
    (700, 4608, 5184, 64, "tile 256 256 64 4 21"),
]

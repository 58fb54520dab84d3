"""Which kernel the tests' sizes take in the scoring call and in the Gram matrix.  test_host_path_cpu.py checks that the library takes these,
test_gpu_parity.py and test_zz_no_alloc.py run them."""
# (candidates, rows, channels): (edge of the tiles, chunk of the contraction in blocks of that edge, (chunk, column block) slots).
# 256 is the DMA kernel; its operands are blocked where the channels are a multiple of 32, and its epilogue is in the loop where they are one of 256.
SCORING_FORMS = {
    (1, 1, 8): (64, 1, 1),  # row-major
    (1, 8, 264): (64, 5, 5),  # row-major
    (1, 64, 64): (64, 1, 1),  # blocked
    (1, 264, 328): (64, 6, 6),  # row-major
    (1, 384, 640): (64, 10, 10),  # blocked
    (1, 512, 512): (64, 8, 8),  # blocked
    (1, 1288, 264): (64, 5, 5),  # row-major
    (2, 65, 72): (64, 2, 2),  # row-major
    (2, 256, 384): (64, 6, 6),  # blocked
    (3, 200, 64): (64, 1, 1),  # blocked
    (8, 63, 520): (64, 9, 9),  # row-major
    (1, 5, 1208): (128, 1, 55),  # row-major, chunks of 1 of 10
    (1, 7, 4096): (128, 2, 272),  # blocked, chunks of 2 of 32
    (1, 96, 2056): (128, 1, 153),  # row-major, chunks of 1 of 17
    (1, 257, 1376): (128, 1, 66),  # blocked, chunks of 1 of 11
    (1, 300, 2312): (128, 2, 100),  # row-major, chunks of 2 of 19
    (1, 1025, 1288): (128, 3, 26),  # row-major, chunks of 3 of 11
    (1, 2056, 768): (128, 2, 12),  # blocked, chunks of 2 of 6
    (1, 16384, 256): (128, 2, 2),  # blocked, whole contractions
    (2, 130, 1000): (128, 1, 36),  # row-major, chunks of 1 of 8
    (2, 264, 3328): (128, 5, 81),  # blocked, chunks of 5 of 26
    (2, 513, 1000): (128, 2, 20),  # row-major, chunks of 2 of 8
    (2, 520, 2048): (128, 3, 51),  # blocked, chunks of 3 of 16
    (2, 768, 640): (128, 1, 15),  # blocked, chunks of 1 of 5
    (2, 9001, 264): (128, 3, 3),  # row-major, whole contractions
    (3, 264, 1504): (128, 2, 42),  # blocked, chunks of 2 of 12
    (4, 130, 1544): (128, 2, 49),  # row-major, chunks of 2 of 13
    (8, 256, 2048): (128, 6, 30),  # blocked, chunks of 6 of 16
    (1, 264, 5024): (256, 2, 110),  # blocked, chunks of 2 of 20
    (1, 264, 6176): (256, 3, 117),  # blocked, chunks of 3 of 25
    (1, 500, 5000): (256, 2, 110),  # row-major, chunks of 2 of 20
    (1, 504, 5000): (256, 2, 110),  # row-major, chunks of 2 of 20
    (2, 264, 2560): (256, 1, 55),  # blocked, epilogue in the loop, chunks of 1 of 10
    (2, 264, 4128): (256, 3, 57),  # blocked, chunks of 3 of 17
    (2, 500, 4104): (256, 3, 57),  # row-major, chunks of 3 of 17
    (2, 500, 5000): (256, 4, 60),  # row-major, chunks of 4 of 20
    (2, 1024, 4096): (256, 5, 34),  # blocked, epilogue in the loop, chunks of 5 of 16
    (3, 250, 4128): (256, 3, 57),  # blocked, chunks of 3 of 17
    (8, 520, 4104): (256, 17, 17),  # row-major, whole contractions
    (8, 1032, 1280): (256, 3, 7),  # blocked, epilogue in the loop, chunks of 3 of 5
    (8, 1536, 1024): (256, 4, 4),  # blocked, epilogue in the loop, whole contractions
}
# (tokens, channels): edge of the Gram matrix's tiles
GRAM_FORMS = {
    (1, 1032): 128,
    (40, 1096): 128,
    (100, 1280): 128,
    (257, 1152): 128,
    (400, 1600): 128,
    (512, 1288): 128,
    (700, 1032): 128,
    (77, 1288): 128,
    (449, 1600): 256,
    (130, 1608): 256,
    (3000, 2056): 256,
    (70, 6144): 256,
    (9999, 3080): 256,
    (4096, 128): 128,
    (1000, 264): 128,
    (8192, 1024): 128,
}

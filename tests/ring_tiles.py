"""Products that the GEMM's cost model gives to each small tile shape, at 256 compute units.

The shapes cannot be forced, so a product stands for each; test_gemm_dispatch.py checks on the host that it
still gets its shape, test_gpu_gemm.py that the shape computes it.
"""
# (rows, columns, LDS stages), M, N and, by output, the K loop's tiles of 128: a single one, around the ring's
# length and past twice that, as far as the model gives the shape such K loops.  N leaves every remainder by 4.
F32, BF16, ACCUM = "f32", "bf16", "accumulate"
RING = [
    ((64, 64, 4), 65, 63, {F32: (1, 3, 4, 5, 6, 9), BF16: (1, 3, 4, 5, 6, 9), ACCUM: (1, 3, 4, 5, 6, 9)}),
    ((128, 64, 3), 8351, 661, {F32: (3, 4, 5, 7), ACCUM: (3, 4, 5, 7)}),
    ((128, 64, 3), 8862, 386, {BF16: (2, 3, 4, 5, 7)}),
    ((128, 64, 6), 68, 8257, {F32: (6, 7, 8, 13), BF16: (5, 6, 7, 8, 13), ACCUM: (6, 7, 8, 13)}),
    ((64, 128, 3), 129, 27693, {F32: (3, 4, 5, 7), BF16: (1, 2, 3, 4, 5, 7), ACCUM: (3, 4, 5, 7)}),
    ((64, 128, 6), 33, 16407, {F32: (6, 7, 8, 13), BF16: (5, 6, 7, 8, 13), ACCUM: (6, 7, 8, 13)}),
    ((128, 128, 2), 198, 26498, {F32: (4, 5), BF16: (1, 2, 3, 4, 5)}),
    ((128, 128, 2), 207, 24739, {ACCUM: (12, 13)}),
    ((128, 128, 4), 65, 25277, {F32: (4, 5, 6, 9), BF16: (3, 4, 5, 6, 9), ACCUM: (18, 21)}),
]
TAILS = (0, 31, 100)  # what the last K tile lacks of 128

"""The tile shape the GEMM picks, read from its launches on the fake HIP runtime (256 compute units)."""
import re

import pytest

from tests.fake_hip import ADDR, calls
from tests.ring_tiles import ACCUM, BF16, RING, TAILS


def launches(qe, hip, products):
    """The kernel and grid of each product (m, n, k, out, ldc)."""
    got = []
    for m, n, k, out, ldc in products:
        hip.clear()
        ld = (k + 15) // 16 * 16
        assert qe.qe_fp8_gemm_tn(ADDR, 0, ld, ADDR, 0, ld, m, n, k, ADDR, ADDR, ADDR, qe.BF16 if out == BF16 else qe.F32, ldc,
                                 qe.ACCUM if out == ACCUM else qe.INIT, stream=0) == "OK"
        (_, _, name, grid), = hip.log("launch")
        got.append([name, int(grid.split("=")[1])])
    return got


@pytest.mark.parametrize("tile,m,n,loops", RING, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else None)
def test_products_get_their_small_tile(tile, m, n, loops):
    products = [[m, n, 128 * t - lack, out, ldc] for out, ts in loops.items() for t in ts for lack in TAILS
                for ldc in ((n + 3) // 4 * 4, (n + 3) // 4 * 4 + 3)]
    bm, bn, _ = tile
    for p, (name, grid) in zip(products, calls(launches, products)):
        shape = re.search(r"gemm_tn_ring_kernelILi0ELi0ELi(\d+)ELi(\d+)ELi(\d+)E", name)
        assert shape and tuple(map(int, shape.groups())) == tile, (p, name)
        assert grid == -(-m // bm) * -(-n // bn)


# products whose small tiles would run in many rounds, with rows a multiple of 4 KB apart
MANY_ROUNDS = [(4096, 28672, 1024, BF16), (4096, 28672, 512, "f32"), (8192, 28672, 512, ACCUM), (4096, 14336, 512, "f32"),
               (4096, 14336, 512, ACCUM), (4096, 4096, 256, BF16), (8192, 8192, 1024, BF16), (4096, 28672, 128, BF16),
               (28672, 4096, 256, ACCUM)]


def test_small_tiles_are_not_taken_for_many_rounds_of_wide_rows():
    """Large outputs after short reductions, rows a multiple of 4 KB apart: on MI355X small tiles take 1.2 to 1.9
    times as long there as the large ones."""
    got = calls(launches, [[*p, p[1]] for p in MANY_ROUNDS])
    assert all("gemm_tn_w4_kernel" in name for name, _ in got), list(zip(MANY_ROUNDS, got))


def test_few_rounds_and_odd_rows_keep_their_small_tiles():
    """The second rule touches neither products of up to two small tiles per unit nor odd rows."""
    products = [[512, 4096, 14336, BF16, 4096], [256, 4096, 4096, BF16, 4096], [128, 256, 256, "f32", 256],
                [1024, 8192, 8192, BF16, 8192], [4100, 4100, 1040, ACCUM, 4103], [1000, 2730, 1365, BF16, 2730]]
    assert all("gemm_tn_ring_kernel" in name for name, _ in calls(launches, products))

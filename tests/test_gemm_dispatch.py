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

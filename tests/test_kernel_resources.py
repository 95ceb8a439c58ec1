"""Registers and scratch of the kernels in the built library, as the launch rules assume them."""
import pytest

from tests.kernel_resources import kernels
from tests.libqe import need_lib


@pytest.fixture(scope="module")
def built():
    found = kernels(need_lib().LIB_PATH)
    assert found
    return found


def test_no_kernel_uses_scratch(built):
    """A spilled register is a load the inline-assembly load counters do not know of: the K loops would wait
    for it, and with it for every load in flight."""
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in built.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad


# name part, workgroups (one wave on each SIMD) a compute unit is to hold; a SIMD has 512 registers, given in eights
OCCUPANCY = [("quantize_kernelILb0ELi0ELi128E", 3), ("quantize_kernelILb1ELi0ELi128E", 3),
             ("quantize_kernelILb0ELi0ELi64E", 6), ("quantize_kernelILb1ELi0ELi64E", 6),
             ("gemm_tn_ring_kernelILi0ELi0ELi64ELi64ELi4E", 2), ("gemm_tn_ring_kernelILi0ELi0ELi128ELi64ELi3E", 2),
             ("gemm_tn_ring_kernelILi0ELi0ELi64ELi128ELi3E", 2), ("gemm_tn_ring_kernelILi0ELi0ELi128ELi128ELi2E", 2)]


@pytest.mark.parametrize("part,workgroups", OCCUPANCY, ids=lambda v: str(v))
def test_workgroups_per_compute_unit(built, part, workgroups):
    """The workgroups a compute unit is meant to hold fit its registers and its 160 KB of LDS."""
    got = [k for n, k in built.items() if part in n]
    assert len(got) == 1
    vgprs = (got[0][".vgpr_count"] + 7) // 8 * 8  # AGPRs included
    assert 512 // vgprs >= workgroups
    assert got[0][".group_segment_fixed_size"] * workgroups <= 160 * 1024

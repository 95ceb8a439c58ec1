"""The hash that ties committed counter runs to the GEMM source they were taken on."""
import os
import shutil

import pytest

import bench


@pytest.fixture
def copy(tmp_path):
    for name in bench.GEMM_SOURCES:
        shutil.copy(os.path.join(bench.CSRC, name), tmp_path)
    return str(tmp_path)


@pytest.mark.parametrize("name", bench.GEMM_SOURCES)
def test_source_hash_follows_code_not_comments(copy, name):
    same = bench.gemm_source_sha256(copy)
    assert same == bench.gemm_source_sha256()
    path = os.path.join(copy, name)
    text = open(path).read()
    open(path, "w").write("// a comment\n/* and\nanother */\n" + text.replace("\n\n", "\n   // x\n\n"))
    assert bench.gemm_source_sha256(copy) == same
    open(path, "w").write(text + "\nstatic int added;\n")
    assert bench.gemm_source_sha256(copy) != same


def test_every_gemm_source_is_hashed():
    built = {f for f in os.listdir(bench.CSRC) if f.startswith("gemm_")}
    assert built == set(bench.GEMM_SOURCES)

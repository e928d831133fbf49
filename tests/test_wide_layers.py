"""Layers of more than 64 MB at up to 64 rows (CPU): which launches load their weights past the caches, and in which plans K is cut for a
workgroup on every compute unit."""
import ctypes
import os
import subprocess

import pytest

import paper_2006_03031_amd as nb
from paper_2006_03031_amd import build

RULE = """
#include "nimble_internal.h"
extern "C" int weights_pass_by(int64_t rows, int64_t N, int64_t K, int64_t slices) { return nimble::weights_pass_by(rows, N, K, slices); }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(RULE)
    lib = str(d / "rule.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    str(d / "rule.cpp"), "-o", lib], check=True)
    lib = ctypes.CDLL(lib)
    lib.weights_pass_by.argtypes = [ctypes.c_int64] * 4
    return lib.weights_pass_by


def test_weights_past_the_caches(rule):
    for rows, N, K, slices, past in (
            # up to 8 rows what is lost where the memory-side cache holds the layer is what is gained where it does not
            (1, 8192, 8192, 1, 1), (8, 8192, 8192, 1, 1), (8, 6144, 6144, 1, 1), (8, 5003, 6400, 1, 1), (8, 4999, 6400, 1, 0),
            # 16 rows of 8192 x 8192 over and over would take 24.2 us in place of 21.1, of 6144 x 6144 18.2 in place of 14.4
            (9, 8192, 8192, 1, 0), (16, 8192, 8192, 1, 0), (16, 6144, 6144, 1, 0), (16, 32000, 4096, 1, 0),
            # what that cache cannot hold
            (16, 8192, 28672, 1, 1), (64, 8192, 28672, 4, 1), (16, 16385, 8192, 1, 1), (16, 16384, 8192, 1, 0),
            # 32-row tiles with a workgroup per compute unit and K in three or more; 64 rows of 6144 x 6144 24.1 in place of 19.5
            (17, 8192, 8192, 3, 1), (32, 4096, 8192, 8, 1), (32, 13824, 5120, 2, 0), (32, 14336, 4096, 4, 0),
            (33, 8192, 8192, 3, 0), (64, 6144, 6144, 5, 0), (64, 4096, 8192, 8, 0)):
        assert rule(rows, N, K, slices) == past, (rows, N, K, slices)


@pytest.mark.parametrize("N,K,slices", [(8192, 8192, 3), (6144, 6144, 5), (4096, 8192, 8), (13824, 5120, 2), (1280, 25600, 16), (2048, 32768, 15)])
def test_the_cut(N, K, slices):
    for M in (17, 32, 33, 64) if (N, K) != (2048, 32768) else (33, 64):   # (up to 32 rows of the last are streamed, without scratch)
        p = nb.dense_plan(M, N, K)
        assert (p.bm, p.split_k) == (32 if M <= 32 else 64, slices), M
        assert p.workspace_bytes == slices * M * N * 4


# what ran without scratch still does, whoever else uses the default workspace at the time
@pytest.mark.parametrize("M,N,K", [(33, 16384, 2048), (64, 16384, 2048), (17, 2048, 28672), (32, 2048, 28672)])
def test_plans_without_scratch_stay_so(M, N, K):
    p = nb.dense_plan(M, N, K)
    assert p.workspace_bytes == 0 and (p.split_k == 1 or p.name == "skinny16"), p


# the rest of a row split is planned by the estimates with which the split was decided
@pytest.mark.parametrize("M,N,K,variant,workspace", [(2081, 4096, 8192, "t32x128", 8 * 33 * 4096 * 4), (2067, 4096, 14336, "t32x128", 16 * 19 * 4096 * 4)])
def test_the_rest_of_a_row_split(M, N, K, variant, workspace):
    p = nb.dense_plan(M, N, K)
    assert p.split_rows == 2048 and nb.variant_name(p.residue_variant) == variant and p.workspace_bytes == workspace

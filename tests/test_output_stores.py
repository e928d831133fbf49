"""Output stores: which launches write through the L2s (CPU, on shapes measured both ways) and the results on either side."""
import ctypes
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")
import paper_2006_03031_amd as nb
from paper_2006_03031_amd import build

RULES = """
#include "nimble_internal.h"
extern "C" int output_stays(int64_t batch, int64_t M, int64_t N, int64_t K, int out_f32, uint64_t address, int64_t slices) {
  nimble::GemmArgs g{};
  g.c = (void*)address;
  g.M = (int)M, g.N = (int)N, g.K = (int)K, g.ldc = (int)N, g.sc = M * N, g.batch = (int)batch, g.out_f32 = out_f32;
  return nimble::output_stays(g, slices);
}
extern "C" int any_output_stays(int64_t tiles, int64_t K, int out_f32) { return nimble::any_output_stays(tiles, K, out_f32 != 0); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(RULES)
    lib = str(d / "rules.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    str(d / "rules.cpp"), "-o", lib], check=True)
    lib = ctypes.CDLL(lib)
    lib.output_stays.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_uint64, ctypes.c_int64]
    lib.any_output_stays.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return lib


def test_small_tiles(rules):
    """Written through: 2 to 9 % faster.  The others would be 3 to 90 % slower."""
    for M, N, K, through in ((515, 1001, 1003, True), (700, 1400, 1399, True), (1433, 241, 251, True), (4610, 212, 52, True),
                             (1287, 1517, 111, True), (724, 1381, 421, False), (3038, 470, 339, False), (3000, 1001, 129, False), (12205, 147, 138, False), (11134, 1861, 277, False), (6000, 4001, 33, False)):
        p = nb.dense_plan(M, N, K, out_dtype=nb.F32)
        assert p.bn == 64
        assert rules.any_output_stays(p.grid[0], K, 1) == (not through), (M, N, K)
        assert rules.any_output_stays(p.grid[0], K, 0) == 1


def test_tiles(rules):
    """Written through: 4 to 17 % faster (the second 5).  The others would be 2 to 80 % slower."""
    f32, bf16 = 1, 0
    for batch, M, N, K, out, through in (
            (1, 4096, 4096, 64, bf16, True), (1, 20000, 10240, 128, bf16, True), (1, 700, 24576, 1536, bf16, True),
            (1, 8658, 696, 128, bf16, True), (1, 835, 8336, 480, bf16, True), (1, 4096, 4104, 64, bf16, True),
            (1, 706, 328, 288, bf16, False), (1, 3767, 4616, 1024, bf16, False), (1, 12869, 2488, 960, bf16, False),
            (1, 10201, 7736, 64, bf16, False), (37, 1916, 912, 64, bf16, False),
            (1, 4736, 2048, 512, f32, True), (1, 4096, 4096, 256, f32, True), (1, 385, 5760, 1280, f32, True),
            (12, 1024, 1024, 64, f32, True), (24, 1024, 1024, 64, f32, False), (12, 2048, 2048, 64, f32, False),
            (1, 2000, 12000, 1536, f32, False), (1, 700, 12288, 1536, f32, False), (1, 466, 19520, 320, f32, False),
            (1, 3000, 4104, 256, f32, False), (1, 10201, 3864, 64, f32, False), (46, 1004, 632, 64, f32, False)):
        assert rules.output_stays(batch, M, N, K, out, 1 << 20, 1) == (not through), (batch, M, N, K, out)
    # rows of whole pieces from an address that is none; slices of K, whatever their size, have a rule of their own
    assert rules.output_stays(1, 20000, 10240, 128, bf16, (1 << 20) + 16, 1) == 1
    assert rules.output_stays(1, 4096, 4096, 64, f32, (1 << 20) + 32, 1) == 1
    assert rules.output_stays(1, 3000, 4104, 8192, f32, 1 << 20, 2) == 0


def check(M, N, K, out, offset=0, batch=1, force=nb.VAR_AUTO):
    from paper_2006_03031_amd import runtime as rt
    print(f"{batch} x {M}x{N}x{K} to {out}, {offset} elements off", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    x = torch.empty((batch, M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((batch, N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    n = batch * M * N
    buf = torch.full((offset + n + 256,), 768.0, dtype=torch.float32 if out == nb.F32 else torch.bfloat16, device="cuda")
    y = buf[offset:offset + n].view(batch, M, N)
    if batch == 1:
        rt.dense(x[0], w[0], None, nb.EPI_NONE, out, out=y[0], force_variant=force)
    else:
        rt.batch_matmul(x, w, True, 1.0, out, out=y)
    assert bool((buf[:offset] == 768.0).all()) and bool((buf[offset + n:] == 768.0).all())
    for b in range(batch):
        wt = w[b].double().t().contiguous()
        for r in range(0, M, 4096):
            xs = x[b, r:r + 4096].double()
            ref = torch.matmul(xs, wt)
            # f32 sums of K products: K eps of the sum of magnitudes at the very most; bf16: half a unit in the last place more
            bound = torch.matmul(xs.abs(), wt.abs()) * (K + 1) * 2.0 ** -24
            if out == nb.BF16:
                bound += ref.abs() * 2.0 ** -8
            assert bool(((y[b, r:r + 4096].double() - ref).abs() <= bound).all()), (b, r)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,M,N,K", [(1, 1023, 1001, 65), (1, 1025, 1001, 129), (2, 1023, 1001, 65), (2, 1025, 1001, 65),
                                         (4, 511, 511, 33), (1, 515, 1001, 1003), (1, 1, 17, 9)])
@pytest.mark.parametrize("out", [nb.BF16, nb.F32])
def test_small_tiles_results(batch, M, N, K, out):
    check(M, N, K, out, batch=batch)


T32, T64, T128, T256X128, T256 = 2, 3, 4, 5, 6
HEIGHTS = (128, 160, 192, 224, 256, 288, 320)


@pytest.mark.gpu
@pytest.mark.parametrize("K", [128, 160, 3072])
@pytest.mark.parametrize("variant,rows", [(T32, 0), (T64, 0), (T128, 0), (T256X128, 0)] + [(T256, h) for h in HEIGHTS])
@pytest.mark.parametrize("out", [nb.BF16, nb.F32])
def test_every_tile_with_rows_in_pieces(variant, rows, K, out):
    """Plain stores of small outputs: eight waves, four of a tile's own, one per SIMD (K = 3072), stages of 64 and of 32 k (160);
    rows of whole tiles from an address between pieces (heights other than 256 are built for those only)."""
    force = variant | (rows // 16 << 16)
    if rows in (0, 256):
        check(517, 1000, K, out, force=force)
    check(509, 1024, K, out, offset=8 if out == nb.BF16 else 4, force=force)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,M,N,K,out,offset", [
    (1, 19001, 1000, 192, nb.BF16, 0), (1, 12869, 2488, 192, nb.BF16, 0), (1, 13003, 2056, 2048, nb.BF16, 0),  # walks of several tiles
    (1, 6145, 6144, 64, nb.BF16, 8), (1, 6144, 6144, 128, nb.BF16, 8), (1, 4352, 4096, 64, nb.F32, 0),         # whole tiles
    (1, 8449, 2048, 1024, nb.F32, 0), (3, 2049, 2104, 64, nb.BF16, 0), (5, 257, 264, 64, nb.F32, 0),
    (1, 1100, 4096, 1024, nb.F32, 4), (1, 3000, 504, 64, nb.BF16, 0)])
def test_tiles_results(batch, M, N, K, out, offset):
    check(M, N, K, out, offset, batch)

"""Tiles of 192 x 256 shared by two workgroups, half the columns each: what the plan says (CPU) and the results
against float64 (GPU) at the edges of tiles, K stages and the chip."""
import ctypes
import os
import random
import subprocess

import pytest

torch = pytest.importorskip("torch")
import paper_2006_03031_amd as nb
from paper_2006_03031_amd import binding, build


def is_halved(p):
    return (p.variant, p.bm, p.bn, p.split_k, p.grid[1]) == (6, 192, 256, 1, 2)


def halved(M, N, K):
    return is_halved(nb.dense_plan(M, N, K))


def test_the_plan():
    for M, N, K in ((1100, 4096, 1024), (1536, 4096, 1024), (4200, 1024, 4096), (6144, 1024, 4096), (6000, 768, 3072)):
        p = nb.dense_plan(M, N, K)
        assert halved(M, N, K) and p.grid[0] == -(-M // 192) * (N // 256) <= 128 and p.block == 512, (M, N, K, p)
        assert p.k * 192 + p.r == M and p.residue_copy == (p.r != 0) and p.workspace_bytes == 0
    # 128-row tiles in one round, more than one round of halves, K or N they are not built for, one workgroup when forced
    for M, N, K in ((1024, 4096, 1024), (1537, 4096, 1024), (4096, 1024, 4096), (6145, 1024, 4096), (1100, 4096, 1056),
                    (1100, 4096 + 128, 1024)):
        assert not halved(M, N, K), (M, N, K)
    assert nb.dense_plan(1100, 4096, 1024, force_variant=6 | (12 << 16)).grid[1] == 1
    # weights from memory, 128-row tiles in one round: faster (336 x 9984 x 3456 37.1 us, 43.6 in halves); not in two rounds
    for M, N, K in ((336, 9984, 3456), (378, 10240, 4288), (321, 10496, 3072), (636, 6400, 5312)):
        p = nb.dense_plan(M, N, K)
        assert (p.variant, p.bm, p.split_k) == (4, 128, 1) and p.grid[0] <= 256, (M, N, K, p)
    for M, N, K in ((259, 11520, 3968), (400, 10240, 3648), (642, 6912, 9856)):
        assert halved(M, N, K), (M, N, K)


PLAN_WITHIN = """
#include "nimble_internal.h"
extern "C" int plan_within(int64_t M, int64_t N, int64_t K, int epilogue, uint64_t workspace, nimble_plan* p) {
  nimble::PlanOptions opt;
  opt.max_workspace = workspace;
  return nimble::plan_dense(1, M, N, K, epilogue, NIMBLE_VAR_AUTO, opt, p);
}
"""


@pytest.fixture(scope="module")
def plan_within(tmp_path_factory):
    """The dispatch function as the entry points call it: within the scratch that the caller brought."""
    d = tmp_path_factory.mktemp("plan")
    (d / "plan_within.cpp").write_text(PLAN_WITHIN)
    lib = str(d / "plan_within.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    str(d / "plan_within.cpp"), os.path.join(build.CSRC, "nimble_host.cpp"), "-o", lib], check=True)
    fn = ctypes.CDLL(lib).plan_within
    fn.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_uint64, ctypes.POINTER(binding._CPlan)]

    def plan(M, N, K, epilogue, workspace):
        c = binding._CPlan()
        assert fn(M, N, K, epilogue, workspace, ctypes.byref(c)) == 0
        return binding._plan(c)
    return plan


def test_halves_run_in_any_workspace(plan_within):
    """Halves need no workspace: where the plan names them they run with none and with the built-in scratch.  The shapes
    are those whose best launch without halves would cut K in four, and random ones with weights beyond the caches."""
    rng = random.Random(3)
    shapes = [(262, 11008, 11136), (280, 11008, 10432), (392, 8960, 12160), (616, 6656, 10752)]
    shapes += [(rng.randint(200, 1000), 256 * rng.randint(16, 48), 64 * rng.randint(100, 191)) for _ in range(20000)]
    n = 0
    for M, N, K in shapes:
        for epilogue in (nb.EPI_NONE, nb.EPI_BIAS_GELU_ERF):
            want = nb.dense_plan(M, N, K, epilogue)
            if is_halved(want):
                n += 1
                for workspace in (0, binding.NOALLOC_SCRATCH_BYTES, 64 << 20):
                    assert plan_within(M, N, K, epilogue, workspace) == want, (M, N, K, epilogue, workspace)
    assert n > 1000
    for M, N, K in shapes[:4]:
        assert halved(M, N, K)


def test_products_with_b_kn_take_the_halves_by_their_own_price():
    """A.B with b [K, N] runs on b transposed where the launch found for that, here halves, is estimated to be done
    sooner than 64 x 64 tiles on b as it is.  Both estimates written out once more, in microseconds."""
    def halves(M, N, K):
        tiles, stages = -(-M // 192) * (N // 128), K // 32
        us = 3.0 + (0.244 + 0.00043 * max(0, tiles - 128)) * stages
        return us + 8.0 + 0.3e-6 * (N * K * 2) + 0.12e-6 * (M * K + N * K + M * N) * 2

    def any_kernel(M, N, K):
        tiles, stages = -(-M // 64) * (N // 64), -(-K // 64)
        four = K >= 512 and tiles <= 256
        lone = 3.5 + 1.14 * -(-stages // 4) if four else 3.0 + 0.67 * stages
        per_cu = tiles / 256 if tiles <= 256 else max(2.0, tiles / 256)
        return max(lone, 3.0 + per_cu * (0.6 + 0.42 * stages))

    rng = random.Random(4)
    shapes = [(rng.randint(200, 2000), 256 * rng.randint(1, 48), 64 * rng.randint(5, 190)) for _ in range(30000)]
    seen = {True: 0, False: 0}
    # (the first five were given to the 64 x 64 tiles by the price of whole tiles)
    for M, N, K in [(480, 8448, 1344), (661, 6400, 768), (370, 10240, 6400), (375, 10496, 5120), (624, 6656, 832)] + shapes:
        if is_halved(nb.batch_matmul_plan(1, M, N, K, True)) and M * N * K >= 32e6:
            p, transposed = nb.batch_matmul_plan(1, M, N, K, False), halves(M, N, K) < any_kernel(M, N, K)
            assert (p.bn == 256) == is_halved(p) == transposed, (M, N, K, p, halves(M, N, K), any_kernel(M, N, K))
            seen[transposed] += 1
    assert seen[True] > 500, seen


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1035, 4096, 768), (1152, 4096, 832), (1153, 4096, 896), (1536, 4096, 768), (2115, 2304, 768),
                                   (4225, 1024, 2112), (5569, 768, 768), (12001, 512, 640)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("epilogue", [nb.EPI_NONE, nb.EPI_BIAS, nb.EPI_BIAS_GELU_ERF])
def test_results(M, N, K, out, epilogue):
    from paper_2006_03031_amd import runtime as rt
    assert is_halved(nb.dense_plan(M, N, K, epilogue))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    dt = torch.float32 if out == "f32" else torch.bfloat16
    buf = torch.full((M * N + 256,), 768.0, dtype=dt, device="cuda")
    y = rt.dense(x, w, None if epilogue == nb.EPI_NONE else b, epilogue, nb.F32 if out == "f32" else nb.BF16,
                 out=buf[:M * N].view(M, N))
    bias = b.double() * (epilogue != nb.EPI_NONE)
    ref = torch.matmul(x.double(), w.double().t().contiguous()) + bias
    # f32 sums of K products: K eps of the sum of magnitudes at the very most; bf16: half a unit in the last place more
    bound = (torch.matmul(x.double().abs(), w.double().abs().t().contiguous()) + bias.abs()) * (K + 1) * 2.0 ** -24
    if epilogue == nb.EPI_BIAS_GELU_ERF:
        # its slope is at most 1.13, its fit 2.5e-5 off, its exponential and reciprocal a few units in the last place
        ref = torch.nn.functional.gelu(ref)
        bound = 1.13 * bound + 2.5e-5 + ref.abs() * 2.0 ** -20
    bound += ref.abs() * 2.0 ** -8 if out == "bf16" else 0
    assert bool(((y.double() - ref).abs() <= bound).all())
    assert bool((buf[M * N:] == 768.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("trans_b", [True, False])
@pytest.mark.parametrize("M,N,K", [(1035, 4096, 768), (1153, 4096, 896), (4225, 1024, 2112)])
def test_single_products(M, N, K, trans_b):
    """A product of one batch, scaled, with b [N, K] or transposed into the workspace."""
    from paper_2006_03031_amd import runtime as rt
    assert is_halved(nb.batch_matmul_plan(1, M, N, K, trans_b, nb.F32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    a = torch.empty((1, M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((1, N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    y = rt.batch_matmul(a, b if trans_b else b.transpose(1, 2).contiguous(), trans_b, 0.375, nb.F32)
    ref = torch.matmul(a[0].double(), b[0].double().t().contiguous()) * 0.375
    mag = torch.matmul(a[0].double().abs(), b[0].double().abs().t().contiguous()) * 0.375
    assert bool(((y[0].double() - ref).abs() <= mag * (K + 1) * 2.0 ** -24).all())

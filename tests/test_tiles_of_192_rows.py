"""Tiles of 192 x 256 shared by two workgroups, half the columns each: what the plan says (CPU) and the results
against float64 (GPU) at the edges of tiles, K stages and the chip."""
import pytest

torch = pytest.importorskip("torch")
import paper_2006_03031_amd as nb


def halved(M, N, K):
    p = nb.dense_plan(M, N, K)
    return (p.variant, p.bm, p.bn, p.split_k, p.grid[1]) == (6, 192, 256, 1, 2)


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


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1035, 4096, 768), (1152, 4096, 832), (1153, 4096, 896), (1536, 4096, 768), (2115, 2304, 768),
                                   (4225, 1024, 2112), (5569, 768, 768), (12001, 512, 640)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_results(M, N, K, out):
    from paper_2006_03031_amd import runtime as rt
    assert halved(M, N, K)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    dt = torch.float32 if out == "f32" else torch.bfloat16
    buf = torch.full((M * N + 256,), 768.0, dtype=dt, device="cuda")
    y = rt.dense(x, w, b, nb.EPI_BIAS, nb.F32 if out == "f32" else nb.BF16, out=buf[:M * N].view(M, N))
    ref = torch.matmul(x.double(), w.double().t().contiguous()) + b.double()
    # f32 sums of K products: K eps of the sum of magnitudes at the very most; bf16: half a unit in the last place more
    mag = torch.matmul(x.double().abs(), w.double().abs().t().contiguous()) + b.double().abs()
    bound = mag * (K + 1) * 2.0 ** -24 + (ref.abs() * 2.0 ** -8 if out == "bf16" else 0)
    assert bool(((y.double() - ref).abs() <= bound).all())
    assert bool((buf[M * N:] == 768.0).all())

"""Tiles run by four waves (one per SIMD) against float64, at the edges of tiles, stages, ring slots and walks."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

T128, T256X128, T256 = 4, 5, 6


@pytest.fixture(scope="module")
def nb():
    import paper_2006_03031_amd as nb
    nb.load()
    return nb


def forced(variant, rows=0, split=1):
    return variant | (split << 8 if split > 1 else 0) | (rows // 16 << 16)


# every height, rows and columns of the last tiles partly empty, an odd number of stages; several tiles per workgroup, as
# many stages as ring slots, one more, a ring that turns from tile to tile; K in two, also of unequal lengths
CASES = [(T256, h, 2 * h + 5, 520 if h == 256 else 512, 2112, 1) for h in (128, 160, 192, 224, 256)] + [
    (T256, 256, 10243, 2056, 1024, 1), (T256, 256, 10240, 2048, 1088, 1), (T256, 160, 6405, 2048, 1088, 1),
    (T256, 128, 16611, 7680, 128, 1), (T256, 128, 16640, 7680, 192, 1), (T256, 256, 300, 512, 4224, 2), (T256, 256, 300, 512, 4160, 2),
    (T256X128, 0, 517, 264, 2112, 1), (T256X128, 0, 13321, 6600, 192, 1), (T256X128, 0, 13312, 6656, 256, 1),
    (T256X128, 0, 13321, 6600, 320, 1), (T256X128, 0, 300, 256, 4224, 2), (T256X128, 0, 300, 256, 4160, 2),
    (T128, 0, 133, 264, 3136, 1), (T128, 0, 1, 128, 3072, 1), (T128, 0, 2048, 2040, 3072, 1)]


@pytest.mark.parametrize("variant,rows,M,N,K,split", CASES)
@pytest.mark.parametrize("epilogue,out", [("none", "bf16"), ("bias", "bf16"), ("gelu", "bf16"), ("bias", "f32")])
def test_four_waves(nb, variant, rows, M, N, K, split, epilogue, out):
    from paper_2006_03031_amd import runtime as rt
    force = forced(variant, rows, split)
    plan = nb.dense_plan(M, N, K, force_variant=force)
    assert plan.block == 256 and plan.split_k == split, plan
    print(f"four waves {variant} {rows} {M}x{N}x{K} {split} {epilogue} {out}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    epi = {"none": nb.EPI_NONE, "bias": nb.EPI_BIAS, "gelu": nb.EPI_BIAS_GELU_ERF}[epilogue]
    dt = torch.float32 if out == "f32" else torch.bfloat16
    buf = torch.full((M * N + 256,), 768.0, dtype=dt, device="cuda")
    y = rt.dense(x, w, b if epilogue != "none" else None, epi, nb.F32 if out == "f32" else nb.BF16, force_variant=force,
                 out=buf[:M * N].view(M, N))
    assert bool((buf[M * N:] == 768.0).all())
    wt, bias = w.double().t().contiguous(), 0 if epilogue == "none" else b.double()
    for r in range(0, M, 4096):
        xs = x[r:r + 4096].double()
        ref = torch.matmul(xs, wt) + bias
        # f32 sums of K products: K eps of the sum of magnitudes at the very most (GELU's slope is below 1.13, its fit
        # within 2.5e-5); bf16: half a unit in the last place more
        bound = (torch.matmul(xs.abs(), wt.abs()) + (0 if epilogue == "none" else bias.abs())) * (K + 1) * 2.0 ** -24
        if epilogue == "gelu":
            ref, bound = torch.nn.functional.gelu(ref), bound * 1.13 + 3e-5
        if out == "bf16":
            bound += ref.abs() * 2.0 ** -8
        assert bool(((y[r:r + 4096].double() - ref).abs() <= bound).all()), r


@pytest.mark.parametrize("variant,rows,M,N,K", [(T256, 256, 8192, 2048, 1024), (T256, 160, 5120, 2048, 1088), (T256X128, 0, 8192, 1024, 1024),
                                                (T128, 0, 4096, 2048, 3072)])
@pytest.mark.parametrize("epilogue,out", [("gelu", "bf16"), ("bias", "f32")])
def test_the_same_bits_as_the_ring_kernels(nb, variant, rows, M, N, K, epilogue, out):
    """One of M rows and twice as many runs four waves, the other a ring kernel: the rows that both have are the same."""
    from paper_2006_03031_amd import runtime as rt
    force = forced(variant, rows)
    few, many = (M, 2 * M) if variant != T128 else (M // 2, M)
    waves = [nb.dense_plan(m, N, K, force_variant=force).grid[0] for m in (few, many)]
    blocks = [nb.dense_plan(m, N, K, force_variant=force).block for m in (few, many)]
    assert waves == [256, 512] and blocks == ([512, 256] if variant != T128 else [256, 256]), (waves, blocks)
    print(f"same bits {variant} {rows} {few} / {many} x {N}x{K} {epilogue} {out}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + K)
    x = torch.empty((many, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    epi, dt = (nb.EPI_BIAS if epilogue == "bias" else nb.EPI_BIAS_GELU_ERF), (nb.F32 if out == "f32" else nb.BF16)
    y = [rt.dense(x[:m], w, b, epi, dt, force_variant=force) for m in (few, many)]
    assert torch.equal(y[0], y[1][:few])


@pytest.mark.parametrize("batch,M,N,K", [(8, 1000, 1000, 2048), (4, 1000, 1024, 4096), (2, 2048, 2048, 2048), (5, 1000, 1032, 2112)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_batches(nb, batch, M, N, K, out):
    from paper_2006_03031_amd import runtime as rt
    dt = nb.F32 if out == "f32" else nb.BF16
    plan = nb.batch_matmul_plan(batch, M, N, K, True, dt)
    assert plan.block == 256 and (plan.bm, plan.bn) in ((256, 128), (128, 128)) and plan.grid[2] == batch, plan
    print(f"batch {batch} {M}x{N}x{K} {out}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    a = torch.empty((batch, M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((batch, N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    n = batch * M * N
    buf = torch.full((n + 256,), 768.0, dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    y = rt.batch_matmul(a, b, True, 0.5, dt, out=buf[:n].view(batch, M, N))
    assert bool((buf[n:] == 768.0).all())
    for z in range(batch):
        az, bz = a[z].double(), b[z].double().t().contiguous()
        ref = 0.5 * torch.matmul(az, bz)
        # as above; the factor is a power of two
        bound = 0.5 * torch.matmul(az.abs(), bz.abs()) * (K + 1) * 2.0 ** -24
        if out == "bf16":
            bound += ref.abs() * 2.0 ** -8
        assert bool(((y[z].double() - ref).abs() <= bound).all()), z


def test_the_dispatch_takes_four_waves_for_long_walks(nb):
    assert nb.dense_plan(16129, 1024, 4096).block == 256 and nb.dense_plan(8192, 1024, 4096).block == 256
    assert nb.dense_plan(2113, 1024, 4096).block == 256
    assert nb.dense_plan(2113, 4096, 1024).block == 512 and nb.dense_plan(2113, 1024, 2048).block == 512

"""Large products that the ring kernels cannot run (K not whole 32-wide stages, output rows not whole 16-byte pieces):
the variant's own tiles with every access bounds-checked, against float64."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    import paper_2006_03031_amd as nb
    nb.load()
    return nb


def _operands(M, N, K, T=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + 7 * N + 13 * K)
    a = torch.empty((T, M, K) if T else (M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((T, N, K) if T else (N, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    bias = torch.empty(N, device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    return a, b, bias


def _check(got, ref, f32, what):
    # f32: sums of K products of magnitude 1/3 in another order; bf16: that and one rounding
    err = ((got.double() - ref).abs() / (ref.abs() + ref.abs().mean())).max().item()
    assert err <= (2.0 ** -14 if f32 else 2.0 ** -8), (what, err)


# 64-row, 128-row, 256 x 128 and 256 x 256 tiles, more of them than workgroups are resident at once for most; K of 8, 16 and
# 24 past whole stages, less than one stage of 64; N whole tiles, a multiple of 8, of 4 and of nothing; a last row of tiles of one row
@pytest.mark.parametrize("M,N,K", [(3130, 1024, 904), (2049, 4104, 40), (1153, 4240, 2648), (10753, 3328, 872), (8505, 8192, 528),
                                   (2561, 3656, 4560), (2900, 3471, 4568), (4097, 4100, 904)])
@pytest.mark.parametrize("epilogue", ["none", "bias", "bias_gelu"])
def test_dense(nb, M, N, K, epilogue):
    from paper_2006_03031_amd import runtime as rt
    x, w, b = _operands(M, N, K)
    epi = {"none": nb.EPI_NONE, "bias": nb.EPI_BIAS, "bias_gelu": nb.EPI_BIAS_GELU_ERF}[epilogue]
    f32 = epilogue == "none"
    print(f"dense {M} x {N} x {K} {epilogue}", flush=True)
    buf = torch.full((M * N + 256,), 768.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    rt.dense(x, w, b, epi, nb.F32 if f32 else nb.BF16, out=buf[:M * N].view(M, N))
    assert bool((buf[M * N:] == 768.0).all())
    rows = torch.cat([torch.arange(0, 3), torch.arange(M // 2, M // 2 + 130), torch.arange(M - 258, M)]).cuda()
    ref = x[rows].double() @ w.double().T.contiguous()
    if not f32:
        ref = ref + b.double()
        ref = torch.nn.functional.gelu(ref) if epilogue == "bias_gelu" else ref
    _check(buf[:M * N].view(M, N)[rows], ref, f32, (M, N, K, epilogue))


@pytest.mark.parametrize("T,M,N,K", [(8, 1000, 1000, 1000), (3, 2049, 1032, 520), (12, 520, 1028, 904)])
def test_batch_matmul(nb, T, M, N, K):
    from paper_2006_03031_amd import runtime as rt
    a, b, _ = _operands(M, N, K, T)
    print(f"batch_matmul {T} x {M} x {N} x {K}", flush=True)
    for od, dt in ((nb.F32, torch.float32), (nb.BF16, torch.bfloat16)):
        buf = torch.full((T * M * N + 256,), 768.0, dtype=dt, device="cuda")
        rt.batch_matmul(a, b, True, 0.5, od, out=buf[:T * M * N].view(T, M, N))
        assert bool((buf[T * M * N:] == 768.0).all())
        for t in (0, T - 1):
            _check(buf[:T * M * N].view(T, M, N)[t], 0.5 * (a[t].double() @ b[t].double().T.contiguous()), od == nb.F32, (t, T, M, N, K))


# b [T, K, N] transposed into the workspace, then the ring kernels (whole and partly empty last tiles) or the tile kernel
@pytest.mark.parametrize("T,M,N,K", [(1, 4096, 1024, 512), (4, 1905, 2048, 1408), (12, 2311, 392, 896), (24, 1590, 1536, 384),
                                     (2, 937, 2464, 1120), (8, 1000, 1000, 1000), (3, 2050, 1032, 1048)])
def test_batch_matmul_on_b_transposed(nb, T, M, N, K):
    from paper_2006_03031_amd import runtime as rt
    p = nb.batch_matmul_plan(T, M, N, K, False)
    assert p.bn != 64 and p.workspace_bytes == 2 * T * N * K, p   # this launch, not the one that reads b as it is
    a, b, _ = _operands(M, N, K, T)
    b = b.transpose(1, 2).contiguous()
    print(f"batch_matmul A.B {T} x {M} x {N} x {K}", flush=True)
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    exact = torch.empty(p.workspace_bytes + 256, dtype=torch.uint8, device="cuda").fill_(77)
    for od, dt in ((nb.F32, torch.float32), (nb.BF16, torch.bfloat16)):
        for ws in (exact[:p.workspace_bytes], none):
            buf = torch.full((T * M * N + 256,), 768.0, dtype=dt, device="cuda")
            rt.batch_matmul(a, b, False, 0.5, od, out=buf[:T * M * N].view(T, M, N), workspace=ws)
            assert bool((buf[T * M * N:] == 768.0).all()) and bool((exact[p.workspace_bytes:] == 77).all())
            rows = torch.cat([torch.arange(0, 3), torch.arange(M - 260, M)]).cuda()
            for t in (0, T - 1):
                _check(buf[:T * M * N].view(T, M, N)[t][rows], 0.5 * (a[t][rows].double() @ b[t].double()), od == nb.F32,
                       (t, T, M, N, K, ws.numel()))


@pytest.mark.parametrize("M,N,K,part", [(4096, 4096, 4104, 0.8),    # K not whole stages: 153 us against 287 in 64 x 64 tiles
                                        (423, 2928, 3648, 0.8)])   # a partly empty last tile column: 20 against 37
def test_large_products_do_not_run_in_small_tiles(nb, M, N, K, part):
    """The automatic plan against the generic variant (64 x 64 tiles), timed."""
    from paper_2006_03031_amd import runtime as rt
    x, w, b = _operands(M, N, K)
    times = {}
    for variant in (nb.VAR_AUTO, 0, nb.VAR_AUTO, 0):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
        for e in ev:
            for _ in range(4):   # (more work than the calls take on the host)
                rt.dense(x, w, b, nb.EPI_BIAS, force_variant=variant)
            e.record()
        torch.cuda.synchronize()
        ts = sorted(ev[i].elapsed_time(ev[i + 1]) for i in range(11))
        times[variant] = min(times.get(variant, 1e9), ts[5])
    assert times[nb.VAR_AUTO] < part * times[0], times

"""Products of any shape and alignment (any_kernel, the 16-row blocks of the generic variant, the last
tile column of the ring kernels) against the CPU oracle, at the edges of tiles, chunks and stages."""
import numpy as np
import pytest

import oracle
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-3                 # normwise, as in test_gpu_parity
GATE_BF16, GATE_F32 = 2.0 ** -7, 2.0 ** -14   # element-wise: half an ulp of bf16 times four; summation order in f32


@pytest.fixture(scope="module")
def nb():
    import paper_2006_03031_amd as nb
    nb.load()
    return nb


def _check(got, ref, what, f32):
    rel = GATE_F32 if f32 else GATE_BF16
    e = oracle.normwise_rel_error(got, ref)
    assert e <= TOL, ("normwise", what, e)
    x = oracle.elementwise_excess(got, ref, rel, rel)
    assert x <= 1.0, ("element-wise", what, x)


def _guarded(shape, dtype):
    """An output with a guard row behind it that the kernel must leave alone."""
    n = int(np.prod(shape))
    buf = torch.full((n + 256,), 768.0, dtype=dtype, device="cuda")
    return buf, buf[:n].view(shape)


# K: shorter than a chunk, a chunk's and a stage's edges, many stages for one and for four groups of waves;
# M and N: one row, edges of the 16-row blocks and of the 64-wide tiles, too many blocks for the row kernel
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (3, 5, 3), (17, 33, 7), (16, 16, 9), (65, 63, 15), (64, 64, 65), (130, 129, 71),
                                   (1, 257, 1003), (16, 9000, 63), (33, 130, 511), (600, 300, 1), (600, 1000, 7), (577, 961, 63),
                                   (577, 961, 129), (515, 1001, 513), (700, 643, 1021), (2100, 1027, 67), (515, 1001, 1000),
                                   (600, 1000, 40), (640, 1001, 64)])
def test_dense_of_any_shape(nb, M, N, K):
    from gpu_util import from_dev, to_dev
    from paper_2006_03031_amd import runtime as rt
    rng = np.random.default_rng([11, M, N, K])
    x, w, b = wl.uniform_bf16(rng, (M, K)), wl.uniform_bf16(rng, (N, K)), wl.uniform_bf16(rng, (N,))
    dx, dw, db = to_dev(x), to_dev(w), to_dev(b)
    print(f"dense {M} x {N} x {K}", flush=True)
    for name, epi, od in (("none", nb.EPI_NONE, nb.F32), ("bias", nb.EPI_BIAS, nb.BF16)):
        buf, out = _guarded((M, N), torch.float32 if od == nb.F32 else torch.bfloat16)
        rt.dense(dx, dw, db if name == "bias" else None, epi, od, out=out)
        got = from_dev(buf)
        assert np.all(got[M * N:] == 768.0), ("wrote past the output", name)
        _check(got[:M * N].reshape(M, N), oracle.dense(x.f32, w.f32, b.f32 if name == "bias" else None, name), (name, M, N, K),
               od == nb.F32)


# K odd (every other row starts at an odd element) and even at the edges of chunks, of stages and of rounds of four stages; one
# group of waves (more than 256 tiles, or one stage) and four, and the 16 x 16 blocks that small grids run in up to K = 576; the last element of the last row is the end of the buffer
@pytest.mark.parametrize("K", [5, 7, 8, 9, 57, 63, 64, 65, 66, 71, 72, 73, 127, 129, 191, 193, 255, 256, 257, 263, 321, 577, 639, 641, 769])
@pytest.mark.parametrize("M,N", [(80, 1001), (129, 1001), (63, 2003), (1100, 1031)])
def test_rows_that_start_at_odd_elements(nb, M, N, K):
    from paper_2006_03031_amd import runtime as rt
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K * 10 + M)
    uniform = lambda *shape: torch.empty(shape, device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    x, w, b = uniform(M, K), uniform(N, K), uniform(N)
    ref = x.double() @ w.double().T.contiguous()
    print(f"odd rows {M} x {N} x {K}", flush=True)
    for epi, od in ((nb.EPI_NONE, nb.F32), (nb.EPI_BIAS, nb.BF16), (nb.EPI_BIAS, nb.F32)):
        buf, out = _guarded((M, N), torch.float32 if od == nb.F32 else torch.bfloat16)
        rt.dense(x, w, b if epi == nb.EPI_BIAS else None, epi, od, out=out)
        assert bool((buf[M * N:] == 768.0).all()), "wrote past the output"
        want = ref + b.double() if epi == nb.EPI_BIAS else ref
        err = ((out.double() - want).abs() / (want.abs() + want.abs().mean())).max().item()
        assert err <= (GATE_F32 if od == nb.F32 else 2.0 ** -8), (M, N, K, epi, od, err)   # summation order; one rounding


def test_more_tiles_than_one_launch_holds(nb):
    """4.4 million tiles of 64 x 64 (an output of 36 GB): two launches."""
    from paper_2006_03031_amd import runtime as rt
    M, N, K = 400_003, 45_001, 40
    p = nb.dense_plan(M, N, K, nb.EPI_NONE)
    assert (p.bm, p.bn) == (64, 64) and p.grid[1] == 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    print(f"dense {M} x {N} x {K}", flush=True)
    buf = torch.empty(M * N + 256, dtype=torch.bfloat16, device="cuda").fill_(768.0)
    y = rt.dense(x, w, None, nb.EPI_NONE, nb.BF16, out=buf[:M * N].view(M, N))
    assert bool((buf[M * N:] == 768.0).all())
    rows = torch.cat([torch.arange(0, 2), torch.arange(M // 2, M // 2 + 2), torch.arange(M - 66, M)]).cuda()
    ref = x[rows].double() @ w.double().T.contiguous()
    assert ((y[rows].double() - ref).abs() / (ref.abs() + ref.abs().mean())).max().item() <= 2.0 ** -8
    for r0 in range(0, M, 20_000):   # every tile was written
        assert bool((y[r0:r0 + 20_000, ::64] != 768.0).all()), r0
    del buf, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,M,N,K", [(3, 65, 64, 33), (2, 64, 63, 64), (2, 1, 1, 1), (3, 70, 7, 9), (2, 129, 65, 257), (1, 63, 72, 600),
                                     (12, 33, 64, 513), (5, 200, 200, 1003), (2, 64, 8, 512)])
@pytest.mark.parametrize("trans_b", [False, True])
def test_batch_matmul_of_any_shape(nb, T, M, N, K, trans_b):
    from gpu_util import from_dev, to_dev
    from paper_2006_03031_amd import runtime as rt
    rng = np.random.default_rng([12, T, M, N, K, trans_b])
    a, b = wl.uniform_bf16(rng, (T, M, K)), wl.uniform_bf16(rng, (T, N, K) if trans_b else (T, K, N))
    print(f"batch_matmul {T} x {M} x {N} x {K} {trans_b}", flush=True)
    for od in (nb.F32, nb.BF16):
        buf, out = _guarded((T, M, N), torch.float32 if od == nb.F32 else torch.bfloat16)
        rt.batch_matmul(to_dev(a), to_dev(b), trans_b, 0.5, od, out=out)
        got = from_dev(buf)
        assert np.all(got[T * M * N:] == 768.0), "wrote past the output"
        _check(got[:T * M * N].reshape(T, M, N), oracle.batch_matmul(a.f32, b.f32, trans_b, 0.5), (T, M, N, K, trans_b, od),
               od == nb.F32)


# a partly empty last tile column in the ring kernels: 1000 and 1032 columns leave 104 and 8 of them in the last tile;
# every tile of the family, both outputs
@pytest.mark.parametrize("name", ["t32x128", "t64x128", "t128x128", "t256x128", "t256x256"])
@pytest.mark.parametrize("N,K", [(1000, 1024), (1032, 1056)])
def test_ring_kernels_mask_the_last_columns(nb, name, N, K):
    from gpu_util import from_dev, to_dev
    from paper_2006_03031_amd import runtime as rt
    M = 5125
    variant = [i for i in range(7) if nb.variant_name(i) == name][0]
    rng = np.random.default_rng([13, N, K])
    x, w, b = wl.uniform_bf16(rng, (M, K)), wl.normal_bf16(rng, (N, K)), wl.uniform_bf16(rng, (N,))
    rows = np.unique(np.concatenate([np.arange(3), rng.integers(0, M, 24), np.arange(5118, M)]))
    dx, dw, db = to_dev(x), to_dev(w), to_dev(b)
    print(f"ring {name} {N} {K}", flush=True)
    for epi, ename, od in ((nb.EPI_BIAS, "bias", nb.BF16), (nb.EPI_BIAS_GELU_ERF, "bias_gelu", nb.BF16), (nb.EPI_BIAS, "bias", nb.F32)):
        buf, out = _guarded((M, N), torch.float32 if od == nb.F32 else torch.bfloat16)
        rt.dense(dx, dw, db, epi, od, force_variant=variant, out=out)
        got = from_dev(buf)
        assert np.all(got[M * N:] == 768.0), "wrote past the output"
        _check(got[:M * N].reshape(M, N)[rows], oracle.dense(x.f32[rows], w.f32, b.f32, ename), (name, N, K, ename, od), od == nb.F32)


# the same where every workgroup walks several tiles and hands its ring to the next one, which may be the partly empty
# column's or the last row's; both ring widths (K = 192 is whole stages of 64, K = 160 is not), bias in LDS and none
@pytest.mark.parametrize("name,rows,resident", [("t32x128", 32, 512), ("t64x128", 64, 512), ("t128x128", 128, 512), ("t256x128", 256, 256),
                                                ("t256x256", 256, 256)])
@pytest.mark.parametrize("K", [192, 160])
def test_ring_kernels_walk_tiles_past_a_partly_empty_column(nb, name, rows, resident, K):
    from paper_2006_03031_amd import runtime as rt
    variant = [i for i in range(7) if nb.variant_name(i) == name][0]
    width = 256 if name == "t256x256" else 128
    N = 3 * width - 56
    M = (2 * resident // 3 + 3) * rows + 1
    assert -(-M // rows) * 3 > 2 * resident
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K + rows)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    ref = x.double() @ w.double().T.contiguous()
    print(f"ring walk {name} {M} {N} {K}", flush=True)
    for epi, od in ((nb.EPI_BIAS, nb.BF16), (nb.EPI_NONE, nb.BF16), (nb.EPI_BIAS, nb.F32)):
        buf, out = _guarded((M, N), torch.float32 if od == nb.F32 else torch.bfloat16)
        rt.dense(x, w, b if epi == nb.EPI_BIAS else None, epi, od, force_variant=variant, out=out)
        assert bool((buf[M * N:] == 768.0).all()), "wrote past the output"
        want = ref + b.double() if epi == nb.EPI_BIAS else ref
        err = ((out.double() - want).abs() / (want.abs() + want.abs().mean())).max().item()
        assert err <= (GATE_F32 if od == nb.F32 else 2.0 ** -8), (name, K, epi, od, err)   # summation order; one rounding

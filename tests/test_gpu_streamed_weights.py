"""Layers of more than 64 MB of weights against float64: up to 16 rows in the streaming kernel, which loads the weights past the caches
(up to 8 rows, and of layers beyond 256 MiB) or through them, the 8-row and the 16-row activation tile, a partly filled last block of weight
rows, the layers just above and just below the line, twice in a row with other weights in the same memory; 17 to 64 rows in one
row of tiles with K cut, past the caches and through them; and such a layer as the rest of a row split."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(8192, 4096), (5003, 6400), (4999, 6400), (515, 64000), (16389, 8192)])
@pytest.mark.parametrize("M", [1, 7, 8, 9, 16])
def test_weights_loaded_past_the_caches(M, N, K):
    import paper_2006_03031_amd as nb
    from paper_2006_03031_amd import runtime as rt
    nb.load()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * 7 + N)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    for rep in range(2):
        w.normal_(0, 0.02, generator=gen)
        print(f"streamed {M} x {N} x {K}", flush=True)
        want = x.double() @ w.double().T.contiguous() + b.double()
        for od, tol in ((nb.F32, 2.0 ** -14), (nb.BF16, 2.0 ** -8)):     # summation order; one rounding
            buf = torch.full((M * N + 256,), 768.0, dtype=torch.float32 if od == nb.F32 else torch.bfloat16, device="cuda")
            rt.dense(x, w, b, nb.EPI_BIAS, od, out=buf[:M * N].view(M, N))
            got = buf[:M * N].view(M, N).double()
            assert ((got - want).abs() / (want.abs() + want.abs().mean())).max().item() <= tol, (rep, od)
            assert bool((buf[M * N:] == 768.0).all())


# K in three, five, eight, six, sixteen and fifteen slices of all rows (32- and 64-row tiles, full and not), the last slice shorter, a layer
# beyond 256 MiB; to f32 the estimates' launch; without scratch theirs too; through the built-in scratch
CUTS = [(M, N, K, slices, to_f32) for N, K, slices, f32 in (
    (8192, 8192, 3, (8, 8, 8, 3)), (6144, 6144, 5, (8, 2, 4, 4)), (4096, 14336, 8, (16, 16, 8, 8)), (5120, 6912, 6, (16, 2, 4, 4)),
    (1280, 25600, 16, (8, 8, 8, 8)), (2048, 32768, 15, (0, 0, 16, 16)), (8192, 16448, 4, (8, 8, 8, 8)))
    for M, to_f32 in zip((17, 32, 33, 64), f32) if to_f32]


@pytest.mark.parametrize("M,N,K,slices,to_f32", CUTS)
def test_all_rows_in_one_tile_with_k_cut(M, N, K, slices, to_f32):
    import paper_2006_03031_amd as nb
    from paper_2006_03031_amd import runtime as rt
    nb.load()
    p = nb.dense_plan(M, N, K, nb.EPI_BIAS)
    assert p.bm == (32 if M <= 32 else 64) and p.split_k == slices
    assert 160 <= p.grid[0] * p.split_k <= 256 and -(-K // 64 // p.split_k) % 32 != 0
    assert nb.dense_plan(M, N, K, nb.EPI_BIAS, nb.F32).split_k == to_f32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * 5 + N)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=gen)
    want = x.double() @ w.double().T.contiguous() + b.double()
    print(f"cut {M} x {N} x {K} in {p.split_k}, to f32 in {to_f32}", flush=True)
    for od, tol in ((nb.F32, 2.0 ** -14), (nb.BF16, 2.0 ** -8)):     # summation order; one rounding
        outs = [torch.full((M, N), 768.0, dtype=torch.float32 if od == nb.F32 else torch.bfloat16, device="cuda") for _ in range(3)]
        rt.dense(x, w, b, nb.EPI_BIAS, od, out=outs[0])
        rt.dense(x, w, b, nb.EPI_BIAS, od, out=outs[1], workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
        nb.nimble_dense_noalloc_dyn(x.data_ptr(), w.data_ptr(), b.data_ptr(), outs[2].data_ptr(), M, N, K, nb.EPI_BIAS, od, rt._stream())
        for out in outs:
            assert ((out.double() - want).abs() / (want.abs() + want.abs().mean())).max().item() <= tol, od
        assert torch.equal(outs[0], outs[2])


# 5 rows streamed, 19 and 33 rows with K cut by the estimates, behind a launch of 2048 or 4096 rows
@pytest.mark.parametrize("M,N,K,rest", [(2053, 4096, 8192, 5), (2067, 4096, 14336, 19), (2081, 4096, 8192, 33), (4111, 8192, 4096, 15)])
def test_the_rest_of_a_row_split(M, N, K, rest):
    import paper_2006_03031_amd as nb
    from paper_2006_03031_amd import runtime as rt
    nb.load()
    p = nb.dense_plan(M, N, K)
    assert M - p.split_rows == rest
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=gen)
    print(f"split {M} x {N} x {K}, the rest {rest}", flush=True)
    got = rt.dense(x, w, b)
    rows = slice(p.split_rows - 64, M)
    want = x[rows].double() @ w.double().T.contiguous() + b.double()
    assert ((got[rows].double() - want).abs() / (want.abs() + want.abs().mean())).max().item() <= 2.0 ** -8     # one rounding

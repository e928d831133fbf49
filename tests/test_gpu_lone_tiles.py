"""Dense launches of at most one tile per compute unit (eight waves per 64- and 128-row tile, four per 32-row
tile) and K cut into three, against float64, at the edges of tiles, stages and ring slots."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

T32, T64, T128 = 2, 3, 4


@pytest.fixture(scope="module")
def nb():
    import paper_2006_03031_amd as nb
    nb.load()
    return nb


# K: one stage, fewer stages than slots, as many, more; the line between three and four slots (2048); the line
# between eight and four waves of the 64-row tile (K > 2048: 224 tiles); one tile, 256, 257; a last row alone, a
# last column tile partly empty; K not in 64-wide stages; three slices
@pytest.mark.parametrize("variant,M,N,K,split", [
    (T32, 1, 128, 64, 1), (T32, 33, 256, 128, 1), (T32, 256, 4096, 192, 1), (T32, 257, 4096, 256, 1), (T32, 95, 384, 1056, 1),
    (T64, 64, 128, 64, 1), (T64, 65, 128, 128, 1), (T64, 127, 384, 192, 1), (T64, 512, 4096, 256, 1), (T64, 513, 4096, 256, 1),
    (T64, 1000, 1792, 2112, 1), (T64, 1024, 1920, 2112, 1), (T64, 200, 256, 96, 1), (T64, 500, 768, 1536, 3),
    (T128, 128, 128, 64, 1), (T128, 129, 256, 128, 1), (T128, 255, 384, 256, 1), (T128, 300, 256, 2048, 1), (T128, 300, 256, 2112, 1),
    (T128, 2048, 2048, 320, 1), (T128, 2049, 2048, 320, 1), (T128, 2040, 2040, 1216, 1), (T128, 200, 256, 160, 1),
    (T128, 1100, 1024, 1536, 3)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_lone_tiles(nb, variant, M, N, K, split, out):
    from paper_2006_03031_amd import runtime as rt
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * N + K)
    x = torch.empty((M, K), device="cuda").uniform_(-1, 1, generator=gen).to(torch.bfloat16)
    w = torch.empty((N, K), device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
    b = torch.empty((N,), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    dt = torch.float32 if out == "f32" else torch.bfloat16
    buf = torch.full((M * N + 256,), 768.0, dtype=dt, device="cuda")
    y = rt.dense(x, w, b, nb.EPI_BIAS, nb.F32 if out == "f32" else nb.BF16,
                 force_variant=variant | (split << 8 if split > 1 else 0), out=buf[:M * N].view(M, N))
    ref = torch.matmul(x.double(), w.double().t().contiguous()) + b.double()
    # f32 sums of K products: K eps of the sum of magnitudes at the very most; bf16: half a unit in the last place more
    mag = torch.matmul(x.double().abs(), w.double().abs().t().contiguous()) + b.double().abs()
    bound = mag * (K + 1) * 2.0 ** -24 + (ref.abs() * 2.0 ** -8 if out == "bf16" else 0)
    assert bool(((y.double() - ref).abs() <= bound).all())
    assert bool((buf[M * N:] == 768.0).all())


def test_the_dispatch_takes_lone_tiles_and_three_slices(nb):
    p = nb.dense_plan(800, 4096, 1024)
    assert (p.variant, p.bm, p.block) == (T128, 128, 512)
    p = nb.dense_plan(509, 2304, 768)
    assert (p.variant, p.block) == (T64, 512)
    p = nb.dense_plan(200, 2304, 768)
    assert (p.variant, p.block) == (T32, 256)
    p = nb.dense_plan(600, 1024, 4096)
    assert p.split_k == 3 and p.workspace_bytes == 3 * 600 * 1024 * 4

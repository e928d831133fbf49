"""Fused attention and the attention chain at the edges of its tiles, key blocks and launch shapes, against float64."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-3        # normwise, as in test_gpu_parity: P and O rounded to bf16


@pytest.fixture(scope="module")
def rt():
    import paper_2006_03031_amd as nb
    nb.load()
    from paper_2006_03031_amd import runtime
    return runtime


# one key block; keys over four and eight groups (and groups left without a block); two and four row waves;
# rings of two slots with odd and even numbers of blocks; last blocks of 1, 63 and 64 keys
@pytest.mark.parametrize("heads,L", [(1, 1), (3, 31), (3, 64), (130, 33), (2, 65), (2, 129), (2, 256), (2, 257), (2, 449), (2, 512),
                                     (90, 100), (60, 129), (65, 256), (2, 513), (1, 577), (40, 333), (12, 641), (30, 577),
                                     (16, 1025), (24, 1089), (100, 320), (90, 513)])
@pytest.mark.parametrize("growing", [False, True])
def test_fused_attention_launch_shapes(rt, heads, L, growing):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * heads + L)
    q, k, v = (torch.empty((heads, L, 64), device="cuda").normal_(0, 1, generator=gen) for _ in range(3))
    if growing:   # scores that grow along the keys: every block moves every maximum; values off zero
        k = k * 0.1 + torch.linspace(0, 2, L, device="cuda")[None, :, None]
        q, v = q.abs(), v + 1
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    buf = torch.full((heads * L * 64 + 512,), 768.0, dtype=torch.bfloat16, device="cuda")
    o = rt.fused_attention(q, k, v, out=buf[:heads * L * 64].view(heads, L, 64))
    s = torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) * 0.125
    ref = torch.matmul(torch.softmax(s, -1), v.double())
    err = ((o.double() - ref).norm() / ref.norm()).item()
    assert err <= TOL, err
    # per row too: a wrong row among many must not hide in the norm
    row = ((o.double() - ref).norm(dim=-1) / (ref.norm(dim=-1) + 1e-2 * ref.norm(dim=-1).mean())).max().item()
    assert row <= 4 * TOL, row
    assert bool((buf[heads * L * 64:] == 768.0).all())


# one, two, four and eight waves; a last wave with 1, 63 and 64 keys and waves without any; a last query tile of one
# row; odd L (rows of S and P at any alignment); 513: the three calls
@pytest.mark.parametrize("heads,L", [(1, 1), (3, 31), (2, 33), (5, 63), (3, 64), (2, 65), (2, 127), (3, 128), (2, 129), (1, 193),
                                     (2, 256), (3, 257), (2, 333), (2, 448), (3, 449), (2, 511), (2, 512), (2, 513),
                                     # more workgroups of 16 rows than find a place at once: 32 rows; the last such that do
                                     (2049, 1), (1025, 31), (683, 33), (513, 63), (512, 64), (513, 64), (205, 65), (129, 127), (129, 128),
                                     (57, 129), (40, 193), (32, 256), (33, 256), (15, 257), (16, 257), (13, 333), (10, 448), (9, 511), (9, 512)])
@pytest.mark.parametrize("alpha", [0.125, -0.25])
def test_attention_chain_edges(rt, heads, L, alpha):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * heads + L)
    q, k, v = (torch.empty((heads, L, 64), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16) for _ in range(3))
    import paper_2006_03031_amd as nb
    n = heads * L * L
    sb = torch.full((n + 256,), 768.0, device="cuda")
    pb = torch.full((n + 256,), 768.0, dtype=torch.bfloat16, device="cuda")
    ob = torch.full((heads * L * 64 + 256,), 768.0, dtype=torch.bfloat16, device="cuda")
    ws = rt.default_workspace(q.device)
    nb.nimble_attention_chain_dyn(q.data_ptr(), k.data_ptr(), v.data_ptr(), sb.data_ptr(), pb.data_ptr(), ob.data_ptr(), heads,
                                  L, L, 64, 64, alpha, ws.data_ptr(), ws.numel(), rt._stream())
    s, p, o = sb[:n].view(heads, L, L), pb[:n].view(heads, L, L), ob[:heads * L * 64].view(heads, L, 64)
    rs = torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) * alpha
    rp = torch.softmax(rs, -1)
    # S: 64 products summed in f32; P: one rounding to bf16 (2^-9) of an f32 softmax; O: its own rounding, from the P given
    assert ((s.double() - rs).abs().max() / rs.abs().max()).item() <= 64 * 2.0 ** -24
    assert ((p.double() - rp).abs() / rp).max().item() <= 2.0 ** -8
    ro = torch.matmul(p.double(), v.double())
    assert ((o.double() - ro).abs() / (ro.abs() + ro.abs().mean())).max().item() <= 2.0 ** -8
    for b, m in ((sb, n), (pb, n), (ob, heads * L * 64)):
        assert bool((b[m:] == 768.0).all())


def test_attention_chain_passes_infinite_values_on(rt):
    """The last key's row of V is infinite: the keys past it, which a wave's tile has too, add nothing."""
    L = 333
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q, k, v = (torch.empty((2, L, 64), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16) for _ in range(3))
    v[:, L - 1] = float("inf")
    _, p, o = rt.attention(q, k, v)
    assert bool((p[:, :, L - 1] > 0).all()) and bool((o == float("inf")).all())


# one to eight waves, and the three calls; all scores of a row equal (up to a row of one huge negative value), or far apart
@pytest.mark.parametrize("L", [1, 64, 130, 512, 513])
@pytest.mark.parametrize("score", [1e5, 2e9, -5e9, 1e10, -1e10, -1e30])
def test_attention_chain_of_large_scores(rt, L, score):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    v = torch.empty((2, L, 64), device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)
    # head 0: query row m's scores are all (1 + m) score, whatever the key; head 1: key j adds a part of its own
    q = torch.zeros((2, L, 64), device="cuda")
    k = torch.zeros((2, L, 64), device="cuda")
    q[:, :, 0] = 1 + torch.arange(L, device="cuda") % 100
    k[:, :, 0] = score
    q[1, :, 1] = 1
    k[1, :, 1] = torch.empty(L, device="cuda").normal_(0, 1, generator=gen) * abs(score) * 0.1
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    s, p, o = rt.attention(q, k, v, alpha=1.0)
    # P against the S that was returned (S's own rounding is a large step at these magnitudes): one rounding to bf16
    rp = torch.softmax(s.double(), -1)
    finite = [bool(torch.isfinite(t).all()) for t in (s, p, o)]
    assert all(finite), finite
    assert ((p.double() - rp).abs() / (rp + 1e-30)).max().item() <= 2.0 ** -8
    if L > 1:
        assert bool((p[0].float() * L - 1).abs().max() <= 2.0 ** -8)
    ro = torch.matmul(p.double(), v.double())
    assert ((o.double() - ro).abs() / (ro.abs() + ro.abs().mean())).max().item() <= 2.0 ** -8

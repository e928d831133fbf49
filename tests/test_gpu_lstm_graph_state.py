"""Every run of a captured token loop starts from zero states, whatever the caller did to the results of the last."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("project", [False, True])
@pytest.mark.parametrize("one_launch", [None, False])
def test_runs_start_from_zero(project, one_launch):
    from paper_2006_03031_amd import runtime as rt
    T, B, H = 20, 9, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    bf = lambda *s: torch.empty(s, device="cuda").uniform_(-0.3, 0.3, generator=gen).to(torch.bfloat16)
    w, b, xs = bf(4 * H, 2 * H), bf(4 * H), bf(T, B, H)
    loop = rt.LstmSequenceGraph(w, b, B, T, H, H, project_inputs=project, one_launch=one_launch)
    h, c = (t.clone() for t in loop.run(xs))
    for _ in range(2):
        again = loop.run(xs)
        assert torch.equal(again[0], h) and torch.equal(again[1], c)
        again[0].fill_(1.0), again[1].fill_(-1.0)
    hp, cp = torch.zeros((B, H), dtype=torch.bfloat16, device="cuda"), torch.zeros((B, H), device="cuda")
    if not project:
        for t in range(T):
            hp, cp = rt.lstm_step(xs[t], hp, w, b, cp)
            assert torch.equal(hp, h[t])
        assert torch.equal(cp, c)

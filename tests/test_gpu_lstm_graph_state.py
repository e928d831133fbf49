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
    assert (loop.workspace is not None) == (one_launch is None)   # (the loop in one launch, the steps)
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


@pytest.mark.parametrize("project", [False, True])
@pytest.mark.parametrize("one_launch", [None, False])
def test_a_replay_goes_on_from_the_callers_state(project, one_launch):
    """`graph`, hs and c are public: a replay starts from what the last part of a sequence left there, or from states of the
    caller's own, whatever runs came before."""
    from paper_2006_03031_amd import runtime as rt
    T, B, H = 20, 9, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    bf = lambda *s: torch.empty(s, device="cuda").uniform_(-0.3, 0.3, generator=gen).to(torch.bfloat16)
    w, b, xs, h0, c0 = bf(4 * H, 2 * H), bf(4 * H), bf(2 * T, B, H), bf(B, H), bf(B, H).float()
    part = rt.LstmSequenceGraph(w, b, B, T, H, H, project_inputs=project, one_launch=one_launch)
    assert (part.workspace is not None) == (one_launch is None)

    def replay(xs, h, c):
        """A replay from these states, against the cell step by step from the gates' input shares that the replay computed."""
        part.hs[0].copy_(h)
        part.c.copy_(c)
        part.xs.copy_(xs)
        want_h, want_c = [], part.c.clone()
        part.graph.replay()
        for t in range(T):
            h, want_c = (rt.lstm_step_pre(part.pre[t], h, part.w_h, want_c) if project else rt.lstm_step(xs[t], h, w, b, want_c))
            want_h.append(h)
        assert torch.equal(part.hs[1:], torch.stack(want_h)) and torch.equal(part.c, want_c)

    for _ in range(2):
        replay(xs[:T], h0, c0)
        h, c = part.run(xs[:T])
        replay(xs[T:], h[-1].clone(), c)
    part.run(xs[:T])
    first_c = part.c.clone()
    part.graph.replay()          # h_0 is zero still, c goes on
    assert not torch.equal(part.c, first_c)


@pytest.mark.parametrize("one_launch", [True, False])
def test_no_steps_give_the_first_state(one_launch):
    from paper_2006_03031_amd import runtime as rt
    B, H = 9, 128
    w, b = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((4 * H, 2 * H), (4 * H,)))
    loop = rt.LstmSequenceGraph(w, b, B, 0, H, H, one_launch=one_launch)
    for _ in range(2):
        h, c = loop.run()
        assert h.shape == (0, B, H) and not c.any()
        c.fill_(3.0)

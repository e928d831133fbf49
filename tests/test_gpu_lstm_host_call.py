"""A sentence through the LSTM as one native call: the same bits as the steps, a loop that gives up, other operands left to Python."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    from paper_2006_03031_amd import runtime
    runtime.default_workspace(torch.device("cuda", torch.cuda.current_device()))
    return runtime


def operands(T, B, Ix, H):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T * 1000 + B + H)
    bf = lambda *s: torch.empty(s, device="cuda").uniform_(-0.2, 0.2, generator=gen).to(torch.bfloat16)
    return [bf(T, B, Ix), bf(4 * H, Ix), bf(4 * H, H), bf(4 * H), bf(B, H), bf(B, H).float()]


@pytest.mark.parametrize("T,B,Ix,H", [(1, 1, 64, 64), (3, 4, 40, 256), (9, 2, 512, 512), (17, 1, 96, 1024)])
def test_the_same_as_the_steps(rt, monkeypatch, T, B, Ix, H):
    ops = operands(T, B, Ix, H)
    native = rt._host_calls.lstm_sequence
    got = native(*ops, rt.LSTM_SEQ_MAX_POLLS)
    h, c, one = rt.lstm_sequence(*ops, one_launch=False)
    assert got[2] is True and one is False and torch.equal(got[0], h) and torch.equal(got[1], c)
    monkeypatch.setattr(rt, "LSTM_SEQ_MAX_POLLS", 0)   # the loop gives up at its first wait: the steps run behind it
    if T > 1:
        assert isinstance(native(*ops, 0), torch.Tensor)
        again = rt.lstm_sequence(*ops)
        assert again[2] is False and torch.equal(again[0], h) and torch.equal(again[1], c)


def test_other_operands_are_left_to_the_steps(rt):
    ops, polls = operands(5, 2, 64, 128), rt.LSTM_SEQ_MAX_POLLS
    native = rt._host_calls.lstm_sequence
    for i, other in ((0, ops[0][:0]), (0, ops[0].float()), (0, ops[0][:, :, :32]), (1, ops[1][:-1]), (2, ops[2].t()), (3, ops[3][:-1]),
                     (3, None), (4, ops[4][:1]), (5, ops[5].bfloat16()), (5, ops[5].cpu())):
        assert native(*ops[:i], other, *ops[i + 1:], polls) is None, i
    assert native(*operands(5, 3, 64, 1024), polls) is None   # not the one-launch loop's by default
    h, c, one = rt.lstm_sequence(*operands(5, 3, 64, 1024))
    assert h.shape == (5, 3, 1024) and c.shape == (3, 1024)
    # a cell state that does not start on 16 bytes: refused by the loop, as before, taken by the steps
    buf = torch.zeros(2 * 128 + 1, device="cuda")
    c0 = buf[1:].view(2, 128)
    assert native(*ops[:5], c0, polls) is None
    with pytest.raises(rt.nb.NimbleError, match="16-byte aligned"):
        rt.lstm_sequence(*ops[:5], c0)
    want = rt.lstm_sequence(*ops[:5], torch.zeros((2, 128), device="cuda"))
    got = rt.lstm_sequence(*ops[:5], c0, one_launch=False)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])

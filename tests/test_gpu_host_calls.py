"""The native one-call sequences (csrc/host_calls.cpp) against the steps in Python: the same bits on plain operands, the same
answers and errors on everything that they leave to the steps."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    from paper_2006_03031_amd import runtime
    runtime.default_workspace(torch.device("cuda", 0))   # from here on the native calls serve the device
    return runtime


@pytest.fixture(scope="module")
def nb():
    import paper_2006_03031_amd as nb
    return nb


def _operands(M=23, N=128, K=64):
    gen = torch.Generator(device="cuda").manual_seed(3)
    return [torch.randn(s, device="cuda", generator=gen).bfloat16() for s in ((M, K), (N, K), (N,))]


def _steps(rt, *args, **kw):
    """The same call through the steps: a workspace of the caller's own is theirs."""
    return rt.dense(*args, workspace=rt.default_workspace(torch.device("cuda", 0)), **kw)


@pytest.mark.parametrize("M,N,K", [(23, 128, 64), (0, 128, 64), (1, 1, 8), (70, 33, 65), (300, 1024, 4096)])
def test_dense_gives_the_bits_of_the_steps(rt, nb, M, N, K):
    x, w, b = _operands(M, N, K)
    native = rt._host_calls.dense
    for bias, epi in ((b, nb.EPI_BIAS), (b, nb.EPI_BIAS_GELU_ERF), (None, nb.EPI_NONE)):
        for out in (nb.BF16, nb.F32):
            y = native(x, w, bias, epi, out)
            ref = _steps(rt, x, w, bias, epi, out)
            assert y.dtype == ref.dtype and y.shape == ref.shape and y.device == ref.device and torch.equal(y, ref)


def test_what_the_native_call_leaves_to_the_steps(rt, nb):
    x, w, b = _operands()
    native, E, F = rt._host_calls.dense, nb.EPI_BIAS, nb.BF16
    want = _steps(rt, x, w, b)
    # taken: parameters, gradients asked for, tensors of inference mode, views that are contiguous
    assert torch.equal(native(x, torch.nn.Parameter(w), b, E, F), want)
    assert torch.equal(native(x.clone().requires_grad_(), w, b, E, F), want)
    with torch.inference_mode():
        assert torch.equal(native(x.clone(), w, b, E, F), want)
    two = torch.cat((x, x))
    assert torch.equal(native(two[23:], w, b, E, F), want)
    # left: other types, strides, ranks, extents, hosts, subclasses, modes
    class Sub(torch.Tensor):
        pass
    wide = torch.cat((x, x), 1)
    for args in ((x.float(), w, b), (wide[:, :64], w, b), (x[0], w, b), (x[:, :32].contiguous(), w, b), (x.cpu(), w, b),
                 (x.as_subclass(Sub), w, b), (x, w, b[:5]), (x, w, b.float()), (None, w, b)):
        assert native(*args, E, F) is None
    assert native(x, w, b, 7, F) is None and native(x, w, b, E, 9) is None and native(x, w, b, True, F) is None
    from torch.overrides import TorchFunctionMode
    seen = []

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    with Mode():
        assert native(x, w, b, E, F) is None
        assert torch.equal(rt.dense(x, w, b), want) and torch.empty in seen   # the steps, as the mode sees them
    with pytest.raises(Exception):   # a batched tensor has no address, before as now
        torch.func.vmap(lambda a: rt.dense(a, w, b))(two.view(2, 23, 64))
    # errors are those of the steps
    for args, code in (((wide[:, :64], w, b), -8), ((x.float(), w, b), -4), ((x[:, :32].contiguous(), w, b), -3), ((x, w, None), -1),
                       ((x, w, b[:5]), -3), ((two.view(-1)[1:1 + 23 * 64].view(23, 64), w, b), -5)):
        with pytest.raises(nb.NimbleError) as e:
            rt.dense(*args)
        assert e.value.code == code, (args[0].shape, e.value)


@pytest.mark.parametrize("L", [1, 65, 333, 600])
def test_attention_gives_the_bits_of_the_steps(rt, L, monkeypatch):
    gen = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn((3, L, 64), device="cuda", generator=gen).bfloat16() for _ in range(3))
    got = rt._host_calls.attention(q, k, v, 0.125) + (rt._host_calls.fused_attention(q, k, v, 0.125),)
    for name in ("attention", "fused_attention"):
        assert getattr(rt._host_calls, name)(q, k, v[:, :0], 0.125) is None
        assert getattr(rt._host_calls, name)(q, k.float(), v, 0.125) is None
    # fused: as many queries as keys, one head width throughout
    assert rt._host_calls.fused_attention(q, k, v[:, :, :32].contiguous(), 0.125) is None

    class Steps:
        attention = fused_attention = staticmethod(lambda *a: None)
    monkeypatch.setattr(rt, "_host_calls", Steps)
    want = rt.attention(q, k, v) + (rt.fused_attention(q, k, v),)
    assert all(torch.equal(a, b) and a.dtype == b.dtype for a, b in zip(got, want))


def test_the_interpreter_through_one_native_call(rt, nb, monkeypatch):
    """The feed-forward program: the same bits and the same place in the pool as through the steps; an error keeps its code."""
    from paper_2006_03031_amd import vm
    gen = torch.Generator(device="cuda").manual_seed(1)
    w1, b1, w2, b2 = (torch.randn(s, device="cuda", generator=gen).mul_(0.05).bfloat16()
                      for s in ((256, 64), (256,), (64, 256), (64,)))
    exe = vm.Executable.from_assembler(vm.ffn_block_program(), [w1, b1, w2, b2])
    x = torch.randn((37, 64), device="cuda", generator=gen).bfloat16()
    pool = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    native = rt._host_calls.vm_run(exe._handle.value, [x], pool, exe._constants, 0)
    got = [(t.data_ptr(), t.shape, t.clone()) for t in native]
    assert native[0].untyped_storage().data_ptr() == pool.untyped_storage().data_ptr()
    small = torch.empty(64, dtype=torch.uint8, device="cuda")
    codes = []
    for _ in range(2):
        with pytest.raises(nb.NimbleError) as e:
            exe.run([x], small)
        codes.append(e.value.code)
        monkeypatch.setattr(rt._host_calls, "vm_run", lambda *a: None)   # the steps from here on
    want = exe.run([x], pool)
    assert codes[0] == codes[1]
    assert all(p == t.data_ptr() and s == t.shape and torch.equal(c, t) for (p, s, c), t in zip(got, want)) and len(got) == len(want)


def test_the_interpreter_keeps_what_it_runs_on(rt, nb, monkeypatch):
    """The lists of inputs and constants are the caller's: another thread may empty them while the interpreter runs. Here
    that happens once the operands have been read, in place of the question for the current stream."""
    from paper_2006_03031_amd import vm
    a = vm.Assembler(1)
    a.ret(a.alloc_adt(0, [0, a.load_const(0)]))
    want = torch.arange(6, dtype=torch.float32, device="cuda").view(2, 3)
    inputs, pool = [want.clone()], torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    exe = vm.Executable.from_assembler(a, [want + 6])
    constants, real, dropped = exe._constants, rt._raw_stream, []

    def drop_and_answer(device):
        inputs.clear(), constants.clear()
        dropped.append([torch.zeros((2, 3), device="cuda") for _ in range(4)])   # where their memory was, had it been freed
        return real(device)
    monkeypatch.setattr(rt, "_raw_stream", drop_and_answer)
    monkeypatch.setattr(rt, "_bound", False)
    rt._bind_host_calls(pool.device)
    try:
        got = rt._host_calls.vm_run(exe._handle.value, inputs, pool, constants, 0)
    finally:
        monkeypatch.undo()
        rt._bound = False
        rt._bind_host_calls(pool.device)
    assert len(dropped) == 1 and not inputs and not constants
    assert torch.equal(got[0], want) and torch.equal(got[1], want + 6)

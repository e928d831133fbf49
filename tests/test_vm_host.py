"""The C++ interpreter without a GPU: load-time verification, the host-only instructions and the
pool arithmetic, checked against the reference interpreter and hand-worked values.  Programs here
never reach a kernel launch; tensor inputs are descriptors whose address is never read."""
import os

import numpy as np
import pytest

import paper_2006_03031_amd as nb
from paper_2006_03031_amd import vm
from oracle import vm_oracle as vo

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")
FAKE = 0x7F0000000000  # never dereferenced: 64-byte aligned


def _golden(name):
    out = {}
    for line in open(os.path.join(GOLDEN, name)):
        if line.startswith("#") or ":" not in line:
            continue
        k, v = line.split(":", 1)
        out[k.strip()] = [int(t) for t in v.split()]
    return out


def _w(op, *operands):
    return [op, len(operands), *operands]


def _flat(prog):
    return [x for ins in prog for x in ins]


def test_opcode_numbers_agree_between_assembler_and_reference():
    # two hand-typed copies of the interface's numbering (Table C.1 order)
    names = ["MOVE", "RET", "IF", "GOTO", "LOAD_CONST", "LOAD_CONSTI", "ALLOC_STORAGE", "ALLOC_TENSOR",
             "ALLOC_TENSOR_REG", "ALLOC_ADT", "ALLOC_CLOSURE", "FREE_STORAGE", "FREE_TENSOR", "INVOKE",
             "INVOKE_CLOSURE", "INVOKE_PACKED", "GET_FIELD", "GET_TAG", "DEVICE_COPY", "SHAPE_OF",
             "RESHAPE_TENSOR", "FATAL"]
    for n in names:
        assert getattr(vm, "OP_" + n) == getattr(vo, n)
    for n in ["SHAPE_DENSE", "SHAPE_LSTM", "SHAPE_ATTENTION", "STORAGE_BYTES", "SHAPE_GET", "INT_ADD", "INT_LESS",
              "INDEX0", "DENSE", "DENSE_BIAS", "DENSE_BIAS_GELU", "LSTM_GATES", "ATTENTION"]:
        assert getattr(vm, "PF_" + n) == getattr(vo, n)
    header = open(os.path.join(os.path.dirname(GOLDEN), "..", "include", "nimble_vm.h")).read()
    assert "NIMBLE_OP_FATAL = 21" in header and "NIMBLE_PF_ATTENTION = 12" in header


def test_count_loop_by_hand_in_the_library():
    g = _golden("vm_count_loop.txt")
    exe = vm.Executable(g["words"], g["registers"][0])
    assert exe.run([], None) == [g["result"][0]]
    prof = exe.profile()
    assert prof["instructions"] == g["executed"][0]
    assert prof["opcodes"]["If"][0] == 6 and prof["opcodes"]["Goto"][0] == 5
    assert prof["packed"]["int_add"][0] == 5


@pytest.mark.parametrize("n", [0, 1, 17])
def test_assembled_loop_matches_reference(n):
    a = vm.Assembler(0)
    limit, t, one = a.load_consti(n), a.load_consti(0), a.load_consti(1)
    acc = a.load_consti(0)
    a.label("top")
    a.if_equal(t, limit, "done", "body")
    a.label("body")
    a.invoke_packed(vm.PF_INT_ADD, [acc, t], [acc])
    a.invoke_packed(vm.PF_INT_ADD, [t, one], [t])
    a.goto("top")
    a.label("done")
    lt = a.reg()
    a.invoke_packed(vm.PF_INT_LESS, [acc, limit], [lt])
    a.ret(a.alloc_adt(9, [acc, lt]))
    exe = vm.Executable.from_assembler(a)
    got = exe.run([], None)
    ref, executed = vo.run(a.words(), a.n_regs, [], [])
    assert got == vo.flatten(ref) == [n * (n - 1) // 2, 1 if n * (n - 1) // 2 < n else 0]
    assert exe.profile()["instructions"] == executed


def _shape_program():
    """ShapeOf -> shape function -> storage_bytes -> AllocStorage -> AllocTensorReg -> ShapeOf:
    everything of Appendix A's listing except the kernel launch."""
    a = vm.Assembler(2)  # x, w
    sixteen, bf16 = a.load_consti(16), a.load_consti(nb.BF16)
    sx, sw = a.shape_of(0), a.shape_of(1)
    out_sh = a.host_shape_tensor(sixteen, 2)
    a.invoke_packed(vm.PF_SHAPE_DENSE, [sx, sw], [out_sh])
    nbytes = a.reg()
    a.invoke_packed(vm.PF_STORAGE_BYTES, [out_sh, bf16], [nbytes])
    buf = a.alloc_storage(nbytes, vm.GPU)
    y = a.alloc_tensor_reg(buf, 0, out_sh, nb.BF16)
    a.ret(a.alloc_adt(0, [a.shape_of(y), nbytes, y]))
    return a


@pytest.mark.parametrize("M", [0, 1, 7, 513, 8191])
def test_shape_function_and_allocation_without_a_launch(M):
    a = _shape_program()
    exe = vm.Executable.from_assembler(a)
    x, w = vm.TensorDesc(FAKE, (M, 1024), nb.BF16), vm.TensorDesc(FAKE + (1 << 30), (4096, 1024), nb.BF16)
    pool = vm.TensorDesc(FAKE + (2 << 30), (1 << 28,), nb.BF16)
    shape, nbytes, y = exe.run([x, w], pool)
    assert shape == [M, 4096] and nbytes == M * 4096 * 2
    assert (y.ptr, y.shape, y.dtype) == (pool.ptr, (M, 4096), nb.BF16)
    ref, _ = vo.run(a.words(), a.n_regs, [], [vo.Tensor(np.zeros((M, 1024), np.float32), vo.BF16),
                                              vo.Tensor(np.zeros((4096, 1024), np.float32), vo.BF16)])
    rs, rn, ry = vo.flatten(ref)
    assert rs.array.tolist() == shape and rn == nbytes and ry.array.shape == y.shape
    prof = exe.profile()
    assert prof["storage_allocs"] == 1 and prof["pool_high_water"] == max(64, (nbytes + 63) // 64 * 64)


def test_run_time_type_error_and_fatal():
    exe = vm.Executable.from_assembler(_shape_program())
    x, w = vm.TensorDesc(FAKE, (5, 1000), nb.BF16), vm.TensorDesc(FAKE, (4096, 1024), nb.BF16)
    with pytest.raises(nb.NimbleError) as e:
        exe.run([x, w], vm.TensorDesc(FAKE, (1 << 20,), nb.BF16))
    assert e.value.code == -3  # K disagrees: the shape function's deferred check
    with pytest.raises(nb.NimbleError) as e:
        vm.Executable(_flat([_w(vm.OP_FATAL)]), 1).run([], None)
    assert e.value.code == -3
    # If on a tensor register
    with pytest.raises(nb.NimbleError) as e:
        vm.Executable(_flat([_w(vm.OP_IF, 0, 0, 1, 1), _w(vm.OP_RET, 0)]), 1).run([x], None)
    assert e.value.code == -8
    # empty result register
    with pytest.raises(nb.NimbleError):
        vm.Executable(_flat([_w(vm.OP_RET, 0)]), 1).run([], None)


def test_instruction_limit_stops_an_endless_loop():
    exe = vm.Executable(_flat([_w(vm.OP_GOTO, 0)]), 1)
    with pytest.raises(nb.NimbleError) as e:
        exe.run([], None, max_instructions=5000)
    assert e.value.code == -8 and "limit" in str(e.value)
    assert exe.profile()["opcodes"]["Goto"][0] == 5000


def test_pool_exhaustion_reuse_and_free():
    # allocate 3 blocks of 1000 bytes (rounded to 1024) from a pool of 2048: third fails
    a = vm.Assembler(0)
    n = a.load_consti(1000)
    a.alloc_storage(n, vm.GPU)
    a.alloc_storage(n, vm.GPU)
    a.alloc_storage(n, vm.GPU)
    a.ret(n)
    exe = vm.Executable.from_assembler(a)
    with pytest.raises(nb.NimbleError) as e:
        exe.run([], vm.TensorDesc(FAKE, (1024,), nb.BF16))  # 2048 bytes
    assert e.value.code == -6
    # with FreeStorage (or an overwritten register) the block comes back and is reused
    a = vm.Assembler(0)
    n = a.load_consti(1000)
    s1 = a.alloc_storage(n, vm.GPU)
    a.free_storage(s1)
    s2 = a.alloc_storage(n, vm.GPU)
    a.move(n, s2)                      # drops the last reference to the second block
    s3 = a.alloc_storage(n, vm.GPU)
    t = a.alloc_tensor(s3, 0, nb.F32, [10, 25])
    a.ret(t)
    exe = vm.Executable.from_assembler(a)
    pool = vm.TensorDesc(FAKE, (512,), nb.BF16)  # 1024 bytes: room for exactly one block
    (res,) = exe.run([], pool)
    assert res.ptr == FAKE and res.shape == (10, 25)
    prof = exe.profile()
    assert prof["storage_allocs"] == 3 and prof["storage_reuses"] == 2 and prof["pool_high_water"] == 1024
    # a tensor carved from freed storage, and a tensor larger than its storage
    a = vm.Assembler(0)
    n = a.load_consti(64)
    s1 = a.alloc_storage(n, vm.GPU)
    a.free_storage(s1)
    a.ret(a.alloc_tensor(s1, 0, nb.F32, [4]))
    with pytest.raises(nb.NimbleError):
        vm.Executable.from_assembler(a).run([], pool)
    a = vm.Assembler(0)
    s1 = a.alloc_storage(a.load_consti(64), vm.GPU)
    a.ret(a.alloc_tensor(s1, 0, nb.F32, [17]))
    with pytest.raises(nb.NimbleError) as e:
        vm.Executable.from_assembler(a).run([], pool)
    assert e.value.code == -6


@pytest.mark.parametrize("words,what", [
    ([99, 0], "unknown opcode"),
    (_w(vm.OP_RET, 5), "register"),
    (_w(vm.OP_GOTO, 7), "jumps outside"),
    (_w(vm.OP_GOTO, -1), "jumps outside"),
    (_w(vm.OP_MOVE, 0, 0), "runs off its end"),
    (_w(vm.OP_MOVE, 0), "operands"),
    (_w(vm.OP_INVOKE, 0, 0) + _w(vm.OP_RET, 0), "not implemented"),
    (_w(vm.OP_ALLOC_CLOSURE, 0) + _w(vm.OP_RET, 0), "not implemented"),
    (_w(vm.OP_DEVICE_COPY, 0, 0) + _w(vm.OP_RET, 0), "not implemented"),
    (_w(vm.OP_INVOKE_PACKED, vm.PF_INT_ADD, 2, 1, 0, 0) + _w(vm.OP_RET, 0), "inputs"),
    (_w(vm.OP_INVOKE_PACKED, 77, 3, 1, 0, 0, 0) + _w(vm.OP_RET, 0), "unknown packed"),
    (_w(vm.OP_LOAD_CONST, 0, 0) + _w(vm.OP_RET, 0), "constant"),
    (_w(vm.OP_ALLOC_STORAGE, 0, 48, 1, 0) + _w(vm.OP_RET, 0), "alignment"),
    (_w(vm.OP_ALLOC_TENSOR, 0, 0, 0, 2, 3, 0) + _w(vm.OP_RET, 0), "malformed"),
    ([vm.OP_RET, 3, 0], "runs past the end"),
    ([vm.OP_RET], "truncated"),
])
def test_load_time_verification(words, what):
    with pytest.raises(nb.NimbleError) as e:
        vm.Executable(words, 1)
    assert e.value.code == -8 and what in str(e.value), str(e.value)


def test_library_programs_assemble_and_load():
    for prog, n_const in ((vm.lstm_sequence_program(), 2), (vm.ffn_block_program(), 4), (vm.attention_program(), 0)):
        vm.Executable.from_assembler(prog, [vm.TensorDesc(FAKE, (8, 8), nb.BF16)] * n_const)


def test_programs_run_without_the_native_host_calls():
    """Importing the runtime and running programs of descriptors needs no more than the HIP library; what hinders the
    native calls (here another torch than they were built for) is told when a GPU call would have used them."""
    import subprocess
    import sys
    import textwrap
    code = textwrap.dedent("""
        import importlib.abc, sys, warnings
        class NoHostCalls(importlib.abc.MetaPathFinder):
            def find_spec(self, name, path=None, target=None):
                if name.endswith("._host_calls"):
                    raise ImportError("undefined symbol: of another torch")
        sys.meta_path.insert(0, NoHostCalls())
        import paper_2006_03031_amd as nb
        from paper_2006_03031_amd import vm, runtime as rt
        a = vm.Assembler(1)
        a.ret(a.shape_of(0))
        x = vm.TensorDesc(0x7F0000000000, (37, 64), nb.BF16)
        assert vm.Executable.from_assembler(a).run([x], None) == [[37, 64]]
        with warnings.catch_warnings(record=True) as seen:
            warnings.simplefilter("always")
            for _ in range(2):
                rt._bind_host_calls(rt.torch.device("cuda", 0))
        assert len(seen) == 1 and "of another torch" in str(seen[0].message), seen
        assert rt._host_calls.dense(None, None, None, 0, 0) is None
    """)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

"""The native list reader against the binding's own checks, on CPU tensors: a list in order
gives the same addresses and sizes, and anything else is left to the checks (None), which
raise what they always raised or read the list themselves."""
import ctypes

import pytest
import torch
from torch.overrides import TorchFunctionMode

import paper_2608_11919_amd as lt
from paper_2608_11919_amd import lazytrain as binding

lt.lib()
reader = binding._lists
CPU = torch.device("cpu")


class Sub(torch.Tensor):
    pass


def _words(b):
    return list((ctypes.c_uint64 * (len(b) // 8)).from_buffer_copy(b))


@pytest.mark.parametrize("tensors", [
    [], (), [torch.zeros(0)], [torch.zeros(3), torch.zeros(5)], (torch.zeros(2, 3),),
    [torch.nn.Parameter(torch.zeros(7)), torch.zeros(4, requires_grad=True)],
    [torch.zeros(64)[16:32], torch.zeros(1, 5, 1)], [torch.zeros(3, 4).t().t()],
    [torch.zeros(0, 3).t()]], ids=str)
@pytest.mark.parametrize("dtype", [torch.float32, None])
def test_lists_in_order(tensors, dtype):
    ptrs, numels, kind = reader.take(tensors, CPU, dtype)
    binding._check_tensors(tensors, CPU, dtype)
    assert _words(ptrs) == [t.data_ptr() for t in tensors]
    assert _words(numels) == [t.numel() for t in tensors]
    assert kind is (torch.float32 if len(tensors) else None)


@pytest.mark.parametrize("tensors, dtype, error", [
    ([torch.zeros(4, 4).t()], torch.float32, ValueError),
    ([torch.zeros(8)[::2]], None, ValueError),
    ([torch.zeros(3), torch.zeros(3, device="meta")], torch.float32, ValueError),
    ([torch.zeros(3, dtype=torch.int8)], torch.float32, TypeError),
    ([torch.zeros(3), torch.zeros(3, dtype=torch.bfloat16)], torch.float32, TypeError),
    ([torch.zeros(3), torch.zeros(3, dtype=torch.bfloat16)], None, None),
    ([torch.zeros(3), None], None, AttributeError),
    ([torch.zeros(3).as_subclass(Sub)], torch.float32, None)], ids=str)
def test_other_lists_take_the_checks(tensors, dtype, error):
    assert reader.take(tensors, CPU, dtype) is None
    if error is None:
        taken = binding._List(tensors, CPU, dtype)
        assert _words(taken.ptrs) == [t.data_ptr() for t in tensors]
        assert _words(taken.numels) == [t.numel() for t in tensors] and taken.dtype is None
    else:
        with pytest.raises(error):
            binding._List(tensors, CPU, dtype)


def test_mixed_gradient_dtypes_are_refused_and_raw_bits_taken():
    mixed = [torch.zeros(3), torch.zeros(3, dtype=torch.bfloat16)]
    with pytest.raises(TypeError):
        binding._grad_code(mixed, binding._List(mixed, CPU))
    for dtype, code in ((torch.float32, lt.LT_DTYPE_F32), (torch.bfloat16, lt.LT_DTYPE_BF16),
                        (torch.int16, lt.LT_DTYPE_BF16), (torch.uint16, lt.LT_DTYPE_BF16)):
        grads = [torch.zeros(3, dtype=dtype)]
        assert binding._grad_code(grads, binding._List(grads, CPU)) == code
    with pytest.raises(TypeError):
        binding._grad_code([torch.zeros(3).half()], binding._List([torch.zeros(3).half()], CPU))


def test_function_modes_see_the_tensors():
    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert reader.take([torch.zeros(3)], CPU, torch.float32) is None


@pytest.mark.parametrize("block", [1, 64, 4096])
def test_absmax_sizes(block):
    numels = [0, 1, block - 1, block, block + 1, 10 * block, (1 << 62) + 1]
    words = lambda v: bytes((ctypes.c_int64 * len(v))(*v))
    need = [-(-n // block) for n in numels]
    assert reader.covers(words(numels), words(need), block)
    for i, n in enumerate(need):
        if n:
            assert not reader.covers(words(numels), words(need[:i] + [n - 1] + need[i + 1:]), block)
    assert not reader.covers(words(numels), words(need[1:]), block)


def test_without_the_native_reader(monkeypatch):
    """Where the reader does not load (another torch or Python) the library still does: with
    a warning, and with the same checks and the same words, read in Python."""
    import sys
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_lists", None)
    monkeypatch.delattr(lt, "_lists", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2608_11919_amd._lists", None)
    with pytest.warns(RuntimeWarning, match="list reader"):
        lt.lib()
    tensors = [torch.zeros(3), torch.zeros(700)]
    plain = binding._List(tensors, CPU, torch.float32)
    assert (plain.ptrs, plain.numels) == reader.take(tensors, CPU, torch.float32)[:2]
    with pytest.raises(TypeError):
        binding._List(tensors, CPU, torch.int8, "codes")
    assert binding._grad_code(tensors, plain) == lt.LT_DTYPE_F32

    def sizes(absmax):
        lists = [tensors] * 4 + [[torch.zeros(n) for n in absmax]] * 2
        binding._check_step_sizes(*lists, 64, [binding._List(x, CPU) for x in
                                               (tensors, tensors, tensors, tensors, lists[4],
                                                lists[5])], lambda n, nb: f"{nb}")
    sizes([1, 11])
    with pytest.raises(ValueError):
        sizes([1, 10])
    copies = [torch.zeros(3, dtype=torch.bfloat16), None]
    assert binding._bf16_list(copies, tensors, CPU, plain.numels) is not None


@pytest.mark.parametrize("block", [0, -64, 65536 + 64, (1 << 32) + 256, 1 << 63, 1 << 64])
def test_block_sizes_out_of_range(block):
    """Also those whose low 32 bits are a block size, and those no 64-bit word holds."""
    n, i8, u8 = torch.zeros(1024), torch.zeros(1024, dtype=torch.int8), \
        torch.zeros(1024, dtype=torch.uint8)
    scale = torch.zeros(4)
    with pytest.raises(lt.LazyTrainError, match="block_size"):
        lt.lt_hybrid8bit_adamw_step([n], [n.clone()], [i8], [scale], [u8], [scale.clone()], block,
                                    1e-3, 0.9, 0.999, 1e-8, 0.0, 1)
    with pytest.raises(lt.LazyTrainError, match="block_size"):
        lt.lt_streamed_hybrid8bit_adamw_step(
            [n], [n.clone()], [i8], [scale], [u8], [scale.clone()], [0, 1], block, 1e-3, 0.9, 0.999,
            1e-8, 0.0, 1, 1.0, 2, torch.zeros(1, dtype=torch.float64), torch.zeros(1),
            torch.zeros(1, dtype=torch.int32))

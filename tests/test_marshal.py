"""The binding's native tensor checks accept and refuse what the checks in
Python do, and name the same fault."""
import pytest
import torch

from paper_2407_00066_amd import _binding as B

CPU = torch.device("cpu")


def _python(t, dtype, shape):
    B._check_tensor(t, "t", CPU, dtype, shape)
    return t.data_ptr() if t.numel() else None


@pytest.mark.parametrize("make,dtype,shape", [
    (lambda: torch.zeros(3, 8), torch.float32, (3, 8)),
    (lambda: torch.zeros(3, 8, dtype=torch.bfloat16), torch.bfloat16, (3, 8)),
    (lambda: torch.zeros(4, 8)[1:], torch.float32, (3, 8)),                  # an offset view
    (lambda: torch.nn.Parameter(torch.zeros(3, 8)), torch.float32, (3, 8)),
    (lambda: torch.zeros(0, 8), torch.float32, (0, 8)),                      # empty
    (lambda: torch.zeros(()), torch.float32, ()),
    (lambda: torch.zeros(5, dtype=torch.uint8), None, None),
    (lambda: torch.zeros(8, 3).t(), torch.float32, (3, 8)),                  # not contiguous
    (lambda: torch.zeros(3, 8), torch.bfloat16, (3, 8)),                     # wrong type
    (lambda: torch.zeros(3, 8), torch.float32, (8, 3)),                      # wrong shape
    (lambda: torch.zeros(3, 8), torch.float32, (3, 8, 1)),
    (lambda: torch.zeros(3, 8, device="meta"), torch.float32, (3, 8)),       # another device
    (lambda: [1.0], torch.float32, (1,)),
    (lambda: None, None, None),
])
def test_address(make, dtype, shape):
    t = make()
    try:
        want = _python(t, dtype, shape)
    except (TypeError, ValueError) as e:
        with pytest.raises(type(e)) as got:
            B._dev(t, "t", CPU, dtype, shape)
        assert str(got.value) == str(e)
        return
    assert B._dev(t, "t", CPU, dtype, shape) == want


def test_a_module_built_for_another_torch_is_not_used(monkeypatch):
    """_marshal.so reads torch's C++ objects: with a torch other than the one it
    was compiled against every call refuses, with what to do."""
    monkeypatch.setattr(torch, "__version__", "1.0.0+other")
    address = B._load_address()
    with pytest.raises(RuntimeError, match="built for torch .*, this is 1.0.0.other.*paper_2407_00066_amd.build"):
        address(torch.zeros(3), CPU, None, None)


class _Raises(torch.Tensor):
    """A wrapper whose attributes are asked for in Python, which raises."""
    @staticmethod
    def __new__(cls):
        return torch.Tensor._make_wrapper_subclass(cls, (3, 8), dispatch_device=True)

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise KeyError(str(func))


def test_a_tensors_own_error_comes_through():
    with pytest.raises(KeyError, match="device"):
        B._check_tensor(_Raises(), "t", CPU, None, None)
    with pytest.raises(KeyError, match="device"):
        B._dev(_Raises(), "t", CPU, None, None)


def test_default_workspaces_are_not_shared():
    """Two calls that are both on their way hold different workspaces."""
    a, b = B._workspace(CPU, 4096, None), B._workspace(CPU, 4096, None)
    assert a.numel() == b.numel() == 4096 and a.data_ptr() != b.data_ptr()

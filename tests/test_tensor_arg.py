"""The native check of a tensor argument says yes to exactly what the binding's Python check accepts."""
import pytest
import torch

from paper_2510_25979_amd import _tensor_arg, binding


class Sub(torch.Tensor):
    pass


def _cases(device):
    x = torch.zeros(3, 4, device=device)
    return [(x, None, None), (x, torch.float32, None), (x, torch.float32, (3, 4)), (x, torch.float16, None),
            (x, None, (4, 3)), (x, None, (3, 4, 1)), (x, None, (3,)), (x, None, ()), (x, None, (3, 2**70)),
            (x.t(), None, None), (x[:, :2], None, None), (x[1:], torch.float32, (2, 4)), (x[:0], None, (0, 4)),
            (torch.zeros((), device=device), None, ()), (x.bfloat16(), torch.bfloat16, (3, 4)),
            (x.int(), torch.int32, torch.Size([3, 4])), (x.requires_grad_(), torch.float32, (3, 4)),
            (torch.nn.Parameter(x.detach().clone()), torch.float32, (3, 4)), (x.detach().as_subclass(Sub), None, (3, 4)),
            (torch.zeros(2, 3, 4, device=device).transpose(0, 1)[:, :1], None, (3, 1, 4))]


def _check(t, dtype, shape):
    """The binding's answer, and the same without the native module."""
    def ask():
        try:
            return binding._dev(t, "x", dtype, shape)
        except ValueError as e:
            return str(e)
    native, address = ask(), binding._address
    binding._address = lambda t, dtype, shape: None
    try:
        return native, ask()
    finally:
        binding._address = address


def test_tensors_that_are_not_on_the_gpu_are_left_to_python():
    for case in _cases("cpu") + [(3, None, None), (None, None, None), (torch.zeros(3, device="meta"), None, (3,))]:
        assert _tensor_arg.address(*case) is None
        native, python = _check(*case)
        assert native == python == "x must be a CUDA tensor"
    with pytest.raises(TypeError):
        _tensor_arg.address(torch.zeros(1))


@pytest.mark.gpu
def test_the_native_check_answers_like_the_python_check():
    yes = 0
    for case in _cases("cuda"):
        native, python = _check(*case)
        assert native == python, case
        yes += _tensor_arg.address(*case) is not None
    assert yes == 10     # plain tensors of the right type and shape (a torch.Size and subclasses go the long way)
    seen = []
    torch.vmap(lambda t: (seen.append(_tensor_arg.address(t, None, None)), t)[1])(torch.zeros(2, 3, device="cuda"))
    assert seen == [None]

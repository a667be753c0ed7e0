"""When a search's start state may be written by one kernel: the check reads private
names of torch, and falls back to tensor operations where they are missing."""
import pytest
import torch

from paper_2410_10447_amd import dock

NAMES = [(torch._C, "_len_torch_dispatch_stack"), (torch._C, "_len_torch_function_stack"), (torch._C, "_functorch"),
         (torch._C, "_get_tracing_state"), (torch.autograd.forward_ad, "_current_level"),
         (torch.compiler, "is_compiling")]


def test_plain_call():
    assert dock._outside_modes()


@pytest.mark.parametrize("owner,name", NAMES, ids=[n for _, n in NAMES])
def test_a_torch_without_the_name(monkeypatch, owner, name):
    with monkeypatch.context() as m:
        m.delattr(owner, name)
        found = dock._outside_modes()
    assert found is False


def test_inside_transforms_and_modes():
    seen = []

    def look(x):
        seen.append(dock._outside_modes())
        return x

    torch.func.vmap(look)(torch.zeros(2, 3))
    torch.func.jvp(look, (torch.zeros(3),), (torch.zeros(3),))
    with torch.autograd.forward_ad.dual_level():
        look(None)
    with torch.overrides.TorchFunctionMode():
        look(None)
    with torch.utils._python_dispatch.TorchDispatchMode():
        look(None)
    torch.jit.trace(look, torch.zeros(2), check_trace=False)
    assert seen == [False] * len(seen) and len(seen) >= 6

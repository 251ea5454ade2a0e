"""Host-side pieces of the binding (CPU)."""
import types

import pytest
import torch

from paper_2607_10611_amd import binding as B


def test_current_stream_with_torch_s_internal_call(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 40 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 2)
    assert B._stream(None) == 42


def test_current_stream_without_torch_s_internal_call(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=7))
    assert B._stream(None) == 7


@pytest.mark.parametrize("hp", [{}, dict(lr_add=2, bias_correction=False, rounding="sr", seed=-1, step=9),
                                dict(rounding=1, seed=2**64 + 3, other="ignored", w_max=4)])
def test_a_dict_of_hyper_parameters_is_the_struct_of_the_class(hp):
    assert bytes(B._hp(hp)) == bytes(B.HParams.from_dict(hp).to_c())

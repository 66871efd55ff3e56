"""Where the native marshalling module cannot be used, calls take the ctypes code (which raises its own
errors here, on host tensors), after one warning.
"""
import types
import warnings

import pytest
import torch

import paper_1701_00485_amd as tbn


def _ctypes_answers():
    t = torch.zeros(8, dtype=torch.bfloat16)
    with pytest.raises(TypeError, match="must be a CUDA"):
        tbn.relu_bwd(t, t)


@pytest.mark.parametrize("content", [None, b"no shared object"])
def test_module_missing_or_broken(monkeypatch, tmp_path, content):
    path = tmp_path / "_tbn_torch.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(tbn, "BINDING_PATH", str(path))
    monkeypatch.setattr(tbn, "_native", None)
    with pytest.warns(UserWarning, match="_tbn_torch.so not loaded"):
        _ctypes_answers()
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        _ctypes_answers()  # warned once


def test_module_built_for_another_torch(monkeypatch):
    other = types.SimpleNamespace(BUILT_FOR="torch 0.0.0, Python 3.10")
    monkeypatch.setattr(tbn.importlib.util, "module_from_spec", lambda spec: other)
    monkeypatch.setattr(tbn.importlib.util, "spec_from_file_location",
                        lambda *a: types.SimpleNamespace(loader=types.SimpleNamespace(exec_module=lambda m: None)))
    monkeypatch.setattr(tbn, "_native", None)
    with pytest.warns(UserWarning, match="built for torch 0.0.0"):
        _ctypes_answers()


def test_built_module_loads(monkeypatch):
    monkeypatch.setattr(tbn, "_native", None)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert not isinstance(tbn._load_native(), tbn._NoBinding)

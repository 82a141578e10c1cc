"""The native calls' module on the CPU: it loads with the installed torch, and
without it (not built, no library, built against another torch, no compiler)
librfq builds and the binding works, with a warning."""
import warnings

import pytest
import torch

from paper_2608_26581_amd import build as rfq_build
from paper_2608_26581_amd import rfq as binding


def _fresh(monkeypatch):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_calls", None)


def test_module_loads_with_the_installed_torch(monkeypatch):
    _fresh(monkeypatch)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        binding.load()
    assert binding._calls.torch_version == torch.__version__


@pytest.mark.parametrize("content", [None, b"", b"no library"])
def test_binding_works_without_the_module(monkeypatch, tmp_path, content):
    path = tmp_path / "_rfq_calls.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(binding, "CALLS_PATH", str(path))
    _check_python_path(monkeypatch)


def test_binding_leaves_a_module_for_another_torch(monkeypatch):
    monkeypatch.setattr(torch, "__version__", "0.0")
    _check_python_path(monkeypatch)


def _check_python_path(monkeypatch):
    _fresh(monkeypatch)
    with pytest.warns(RuntimeWarning, match="cannot be used"):
        binding.load()
    assert binding.rfq_status_str(0) == "ok"
    with pytest.raises(ValueError, match="device tensor"):
        binding.rfq_quantize_act(torch.zeros(4, 64))


def test_build_without_a_host_compiler(monkeypatch, tmp_path):
    path = tmp_path / "_rfq_calls.so"
    path.write_bytes(b"of an earlier build")
    monkeypatch.setattr(rfq_build, "CALLS_PATH", str(path))
    monkeypatch.setattr(rfq_build, "CXX", str(tmp_path / "no-compiler"))
    with pytest.warns(RuntimeWarning, match="not built"):
        assert rfq_build.build_calls_if_possible() is None
    assert not path.exists()

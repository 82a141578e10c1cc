"""The native calls' module on the CPU: it loads with the installed torch, and
without it (not built, no library, built against another torch, no compiler)
librfq builds and the binding works, with a warning."""
import threading
import time
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


def test_module_is_published_bound(monkeypatch):
    """Another thread's first call may come at any point of the load: it must not
    find the module before its entry points are set, nor load a second one."""
    seen, modules = [], []

    class Calls:
        def bind(self, *entries):
            seen.append(binding._calls)
            assert len(entries) == len(binding._NATIVE_ENTRIES) and all(entries)

        def hif4_quantize(self, x, residual):
            return "served"

    def load_calls():
        modules.append(Calls())
        time.sleep(0.05)
        return modules[-1]

    _fresh(monkeypatch)
    monkeypatch.setattr(binding, "_load_calls", load_calls)
    results = []
    threads = [threading.Thread(target=lambda: results.append(binding._native(
        "hif4_quantize", None, True))) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert results == ["served"] * 4
    assert seen == [None] and len(modules) == 1
    assert binding._calls is modules[0] and binding._lib is not None

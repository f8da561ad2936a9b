"""The Python module over the library: when it is built anew, what it is asked for, and a process that cannot load it."""
import os
import warnings

import pytest
import torch

from paper_1911_03458_amd import binding as mb
from paper_1911_03458_amd import build


def test_the_module_names_its_operations():
    assert mb._native() and mb._calls.TORCH == torch.__version__
    entries = [n for n in mb._ops if callable(getattr(mb, n))]
    assert len(entries) == len(mb._ops) == 9 and sorted(mb._ops.values()) == list(range(9))


def test_staleness(tmp_path, monkeypatch):
    deps = [tmp_path / "torch_calls.cpp", tmp_path / "merit.h"]
    module = tmp_path / "_torch_calls.so"
    monkeypatch.setattr(build, "CALLS_DEPS", [str(d) for d in deps])
    monkeypatch.setattr(build, "CALLS_PATH", str(module))
    for d in deps:
        d.write_text("")
        os.utime(d, (1000, 1000))
    assert build.calls_are_stale()                      # there is none
    module.write_text("")
    os.utime(module, (2000, 2000))
    assert not build.calls_are_stale()
    for d in deps:                                      # its source, or the header it calls through
        os.utime(d, (3000, 3000))
        assert build.calls_are_stale()
        os.utime(d, (1000, 1000))


def test_build_all_looks_at_both(monkeypatch):
    done = []
    monkeypatch.setattr(build, "build_library", lambda force=True: done.append(("library", force)))
    monkeypatch.setattr(build, "build_torch_calls", lambda force=True: done.append(("calls", force)))
    build.build_all(force=False)
    assert done == [("library", False), ("calls", False)]


def test_the_library_needs_no_pytorch(tmp_path, monkeypatch):
    """Building libmerit.so runs the HIP compiler and nothing of the module's build."""
    ran = []

    class Done:
        returncode, stdout, stderr = 0, "", ""

    def run(cmd, **kw):
        ran.append(cmd[0])
        return Done()

    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build, "_HERE", str(tmp_path))
    monkeypatch.setattr(build, "build_torch_calls", lambda force=True: pytest.fail("built the module"))
    build.build_library(force=True)
    assert len(ran) == len(build.SOURCES) + 1 and set(ran) == {build.hipcc_path()}


def test_a_module_that_does_not_load_costs_a_warning_and_no_call(tmp_path, monkeypatch):
    broken = tmp_path / "_torch_calls.so"
    broken.write_text("not a module")
    monkeypatch.setattr(build, "CALLS_PATH", str(broken))
    monkeypatch.setattr(mb, "_calls", None)
    monkeypatch.setattr(mb, "_ops", {})
    plan = mb.merit_plan_pool2d(1, 3, 8, 8, 3, 3, 2, 2, 1, 1, 0)
    x = torch.zeros((1, 3, 8, 8))
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert mb._ordinary("merit_pool2d", plan, x) is None
    with warnings.catch_warnings():                     # said once
        warnings.simplefilter("error")
        with pytest.raises(TypeError, match="device tensor"):       # the general path judges the call
            mb.merit_pool2d(plan, x)
    plan.destroy()
    with pytest.raises(ValueError):
        mb.merit_pool2d(plan, x)


def test_a_module_of_another_pytorch_is_not_used(monkeypatch):
    monkeypatch.setattr(mb, "_calls", None)
    monkeypatch.setattr(mb, "_ops", {})
    monkeypatch.setattr(torch, "__version__", "0.0")
    plan = mb.merit_plan_pool2d(1, 3, 8, 8, 3, 3, 2, 2, 1, 1, 0)
    with pytest.warns(RuntimeWarning, match="built for PyTorch"):
        assert mb._ordinary("merit_pool2d", plan, torch.zeros(1)) is None

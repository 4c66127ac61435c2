"""The native autograd node is tied to the Python and torch it was built against: a change of either rebuilds it, and a stale one is
refused with the command that rebuilds it."""
import pytest

from paper_2312_03415_amd import build, module


def test_a_change_of_torch_rebuilds_the_native_node(monkeypatch):
    if not build._ext_is_current():   # (built for another torch)
        build.build()
    assert build._ext_is_current()    # the library itself says what it was built for: no second file to lose
    calls = []
    monkeypatch.setattr(build, "_compile", lambda src: calls.append(src) or src)
    monkeypatch.setattr(build, "_compile_ext", lambda: calls.append("ext"))
    monkeypatch.setattr(build.subprocess, "run", lambda *a, **k: None)
    monkeypatch.setattr(build.os.path, "getmtime", lambda f: 1.0 if "csrc" in f or f.endswith(".h") else 2.0)   # libraries newer than their sources
    build.build()
    assert not calls
    monkeypatch.setattr(build, "_ext_abi", lambda: "python cpython-310 torch 99.0")
    build.build()
    assert "ext" in calls


def test_a_stale_native_node_is_refused(monkeypatch):
    pytest.importorskip("torch")
    monkeypatch.setattr(build, "_ext_abi", lambda: "python cpython-310 torch 99.0")
    monkeypatch.setattr(module, "_native_module", None)
    with pytest.raises(ImportError, match="paper_2312_03415_amd.build"):
        module._native()

"""CPU checks of build.py with the compilers replaced: the C libraries do not depend on torch or on the binding."""
import importlib.util
import os

import pytest

from paper_2603_05451_amd import build


@pytest.fixture
def places(monkeypatch, tmp_path):
    """Every command writes its output file; those of binding.cpp fail with `fails` set."""
    for name in ("LIB", "PROBES_LIB", "BINDING"):
        monkeypatch.setattr(build, name, str(tmp_path / (name + ".so")))
    state = {"fails": False, "commands": []}

    def run(cmd, verbose):
        state["commands"].append(cmd)
        if state["fails"] and any(c.endswith("binding.cpp") for c in cmd):
            raise RuntimeError("no binding")
        open(cmd[cmd.index("-o") + 1], "w").close()

    monkeypatch.setattr(build, "_run", run)
    state["there"] = lambda: sorted(f for f in os.listdir(tmp_path))
    return state


def test_everything_is_built(places):
    assert build.build_library() == build.LIB and places["there"]() == ["BINDING.so", "LIB.so", "PROBES_LIB.so"]
    assert not any("-w" in c for c in places["commands"])


def test_a_binding_that_does_not_compile_leaves_the_libraries(places):
    places["fails"] = True
    with pytest.raises(RuntimeError, match="no binding"):
        build.build_library()
    assert places["there"]() == ["LIB.so", "PROBES_LIB.so"]


def test_the_libraries_without_torch(places, monkeypatch):
    find = importlib.util.find_spec
    monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find(name, *a))
    with pytest.raises(RuntimeError, match="needs torch"):
        build.build_library()
    assert places["there"]() == ["LIB.so", "PROBES_LIB.so"]

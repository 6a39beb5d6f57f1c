"""The binding's extension saves host time and nothing else: where it is missing, no library, or built for something
else, the library loads, says so once, and the calls that it has go through ctypes."""

import ctypes
import os
import subprocess
import warnings

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture()
def binding(monkeypatch):
    """The binding as before its first call."""
    from paper_2605_29986_amd import binding, build
    if not (os.path.exists(binding.library_path()) and os.path.exists(binding.stepcall_path())):
        build.build()
    for name in ("_lib", *CALLS):
        monkeypatch.setattr(binding, name, None)
    return binding


# the extension's calls, and how many arguments each takes
CALLS = {"_decode_step": 9, "_engine_step": 10, "_signatures": 9, "_build_classes": 9, "_displacements": 10, "_nfa_signatures": 5}


def _goes_through_ctypes(binding):
    with pytest.warns(RuntimeWarning, match="through ctypes"):
        lib = binding.load_library()
    assert isinstance(lib, ctypes.CDLL) and binding.cfgzip_version() >= 100
    for name, n in CALLS.items():
        assert getattr(binding, name) is binding._by_ctypes and getattr(binding, name)(*range(n)) is None
    logits = torch.zeros((1, 8))
    ids = torch.zeros(8, dtype=torch.int32)
    with pytest.raises(ValueError, match="GPU tensor"):
        binding.cfgzip_decode_step(logits, ids[:1].view(1, 1), ids, 1, ids[:1], ids[:1])
    with pytest.raises(ValueError, match="GPU tensor"):
        binding.cfgzip_engine_step(logits, ids[:1].view(1, 1), 1, ids, None, None, ids[:1])


def test_the_extension_is_used_where_it_is_there(binding):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        binding.load_library()
    assert list(CALLS) == ["_" + name for name in binding._CALLS]
    for name, n in CALLS.items():
        assert getattr(binding, name).__module__ == "cfgzip_stepcall"
        assert getattr(binding, name)(*range(n)) is None  # what is not plain tensors in GPU memory is left to ctypes


def test_without_the_extension(binding, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_STEPCALL_PATH", str(tmp_path / "cfgzip_stepcall.so"))
    _goes_through_ctypes(binding)


def test_an_extension_that_is_no_library(binding, monkeypatch, tmp_path):
    path = tmp_path / "cfgzip_stepcall.so"
    path.write_bytes(b"not a library")
    monkeypatch.setattr(binding, "_STEPCALL_PATH", str(path))
    _goes_through_ctypes(binding)


@pytest.mark.parametrize("built_for", ["2.9.1+rocm6.4", "2.10.1", "3.0.0a0+git"])
def test_an_extension_of_another_torch(binding, monkeypatch, built_for):
    monkeypatch.setattr(binding.torch, "__version__", built_for)
    _goes_through_ctypes(binding)


def test_a_build_without_a_compiler_for_the_extension(monkeypatch, tmp_path):
    """The library is built all the same, and an extension of an older source does not stay beside it."""
    from paper_2605_29986_amd import build
    for name in ("LIB_PATH", "STEPCALL_PATH", "TOOL_PATH"):
        monkeypatch.setattr(build, name, str(tmp_path / os.path.basename(getattr(build, name))))
    (tmp_path / os.path.basename(build.STEPCALL_PATH)).write_bytes(b"older")
    ran = []

    def check_call(cmd):
        if cmd[0] == "no-such-compiler":
            raise FileNotFoundError(cmd[0])
        ran.append(cmd)
        open(cmd[cmd.index("-o") + 1], "wb").close()

    monkeypatch.setenv("CXX", "no-such-compiler")
    monkeypatch.setattr(build, "find_hipcc", lambda: "hipcc")
    monkeypatch.setattr(subprocess, "check_call", check_call)
    assert build.build() == build.LIB_PATH and len(ran) == 2
    assert os.path.exists(build.LIB_PATH) and os.path.exists(build.TOOL_PATH)
    assert not os.path.exists(build.STEPCALL_PATH)

"""The binding's native host path (csrc_host/fsa_host.cpp) without a GPU: built with a header that lets CPU tensors
through, its library calls answered by Python functions."""
import ctypes
import importlib.machinery
import importlib.util
import os
import subprocess
import sys

import pytest
import torch

from paper_2511_13645_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
B, N, E, D, K1, K2 = 5, 9, 20, 8, 3, 2


class Host:
    """The module, the calls that reached the library, and what they are to return."""
    def __init__(self, path):
        spec = importlib.util.spec_from_loader("_fsa_host", importlib.machinery.ExtensionFileLoader("_fsa_host", path))
        self.module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.module)
        self.shim = ctypes.CDLL(path)
        self.calls, self.status, self.keep = [], 0, []
        addresses = {}
        for name in binding._HOST_ENTRIES:
            fn = ctypes.CFUNCTYPE(ctypes.c_int, *getattr(binding.lib(), name).argtypes)(self._answer(name))
            self.keep.append(fn)
            addresses[name] = ctypes.cast(fn, ctypes.c_void_p).value
        self.module.bind(lambda device: 4711, addresses)

    def _answer(self, name):
        def call(*args):
            self.calls.append((name, args))
            return self.status
        return call

    def count(self, name):
        return ctypes.c_int.in_dll(self.shim, name).value


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "_fsa_host_on_cpu.so")
    build.build_host(("-include", os.path.join(ROOT, "tests", "native", "host_path_shim.h")), out=out)
    return Host(out)


def _graph():
    i32 = dict(dtype=torch.int32)
    return dict(indptr=torch.zeros(N + 1, **i32), indices=torch.zeros(E, **i32), w=torch.zeros(E), x=torch.zeros(N, D),
                seeds=torch.zeros(B, **i32), ids1=torch.zeros((B, K1), **i32), ids2=torch.zeros((B, K1, K2), **i32))


@pytest.mark.parametrize("fan", [[K1], [K1, K2]])
def test_outputs_are_allocated_without_the_interpreter_lock(host, fan):
    """An allocation may wait for the driver; other threads run meanwhile, as they do in torch's own allocating calls."""
    g, two = _graph(), len(fan) == 2
    before, held = host.count("allocations"), host.count("allocations_with_gil")
    for w in (None, g["w"]):
        out = host.module.sample_fwd(g["indptr"], g["indices"], w, g["x"], g["seeds"], fan, 1, True, True)
        assert out[0].shape == (B, D) and out[2].shape == (B, K1)
    out = host.module.replay_fwd(g["x"], g["ids1"], g["ids2"] if two else None, True)
    assert out[0].shape == (B, D)
    assert host.count("allocations") - before == (4 + 6 + 2 if two else 2 + 3 + 1)
    assert host.count("allocations_with_gil") == held


@pytest.mark.parametrize("found", ["nothing", "something else"])
def test_the_library_loads_without_the_host_path(tmp_path, found):
    """The host path only saves time: where it is missing, or what lies there is no module of this Python, the binding
    says so and takes every call itself."""
    path = tmp_path / "host.so"
    if found == "something else":
        path.write_bytes(b"not a shared object")
    code = ("import warnings\n"
            "from paper_2511_13645_amd import binding\n"
            "binding.HOST_PATH = %r\n"
            "with warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always')\n"
            "    assert binding.lib() and binding._host is None\n"
            "assert [x for x in w if issubclass(x.category, RuntimeWarning) and binding.HOST_PATH in str(x.message)]\n"
            "assert binding.fsa_mean_bwd_workspace_bytes(1024, 25, 10, 602) > 0\n" % str(path))
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr


def test_the_host_path_belongs_to_one_python_and_one_torch():
    """It uses what neither keeps stable: a build for another one has another name and is not loaded."""
    name = os.path.basename(binding.HOST_PATH)
    assert sys.implementation.cache_tag in name and torch.__version__ in name
    assert binding.lib() and binding._host.__file__ == binding.HOST_PATH


def _sources(tmp_path, change=lambda text: text):
    """A copy of fsa_host.cpp with include/fsa.h where it looks for it, the header changed."""
    src = tmp_path / "package" / "csrc_host" / "fsa_host.cpp"
    for path, text in ((src, open(build.HOST_SOURCE).read()),
                       (tmp_path / "include" / "fsa.h", change(open(os.path.join(ROOT, "include", "fsa.h")).read()))):
        path.parent.mkdir(parents=True, exist_ok=True)
        path.write_text(text)
    return str(src)


def test_a_changed_declaration_of_the_library_does_not_compile(tmp_path, monkeypatch, capfd):
    declared = "int fsa_mean_bwd(const float* grad_out, "
    def change(text):
        assert declared in text
        return text.replace(declared, declared + "int64_t first_root, ")
    monkeypatch.setattr(build, "HOST_SOURCE", _sources(tmp_path, change))
    with pytest.raises(subprocess.CalledProcessError):
        build.build_host(("-fsyntax-only",), out=str(tmp_path / "host.so"))
    assert "abi.fsa_mean_bwd(" in capfd.readouterr().err


def test_the_host_path_is_stale_after_a_change_of_the_header(tmp_path, monkeypatch):
    header = os.path.join(ROOT, "include", "fsa.h")
    at = os.path.getmtime(header)
    files = {}
    for name, mtime in (("LIB", at + 1e6), ("HOST_SOURCE", at - 20), ("host", at - 10)):
        files[name] = str(tmp_path / name)
        open(files[name], "w").close()
        os.utime(files[name], (mtime, mtime))
    monkeypatch.setattr(build, "LIB", files["LIB"])
    monkeypatch.setattr(build, "HOST_SOURCE", files["HOST_SOURCE"])
    monkeypatch.setattr(build, "host_lib", lambda: files["host"])
    assert build.is_stale()
    os.utime(files["host"], (at + 10, at + 10))
    assert not build.is_stale()

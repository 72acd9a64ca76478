"""The short way from Python into the library, built for CPU tensors and calling functions of the test instead of the library's."""
import ctypes
import importlib.util
import shutil
import subprocess
import sys

import pytest

FUNCTIONS = r"""
#include <new>
#include <vector>
static std::vector<const void*> seen;
extern "C" int record(void* plan, const float* x, const float* w, const float* b, float* y, void* s) { seen = {plan, x, w, b, y, s}; y[0] = x[0] + w[0]; return 0; }
extern "C" int refuse(void*, const float*, const float*, const float*, float*, void*) { return -3; }
extern "C" int throws(void*, const float*, const float*, const float*, float*, void*) { throw std::bad_alloc(); }
extern "C" int throws_static(const void*, const void*, int, const float*, const float*, const float*, float*, void*) { throw std::bad_alloc(); }
extern "C" int record_static(const int* shape, const int* geom, int tile, const float* x, const float*, const float*, float* y, void*)
{
    for (int i = 0; i < 7; ++i) y[i] = (float)shape[i];
    for (int i = 0; i < 6; ++i) y[7 + i] = (float)geom[i];
    y[13] = (float)tile;
    return 0;
}
"""
SHAPES = ((1, 2, 3, 3), (2, 2, 1, 1), (2,), (1, 2, 3, 3))


@pytest.fixture(scope="module")
def fast(tmp_path_factory):
    """(the module, address of a named function)"""
    pytest.importorskip("torch")
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    from paper_2002_12418_amd.build import fast_call_command
    d = tmp_path_factory.mktemp("fast_call")
    subprocess.run(fast_call_command(str(d / "_fast_call.so"), "-DFAST_CALL_ON_CPU", "-O0"), check=True, timeout=300)
    (d / "functions.cpp").write_text(FUNCTIONS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", str(d / "functions.cpp"), "-o", str(d / "functions.so")], check=True, timeout=120)
    spec = importlib.util.spec_from_file_location("_fast_call", str(d / "_fast_call.so"))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    functions = ctypes.CDLL(str(d / "functions.so"))
    yield module, lambda name: ctypes.cast(getattr(functions, name), ctypes.c_void_p).value


def tensors():
    import torch
    return [torch.rand(s) for s in SHAPES]


def test_an_exception_leaves_the_interpreter_whole(fast):
    """In a process of its own: without the GIL the interpreter ends where it next looks for it."""
    module, _ = fast
    d = module.__file__.rsplit("/", 1)[0]
    code = f"""
import ctypes, importlib.util, threading, torch
spec = importlib.util.spec_from_file_location("_fast_call", {module.__file__!r})
m = importlib.util.module_from_spec(spec)
spec.loader.exec_module(m)
f = ctypes.CDLL({d + "/functions.so"!r})
address = lambda n: ctypes.cast(getattr(f, n), ctypes.c_void_p).value
x, w, b, y = [torch.rand(s) for s in {SHAPES!r}]
r = m.Runner(address("throws"), 1, *{SHAPES!r})
r.remember(w)
class L: n = c_in = h = w = c_out = kh = kw = stride = pad = dil = 1
for _ in range(3):
    assert r(x, w, b, y) is None
    assert m.run_static(address("throws_static"), L, 2, x, w, b, y) is None
    t = threading.Thread(target=lambda: [list(range(10)) for _ in range(1000)])
    t.start()
    t.join()
print("whole")
"""
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and "whole" in p.stdout, p.stderr[-2000:]


def test_a_plan_that_its_weights_hold_is_collected(fast):
    """weight -> plan -> runner -> weight, as where a module keeps the plan with its parameter."""
    import gc
    import weakref
    module, address = fast

    class Plan:
        pass

    x, w, b, y = tensors()
    plan = Plan()
    plan.fast = module.Runner(address("record"), 1, *SHAPES)
    plan.fast.remember(w)
    assert plan.fast(x, w, b, y) == 0
    w.plan = plan
    gone = weakref.ref(plan)
    assert gc.is_tracked(plan.fast)
    del plan, w
    gc.collect()
    assert gone() is None


def test_the_last_reference_to_a_remembered_tensor(fast):
    """Forgetting a tensor may run Python code, which may use the runner again."""
    module, address = fast
    x, w, b, y = tensors()
    other, third = w * 2, w * 3
    r = module.Runner(address("record"), 1, *SHAPES)

    class Last:
        def __del__(self):
            r.remember(other)

    w.last = Last()
    r.remember(w)
    del w
    r.remember(third)                       # w's last reference goes here, and the runner is told of another
    assert r(x, other, b, y) == 0 and r(x, third, b, y) is None
    assert float(y.view(-1)[0]) == float(x.view(-1)[0] + other.view(-1)[0])
    r.close()
    assert r(x, other, b, y) is None
    assert sys.getrefcount(other) == 2 and sys.getrefcount(third) == 2       # the name and the argument


def test_the_built_file_is_for_this_torch_and_source(monkeypatch, tmp_path):
    """A module built against other headers reads tensors at other places: it is not the file that the binding looks for."""
    import paper_2002_12418_amd.build as build
    path = build.fast_call_path()
    assert path.startswith(build.PKG) and path.endswith(".so") and path == build.fast_call_path()
    # the binding loads that file and no other
    import paper_2002_12418_amd.binding as binding
    monkeypatch.setattr(build, "fast_call_path", lambda: str(tmp_path / "other.so"))
    with pytest.warns(RuntimeWarning):
        assert binding._load_fast_call() is None
    monkeypatch.undo()
    # another torch, another Python, another source, another interface
    root = tmp_path / "torch"
    root.mkdir()
    (root / "version.py").write_text("__version__ = '0.0'\n")
    monkeypatch.setattr(build, "_torch_dir", lambda: str(root))
    other = {path, build.fast_call_path()}
    monkeypatch.undo()
    monkeypatch.setattr(build.sys, "version", "9.9")
    other.add(build.fast_call_path())
    monkeypatch.undo()
    for name in ("CSRC", "INCLUDE"):
        changed = tmp_path / name
        shutil.copytree(getattr(build, name), changed)
        for f in ("fast_call.cpp", "mnn_conv.h"):
            if (changed / f).exists():
                (changed / f).write_text((changed / f).read_text() + "\n")
        monkeypatch.setattr(build, name, str(changed))
        other.add(build.fast_call_path())
        monkeypatch.undo()
    assert len(other) == 5
    monkeypatch.setattr(build, "CSRC", str(tmp_path / "nowhere"))
    assert build.fast_call_path() is None


def test_without_torch_or_a_compiler_the_library_is_built(monkeypatch, tmp_path, capsys):
    import paper_2002_12418_amd.build as build
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build, "_hipcc", lambda: "true")
    real = subprocess.run

    def run(cmd, *args, **kw):
        if cmd[0] == "true":
            open(cmd[cmd.index("-o") + 1], "w").close()
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        return real(cmd, *args, **kw)

    monkeypatch.setattr(build.subprocess, "run", run)
    assert build.build_library(verbose=False) == str(tmp_path / "lib.so")
    assert "g++" in capsys.readouterr().err
    find = importlib.util.find_spec
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find(name, *a))
    assert build.build_library(verbose=False) == str(tmp_path / "lib.so")


def test_builds_at_the_same_time_write_files_of_their_own(monkeypatch, tmp_path):
    import os

    import paper_2002_12418_amd.build as build
    written = []

    def run(cmd, *args, **kw):
        written.append(cmd[cmd.index("-o") + 1])
        open(written[-1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    for pid in (11, 12):
        monkeypatch.setattr(build.os, "getpid", lambda: pid)
        build.build_fast_call()
    assert len(set(written)) == 2 and all(os.path.dirname(f) == str(tmp_path) for f in written)
    assert os.listdir(tmp_path) == [os.path.basename(build.fast_call_path())]

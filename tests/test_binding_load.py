"""Building and loading the library from Python: what other threads may see meanwhile, and what works without the native calls."""
import os
import subprocess
import sys
import time

import pytest


@pytest.fixture
def binding(monkeypatch):
    from paper_2407_08330_amd import binding as b
    b.load_library()
    monkeypatch.setattr(b, "_lib", None)
    monkeypatch.setattr(b, "_calls", None)
    return b


def test_a_loaded_library_has_its_native_calls(binding):
    """Between any two steps of load_library: who sees _lib goes on to use _calls without a look at it."""
    seen = set()

    def step(frame, event, arg):
        frame.f_trace_opcodes = True
        seen.add((binding._lib is not None, binding._calls is not None))
        return step

    def trace(frame, event, arg):
        return step(frame, event, arg) if frame.f_code is binding.load_library.__code__ else None

    before = sys.gettrace()
    sys.settrace(trace)
    try:
        binding.load_library()
    finally:
        sys.settrace(before)
    assert (True, True) in seen and (True, False) not in seen


def fresh_package(tmp_path, module=None):
    """A copy of the package with libhdt.so and, as its Python module, what `module` writes."""
    import shutil
    from paper_2407_08330_amd import binding as b
    b.load_library()  # (built by now, or this fails)
    src = os.path.dirname(b.__file__)
    pkg = tmp_path / os.path.basename(src)
    pkg.mkdir()
    for name in ("__init__.py", "binding.py", "build.py", "libhdt.so"):
        shutil.copy(os.path.join(src, name), pkg)
    if module:
        (pkg / "_hdt_pycall.py").write_text(module)
    return tmp_path


CALLS = r"""
import warnings
with warnings.catch_warnings(record=True) as told:
    warnings.simplefilter("always")
    import torch
    import paper_2407_08330_amd as hdt
    lib = hdt.load_library()
    hdt.load_library()
print(lib.hdt_index_vectors_workspace_bytes(1, 64) > 0, sum("_hdt_pycall" in str(w.message) for w in told))
ids = torch.zeros((1, 8), dtype=torch.int32)
q = torch.zeros((1, 1, 8, 64))
for call in (lambda: hdt.hdt_build_layout(ids, ids), lambda: hdt.hdt_attn_fwd(hdt.Layout(0, 1, 8), q, q, q, 0.125),
             lambda: hdt.hdt_attn_bwd(hdt.Layout(0, 1, 8), q, q, q, q, q, q, 0.125)):
    try:
        call()
    except ValueError as e:
        print("general path:", e)
"""


@pytest.mark.parametrize("module", [None, "raise ImportError('undefined symbol')", "def bind(*a): raise AssertionError\ntorch_version = '1.0'"],
                         ids=["missing", "does not load", "another torch"])
def test_the_library_alone_is_enough(tmp_path, module):
    """libhdt.so takes any Python and torch; the module that saves host time is compiled for one of each."""
    run = subprocess.run([sys.executable, "-c", CALLS], cwd=fresh_package(tmp_path, module), stdout=subprocess.PIPE,
                         stderr=subprocess.STDOUT, text=True)
    assert run.returncode == 0, run.stdout[-2000:]
    out = run.stdout.split("\n")
    assert out[0] == "True 1" and sum(line.startswith("general path: ") for line in out) == 3, run.stdout[-2000:]


@pytest.mark.parametrize("command", [["false"], ["/no/such/compiler"], None], ids=["fails", "no compiler", "no torch"])
def test_the_library_is_linked_without_the_module(tmp_path, monkeypatch, command):
    """A host compiler or torch headers that are missing: libhdt.so is there, and build() says what is not."""
    from paper_2407_08330_amd import build as b
    hipcc = tmp_path / "hipcc"
    hipcc.write_text("#!/bin/sh\nwhile [ $# -gt 1 ]; do [ \"$1\" = -o ] && : > \"$2\"; shift; done\n")
    hipcc.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setattr(b, "CSRC", str(tmp_path))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "libhdt.so"))
    monkeypatch.setattr(b, "PYCALL", str(tmp_path / "_hdt_pycall.so"))
    (tmp_path / "_hdt_pycall.so").write_text("of an earlier build")

    def pycall():
        if command is None:
            raise ImportError("No module named 'torch'")
        return command

    monkeypatch.setattr(b, "_pycall_command", pycall)
    with pytest.raises(RuntimeError, match="_hdt_pycall"):
        b.build()
    assert (tmp_path / "libhdt.so").exists() and not (tmp_path / "_hdt_pycall.so").exists()


def test_a_call_that_is_not_plain_is_refused_quickly():
    """The general path pays for every refusal.  Against one by the number of arguments alone, 0.05 us; a C++ exception on the way
    takes thirty times that, a dozen looks at arguments three times."""
    import numpy as np
    import torch
    from paper_2407_08330_amd import binding as b
    b.load_library()
    q, ids = torch.zeros((1, 1, 8, 64)), torch.zeros((1, 8), dtype=torch.int32)
    fwd = [8, 1, 8, 8, q, q, q, 0.125, None, None, None, None]
    bwd = [*fwd[:8], q, q, q, None, None, None, None, None]
    build = [ids, ids, 0, 0, False, False, False, 0, True, 0, None]
    assert b._calls.attn_fwd() is b._calls.attn_bwd() is b._calls.build_layout() is None

    def us(f, args):
        def once():
            t = time.perf_counter()
            for _ in range(500):
                assert f(*args) is None
            return (time.perf_counter() - t) / 500 * 1e6
        return min(once() for _ in range(40))

    class Own(torch.Tensor):
        pass

    forms = [(b._calls.attn_fwd, fwd, {}), (b._calls.attn_fwd, fwd, {7: np.float64(0.125)}), (b._calls.attn_fwd, fwd, {7: 1}),
             (b._calls.attn_fwd, fwd, {4: q.as_subclass(Own)}), (b._calls.attn_bwd, bwd, {7: np.float64(0.125)}),
             (b._calls.attn_bwd, bwd, {15: 64}), (b._calls.build_layout, build, {}), (b._calls.build_layout, build, {7: np.int64(7)}),
             (b._calls.build_layout, build, {5: 0}), (b._calls.build_layout, build, {9: 1 << 70})]
    for f, args, other in forms:
        args = [other.get(i, x) for i, x in enumerate(args)]
        assert us(f, args) < 10 * us(f, ()), (f.__name__, other)

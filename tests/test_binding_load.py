"""Loading the library from Python: what other threads may see meanwhile."""
import sys

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

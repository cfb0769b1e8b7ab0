"""The native form of the hot calls (csrc/hdt_pycall.cpp) against binding.py's general path: the same results to the bit and
the same errors, over the forms of arguments that a program uses."""
import math

import numpy as np
import pytest

import gpu_common as gc
from paper_2407_08330_amd import inputs

pytestmark = pytest.mark.gpu


class General:
    """What takes no call: binding.py's own path does."""
    build_layout = attn_fwd = attn_bwd = staticmethod(lambda *a: None)


class Counting:
    """The native calls, and which of them were taken."""

    def __init__(self, calls):
        self.calls, self.taken = calls, set()

    def __getattr__(self, name):
        f = getattr(self.calls, name)

        def call(*a):
            r = f(*a)
            if r is not None:
                self.taken.add(name)
            return r
        return call


BUILD, FWD, BWD = "build_layout", "attn_fwd", "attn_bwd"


def both(monkeypatch, f, taken, raises=False):
    """f() on the general path, then with the native calls, which must have taken exactly those of `taken`.  ``raises``: what
    the library and the binding raise is the result; a failed assertion is one in any case."""
    from paper_2407_08330_amd import binding
    binding.load_library()
    calls = Counting(binding._calls)
    out = []
    for c in (General, calls):
        with monkeypatch.context() as m:
            m.setattr(binding, "_calls", c)
            if not raises:
                out.append(f())
                continue
            with pytest.raises(Exception) as caught:
                f()
            assert not issubclass(caught.type, AssertionError)
            out.append((caught.type, str(caught.value)))
    assert calls.taken == set(taken)
    return out


def equal(a, b):
    import torch
    torch.cuda.synchronize()
    assert len(a) == len(b)
    for x, y in zip(a, b):
        if isinstance(x, torch.Tensor):
            assert type(x) is type(y) and x.dtype == y.dtype and x.device == y.device and x.requires_grad == y.requires_grad
            assert x.stride() == y.stride() and torch.equal(x, y)
        else:
            assert x == y


def state(n=300, heads=2, d=64, dtype="bf16", batch=2):
    level, parent = map(np.stack, zip(*(inputs.listops_like_tree(np.random.default_rng(b), n) for b in range(batch))))
    _, x = gc.make_inputs(batch, heads, n, d, 5, dtype, 4)
    return gc.to_dev_i32(level), gc.to_dev_i32(parent), x


@pytest.mark.parametrize("dtype,d,tile", [("bf16", 64, (0, 0)), ("bf16", 128, (64, 32)), ("f32", 64, (0, 0))])
@pytest.mark.parametrize("form", ["plain", "outputs", "stream", "deferred", "grad", "subclass"])
def test_same_results(monkeypatch, dtype, d, tile, form):
    import torch
    import paper_2407_08330_amd as hdt
    level, parent, (q, k, v, d_o) = state(d=d, dtype=dtype)
    scale = 1 / math.sqrt(d)
    if form == "grad":
        q = torch.nn.Parameter(q)
    if form == "subclass":
        q = q.as_subclass(type("Own", (torch.Tensor,), {}))
    stream = torch.cuda.Stream() if form == "stream" else None
    torch.cuda.synchronize()

    def run():
        lay = hdt.hdt_build_layout(level, parent, *tile, edges=6, deferred=form == "deferred", stream=stream)
        assert (lay.batch, lay.n_pos, lay.n_kv) == (level.shape[0], level.shape[1], level.shape[1])
        kw = dict(stream=stream)
        if form == "outputs":
            kw.update(o=torch.empty_like(q), lse=torch.empty(q.shape[:3], device="cuda"))
        o, lse = hdt.hdt_attn_fwd(lay, q, k, v, scale, **kw)
        if form == "outputs":
            assert o is kw["o"] and lse is kw["lse"]
            n = hdt.hdt_attn_bwd_workspace_bytes(lay, q.shape[1], d, 0 if dtype == "bf16" else 1)
            ws = gc.GuardedWorkspace(n)
            kw = dict(dq=torch.empty_like(q), dk=torch.empty_like(k), dv=torch.empty_like(v), workspace=ws.view)
        g = hdt.hdt_attn_bwd(lay, q, k, v, o, lse, d_o, scale, **{n: t for n, t in kw.items() if n not in ("o", "lse")})
        if form == "outputs":
            assert g[0] is kw["dq"] and g[1] is kw["dk"] and g[2] is kw["dv"]
            torch.cuda.synchronize()
            ws.check()
        torch.cuda.synchronize()
        lay.destroy()
        return [t.detach() if form == "grad" else t for t in (o, lse, *g)]

    # (on another stream a temporary workspace is the general path's business)
    equal(*both(monkeypatch, run, {"stream": {BUILD, FWD}, "subclass": {BUILD}}.get(form, {BUILD, FWD, BWD})))


def test_cross_attention_with_a_workspace(monkeypatch):
    import torch
    import paper_2407_08330_amd as hdt
    level = gc.to_dev_i32(np.random.default_rng(1).integers(-1, 4, (2, 2100)))
    q, d_o = (torch.randn((2, 2, 70, 64), device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((2, 2, 2100, 64), device="cuda").bfloat16() for _ in range(2))
    lay = hdt.hdt_build_cross_layout(level, 70, 14)
    need = hdt.hdt_attn_fwd_workspace_bytes(lay, 2, 64, 0)
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")

    def run():
        o, lse = hdt.hdt_attn_fwd(lay, q, k, v, 0.125, workspace=ws)
        return [o, lse, *hdt.hdt_attn_bwd(lay, q, k, v, o, lse, d_o, 0.125)]

    equal(*both(monkeypatch, run, {FWD, BWD}))


ERRORS = {
    "shape": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q[:, :, :-1].contiguous(), s.k, s.v, 0.125), ()),
    "kv shape": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q, s.k[:, :, :-1].contiguous(), s.v, 0.125), ()),
    "three dimensions": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q[0], s.k, s.v, 0.125), ()),
    "dtypes differ": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q, s.k.float(), s.v, 0.125), ()),
    "float64": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q.double(), s.k.double(), s.v.double(), 0.125), ()),
    "strided": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q.transpose(2, 3), s.k, s.v, 0.125), ()),
    "on the host": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q.cpu(), s.k, s.v, 0.125), ()),
    "scale": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q, s.k, s.v, -1.0), {FWD}),
    "aliased": (lambda h, s: h.hdt_attn_fwd(s.lay, s.q, s.k, s.v, 0.125, o=s.q), {FWD}),
    "d_o shape": (lambda h, s: h.hdt_attn_bwd(s.lay, s.q, s.k, s.v, s.q, s.lse, s.d_o[:, :1].contiguous(), 0.125), ()),
    "small workspace": (lambda h, s: h.hdt_attn_bwd(s.lay, s.q, s.k, s.v, s.d_o, s.lse, s.d_o, 0.125, workspace=s.lse[:0]), {BWD}),
    "ids on the host": (lambda h, s: h.hdt_build_layout(s.level.cpu(), s.parent), ()),
    "int64 ids": (lambda h, s: h.hdt_build_layout(s.level.long(), s.parent), ()),
    "ids' shapes": (lambda h, s: h.hdt_build_layout(s.level, s.parent[:, :-1].contiguous()), ()),
    "tile": (lambda h, s: h.hdt_build_layout(s.level, s.parent, 48, 64), {BUILD}),
    "hierarchy": (lambda h, s: h.hdt_build_layout(s.level, s.level + 400), {BUILD}),
    "destroyed": (lambda h, s: h.hdt_attn_fwd(s.dead, s.q, s.k, s.v, 0.125), {FWD}),
}


@pytest.mark.parametrize("name", list(ERRORS))
def test_same_errors(monkeypatch, name):
    import types
    import torch
    import paper_2407_08330_amd as hdt
    level, parent, (q, k, v, d_o) = state()
    s = types.SimpleNamespace(level=level, parent=parent, q=q, k=k, v=v, d_o=d_o, lse=torch.zeros(q.shape[:3], device="cuda"),
                              lay=hdt.hdt_build_layout(level, parent), dead=hdt.hdt_build_layout(level, parent))
    s.dead.destroy()
    call, taken = ERRORS[name]
    general, here = both(monkeypatch, lambda: call(hdt, s), taken, raises=True)
    assert general == here


@pytest.mark.parametrize("scale", [1, np.float64(0.125), "tensor"])
def test_other_numbers_take_the_general_path(monkeypatch, scale):
    import torch
    import paper_2407_08330_amd as hdt
    level, parent, (q, k, v, _) = state()
    lay = hdt.hdt_build_layout(level, parent)
    scale = torch.tensor(0.25) if scale == "tensor" else scale
    equal(*both(monkeypatch, lambda: hdt.hdt_attn_fwd(lay, q, k, v, scale), ()))

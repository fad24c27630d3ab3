"""The binding's native marshalling: it takes calls of the plain form, with the results of the Python path, and leaves every other call
to that path and its errors."""
import sys

import numpy as np
import pytest
import torch

import paper_2210_06223_amd as pkg
from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import build, synth
from tests import _util as U


def test_tensors_that_are_not_on_the_gpu_are_left_to_the_python_path():
    L = B.lib()
    x, f, i = torch.zeros(1, 4, 4, 8), torch.zeros(8), torch.zeros(4, dtype=torch.int32)
    w = (torch.zeros(2, 8), torch.zeros(2), torch.zeros(2, 3, 3, 2), torch.zeros(2), torch.zeros(8, 2), f)
    assert B._marshal.masker_ex(L.at_masker_ex, x, f, 0.0, 2, 0.0, i, i, i, None) is None
    assert B._marshal.block_ex(L.at_ex, x, i, i, 2, *w, x, 0) is None
    assert B._marshal.block_dense(L.at_dense, x, *w, x, 0) is None
    assert B._marshal.block_packed(L.at_packed, x, i, i, 2, 2, f, L.at_packed_bytes, f, f, f, x, 0) is None
    assert B._marshal.block_planned(L.at_planned, x, i, i, None, 2, 2, f, f, f, f, x, None, 0) is None
    for junk in (None, 3, "x", [1]):
        assert B._marshal.masker_ex(L.at_masker_ex, junk, f, 0.0, 2, 0.0, i, i, i, None) is None
    with pytest.raises(TypeError):
        B._marshal.block_dense(L.at_dense, x)
    with pytest.raises(ValueError, match="device memory"):
        B.lasnet_masker(x, f, 0.0, 2, mask=i, idx=i, count=i)
    with pytest.raises(ValueError, match="device memory"):
        B.lasnet_dense_bottleneck(x, *w, out=x)


def test_calls_that_leave_their_outputs_out_are_not_offered(monkeypatch):
    """(The attempt could only fail.)"""
    B.lib()

    class Never:
        def __getattr__(self, name):
            raise AssertionError(name)
    monkeypatch.setattr(B, "_marshal", Never())
    x, f, i = torch.zeros(1, 4, 4, 8), torch.zeros(8), torch.zeros(4, dtype=torch.int32)
    w = (torch.zeros(2, 8), torch.zeros(2), torch.zeros(2, 3, 3, 2), torch.zeros(2), torch.zeros(8, 2), f)
    for call in (lambda: B.lasnet_masker(x, f, 0.0, 2), lambda: B.lasnet_masker_ex(x, f, 0.0, 2, mask=i, idx=i, pass_out=x),
                 lambda: B.lasnet_sparse_bottleneck(x, i, i, 2, *w), lambda: B.lasnet_dense_bottleneck(x, *w),
                 lambda: B.lasnet_sparse_bottleneck_packed(x, i, i, 2, 2, f, f, f, f)):
        with pytest.raises(ValueError, match="device memory"):
            call()


class _Refuses:
    """An import hook: the extension does not load."""
    def find_spec(self, name, path=None, target=None):
        if name == pkg.__name__ + "._marshal":
            raise ImportError("undefined symbol: of_another_torch")


@pytest.fixture(params=["missing", "of another torch"])
def without(request, monkeypatch):
    """The binding in a process where the extension is not there, or does not load."""
    name = pkg.__name__ + "._marshal"
    monkeypatch.delattr(pkg, "_marshal", raising=False)
    if request.param == "missing":
        monkeypatch.setitem(sys.modules, name, None)
    else:
        monkeypatch.delitem(sys.modules, name, raising=False)
        monkeypatch.setattr(sys, "meta_path", [_Refuses()] + sys.meta_path)
    monkeypatch.setattr(B, "_marshal", None)
    with pytest.warns(RuntimeWarning, match="undefined symbol" if request.param != "missing" else "_marshal"):
        monkeypatch.setattr(B, "_lib", B.load_library(build.LIB))


def test_the_library_loads_without_the_extension(without):
    assert B.lasnet_version() == 100
    x, f, i = torch.zeros(1, 4, 4, 8), torch.zeros(8), torch.zeros(4, dtype=torch.int32)
    with pytest.raises(ValueError, match="device memory"):
        B.lasnet_masker(x, f, 0.0, 2, mask=i, idx=i, count=i)


class _Case:
    def __init__(self, dtype):
        shape = (3, 14, 14, 1024, 256, 2) if dtype == "bf16" else (2, 8, 12, 64, 32, 4)
        self.cfg = synth.BlockConfig("marshal", *shape, dtype, 0.5, 161)
        self.d = U.dev_inputs(synth.make_block_inputs(self.cfg, want_f64=False))
        self.x, self.w = self.d["x"], U.weights(self.d)
        N, H, W, C, M, S = shape
        self.S, self.M, self.P = S, M, self.cfg.P
        self.masker = (torch.zeros((N, H // S, W // S), dtype=torch.uint8, device="cuda"), torch.zeros(self.P, dtype=torch.int32, device="cuda"),
                       torch.zeros(1, dtype=torch.int32, device="cuda"))


def _calls(c):
    """name, the marshalled call (its arguments), the binding's function with a stream (never marshalled)"""
    mask, idx, count = c.masker
    kw = dict(mask=mask, idx=idx, count=count)
    yield "masker", lambda o, **k: B.lasnet_masker(c.x, c.d["Wm"], -1, c.S, 0, **kw, **k)
    yield "masker_ex", lambda o, **k: B.lasnet_masker_ex(c.x, c.d["Wm"], -1.0, c.S, 0.0, pass_out=o, **kw, **k)
    yield "ex", lambda o, **k: B.lasnet_sparse_bottleneck(c.x, idx, count, c.S, *c.w, out=o, flags=B.LASNET_POST_RELU, **k)
    yield "all cells", lambda o, **k: B.lasnet_sparse_bottleneck(c.x, None, None, c.S, *c.w, out=o, **k)
    yield "dense", lambda o, **k: B.lasnet_dense_bottleneck(c.x, *c.w, out=o, **k)
    if c.cfg.dtype == "bf16":
        p = B.lasnet_pack_weights(c.S, c.w[0], c.w[2], c.w[4])
        b = (c.d["b1"], c.d["b2"], c.d["b3"])
        yield "packed", lambda o, **k: B.lasnet_sparse_bottleneck_packed(c.x, idx, count, c.S, c.M, p, *b, out=o, **k)
        ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
        yield "planned", lambda o, **k: B.lasnet_sparse_bottleneck_planned(c.x, idx, count, mask, c.S, c.M, p, *b, o, ws, **k)
        yield "planned without", lambda o, **k: B.lasnet_sparse_bottleneck_planned(c.x, idx, count, None, c.S, c.M, p, *b, o, None, **k)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_same_results_as_the_python_path(dtype, monkeypatch):
    c = _Case(dtype)
    B.lib()
    handled = []
    real = B._marshal

    class Spy:
        def __getattr__(self, name):
            def f(*a):
                r = getattr(real, name)(*a)
                handled.append(r is not None)
                return r
            return f
    monkeypatch.setattr(B, "_marshal", Spy())
    side = torch.cuda.Stream()
    for name, call in _calls(c):
        handled.clear()
        outs = []
        for where in ("marshalled", "python", "another stream"):
            o = torch.full_like(c.x, 777.0)
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side if where == "another stream" else torch.cuda.current_stream()):
                r = call(o, **({"stream": torch.cuda.current_stream()} if where == "python" else {}))
            torch.cuda.synchronize()
            outs.append([U.bits(t) for t in (r if isinstance(r, tuple) else (r,))] + [U.bits(o)])
        assert handled == [True, True], name                 # (with a stream the marshalling is not asked)
        for other in outs[1:]:
            assert all(np.array_equal(a, b) for a, b in zip(outs[0], other)), name


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_same_results_without_the_extension(dtype, without):
    c = _Case(dtype)
    for name, call in _calls(c):
        o, p = torch.full_like(c.x, 777.0), torch.full_like(c.x, 777.0)
        call(o)
        call(p, stream=torch.cuda.current_stream())
        assert np.array_equal(U.bits(o), U.bits(p)), name


@pytest.mark.gpu
def test_other_forms_are_converted_or_refused_as_ever():
    c = _Case("f32")
    mask, idx, count = c.masker
    m, i, n = B.lasnet_masker(c.x, c.d["Wm"], np.float32(-1), np.int64(c.S))          # (outputs made, numbers converted)
    m2, i2, n2 = B.lasnet_masker(c.x, c.d["Wm"], -1.0, c.S, 0.0, mask, idx, count)
    assert torch.equal(m, m2) and torch.equal(n, n2) and torch.equal(i[:int(n)], i2[:int(n)])
    out = torch.empty_like(c.x)
    with pytest.raises(ValueError, match="NHWC"):
        B.lasnet_dense_bottleneck(c.x.transpose(1, 2), *c.w, out=out)
    with pytest.raises(ValueError, match="dtype must be"):
        B.lasnet_dense_bottleneck(c.x.half(), *c.w, out=out)
    with pytest.raises(ValueError, match="of x's dtype"):
        B.lasnet_dense_bottleneck(c.x, c.w[0].bfloat16(), *c.w[1:], out=out)
    with pytest.raises(ValueError, match="b1 must be"):
        B.lasnet_sparse_bottleneck(c.x, idx, count, c.S, c.w[0], c.w[1].double(), *c.w[2:], out=out)
    with pytest.raises(ValueError, match="room for all"):
        B.lasnet_sparse_bottleneck(c.x, idx[:c.P - 1], count, c.S, *c.w, out=out)
    with pytest.raises(ValueError, match="int32"):
        B.lasnet_sparse_bottleneck(c.x, idx.long(), count, c.S, *c.w, out=out)
    with pytest.raises(ValueError, match="biases"):
        B.lasnet_sparse_bottleneck(c.x, idx, count, c.S, *c.w[:5], c.w[5][:8], out=out)
    with pytest.raises(B.LasnetError):
        B.lasnet_sparse_bottleneck(c.x, idx, count, 3, *c.w, out=out)
    with pytest.raises(B.LasnetError):
        B.lasnet_dense_bottleneck(c.x, *c.w, out=c.x)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [-1, -256])
def test_a_negative_mid_width_is_refused_as_in_the_python_path(M):
    """(Both before anything is enqueued.)"""
    c = _Case("bf16")
    mask, idx, count = c.masker
    p = B.lasnet_pack_weights(c.S, c.w[0], c.w[2], c.w[4])
    b, out = (c.d["b1"], c.d["b2"], c.d["b3"]), torch.empty_like(c.x)
    for stream in (None, torch.cuda.current_stream()):
        with pytest.raises(ValueError, match="biases"):
            B.lasnet_sparse_bottleneck_packed(c.x, idx, count, c.S, M, p, *b, out=out, stream=stream)
        with pytest.raises(ValueError, match="biases"):
            B.lasnet_sparse_bottleneck_planned(c.x, idx, count, mask, c.S, M, p, *b, out, None, stream=stream)

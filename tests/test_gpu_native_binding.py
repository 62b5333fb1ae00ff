"""The natively marshalled calls against the Python functions: the same outputs, and for every call that either refuses the same
exception (the native path hands what it does not take to the Python one)."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nf():
    import paper_2009_13062_amd as nf
    assert nf._native is not None, "the binding was not built, or for another torch"
    return nf


def _t(*s, dt=torch.float32):
    return torch.randn(*s, device="cuda").to(dt)


def _calls(nf, dt):
    f = torch.float32
    x, w, wp = _t(2, 128, 256, dt=dt), _t(2, 256, 384, dt=dt), None
    b, r, g = _t(2, 384, dt=f), _t(2, 128, 384, dt=dt), _t(2 * 256, dt=f)
    qkv, kr, mask = _t(2, 2 * 8, 3 * 128, dt=dt), _t(2, 16, 128, dt=dt), _t(2, 2, 8, dt=f)
    cx, cw, s = _t(2, 2 * 6, 9, 7, dt=dt), _t(2 * 8, 3, 3, 3, dt=dt), _t(16, dt=f)
    calls = [
        (nf.linear, (x, w), {}), (nf.linear, (x, w), dict(bias=b, residual=r, act=2)), (nf.linear, (x, w), dict(out=torch.empty_like(r))),
        (nf.linear, (x, w), dict(act=True)), (nf.linear, (x[:, ::2], w), {}), (nf.linear, (x, w[:1]), {}), (nf.linear, (x.cpu(), w), {}),
        (nf.linear, (x, w.double()), {}), (nf.linear, (x, w), dict(bias=b.bfloat16())), (nf.linear, (x, w), dict(act=7)),
        (nf.linear, (x, w), dict(out=torch.empty(2, 384, 128, device="cuda", dtype=dt).transpose(1, 2))), (nf.linear, (x[0], w), {}),
        (nf.linear, (x[:, :0], w), {}), (nf.linear, (torch.nn.Parameter(x), w), {}),
        (nf.layernorm, (x, g, g, 2), dict(residual=x)), (nf.layernorm, (x[0], g[:256], g[:256], 2), dict(layout=nf.MERGE_CHANNEL)),
        (nf.layernorm, (x, g, g, 2), dict(eps=1)), (nf.layernorm, (x, g, g.to(torch.float64), 2), {}), (nf.layernorm, (x, g, g, 0), {}),
        (nf.layernorm, (x, g, g, 2), dict(layout=5)), (nf.layernorm, (x[0], g, g, 2), {}),
        (nf.attention_packed, (qkv, 2, 8, 2), dict(mask=mask)), (nf.attention_packed, (qkv, 2, 8, 2), dict(scale=0.5)),
        (nf.attention_packed, (qkv, 2, 8, 2), dict(scale=1)), (nf.attention_packed, (qkv, 3, 8, 2), {}), (nf.attention_packed, (qkv, 2, 8, 5), {}),
        (nf.attention_packed, (qkv, 2, 8, 0), {}), (nf.attention_packed, (qkv, 2, 8, 2), dict(out=torch.empty(2, 16, 128, device="cuda", dtype=torch.float16))),
        (nf.attention_relpos_packed, (qkv, kr, 2, 8, 2), dict(bias_w=_t(2, 128), bias_r=_t(2, 128))), (nf.attention_relpos_packed, (qkv, kr[:, :9], 2, 8, 2), {}),
        (nf.conv2d, (cx, cw, 2), dict(g=2, pad=1, scale=s, shift=s, act=1)), (nf.conv2d, (cx, cw, 2), dict(g=2, stride=2, dil=2, pad=2, bias=s)),
        (nf.conv2d, (cx, cw, 2), dict(g=2, scale=s)), (nf.conv2d, (cx, cw, 5), {}), (nf.conv2d, (cx, cw, 2), dict(g=3)), (nf.conv2d, (cx, cw, 2), dict(g=2, stride=0)),
        (nf.conv2d, (cx[:, :, :2], cw, 2), dict(g=2)), (nf.conv2d, (cx.contiguous(memory_format=torch.channels_last), cw, 2), dict(g=2, pad=1)),
    ]
    if dt == torch.bfloat16:
        wp = nf.linear_pack_weight(w)
        calls += [(nf.linear_packed, (x, wp), dict(bias=b, residual=r, act=1)), (nf.linear_packed, (x[:, :100].contiguous(), wp), {}),
                  (nf.linear_packed, (x, wp[:, :128]), {})]
    return calls


def _outcome(call):
    fn, args, kw = call
    try:
        return fn(*args, **kw)
    except Exception as e:                                    # compared below
        return type(e), str(e)


# What the native path does with each of the calls above: T takes it, E raises the entry point's error, - hands it on, . is not asked.
OUTCOMES = "TTT-" "--.-" "-E--" "E." "TT---" "--" "TT" "-----" "T-" "TT" "E---" "--"


class Recorder:
    def __init__(self, native):
        self.native, self.seen = native, "."

    def __getattr__(self, name):
        def call(*args):
            self.seen = "E"
            out = getattr(self.native, name)(*args)
            self.seen = "-" if out is None else "T"
            return out
        return call


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_takes_the_ordinary_calls(nf, dt, monkeypatch):
    rec, seen = Recorder(nf._native), []
    monkeypatch.setattr(nf, "_native", rec)
    for c in _calls(nf, dt):
        rec.seen = "."
        _outcome(c)
        seen.append(rec.seen)
    assert "".join(seen) == OUTCOMES + ("TE-" if dt == torch.bfloat16 else "")


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_same_as_the_python_path(nf, dt, monkeypatch):
    calls = _calls(nf, dt)
    native = [_outcome(c) for c in calls]
    native = [n.clone() if isinstance(n, torch.Tensor) else n for n in native]
    monkeypatch.setattr(nf, "_native", None)
    for i, (c, a) in enumerate(zip(calls, native)):
        b = _outcome(c)
        if isinstance(b, torch.Tensor):
            assert isinstance(a, torch.Tensor) and a.dtype == b.dtype and a.shape == b.shape, (i, c[0].__name__, a)
            assert torch.equal(a, b) or torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num()), (i, c[0].__name__)
        else:
            assert a == b, (i, c[0].__name__, a, b)


def test_runs_on_the_current_stream_and_returns_the_output_given(nf):
    x, w, out = _t(2, 8, 64), _t(2, 64, 64), torch.zeros(2, 8, 64, device="cuda")
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    nf.linear(x, w, out=out)
    want = out.clone()
    out.zero_()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=s):                   # a launch on any other stream would fail the capture
        assert nf.linear(x, w, out=out) is out
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def test_other_python_threads_run_during_a_call(nf):
    """With the interpreter's own "does this thread hold the lock" (1 or 0, read as a status) in the place of every entry point."""
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    native, stream, x, g = nf._native, 0, _t(2, 16, 64), _t(2 * 64)
    w, qkv, kr, image, taps = _t(2, 64, 32), _t(2, 16, 3 * 64), _t(2, 16, 64), _t(1, 4, 5, 5), _t(4, 2, 3, 3)
    calls = [(native.linear, (x, w, None, None, 0)), (native.linear_packed, (x, w, None, None, 0)), (native.layernorm, (x, g, g, 2, None, 1e-5, 0)),
             (native.attention_packed, (qkv, 2, 8, 2, None, None)), (native.attention_relpos_packed, (qkv, kr, 2, 8, 2, None, None, None, None)),
             (native.conv2d, (image, taps, 2, 1, None, None, None, None, 1, 0, 1, 0))]
    native.bind(nf._check, *[address(ctypes.pythonapi.PyGILState_Check)] * 6)
    try:
        for fn, args in calls:
            made = fn(*args, None, stream)                    # raises if the lock was held
            assert isinstance(made, torch.Tensor), fn.__name__
            assert fn(*args, made, stream) is made
    finally:
        lib = nf.lib
        native.bind(nf._check, *(address(f) for f in (lib.netfuse_linear, lib.netfuse_linear_packed, lib.netfuse_layernorm, lib.netfuse_attention,
                                                      lib.netfuse_attention_relpos, lib.netfuse_conv2d)))

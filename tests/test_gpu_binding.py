"""The extension module behind the layer calls against the Python code that it stands in for: the same results for every call that it
takes, and None, so that the Python code does the call or refuses it, for everything else."""
import ctypes

import pytest
import torch

from paper_2307_09782_amd import zqfp

pytestmark = pytest.mark.gpu


class Nothing:
    """In the module's place: leaves every call to the Python code."""
    quantize = gemm = linear = staticmethod(lambda *a: None)


class Recorder:
    """In the module's place: the module, and whether it took each call."""

    def __init__(self, native):
        self.native, self.took = native, []

    def __getattr__(self, name):
        def call(*a):
            done = getattr(self.native, name)(*a)
            self.took.append(done is not None)
            return done
        return call


def _both(call, monkeypatch, taken=True):
    """The public call with the module, which has to do it itself (or, not `taken`, to leave it), and with the Python code alone."""
    zqfp.lib()
    native = Recorder(zqfp._native)
    with monkeypatch.context() as m:
        m.setattr(zqfp, "_native", native)
        got = call()
    assert native.took == [taken]
    with monkeypatch.context() as m:
        m.setattr(zqfp, "_native", Nothing)
        want = call()
    got, want = (x if isinstance(x, tuple) else (x,) for x in (got, want))
    assert len(got) == len(want)
    for a, b in zip(got, want):
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device and not a.requires_grad
        assert torch.equal(a, b)


def _state(M=20, K=512, N=272, r=8):
    gen = torch.Generator(device="cuda").manual_seed(1)
    f = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    return dict(X=f(M, K).bfloat16(), R=f(M, K).bfloat16(), g=f(K).bfloat16(), b=f(K).bfloat16(), U=(f(K, r) * .01).half(), V=(f(r, N) * .01).half(),
                W=(f(K, N) * .02).bfloat16(), N=N)


@pytest.mark.parametrize("M", [1, 20, 200])
@pytest.mark.parametrize("rank", [0, 8])
def test_same_results(M, rank, monkeypatch):
    s = _state(M)
    X, R, g, b, U = s["X"], s["R"], s["g"], s["b"], s["U"] if rank else None
    for call in (lambda: zqfp.quantize_act_fp8(X, U), lambda: zqfp.rmsnorm_quantize_act_fp8(X, g, 1e-5, U),
                 lambda: zqfp.layernorm_quantize_act_fp8(X, g, b, 1e-5, U), lambda: zqfp.relu_quantize_act_fp8(X, U), lambda: zqfp.swiglu_quantize_act_fp8(X, R, U),
                 lambda: zqfp.add_norm_quantize_act_fp8(X, R, g, 1e-5, None, U), lambda: zqfp.add_norm_quantize_act_fp8(X, R, g, 1e-5, b, U),
                 lambda: zqfp.relu_quantize_act_fp8(torch.cat([X, R], 1)[:, :X.shape[1]], U)):
        _both(call, monkeypatch)
    _both(lambda: zqfp.rmsnorm_quantize_act_fp8(X, g, 1, U), monkeypatch, taken=False)  # eps is no float
    T = zqfp.quantize_act_fp8(X, s["U"])[2] if rank else None
    V = s["V"] if rank else None
    Xq, sx = zqfp.quantize_act_fp8(X)
    p4, p8 = zqfp.pack_weight_fp4(s["W"], 128, 1), zqfp.pack_weight_fp8(s["W"], 128, 1)
    for out in (torch.float32, torch.bfloat16):
        for accum in (0, 1):
            _both(lambda: zqfp.w8a8_gemm(Xq, sx, p8, s["N"], 128, T, V, out_dtype=out, accum=accum), monkeypatch)
            _both(lambda: zqfp.w4a8_linear(X, p4, s["N"], 128, U, V, out_dtype=out, accum=accum), monkeypatch)
            if rank:
                _both(lambda: zqfp.w4a8_gemm_lorc(Xq, sx, p4, s["N"], 128, T, V, out_dtype=out, accum=accum), monkeypatch)
            else:
                _both(lambda: zqfp.w4a8_gemm(Xq, sx, p4, s["N"], 128, out_dtype=out, accum=accum), monkeypatch)


def test_what_was_refused_is_refused():
    s = _state()
    X, packed = s["X"], zqfp.pack_weight_fp4(s["W"], 128, 1)
    Xq, sx = zqfp.quantize_act_fp8(X)
    for call, error in ((lambda: zqfp.quantize_act_fp8(X.float()), TypeError), (lambda: zqfp.quantize_act_fp8(X.t()), TypeError),
                        (lambda: zqfp.quantize_act_fp8(X.cpu()), TypeError), (lambda: zqfp.quantize_act_fp8(X[:, :500].contiguous()), zqfp.ZqfpError),
                        (lambda: zqfp.rmsnorm_quantize_act_fp8(X, s["g"], 0.0), zqfp.ZqfpError), (lambda: zqfp.rmsnorm_quantize_act_fp8(X, s["g"][:-1], 1e-5), zqfp.ZqfpError),
                        (lambda: zqfp.swiglu_quantize_act_fp8(X, s["R"][:-1]), zqfp.ZqfpError), (lambda: zqfp.add_norm_quantize_act_fp8(X, s["R"][:-1], s["g"], 1e-5), zqfp.ZqfpError),
                        (lambda: zqfp.w4a8_gemm(Xq, sx, packed, 256, 128), zqfp.ZqfpError), (lambda: zqfp.w4a8_gemm(Xq, sx, packed, 272.0, 128), TypeError), (lambda: zqfp.w4a8_gemm(Xq, sx, packed, 272, 128.0), ctypes.ArgumentError),
                        (lambda: zqfp.w4a8_gemm(Xq, sx[:-1].contiguous(), packed, 272, 128), zqfp.ZqfpError), (lambda: zqfp.w4a8_gemm(Xq, sx, packed, 272, 128, accum=7), zqfp.ZqfpError),
                        (lambda: zqfp.w4a8_gemm(Xq, sx, packed, 272, 128, out_dtype=torch.float16), zqfp.ZqfpError),
                        (lambda: zqfp.w4a8_gemm_lorc(Xq, sx, packed, 272, 128, sx[:, None].contiguous(), s["V"]), zqfp.ZqfpError),
                        (lambda: zqfp.w4a8_gemm(None, sx, packed, 272, 128), TypeError), (lambda: zqfp.w4a8_linear(X, packed[:-256], 272, 128), zqfp.ZqfpError)):
        with pytest.raises(error):
            call()


@pytest.mark.parametrize("M, K, rank", [(16, 4096, 0), (17, 4096, 0), (16, 4224, 0), (16, 4096, 8), (1, 4096, 0)])
def test_linear_with_and_without_codes(M, K, rank, monkeypatch):
    """At the edges of the form that needs no room for codes: the library refuses the module's call if the module made none where it should."""
    s = _state(M, K, 272, rank or 8)
    p4 = zqfp.pack_weight_fp4(s["W"], 128, 1)
    _both(lambda: zqfp.w4a8_linear(s["X"], p4, s["N"], 128, *((s["U"], s["V"]) if rank else ())), monkeypatch)


def _captured_calls(s):
    """Each call that the module does itself, once: what it reads is s["X"], or the codes behind it."""
    native, X, N, f32 = zqfp._native, s["X"], s["N"], torch.float32
    return [native.quantize(0, X, None, None, None, None, s["U"]), native.quantize(1, X, s["R"], s["g"], None, 1e-5, None),
            (native.gemm(4, s["Xq"], s["sx"], s["p4"], N, 128, None, None, f32, 0),), (native.gemm(8, s["Xq"], s["sx"], s["p8"], N, 128, None, None, f32, 0),),
            (native.linear(X, s["p4"], N, 128, s["U"], s["V"], f32, 0),)]


def test_on_a_side_stream():
    """Captured on a side stream and replayed with other inputs: a launch on any other stream would be refused there, or would be missing from
    the replay."""
    s = _state(200)
    s["p4"], s["p8"] = zqfp.pack_weight_fp4(s["W"], 128, 1), zqfp.pack_weight_fp8(s["W"], 128, 1)
    s["Xq"], s["sx"] = zqfp.quantize_act_fp8(s["X"])
    assert all(x is not None for done in _captured_calls(s) for x in done)  # kernels loaded
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        got = _captured_calls(s)
    assert all(done is not None and done[0] is not None for done in got)
    for scale in (0.5, 3.0):
        other = (s["X"].flip(0) * scale).contiguous()
        codes, sx = zqfp.quantize_act_fp8(other)
        s["X"].copy_(other), s["Xq"].copy_(codes), s["sx"].copy_(sx)
        graph.replay()
        torch.cuda.synchronize()
        for done, want in zip(got, _captured_calls(s)):
            assert len(done) == len(want) and all(torch.equal(a, b) for a, b in zip(done, want))


def test_under_a_function_mode(monkeypatch):
    """A torch function mode: the Python code, whose allocations it may see."""
    s = _state(200)

    def call():
        with torch.device("cuda"):
            return zqfp.quantize_act_fp8(s["X"], s["U"])
    _both(call, monkeypatch, taken=False)


# in the order in which the module takes them; the others are host arithmetic
_QUERIES = ("packed_weight_bytes", "packed_weight_fp8_bytes", "gemm_workspace_bytes")


def test_the_interpreter_lock_is_not_held_inside_the_library():
    """In the place of every entry point that launches something stands the interpreter's own question whether this thread holds its
    lock: 0, which is the library's success, where it does not, and 1, an error that makes the module decline the call, where it does."""
    s = _state()
    X, R, g, b, U, V, N = (s[k] for k in ("X", "R", "g", "b", "U", "V", "N"))
    Xq, sx, T = zqfp.quantize_act_fp8(X, U)
    p4, p8 = zqfp.pack_weight_fp4(s["W"], 128, 1), zqfp.pack_weight_fp8(s["W"], 128, 1)
    native, address = zqfp._native, lambda f: ctypes.cast(f, ctypes.c_void_p).value
    real = {name: address(getattr(zqfp.lib(), "zqfp_" + name)) for name in zqfp._NATIVE_CALLS}
    assert ctypes.pythonapi.PyGILState_Check() == 1
    held = address(ctypes.pythonapi.PyGILState_Check)
    native.use(tuple(real[name] if name in _QUERIES else held for name in zqfp._NATIVE_CALLS))
    try:
        done = [native.quantize(0, X, None, None, None, None, U), native.quantize(1, X, None, g, None, 1e-5, U), native.quantize(2, X, None, g, b, 1e-5, U),
                native.quantize(1, X, R, g, None, 1e-5, None), native.quantize(2, X, R, g, b, 1e-5, None), native.quantize(3, X, None, None, None, None, U),
                native.quantize(4, X, R, None, None, None, U), native.gemm(4, Xq, sx, p4, N, 128, None, None, torch.float32, 0),
                native.gemm(4, Xq, sx, p4, N, 128, T, V, torch.float32, 0), native.gemm(8, Xq, sx, p8, N, 128, None, None, torch.float32, 0),
                native.linear(X, p4, N, 128, U, V, torch.float32, 0)]
    finally:
        native.use(tuple(real[name] for name in zqfp._NATIVE_CALLS))
    assert [i for i, d in enumerate(done) if d is None] == []


def test_an_allocation_that_fails_is_reported():
    """Both paths meet it; the module's lock is back when its exception leaves."""
    with pytest.raises(torch.OutOfMemoryError):
        zqfp.relu_quantize_act_fp8(torch.zeros(1, 128, dtype=torch.bfloat16, device="cuda").expand(1 << 40, 128))
    assert zqfp.relu_quantize_act_fp8(torch.zeros(1, 128, dtype=torch.bfloat16, device="cuda"))[0].shape == (1, 128)

"""The Python binding's argument checks and marshalling, on the CPU.

The library itself is replaced by a recorder (no pointer is dereferenced and
nothing is launched), and host tensors stand in for device tensors: every
wrapper of a layer call must accept tensors of exactly the sizes its dims
describe, pass one argument per parameter of the C declaration, and refuse
a tensor that is too small or of the wrong dtype before calling the library.
"""
import ctypes

import pytest
import torch

from paper_2502_02414_amd import binding as B


class _Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return B.PA_OK
        return call

    def pa_last_error(self):
        return b""


@pytest.fixture
def fake(monkeypatch):
    rec = _Recorder()
    monkeypatch.setattr(B, "load", lambda *a, **k: rec)
    monkeypatch.setattr(B, "_ptr", lambda t: None if t is None else 4096)
    monkeypatch.setattr(B, "_stream", lambda s=None: None)
    return rec


N, C, H, M = 100, 32, 2, 8


def _t(*shape, dt=torch.float32):
    return torch.zeros(*shape, dtype=dt)


@pytest.mark.parametrize("dt", [B.PA_F32, B.PA_BF16])
def test_layer_calls_accept_their_shapes(fake, dt):
    tdt = torch.bfloat16 if dt == B.PA_BF16 else torch.float32
    d = B.make_dims(N, C, H, M, 0.5, 0.01, 1e-5, dt)
    x, G, y = _t(N, C, dt=tdt), _t(N, M, dt=tdt), _t(N, C, dt=tdt)
    sp = B.make_slice_params(_t(C, M, dt=tdt), _t(M), _t(C, dt=tdt), 0.1, _t(1))
    ap = B.make_attn_params(_t(C, C), _t(C, C), _t(C, C), _t(C), _t(C), _t(C), _t(C, C), _t(C))
    mc, m = _t(M, C), _t(M)
    ws = _t(64, dt=torch.uint8)
    gr = B.make_slice_grads(_t(C, M), _t(M), _t(C), _t(1), _t(1))
    ag = B.make_attn_grads(*[_t(C, C) if i % 2 == 0 else _t(C) for i in range(8)])
    B.pa_slice_weights(d, x, G, sp, _t(N, M), _t(N), ws)
    B.pa_slice_aggregate(d, x, G, sp, mc, m, mc, ws)
    B.pa_token_attention(d, mc, ap, mc, ws)
    B.pa_deslice(d, x, G, sp, mc, y, ws)
    B.pa_deslice_backward(d, x, G, sp, y, mc, ws)
    B.pa_token_attention_backward(d, mc, ap, mc, mc, ag, ws)
    B.pa_slice_aggregate_backward(d, x, G, sp, mc, m, mc, mc, y, y, gr, ws)
    B.pa_slice_weights_backward(d, x, G, sp, _t(N, M), _t(N), y, gr, ws)
    B.pa_slice_aggregate_w(d, x, G, sp, mc, m, mc, _t(N, M, dt=tdt), ws)
    B.pa_deslice_w(d, _t(N, M, dt=tdt), mc, y, ws)
    B.pa_deslice_backward_w(d, _t(N, M, dt=tdt), y, mc, ws)
    B.pa_slice_aggregate_noalloc(d, x, G, sp, mc, m, mc)
    # one argument per parameter of each C declaration
    nargs = {name: len(args) for name, args in fake.calls}
    assert nargs == {"pa_slice_weights": 9, "pa_slice_aggregate": 10, "pa_token_attention": 7,
                     "pa_deslice": 9, "pa_deslice_backward": 9,
                     "pa_token_attention_backward": 9, "pa_slice_aggregate_backward": 14,
                     "pa_slice_weights_backward": 11, "pa_slice_aggregate_w": 11,
                     "pa_deslice_w": 7, "pa_deslice_backward_w": 7,
                     "pa_slice_aggregate_noalloc": 8}


def test_heads_calls_accept_their_shapes(fake):
    heads, D = 4, 32
    d = B.make_dims(N, D, 1, M, 0.5, 0.01, 1e-5, B.PA_F32)
    x, G = _t(heads, N, D), _t(heads, N, M)
    hp = B.make_heads_params(_t(heads, D, M), _t(heads, M), _t(heads, D), _t(heads))
    mc, m, ws = _t(heads, M, D), _t(heads, M), _t(64, dt=torch.uint8)
    gr = B.make_slice_grads(_t(heads, D, M), _t(heads, M), _t(heads, D), _t(heads), _t(heads))
    B.pa_heads_slice_aggregate(d, heads, x, G, hp, mc, m, mc, ws)
    B.pa_heads_deslice(d, heads, x, G, hp, mc, x, ws)
    B.pa_heads_deslice_backward(d, heads, x, G, hp, x, mc, ws)
    B.pa_heads_slice_aggregate_backward(d, heads, x, G, hp, mc, m, mc, mc, x, x, gr, ws)
    shared = B.make_heads_params(_t(D, M), _t(M), _t(D), _t(1), shared=True)
    B.pa_heads_slice_aggregate(d, heads, x, G, shared, mc, m, mc, ws)
    # a per-head parameter block too small for the heads
    small = B.make_heads_params(_t(heads - 1, D, M))
    with pytest.raises(ValueError, match="A"):
        B.pa_heads_slice_aggregate(d, heads, x, G, small, mc, m, mc, ws)
    with pytest.raises(ValueError, match="x"):
        B.pa_heads_deslice(d, heads, x[:2], G, hp, mc, x, ws)
    # per-head gradients are stacked head after head
    gr1 = B.make_slice_grads(_t(D, M))
    with pytest.raises(ValueError, match="dA"):
        B.pa_heads_slice_aggregate_backward(d, heads, x, G, hp, mc, m, mc, mc, x, x, gr1, ws)


def test_small_or_mistyped_tensors_refused_before_the_call(fake):
    d = B.make_dims(N, C, H, M, 0.5, 0.01, 1e-5, B.PA_BF16)
    bf = torch.bfloat16
    x, G, ws = _t(N, C, dt=bf), _t(N, M, dt=bf), _t(64, dt=torch.uint8)
    sp = B.make_slice_params(_t(C, M, dt=bf))
    mc, m = _t(M, C), _t(M)
    with pytest.raises(ValueError, match="x"):
        B.pa_slice_aggregate(d, x[:-1], G, sp, mc, m, mc, ws)
    with pytest.raises(ValueError, match="dtype"):
        B.pa_slice_aggregate(d, x.float(), G, sp, mc, m, mc, ws)
    with pytest.raises(ValueError, match="den"):
        B.pa_slice_aggregate(d, x, G, sp, mc, m[:-1], mc, ws)
    with pytest.raises(ValueError, match="A"):
        B.pa_slice_aggregate(d, x, G, B.make_slice_params(_t(C, M)), mc, m, mc, ws)
    with pytest.raises(ValueError, match="Wq"):
        B.pa_token_attention(d, mc, B.make_attn_params(_t(C, C - 1), _t(C, C), _t(C, C)), mc, ws)
    with pytest.raises(ValueError, match="dA"):
        B.pa_slice_aggregate_backward(d, x, G, sp, mc, m, mc, None, None, x,
                                      B.make_slice_grads(dA=_t(C * M - 1)), ws)
    assert fake.calls == []


# every tensor of every parameter and gradient struct: (helper, its keyword,
# elements at the test's dims, in the storage dtype?), for one layer
_CM, _CC = C * M, C * C
STRUCT_FIELDS = (
    [("make_slice_params", k, n, st) for k, n, st in
     (("A", _CM, True), ("b", M, False), ("a", C, True), ("b_t_dev", 1, False))] +
    [("make_slice_grads", k, n, False) for k, n in
     (("dA", _CM), ("db", M), ("da", C), ("db_t", 1), ("dtau0", 1))] +
    [("make_attn_params", k, _CC if k[0] == "W" else C, False) for k in
     ("Wq", "Wk", "Wv", "Wo", "bq", "bk", "bv", "bo")] +
    [("make_attn_grads", k, _CC if k[1] == "W" else C, False) for k in
     ("dWq", "dWk", "dWv", "dWo", "dbq", "dbk", "dbv", "dbo")])
HEADS = 3
HEAD_FIELDS = [("A", _CM, True), ("b", M, False), ("a", C, True), ("b_t", 1, False)]


def _struct(maker, key, t):
    kw = {key: t}
    if maker == "make_attn_params":  # (the three weights are positional)
        kw = {**{w: _t(C, C) for w in ("Wq", "Wk", "Wv")}, **kw}
    if maker in ("make_slice_params", "make_heads_params") and key != "A":
        kw["A"] = _t(HEADS * _CM, dt=torch.bfloat16)
    return getattr(B, maker)(**kw)


def _refuses(st, key, dims, *args):
    with pytest.raises(ValueError, match=rf"^{key}: "):
        B._check_struct(st, dims, *args)


@pytest.mark.parametrize("maker,key,n,storage", STRUCT_FIELDS,
                         ids=[f"{f[0]}-{f[1]}" for f in STRUCT_FIELDS])
def test_every_struct_field_is_checked(fake, maker, key, n, storage):
    """One element short or of another type: refused by name; the exact size
    and larger: taken.  Gradients of a per-head call: stacked head on head."""
    dims = B.make_dims(N, C, H, M, 0.5, 0.01, 1e-5, B.PA_BF16)
    dt, other = (torch.bfloat16, torch.float32) if storage else (torch.float32, torch.bfloat16)
    for heads in (1, HEADS) if maker == "make_slice_grads" else (1,):
        m, args = heads * n, (dims, heads, heads > 1)
        for size in (m, m + 1):
            B._check_struct(_struct(maker, key, _t(size, dt=dt)), *args)
        _refuses(_struct(maker, key, _t(m - 1, dt=dt)), key, *args)
        _refuses(_struct(maker, key, _t(m, dt=other)), key, *args)
        with pytest.raises(ValueError, match="unsupported dtype"):
            B._check_struct(_struct(maker, key, _t(m, dt=torch.float16)), *args)


@pytest.mark.parametrize("key,n,storage", HEAD_FIELDS, ids=[f[0] for f in HEAD_FIELDS])
@pytest.mark.parametrize("shared", [False, True])
def test_every_head_parameter_is_checked(fake, key, n, storage, shared):
    """A block per head, or one for all."""
    dims = B.make_dims(N, C, 1, M, 0.5, 0.01, 1e-5, B.PA_BF16)
    dt, other = (torch.bfloat16, torch.float32) if storage else (torch.float32, torch.bfloat16)
    m = n if shared else HEADS * n

    def make(t):
        kw = {"A": _t(HEADS * _CM, dt=torch.bfloat16), key: t}
        return B.make_heads_params(**kw, shared=shared)
    for size in (m, m + 1):
        B._check_struct(make(_t(size, dt=dt)), dims, HEADS)
    _refuses(make(_t(m - 1, dt=dt)), key, dims, HEADS)
    _refuses(make(_t(m, dt=other)), key, dims, HEADS)


def test_argument_checks(fake):
    assert B._arg(None, 10, B.PA_F32, "x") is None
    assert B._arg(_t(10), 10, B.PA_F32, "x") == 4096
    assert B._arg(_t(10, dt=torch.float16), 10, None, "x") == 4096  # (type not asked for)
    with pytest.raises(ValueError, match="^x: 9 elements, the call needs 10"):
        B._arg(_t(9), 10, B.PA_F32, "x")
    with pytest.raises(ValueError, match="^x: dtype torch.float32 does not match the call's bf16"):
        B._arg(_t(10), 10, B.PA_BF16, "x")
    with pytest.raises(ValueError, match="unsupported dtype torch.float16"):
        B._arg(_t(10, dt=torch.float16), 10, B.PA_F32, "x")


def test_host_and_strided_tensors_refused():
    with pytest.raises(ValueError, match="GPU"):
        B._arg(_t(10), 10, B.PA_F32, "x")

    class Strided:
        is_cuda, dtype = True, torch.float32

        def numel(self):
            return 10

        def is_contiguous(self):
            return False
    with pytest.raises(ValueError, match="contiguous"):
        B._arg(Strided(), 10, B.PA_F32, "x")


def test_no_stream_without_a_gpu(monkeypatch):
    """torch's own error, every time: nothing is kept from a first call that
    found no GPU."""
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda *a: (_ for _ in ()).throw(RuntimeError("no GPU")))
    for _ in range(2):
        with pytest.raises(RuntimeError, match="no GPU"):
            B._stream()
    assert B._raw_stream is None


@pytest.mark.gpu
def test_calls_go_to_the_current_stream():
    """Without a stream, torch's current one at the time of the call, of the
    calling thread; with one, that one."""
    import threading
    say = lambda: torch.cuda.current_stream().cuda_stream
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    seen = []

    def look():
        seen.append((B._stream(), say()))
    for _ in range(2):
        look()
        with torch.cuda.stream(a):
            look()
            with torch.cuda.stream(b):
                look()
                t = threading.Thread(target=look)
                t.start()
                t.join()
            look()
            assert B._stream(b) == b.cuda_stream
        look()
    assert all(got == want for got, want in seen), seen
    assert len({got for got, _ in seen}) == 3


def test_wrapper_calls_match_argtypes():
    """Every load().pa_*(...) call in the binding passes exactly as many
    arguments as the symbol's ctypes argtypes declare (read from the source,
    no GPU needed)."""
    import ast
    import inspect
    from paper_2502_02414_amd import binding as B
    lib = B.load()
    tree = ast.parse(inspect.getsource(B))
    calls = 0
    for node in ast.walk(tree):
        if not (isinstance(node, ast.Call) and isinstance(node.func, ast.Attribute)):
            continue
        f = node.func
        if isinstance(f.value, ast.Call) and getattr(f.value.func, "id", "") == "load" \
                and f.attr.startswith("pa_"):
            calls += 1
            assert len(node.args) == len(getattr(lib, f.attr).argtypes or []), f.attr
    assert calls > 30
    # pa_gemm and pa_gemm_prepare are called through a chosen function
    assert lib.pa_gemm.argtypes == lib.pa_gemm_prepare.argtypes
    src = inspect.getsource(B.pa_gemm)
    call = next(n for n in ast.walk(ast.parse(src.strip()))
                if isinstance(n, ast.Call) and getattr(n.func, "id", "") == "fn")
    assert len(call.args) == len(lib.pa_gemm.argtypes)

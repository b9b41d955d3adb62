"""The C++ marshalling of the plain calls: it takes only what it can handle, and gives what the ctypes calls give."""
import ctypes as C
import os
import sys
import threading
import types

import pytest
import torch

from paper_2407_09105_amd import binding, workloads as wl
from tests.gpu_util import DEV, assert_close, run_gpu, run_oracle, to_dev


def _lib():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("library is not built")
    binding.lib()
    assert binding._native is not None, "the library is built, its C++ marshalling is not"
    return binding._native


@pytest.fixture(params=["absent", "another torch", "older"])
def without_native(request, monkeypatch):
    """A binding that finds no C++ marshalling, or one built for another torch, or one that does not say for which."""
    _lib()
    package = sys.modules[binding.__package__]
    other = types.ModuleType("_va_native")
    if request.param == "another torch":
        other.torch_version = torch.__version__ + ".1"
    monkeypatch.delattr(package, "_va_native", raising=False)
    monkeypatch.setitem(sys.modules, binding.__package__ + "._va_native", None)   # an import of it raises
    if request.param != "absent":
        monkeypatch.setattr(package, "_va_native", other, raising=False)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)


def test_library_serves_without_cpp_marshalling(without_native, caplog):
    assert binding.lib().va_plan_bytes(1, 16) > 0
    assert binding._native is None and "ctypes" in caplog.text
    with pytest.raises(ValueError, match="GPU"):
        binding.pack_to_cu_seqlens(torch.zeros(1, 8, dtype=torch.int64))


@pytest.mark.gpu
def test_same_results_without_cpp_marshalling(without_native):
    w = wl.make_custom([[129, 40], [100, 69]], 4, 2, 80, "bf16", seed=5)
    got = run_gpu(w)
    assert binding._native is None
    assert_close(got, run_oracle(w), "bf16", bf16_stored=("dQ", "dK", "dV"))


def test_leaves_what_is_not_on_the_gpu():
    native = _lib()
    c = binding.VaSegments()
    q, k = torch.zeros(8, 2, 16), torch.zeros(8, 1, 16)
    addr = C.addressof(c)
    assert native.pack(torch.zeros(1, 8, dtype=torch.int64), addr, 0) is None
    assert native.fwd(q, k, k, addr, 1, 8, 0.0, 0) is None
    assert native.bwd(q, q, k, k, q, torch.zeros(2, 8), addr, 1, 8, 0.0, False, 0) is None
    assert native.fwd(None, "k", 3, addr, 1, 8, 0.0, 0) is None
    assert c.cu_seqlens is None
    with pytest.raises(ValueError, match="GPU"):
        binding.pack_to_cu_seqlens(torch.zeros(1, 8, dtype=torch.int64))
    with pytest.raises(TypeError):
        native.connect(1, 2)


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("stages", [None, binding.STAGE_D, binding.STAGE_DQ, binding.STAGE_DKDV, "noalloc"])
def test_short_dO_and_O_are_refused(stages, monkeypatch):
    # The kernels read as many elements of dO and O as Q has.  The tensors have no memory behind them: a call that passes the
    # binding's checks ends at the library's, which refuses null pointers.
    from torch._subclasses.fake_tensor import FakeTensorMode
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("library is not built")
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    seg = binding.Segments._of(2, 16, torch.empty(0), binding.VaSegments())
    with FakeTensorMode():
        of = lambda *shape: torch.empty(shape, device="cuda", dtype=torch.bfloat16)  # noqa: E731
        q, k, lse = of(32, 4, 64), of(32, 2, 64), torch.empty((4, 32), device="cuda")

        def bwd(do, o):
            if stages == "noalloc":
                return binding.varlen_attn_bwd_noalloc(do, q, k, k, o, lse, seg, q, k, k)
            return binding.varlen_attn_bwd(do, q, k, k, o, lse, seg, stages=stages)

        for short in (of(31, 4, 64), of(32, 2, 64), of(0, 4, 64)):
            with pytest.raises(ValueError, match="must hold"):
                bwd(short, q)
            if stages != binding.STAGE_DKDV:   # it reads no O
                with pytest.raises(ValueError, match="must hold"):
                    bwd(q, short)
        for enough in (q, of(32, 256), of(33, 4, 64)):
            with pytest.raises(binding.VarlenAttnError, match="null pointer"):
                bwd(enough, enough)


@pytest.fixture
def taken(monkeypatch):
    """What the C++ functions returned to the binding, in order: "tuple", "NoneType" or "int" after the function's name."""
    native, calls = _lib(), []

    def spy(name):
        def call(*args):
            got = getattr(native, name)(*args)
            calls.append((name, type(got).__name__))
            return got
        return call

    monkeypatch.setattr(binding, "_native", types.SimpleNamespace(**{name: spy(name) for name in ("pack", "fwd", "bwd")}))
    return calls


TAKEN = [(name, "tuple") for name in ("pack", "fwd", "bwd")]


def _inputs(dtype="bf16", lengths=((300, 45, 1, 1, 200, 93),), hq=4, hkv=2, d=128, seed=41):
    w = wl.make_custom([list(row) for row in lengths], hq, hkv, d, dtype, seed=seed)
    return (torch.from_numpy(w.position_ids).to(DEV), *(to_dev(a, dtype) for a in (w.do, w.q, w.k, w.v)))


def _pass(pos, do, q, k, v):
    seg = binding.pack_to_cu_seqlens(pos)
    o, lse = binding.varlen_attn_fwd(q, k, v, seg)
    return [seg.seg_start, seg.q_tile_order, o, lse, *binding.varlen_attn_bwd(do, q, k, v, o, lse, seg)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,grads,d,lengths", [
    ("f32", None, 16, [[6, 1, 5, 4]]), ("bf16", None, 80, [[129, 40], [100, 69]]), ("bf16", torch.float32, 64, [[300]]),
    ("f16", torch.float16, 128, [[1100]]), ("f32", torch.bfloat16, 32, [[33, 7]])])
def test_same_as_ctypes(dtype, grads, d, lengths, taken):
    w = wl.make_custom(lengths, 4, 2, d, dtype, seed=5)
    q, k, v, do = (to_dev(a, dtype) for a in (w.q, w.k, w.v, w.do))
    for ids in (torch.int64, torch.int32):
        pos = torch.from_numpy(w.position_ids).to(DEV).to(ids)
        seg = binding.pack_to_cu_seqlens(pos)
        given = binding.pack_to_cu_seqlens(pos, binding.Segments(*pos.shape, pos.device))
        assert (seg.rows, seg.tokens_per_row, seg.n_tokens) == (given.rows, given.tokens_per_row, given.n_tokens)
        a, b = seg.host(), given.host()
        assert all((x == y).all() if hasattr(x, "all") else x == y for x, y in zip(a.values(), b.values()))
    q.requires_grad_()
    o, lse = binding.varlen_attn_fwd(q, k, v, seg, 0.2)
    assert not o.requires_grad and not lse.requires_grad
    o2, lse2 = binding.varlen_attn_fwd(q, k, v, given, 0.2, out=torch.empty_like(o), lse=torch.empty_like(lse))
    assert o.dtype == q.dtype and torch.equal(o, o2) and torch.equal(lse, lse2)
    got = binding.varlen_attn_bwd(do, q, k, v, o, lse, seg, 0.2, grad_dtype=grads)
    ref = binding.varlen_attn_bwd(do, q, k, v, o, lse, given, 0.2, grad_dtype=grads, workspace=binding.bwd_workspace(q, k))
    for x, y, like in zip(got, ref, (q, k, v)):
        assert x.shape == like.shape and x.dtype == (grads or q.dtype) and torch.equal(x, y)
    # one call of each went to C++ (two of pack), but gradients in a third type are left to ctypes
    left = grads is torch.bfloat16
    assert taken == [("pack", "tuple"), *TAKEN[:2]] + ([] if left else TAKEN[2:])


@pytest.mark.gpu
def test_on_another_stream(taken):
    args = _inputs()
    ref = _pass(*args)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        # the inputs arrive on this stream only: a launch on another one would read the old values
        late = [torch.zeros_like(x) for x in args]
        torch.cuda._sleep(20_000_000)
        for x, y in zip(late, args):
            x.copy_(y)
        got = _pass(*late)
    side.synchronize()
    assert taken == 2 * TAKEN
    for x, y in zip(got, ref):
        assert torch.equal(x, y)


@pytest.mark.gpu
def test_under_capture(taken):
    args = _inputs(lengths=((513, 31, 480),), hq=5, hkv=1, seed=42)
    pos, do, q, k, v = args
    _pass(*args)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = _pass(*args)   # outputs and workspace come from the graph's pool
    assert taken == 2 * TAKEN
    for rep in range(3):
        if rep:
            q.mul_(-1.0)
            do.mul_(0.5)
        eager = _pass(*args)
        for x in outs[2:]:
            x.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(outs, eager):
            assert torch.equal(x, y), rep


@pytest.mark.gpu
def test_from_two_threads(taken):
    work = [_inputs(), _inputs("f16", ((700, 60), (1, 759)), 8, 2, 64, seed=43)]
    ref = [_pass(*args) for args in work]
    torch.cuda.synchronize()
    wrong = [None, None]

    def run(i):
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            for _ in range(50):
                got = _pass(*work[i])
                side.synchronize()
                wrong[i] = (wrong[i] or 0) + sum(not torch.equal(x, y) for x, y in zip(got, ref[i]))

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert wrong == [0, 0]
    assert len(taken) == 3 * 102 and {kind for _, kind in taken} == {"tuple"}


@pytest.mark.gpu
def test_modes_that_ask_for_the_python_calls_see_them(taken):
    from torch.overrides import TorchFunctionMode

    class Record(TorchFunctionMode):
        def __init__(self):
            super().__init__()
            self.seen = []

        def __torch_function__(self, func, types_, args=(), kwargs=None):
            self.seen.append(func)
            return func(*args, **(kwargs or {}))

    args = _inputs()
    ref = _pass(*args)
    with Record() as mode:
        got = _pass(*args)
    assert mode.seen.count(torch.empty) >= 5 and torch.empty_like in mode.seen   # plan, LSE, gradients; O
    assert taken == TAKEN + [(name, "NoneType") for name in ("pack", "fwd", "bwd")]
    for x, y in zip(got, ref):
        assert torch.equal(x, y)


@pytest.mark.gpu
def test_what_is_left_to_python_and_what_the_library_refuses():
    native = _lib()
    pos, do, q, k, v = _inputs(lengths=((20, 12),), d=64)
    seg = binding.pack_to_cu_seqlens(pos)
    o, lse = binding.varlen_attn_fwd(q, k, v, seg)
    at, s = (C.addressof(seg.c), 1, 32, 0.0), binding._stream()
    class Sub(torch.Tensor):
        pass
    fwd = lambda *qkv: native.fwd(*qkv, *at, s)  # noqa: E731
    bwd = lambda *t: native.bwd(*t, *at, False, s)  # noqa: E731
    c = binding.VaSegments()   # written by pack: it has to outlive the calls
    pack = lambda x: native.pack(x, C.addressof(c), s)  # noqa: E731
    assert [type(pack(x)) for x in (pos, pos.to(torch.int32))] == [tuple, tuple]
    for x in (pos[0], pos.float(), pos[:, ::2], pos.as_subclass(Sub), pos.cpu()):
        assert pack(x) is None
    assert type(fwd(q, k, v)) is tuple and type(bwd(do, q, k, v, o, lse)) is tuple
    for qkv in ((q, k, v.float()), (q.transpose(0, 1), k, v), (q[:16], k[:16], v[:16]), (q.double(), k.double(), v.double()),
                (q.as_subclass(Sub), k, v), (q, k, v[:, :1].contiguous())):
        assert fwd(*qkv) is None
    for t in ((do.float(), q, k, v, o, lse), (do[:16], q, k, v, o, lse), (do, q, k, v, o[:, :2].contiguous(), lse),
              (do, q, k, v, o, lse[:1]), (do, q, k, v, o, lse.double())):
        assert bwd(*t) is None
    assert fwd(q[:, :3].contiguous(), k, v) == 2   # 3 query heads on 2 KV heads: VA_ERR_SHAPE


@pytest.mark.gpu
def test_the_interpreter_is_free_during_the_calls():
    # Allocations and launches can block: other Python threads run meanwhile, as they do around a ctypes call.  The three
    # calls reach an interpreter function that says whether the calling thread holds the interpreter lock (1: held, which
    # arrives as a status; 0 is taken for success) in place of the library's, so nothing is launched.
    native, L = _lib(), binding.lib()
    w = wl.make_custom([[20, 12]], 4, 2, 64, "bf16", seed=6)
    q, k, v, do = (to_dev(a, "bf16") for a in (w.q, w.k, w.v, w.do))
    pos = torch.from_numpy(w.position_ids).to(DEV)
    o, lse = torch.empty_like(q), torch.empty((4, 32), device=DEV)
    c = binding.VaSegments()
    plan_bytes, segments_bind, _, workspace_bytes, _, _ = binding.native_addresses(L)
    held = C.cast(C.pythonapi.PyGILState_Check, C.c_void_p).value
    native.connect(plan_bytes, segments_bind, held, workspace_bytes, held, held)
    try:
        assert type(native.pack(pos, C.addressof(c), 0)) is tuple
        assert type(native.fwd(q, k, v, C.addressof(c), 1, 32, 0.0, 0)) is tuple
        assert type(native.bwd(do, q, k, v, o, lse, C.addressof(c), 1, 32, 0.0, False, 0)) is tuple
    finally:
        native.connect(*binding.native_addresses(L))


@pytest.mark.gpu
def test_refuses_the_same_calls():
    _lib()
    w = wl.make_custom([[20, 12]], 4, 2, 64, "bf16", seed=6)
    q, k, v, do = (to_dev(a, "bf16") for a in (w.q, w.k, w.v, w.do))
    pos = torch.from_numpy(w.position_ids).to(DEV)
    seg = binding.pack_to_cu_seqlens(pos)
    o, lse = binding.varlen_attn_fwd(q, k, v, seg)
    fwd = binding.varlen_attn_fwd
    bwd = binding.varlen_attn_bwd
    for call, error in [
            (lambda: binding.pack_to_cu_seqlens(pos[0]), ValueError), (lambda: binding.pack_to_cu_seqlens(pos.float()), TypeError),
            (lambda: binding.pack_to_cu_seqlens(pos[:, ::2]), ValueError),
            (lambda: fwd(q, k, v.float(), seg), TypeError), (lambda: fwd(q.transpose(0, 1), k, v, seg), ValueError),
            (lambda: fwd(q[:16], k[:16], v[:16], seg), ValueError), (lambda: fwd(q, k.cpu(), v, seg), ValueError),
            (lambda: fwd(q.double(), k.double(), v.double(), seg), TypeError),
            (lambda: fwd(q[:, :3].contiguous(), k, v, seg), binding.VarlenAttnError),   # 3 query heads on 2 KV heads
            (lambda: bwd(do[:16], q, k, v, o, lse, seg), ValueError), (lambda: bwd(do, q, k, v, o[:, :2].contiguous(), lse, seg), ValueError),
            (lambda: bwd(do.float(), q, k, v, o, lse, seg), TypeError), (lambda: bwd(do, q, k, v, o, lse[:1], seg), ValueError),
            (lambda: bwd(do, q, k, v, o, lse, seg, grad_dtype=torch.float16), binding.VarlenAttnError),
            (lambda: bwd(do, q, k, v, o, lse, seg, grad_dtype=torch.float64), TypeError)]:
        with pytest.raises(error):
            call()

"""The native binding answers as the general path through ctypes does: the same refusals (no GPU needed), the same results."""
import os
import shutil
import subprocess
import sys
import types

import pytest
import torch

from paper_2301_10936_amd import pit

NAMES = ["build_index", "relu_channel_major_index", "sread_gemm", "select_and_run_gemm", "moe_dispatch_gemm", "sparse_attn"]


class Sub(torch.Tensor):
    pass


def _outcome(call):
    try:
        r = call()
        return "ok", r if isinstance(r, tuple) else type(r).__name__
    except Exception as e:       # noqa: BLE001 -- whatever it is, both paths raise the same
        return type(e).__name__, str(e)


def _both(monkeypatch, call):
    native = _outcome(call)
    with monkeypatch.context() as m:
        m.setattr(pit, "_native", types.SimpleNamespace(**{n: lambda *a: None for n in NAMES}))
        general = _outcome(call)
    return native, general


def _calls(dev="cpu"):
    """Calls that end at a check on the host (N % 128, a micro-tile that does not divide, ...), and malformed ones."""
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(s, dtype=dtype, device=dev)
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)
    ix = pit.PitIndex(i32(3), i32(1024), None, 2, 1024)
    X, W, C, ws = z(512, 256), z(512, 100), z(256, 128, dtype=torch.float32), z(4096, dtype=torch.uint8)
    sub, param = X.as_subclass(Sub), torch.nn.Parameter(X, requires_grad=True)
    for src in (X, sub, param, X.t(), X[0], X.double(), X[:1], X[:0], X[:, :0], z(4, 4, 4), None, 3, X.to(torch.int64)):
        for args in ((3, 128, 0), (1, 100, 0), (1, 128, 7), (0, 128, 0), (1, 2 ** 40, 0), (1.0, 128, 0), (True, 128, 5)):
            yield lambda s=src, a=args: pit.pit_build_index(s, *a, out=ix, ws=ws)
            yield lambda s=src, a=args: pit.pit_build_index(s, *a, out=pit.PitIndex(i32(3), None, None, 2, 1024), ws=ws)
        yield lambda s=src: pit.pit_relu_channel_major_index(s, out_xt=z(256, 512), out=ix, ws=ws)
        yield lambda s=src: pit.pit_relu_channel_major_index(X, out_xt=s, out=ix, ws=ws)
        yield lambda s=src: pit.pit_sread_gemm(1, s, W, ix, 128, 256, 100, 512, out=C)
        yield lambda s=src: pit.pit_sread_gemm(1, X, s, ix, 100, 256, 128, 512, out=C)
        yield lambda s=src: pit.pit_sread_gemm(1, X, W, ix, 128, 256, 100, 512, out=s)
        yield lambda s=src: pit.pit_sread_gemm(9, X, s, None, 100, 256, 128, 512, out=C, zero_uncovered=False)
        yield lambda s=src: pit.pit_moe_dispatch_gemm(s, i32(512), None, z(2, 256, 100), z(2, 100, 256), out=C, ws=ws)
        yield lambda s=src: pit.pit_moe_dispatch_gemm(X, i32(512), s, z(2, 256, 100), z(2, 100, 256), out=s, ws=ws)
        yield lambda s=src: pit.pit_sparse_attn(s, s, s, z(256, 256, dtype=torch.uint8), 1.0, out=C, ws=ws)
        yield lambda s=src: pit.pit_sparse_attn(z(2, 256, 48), z(2, 256, 48), z(2, 256, 48), s, 1, out=C, ws=ws)
        for cand in ([{"mt_rows": 1, "mt_cols": 100, "tile_cost": 1.0}], [{"mt_rows": 1, "mt_cols": 128, "tile_cost": 1, "dense": True}],
                     [{"mt_rows": 1, "mt_cols": 128}], [], None):
            yield lambda s=src, c=cand: pit.pit_select_and_run_gemm(c, [[1]], [[2]], s, W, 256, 100, 512, out=C, ws=ws)
            yield lambda s=src, c=cand: pit.pit_select_and_run_gemm(c, [[-1]], [[2]], X, s, 256, 128, 512, out=C, ws=ws)
            yield lambda s=src, c=cand: pit.pit_select_and_run_gemm(c, [[1, 2]], [], X, W, 256, 128, 512, out=s, ws=ws)


@pytest.mark.skipif(torch.cuda.is_available(), reason="host memory, and some of the calls get as far as a launch")
def test_the_same_refusals(monkeypatch):
    monkeypatch.setattr(pit, "_stream", lambda: 0)
    seen, n = set(), 0
    for call in _calls():
        native, general = _both(monkeypatch, call)
        assert native == general
        seen.add(native[0])
        n += 1
    assert n > 500 and {"PitError", "AssertionError", "AttributeError", "KeyError"} <= seen


@pytest.mark.parametrize("native,says", [(None, "cannot import name"), (b"not a library", "file too short")])
def test_the_package_loads_without_the_native_module(tmp_path, native, says):
    """The ctypes path needs the library alone: without the module, or with one that does not load, calls take that path and a
    warning says what the loader said."""
    here = os.path.dirname(os.path.abspath(pit.__file__))
    to = tmp_path / "paper_2301_10936_amd"
    to.mkdir()
    for name in ("__init__.py", "pit.py", "libpit_hip.so"):
        shutil.copy(os.path.join(here, name), to / name)
    if native is not None:
        (to / "_pit_native.so").write_bytes(native)
    code = """if True:
        import warnings
        with warnings.catch_warnings(record=True) as seen:
            warnings.simplefilter("always")
            from paper_2301_10936_amd import pit
        import torch
        print(pit.__file__, [str(w.message) for w in seen if "native binding" in str(w.message)])
        print(pit.pit_select_kernel([{"mt_rows": 1, "mt_cols": 128, "tile_cost": 1.0}], [[1]], [[2]]))
        pit._stream = lambda: 0
        ix = pit.PitIndex(torch.zeros(3, dtype=torch.int32), torch.zeros(8, dtype=torch.int32), None, 2, 8)
        try:
            pit.pit_build_index(torch.zeros((4, 256), dtype=torch.bfloat16), 1, 100, 0, out=ix, ws=torch.zeros(64, dtype=torch.uint8))
        except pit.PitError as e:
            print(e)
    """
    p = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path)}, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
    assert str(tmp_path) in p.stdout and "(0, [1.0])" in p.stdout and "pit_build_index: PIT_ESHAPE" in p.stdout
    assert says in p.stdout, p.stdout


@pytest.mark.gpu
def test_the_same_results(monkeypatch):
    """Every call of the binding, both paths, the same bits; a Parameter and a subclass among the operands."""
    g = torch.Generator(device="cuda").manual_seed(1)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    dev = torch.device("cuda:0")
    X, W, H = r(512, 256) * (r(512, 256) > 1), r(512, 128), r(256, 512)
    ws = torch.empty(1 << 24, dtype=torch.uint8, device=dev)
    eid = torch.randint(0, 4, (96,), generator=g, device="cuda").to(torch.int32)
    Xm, W1, W2, gate, status = r(96, 128), r(4, 128, 256), r(4, 256, 128), torch.rand(96, generator=g, device="cuda"), torch.zeros(1, dtype=torch.int32, device=dev)
    Q = r(2, 256, 64)
    mask = (torch.rand((256, 256), generator=g, device="cuda") < 0.2).to(torch.uint8)
    cands = [{"mt_rows": 1, "mt_cols": 128, "tile_cost": 1.0}, {"mt_rows": 1, "mt_cols": 64, "tile_cost": 0.1, "fixed_cost": 2.0}]

    def everything(wrap):
        ix, ix2 = (pit.PitIndex.empty(2, 1024) for _ in range(2))
        ix.idx.zero_(), ix2.idx.zero_()
        Xt, C, C2, Y, O = torch.zeros((512, 256), dtype=torch.bfloat16, device=dev), *(torch.zeros(s, device=dev) for s in ((256, 128), (256, 128), (96, 128), (2, 256, 64)))
        pit.pit_build_index(wrap(X), 1, 128, 0, out=ix, ws=ws)
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_K, wrap(X), W, ix, 128, 256, 128, 512, out=C)
        pit.pit_relu_channel_major_index(wrap(H), out_xt=Xt, out=ix2, ws=ws)
        _, best = pit.pit_select_and_run_gemm(cands, [[900, 1500]], [[1024, 2048]], wrap(X), W, 256, 128, 512, out=C2, ws=ws)
        pit.pit_moe_dispatch_gemm(wrap(Xm), eid, gate, W1, W2, out=Y, status=status, ws=ws)
        pit.pit_sparse_attn(wrap(Q), Q, Q, mask, 0.125, out=O, ws=ws)
        torch.cuda.synchronize()
        return [t.clone() for t in (ix.seg_ptr, ix.idx, C, ix2.seg_ptr, ix2.idx, Xt, C2, Y, O, status)] + [best]

    native = everything(lambda t: t)
    assert native[-1] == 1 and bool(native[2].any())
    for got in (everything(lambda t: torch.nn.Parameter(t)), everything(lambda t: t.as_subclass(Sub))):
        assert all(torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b for a, b in zip(native, got))
    monkeypatch.setattr(pit, "_native", types.SimpleNamespace(**{n: lambda *a: None for n in NAMES}))
    got = everything(lambda t: t)
    assert all(torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b for a, b in zip(native, got))


class Recorder:
    """_native with what each call of it answered"""
    def __init__(self, native):
        self.answers = []
        for n in NAMES:
            setattr(self, n, lambda *a, f=getattr(native, n): self.answers.append(f(*a)) or self.answers[-1])


def _refused(wrap, dev="cpu"):
    """One call of each function that ends at the library's own checks."""
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(s, dtype=dtype, device=dev)
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)
    ix = pit.PitIndex(i32(3), i32(1024), None, 2, 1024)
    X, W, C, ws = wrap(z(512, 256)), z(512, 100), z(256, 128, dtype=torch.float32), z(4096, dtype=torch.uint8)
    yield lambda: pit.pit_build_index(X, 1, 100, 0, out=ix, ws=ws)
    yield lambda: pit.pit_relu_channel_major_index(wrap(z(512, 100)), out_xt=z(100, 512), out=ix, ws=ws)
    yield lambda: pit.pit_sread_gemm(1, X, W, ix, 128, 256, 100, 512, out=C)
    yield lambda: pit.pit_select_and_run_gemm([{"mt_rows": 1, "mt_cols": 100, "tile_cost": 1.0}], [[1]], [[2]], X, W, 256, 100, 512, out=C, ws=ws)
    yield lambda: pit.pit_moe_dispatch_gemm(X, i32(512), None, z(2, 256, 100), z(2, 100, 256), out=C, ws=ws)
    yield lambda: pit.pit_sparse_attn(wrap(z(2, 256, 48)), z(2, 256, 48), z(2, 256, 48), z(256, 256, dtype=torch.uint8), 1.0, out=C, ws=ws)


def test_ordinary_calls_are_answered_natively(monkeypatch):
    """An ordinary call gets the library's status from the native side; a subclass of Tensor gets None there and the same refusal from the
    general path.  (Without a native binding every call would pass the tests of equal results.)"""
    monkeypatch.setattr(pit, "_stream", lambda: 0)
    for wrap, native in ((lambda t: t, True), (torch.nn.Parameter, True), (lambda t: t.as_subclass(Sub), False)):
        for name, call in zip(NAMES, _refused(wrap)):
            with monkeypatch.context() as m:
                rec = Recorder(pit._native)
                m.setattr(pit, "_native", rec)
                with pytest.raises(pit.PitError):
                    call()
            assert len(rec.answers) == 1, name
            status = rec.answers[0][0] if isinstance(rec.answers[0], tuple) else rec.answers[0]
            assert (status in (pit.PIT_EINVAL, pit.PIT_ESHAPE, pit.PIT_ECAPACITY)) if native else status is None, (name, rec.answers)


@pytest.mark.gpu
def test_ordinary_calls_are_answered_natively_on_the_device(monkeypatch):
    """The handle of the current stream is what the native side takes, and each function answers PIT_OK."""
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(s, dtype=dtype, device="cuda")
    ix, ws = pit.PitIndex(z(3, dtype=torch.int32), z(1024, dtype=torch.int32), None, 2, 1024), z(1 << 22, dtype=torch.uint8)
    X, W, C = z(512, 256), z(512, 128), z(256, 128, dtype=torch.float32)
    cands = [{"mt_rows": 1, "mt_cols": 128, "tile_cost": 1.0}]
    rec = Recorder(pit._native)
    monkeypatch.setattr(pit, "_native", rec)
    pit.pit_build_index(X, 1, 128, 0, out=ix, ws=ws)
    pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_K, X, W, ix, 128, 256, 128, 512, out=C)
    pit.pit_relu_channel_major_index(z(256, 512), out_xt=X, out=ix, ws=ws)
    pit.pit_select_and_run_gemm(cands, [[900]], [[1024]], X, W, 256, 128, 512, out=C, ws=ws)
    pit.pit_moe_dispatch_gemm(z(96, 128), z(96, dtype=torch.int32), None, z(4, 128, 256), z(4, 256, 128), out=z(96, 128, dtype=torch.float32), ws=ws)
    pit.pit_sparse_attn(z(2, 256, 64), z(2, 256, 64), z(2, 256, 64), z(256, 256, dtype=torch.uint8), 0.125, out=z(2, 256, 64, dtype=torch.float32), ws=ws)
    torch.cuda.synchronize()
    assert rec.answers == [0, 0, 0, (0, 0), 0, 0]

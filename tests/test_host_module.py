"""The native marshalling of the binding's ordinary calls (csrc/host.cpp) against the Python marshalling: the same results
for the calls it takes, nothing done for the ones it leaves alone, the same errors."""
import ctypes
import os
import sys
import warnings

import pytest
import torch

from host_on_cpu import host_cpu, stand_in  # noqa: F401 (fixtures)
from paper_2503_03588_amd import binding as pa
from paper_2503_03588_amd import build

PAT = pa.Pattern(64, 3, 1)


def bound_host():
    from paper_2503_03588_amd import _host
    L = pa.lib()
    _host.bind(*(ctypes.cast(getattr(L, "powattn_" + n), ctypes.c_void_p).value for n in pa._NATIVE_ENTRY_POINTS), torch.Tensor,
               torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, pa._check)
    return _host


def test_out_of_the_ordinary_is_left_alone():
    if not hasattr(torch._C, "_cuda_getCurrentRawStream"):
        pytest.skip("this torch has no GPU support")
    host = bound_host()

    class Sub(torch.Tensor):
        pass

    x = torch.zeros(1, 2, 64, 64)
    for q in (x, x.as_subclass(Sub), torch.nn.Parameter(x), x.transpose(1, 2), x.data_ptr(), None):
        assert host.prefill(PAT._values, None, None, q, x, x, None, None, 0.0, True) is NotImplemented
        assert host.decode(PAT._values, q, x, x, x, None, None, 0.0, x, True) is NotImplemented
    assert host.mask_build(PAT._values, -1) is NotImplemented
    assert host.mask_build((64, 3, 1), 128) is NotImplemented
    assert host.mask_build(PAT._values, 128.0) is NotImplemented
    with pytest.raises(TypeError):
        host.prefill(PAT._values)


def test_a_refusal_inside_the_call_comes_back_to_python(stand_in):
    """Sizes that do not fit the library's integers are found while its arguments are formed, with other threads running."""
    huge = 2 ** 31
    q, k = torch.empty(1, huge, 0, 64), torch.empty(1, 2, 0, 64)
    q1, k1 = torch.empty(0, huge, 64), torch.empty(0, 2, 64, 64)
    none = torch.empty(0, dtype=torch.int32)
    cnt, idx = torch.zeros(4, dtype=torch.int32), torch.zeros(4, 4, dtype=torch.int32)
    table = torch.zeros(1, 4, dtype=torch.int32)
    one = torch.zeros(1, dtype=torch.int32)
    pages = torch.empty(0, 2, 64, 64)
    ws = torch.empty(256, dtype=torch.uint8)
    host, v = pa._native, PAT._values
    for args in [
        (host.prefill, v, cnt, idx, q, k, k, None, None, 0.0, True),
        (host.prefill_chunk, v, cnt, idx, q, k, k, 0, None, None, 0.0, True),
        (host.prefill_chunk_paged, v, cnt, idx, q, pages, pages, table, 0, None, None, 0.0, True),
        (host.prefill_batch_paged, v, cnt, idx, q, pages, pages, table, one, one, None, None, 0.0, True),
        (host.prefill_varlen, v, cnt, idx, q, k, k, one, None, None, 0.0, True),
        (host.decode, v, q1, k1, k1, none, None, None, 0.0, ws, True),
        (host.decode_paged, v, q1, pages, pages, torch.empty(0, 4, dtype=torch.int32), none, None, None, 0.0, ws, True),
        (host.backward, v, cnt, idx, q, k, k, q, torch.empty(1, huge, 0), q, None, None, None, 0.0, ws),
    ]:
        assert args[0](*args[1:]) is NotImplemented, args[0].__name__
    assert not stand_in.seen


def test_the_library_is_called_once_and_its_status_raised(stand_in):
    q, ws = torch.zeros(1, 2, 64, 64), torch.empty(1 << 20, dtype=torch.uint8)
    cnt, idx = torch.zeros(1, dtype=torch.int32), torch.zeros(1, 4, dtype=torch.int32)
    one, table, q1 = torch.ones(1, dtype=torch.int32), torch.zeros(1, 1, dtype=torch.int32), q[:, :, 0].contiguous()
    for name, call in [
        ("prefill", lambda: pa.prefill(PAT, cnt, idx, q, q, q)),
        ("prefill_chunk", lambda: pa.prefill_chunk(PAT, cnt, idx, q, q, q, 0)),
        ("prefill_chunk_paged", lambda: pa.prefill_chunk_paged(PAT, cnt, idx, q, q, q, table, 0)),
        ("prefill_batch_paged", lambda: pa.prefill_batch_paged(PAT, cnt, idx, q, q, q, table, one, one)),
        ("prefill_varlen", lambda: pa.prefill_varlen(PAT, cnt, idx, q, q, q, one)),
        ("decode", lambda: pa.decode(PAT, q1, q, q, one, workspace=ws)),
        ("decode_paged", lambda: pa.decode_paged(PAT, q1, q, q, table, one, workspace=ws)),
        ("backward", lambda: pa.backward(PAT, cnt, idx, q, q, q, q, q[..., 0].contiguous(), q, workspace=ws)),
        ("mask_build", lambda: pa._native.mask_build(PAT._values, 64)),
    ]:
        for status in (pa.HIP_ERROR, pa.WORKSPACE_TOO_SMALL):
            stand_in.seen.clear()
            stand_in.answers[:] = [status]
            with pytest.raises(pa.PowattnError, match="powattn_" + name + ": status"):
                call()
            assert len(stand_in.seen) == 1 and not stand_in.answers, name


def test_other_threads_run_while_outputs_are_allocated(stand_in):
    watch = ctypes.CDLL(pa._native.__file__)
    q, ws = torch.zeros(1, 2, 64, 64), torch.empty(1 << 20, dtype=torch.uint8)
    cnt, idx = torch.zeros(1, dtype=torch.int32), torch.zeros(1, 4, dtype=torch.int32)
    one, table, q1, lse = torch.ones(1, dtype=torch.int32), torch.zeros(1, 1, dtype=torch.int32), q[:, :, 0].contiguous(), q[..., 0].contiguous()
    for new, call in [
        (2, lambda: pa._native.mask_build(PAT._values, 64)),
        (2, lambda: pa.prefill(PAT, cnt, idx, q, q, q)),
        (2, lambda: pa.prefill_chunk(PAT, cnt, idx, q, q, q, 0)),
        (2, lambda: pa.prefill_chunk_paged(PAT, cnt, idx, q, q, q, table, 0)),
        (2, lambda: pa.prefill_batch_paged(PAT, cnt, idx, q, q, q, table, one, one)),
        (2, lambda: pa.prefill_varlen(PAT, cnt, idx, q, q, q, one)),
        (2, lambda: pa.decode(PAT, q1, q, q, one, workspace=ws)),
        (1, lambda: pa.decode_paged(PAT, q1, q, q, table, one, workspace=ws, want_lse=False)),
        (4, lambda: pa.backward(PAT, cnt, idx, q, q, q, q, lse, q)),
    ]:
        watch.watch_allocations(1)
        try:
            call()
        finally:
            watch.watch_allocations(0)
        assert (watch.allocations_with_gil(), watch.allocations_without_gil()) == (0, new)


@pytest.mark.parametrize("compiler,why", [("/nonexistent/compiler", "No such file"), ("false", "failed to build")])
def test_the_build_does_without_a_host_module(monkeypatch, tmp_path, capsys, compiler, why):
    old = tmp_path / "_host.so"
    old.write_bytes(b"of an earlier build")
    monkeypatch.setattr(build, "HOST_OUT", str(old))
    monkeypatch.setenv("CXX", compiler)
    assert build.build_host_or_do_without() is None
    assert not old.exists()
    said = capsys.readouterr().err
    assert "_host.so was not built" in said and why in said


def test_a_host_module_that_cannot_be_loaded_is_reported(monkeypatch, tmp_path):
    monkeypatch.setattr(pa, "_native", None)
    monkeypatch.setattr(pa, "_native_tried", False)
    monkeypatch.setitem(sys.modules, "paper_2503_03588_amd._host", None)     # its import fails
    monkeypatch.delattr("paper_2503_03588_amd._host", raising=False)
    broken = tmp_path / "_host.so"
    broken.write_bytes(b"")
    monkeypatch.setattr(pa, "HOST_PATH", str(broken))
    with pytest.warns(RuntimeWarning, match="cannot be loaded"):
        pa._enable_native()
    assert pa._native is None and pa._native_tried
    monkeypatch.setattr(pa, "HOST_PATH", str(tmp_path / "not built"))
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        pa._enable_native()
    assert pa._native is None


def test_a_forked_child_starts_without_the_native_way(monkeypatch):
    monkeypatch.setattr(pa, "_native", object())
    monkeypatch.setattr(pa, "_native_tried", True)
    r, w = os.pipe()
    child = os.fork()
    if child == 0:
        os.write(w, repr((pa._native, pa._native_tried)).encode())
        os._exit(0)
    os.waitpid(child, 0)
    assert os.read(r, 100) == b"(None, False)"
    os.close(r)
    os.close(w)
    assert pa._native is not None and pa._native_tried


def calls():
    """(name, function of no arguments) of every entry point that is marshalled natively; fresh outputs each time."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    n, hq, hkv, d, b = 200, 4, 2, 64, 2
    q, k, v = normal(b, hq, n, d), normal(b, hkv, n, d), normal(b, hkv, n, d)
    cnt, idx, _ = pa.mask_build(PAT, 256)
    pk, pv = normal(9, hkv, 64, d), normal(9, hkv, 64, d)
    table = torch.arange(8, dtype=torch.int32, device="cuda").reshape(b, 4)
    lens = torch.tensor([n, 77], dtype=torch.int32, device="cuda")
    start = torch.tensor([30, 0], dtype=torch.int32, device="cuda")
    rows = torch.tensor([100, 3], dtype=torch.int32, device="cuda")
    ws = pa.decode_workspace(PAT, b, hq, hkv, d, 256)
    q1, o1 = q[:, :, 0].contiguous(), torch.empty_like(q[:, :, 0].contiguous())
    nosink = pa.Pattern(64, 3, 0)                # (sums over a sink block's column depend on the order of arrival)
    cnt0, idx0, _ = pa.mask_build(nosink, 256)
    saved = pa.prefill(nosink, cnt0, idx0, q, k, v)
    zo, zl = torch.zeros_like(q), torch.zeros(q.shape[:3], device="cuda")
    return [
        ("mask_build", lambda: pa.mask_build(PAT, 1000)[:2]),
        ("prefill", lambda: pa.prefill(PAT, cnt, idx, q, k, v)),
        ("prefill without lse, scale given", lambda: pa.prefill(PAT, cnt, idx, q, k, v, softmax_scale=0.3, want_lse=False)[:1]),
        ("prefill fp32", lambda: pa.prefill(PAT, cnt, idx, q.float(), k.float(), v.float())),
        ("prefill dense", lambda: pa.prefill(pa.Pattern(64, 1, 0, pa.DENSE | pa.POWER), None, None, q, k, v)),
        ("chunk", lambda: pa.prefill_chunk(PAT, cnt, idx, q[:, :, :50].contiguous(), k, v, 31)),
        ("chunk paged", lambda: pa.prefill_chunk_paged(PAT, cnt, idx, q[:, :, :50].contiguous(), pk, pv, table, 31)),
        ("batch paged", lambda: pa.prefill_batch_paged(PAT, cnt, idx, q, pk, pv, table, start, rows, o=zo.clone(), lse=zl.clone())),
        ("varlen", lambda: pa.prefill_varlen(PAT, cnt, idx, q, k, v, lens)),
        ("decode", lambda: pa.decode(PAT, q1, k, v, lens, workspace=ws)),
        ("decode, outputs given", lambda: pa.decode(PAT, q1, k, v, lens, o=o1, workspace=ws)),
        ("decode paged", lambda: pa.decode_paged(PAT, q1, pk, pv, table, lens, workspace=ws)),
        ("backward", lambda: pa.backward(nosink, cnt0, idx0, q, k, v, *saved, q)),
        ("backward, outputs given", lambda: pa.backward(nosink, cnt0, idx0, q, k, v, *saved, q, dq=zo.clone(), dv=v.clone(), softmax_scale=0.2)),
    ]


@pytest.mark.gpu
def test_the_same_results_as_through_python(monkeypatch):
    pa.mask_build(PAT, 64)                       # (the first call enables the native ones)
    host = pa._native
    assert host is not None, "the host module is not built"
    for name, call in calls():
        results = []
        for native in (host, None):
            monkeypatch.setattr(pa, "_native", native)
            side = torch.cuda.Stream()           # the current stream is the one that counts
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                out = call()
            side.synchronize()
            results.append([t.clone() for t in out])
        for a, b in zip(*results):
            assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b), name
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_every_ordinary_call_goes_the_native_way(monkeypatch):
    pa.mask_build(PAT, 64)
    host, seen = pa._native, []

    class Spy:
        def __getattr__(self, name):
            def f(*a):
                r = getattr(host, name)(*a)
                seen.append((name, r is not NotImplemented))
                return r
            return f

    todo = calls()
    monkeypatch.setattr(pa, "_native", Spy())
    for name, call in todo:
        call()
    torch.cuda.synchronize()
    assert len(seen) == len(todo) and all(ok for _, ok in seen), seen


@pytest.mark.gpu
def test_errors_are_the_python_ways_own():
    pa.mask_build(PAT, 64)
    q = torch.zeros(1, 2, 64, 64, dtype=torch.bfloat16, device="cuda")
    cnt, idx, _ = pa.mask_build(PAT, 64)
    with pytest.raises(ValueError, match="dtype"):
        pa.prefill(PAT, cnt, idx, q, q.float(), q)
    with pytest.raises(ValueError, match="shape"):
        pa.prefill(PAT, cnt, idx, q, q[:, :, :32].contiguous(), q)
    with pytest.raises(ValueError, match="contiguous"):
        pa.prefill(PAT, cnt, idx, q.transpose(1, 2), q.transpose(1, 2), q.transpose(1, 2))
    with pytest.raises(pa.PowattnError):
        pa.prefill(pa.Pattern(72, 3, 1), cnt, idx, q, q, q)
    with pytest.raises(pa.PowattnError):
        pa.mask_build(PAT, -3)
    with pytest.raises(pa.PowattnError):
        pa.decode(PAT, q[:, :, 0].contiguous(), q, q, cnt, workspace=torch.empty(1, dtype=torch.uint8, device="cuda"))

"""The two ways the enqueue calls take into the library (the extension module and ctypes): the same conversions, the same
status codes, the same refusals.  No GPU: the graph is host-only, and the library's own argument checks show what it was given."""
import ctypes
import importlib

import numpy as np
import pytest

import paper_2412_20379_amd as ntp
from paper_2412_20379_amd import binding, build

N, F = 50, 8


@pytest.fixture(scope="module")
def graph():
    v = np.arange(N, dtype=np.int32)
    g = ntp.ntp_graph_build(N, v, (v + 1) % N, flags=ntp.NTP_GCN_FLAGS | ntp.NTP_HOST_ONLY)
    yield g
    g.close()


@pytest.fixture(params=["native", "ctypes"])
def calls(request):
    if request.param == "ctypes":
        return binding.CtypesCalls(ntp.lib())
    if build.native_command("") is None:
        pytest.skip("no Python.h")
    ntp.lib()
    return importlib.import_module("paper_2412_20379_amd._native")


class Stream:
    def __init__(self, cuda_stream):
        self.cuda_stream = cuda_stream


def _forms(array):
    import torch
    t = torch.from_numpy(array)
    return [array, t, array.ctypes.data, ctypes.c_void_p(array.ctypes.data)]


def test_every_enqueue_call_is_there(calls):
    for name in binding.ENQUEUE_CALLS:
        assert callable(getattr(calls, name))
        with pytest.raises(TypeError):
            getattr(calls, name)()


def test_pointers(calls, graph):
    """an address arrives as it is: the library finds two forms of one buffer overlapping, and a neighbour not"""
    both = np.zeros((2 * N, F), np.float32)
    x, y = both[:N], both[N:]
    for a in _forms(x):
        for b in _forms(y):
            assert calls.ntp_aggregate_fwd(graph.addr, a, b, F, F, F, ntp.NTP_F32, None) == ntp.NTP_EBUDGET      # host-only
        for b in _forms(both[N - 1:2 * N - 1]):                                                                  # one row shared
            assert calls.ntp_aggregate_fwd(graph.addr, a, b, F, F, F, ntp.NTP_F32, None) == ntp.NTP_EINVAL
            assert "overlap" in ntp.ntp_last_error()
        assert calls.ntp_aggregate_fwd(graph.addr, a, None, F, F, F, ntp.NTP_F32, None) == ntp.NTP_EINVAL
    assert calls.ntp_aggregate_fwd(None, x, y, F, F, F, ntp.NTP_F32, None) == ntp.NTP_EINVAL
    for wrong in ("x", 1.5, object()):
        with pytest.raises((AttributeError, TypeError)):
            calls.ntp_aggregate_fwd(graph.addr, wrong, y, F, F, F, ntp.NTP_F32, None)


def test_streams(calls, graph):
    x, y = np.zeros((N, F), np.float32), np.zeros((N, F), np.float32)
    for s in (None, 0, 1 << 40, Stream(0), Stream(1 << 40)):
        assert calls.ntp_aggregate_fwd(graph.addr, x, y, F, F, F, ntp.NTP_F32, s) == ntp.NTP_EBUDGET
        assert calls.ntp_chunked_aggregate(graph.addr, ntp.NTP_FWD, x, y, F, F, F, ntp.NTP_F32, s, Stream(7)) == ntp.NTP_EBUDGET
    with pytest.raises(AttributeError):
        calls.ntp_aggregate_fwd(graph.addr, x, y, F, F, F, ntp.NTP_F32, object())


def test_numbers(calls, graph):
    x, y = np.zeros((N, F), np.float32), np.zeros((N, F), np.float32)
    ok = lambda f, code: calls.ntp_aggregate_fwd(graph.addr, x, y, f, np.int64(F), np.int32(F), code, None)
    for f in (F, np.int64(F), np.int32(F), np.uint8(F), float(F), True):
        assert ok(f, ntp.NTP_F32) == ntp.NTP_EBUDGET
    assert ok(F + 1, ntp.NTP_F32) == ntp.NTP_EINVAL and "stride" in ntp.ntp_last_error()
    assert ok(-1, ntp.NTP_F32) == ntp.NTP_EINVAL and "-1" in ntp.ntp_last_error()
    assert ok(F, 7) == ntp.NTP_EINVAL and "dtype 7" in ntp.ntp_last_error()
    assert calls.ntp_chunked_aggregate(graph.addr, 5, x, y, F, F, F, ntp.NTP_F32, None, 7) == ntp.NTP_EINVAL
    for slope in (0.2, 1, np.float32(0.2), np.float64(0.2)):
        assert calls.ntp_edge_softmax(graph.addr, x, y, slope, x, None, None) == ntp.NTP_EBUDGET
    for wrong in ("width", None, object()):
        with pytest.raises((TypeError, ValueError)):
            ok(wrong, ntp.NTP_F32)
        with pytest.raises((TypeError, ValueError)):
            calls.ntp_edge_softmax(graph.addr, x, y, wrong, x, None, None)


def test_ctypes_takes_over_where_the_module_is_missing(monkeypatch, graph):
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": "/nonexistent"})
    assert build.native_command("out.so") is None
    native = binding._native

    def missing(name, package=None):
        raise ImportError(name)

    monkeypatch.setattr(importlib, "import_module", missing)
    monkeypatch.setattr(build, "NATIVE", "/nonexistent/_native.so")
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", native)
    binding.lib()
    assert isinstance(binding._native, binding.CtypesCalls)
    x, y = np.zeros((N, F), np.float32), np.zeros((N, F), np.float32)
    with pytest.raises(ntp.NtpError) as e:
        ntp.ntp_aggregate_fwd(graph, x, y, F, F, F)
    assert e.value.code == ntp.NTP_EBUDGET


def test_hipcc_builds_the_module_where_there_is_no_gxx(monkeypatch, tmp_path):
    import subprocess
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    out = str(tmp_path / "module.so")
    cmd = build.native_command(out)
    if cmd is None:
        pytest.skip("no Python.h")
    assert "hipcc" in cmd[0]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

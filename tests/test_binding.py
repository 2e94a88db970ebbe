"""The native argument marshalling of the Python entry points against the ctypes calls it took the place of, on a
stand-in library that writes its arguments down (no GPU)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2507_11830_amd as sp

HERE = os.path.dirname(os.path.abspath(__file__))


class T:  # what the binding asks of a tensor
    def __init__(self, ptr, *shape, size=2):
        self.ptr, self.shape, self.size = ptr, shape, size

    def data_ptr(self):
        return self.ptr

    def numel(self):
        return int(np.prod(self.shape, dtype=np.int64))

    def element_size(self):
        return self.size


class Cache:
    desc = sp.sp_cache_desc(0x7000_0000_1000, 0x7000_0000_2000, 77, 16, 2, 128)


class Stream:
    cuda_stream = 0x7FFF_0000_1234


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "stub.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-I", os.path.join(HERE, "..", "include"), os.path.join(HERE, "binding_stub.c"), "-o", so])
    L, real = ctypes.CDLL(so), sp.lib()
    for name in ("sp_kv_append", "sp_attn_prefill", "sp_chunk_step", "sp_attn_decode", "sp_attn_decode_static", "sp_decode_step"):
        getattr(L, name).argtypes = getattr(real, name).argtypes
    L.stub_seen.restype, L.stub_size.restype = ctypes.c_void_p, ctypes.c_size_t
    sp._bind(L)
    yield L, lambda: ctypes.string_at(L.stub_seen(), L.stub_size())
    sp._bind(real)


def test_the_file_is_named_for_its_interpreter():
    """Another one does not find it, rather than load code made for other object layouts."""
    import sysconfig

    assert os.path.basename(sp.BINDING_PATH) == "_binding" + sysconfig.get_config_var("EXT_SUFFIX")


def by_ctypes(L, name, desc, *args):
    return getattr(L, name)(ctypes.byref(desc), *args)


class AsParameter:  # ctypes' own way to pass an object of the caller's
    def __init__(self, value):
        self._as_parameter_ = value


I32S = (5, np.int64(9), np.int32(-3), True, 2**32 + 7, -1, ctypes.c_int32(4), AsParameter(6), AsParameter(ctypes.c_int32(8)))
STREAMS = ((0, 0), (0x1234_5678_9ABC, 0x1234_5678_9ABC), (Stream(), Stream.cuda_stream))


SCALES = (0.125, 1, np.float32(0.3), np.float64(1e-9))
SPACES = (None, T(0x7777_0000, 3, 5, size=1), T(0, 0), T(2**47, 1 << 33, size=4))


@pytest.mark.parametrize("n", range(len(I32S)))
def test_same_arguments_as_ctypes(stub, n):
    L, seen = stub
    (stream, raw), scale, ws = STREAMS[n % 3], SCALES[n % 4], SPACES[(n // 2) % 4]
    N = sp._native
    a, b = I32S[n], I32S[(n + 1) % len(I32S)]
    table, q, k = T(0x10_0000_0000, 6, 11, size=4), T(0x7FEE_0000_0000, 40, 8, 128), T(2**48 - 16, 40, 2, 128)
    v, out, lens, cu = T(0x30, 40, 2, 128), T(0x40, 40, 8, 128), T(0, 0, size=4), T(0x60, 7, size=4)
    p = lambda t: None if t is None else t.data_ptr()
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    d = Cache.desc
    for got, want in (
        (lambda: N.kv_append(Cache, k, v, cu, lens, table, stream), ("sp_kv_append", p(k), p(v), p(cu), p(lens), p(table), 6, 11, 40, raw)),
        (lambda: N.kv_append(Cache, k, None, None, lens, table, stream), ("sp_kv_append", p(k), None, None, p(lens), p(table), 6, 11, 40, raw)),
        (lambda: N.attn_prefill(Cache, q, out, cu, lens, table, a, b, scale, 1, ws, stream),
         ("sp_attn_prefill", p(q), p(out), p(cu), p(lens), p(table), 6, 11, 40, a, b, 8, float(scale), 1, p(ws), nbytes, raw)),
        (lambda: N.chunk_step(Cache, k, v, q, out, cu, lens, table, a, b, scale, ws, stream),
         ("sp_chunk_step", p(k), p(v), p(q), p(out), p(cu), p(lens), p(table), 6, 11, 40, a, b, 8, float(scale), p(ws), nbytes, raw)),
        (lambda: N.attn_decode(Cache, q, out, lens, table, a, scale, ws, stream),
         ("sp_attn_decode", p(q), p(out), p(lens), p(table), 6, 11, a, 8, float(scale), p(ws), nbytes, raw)),
        (lambda: N.attn_decode_static(Cache, q, out, lens, table, a, scale, stream),
         ("sp_attn_decode_static", p(q), p(out), p(lens), p(table), 6, 11, a, 8, float(scale), raw)),
        (lambda: N.decode_step(Cache, k, v, q, out, lens, table, a, scale, ws, stream),
         ("sp_decode_step", p(k), p(v), p(q), p(out), p(lens), p(table), 6, 11, a, 8, float(scale), p(ws), nbytes, raw)),
    ):
        status = by_ctypes(L, want[0], d, *want[1:])
        record = seen()
        assert got() == status and seen() == record, want


def test_refuses_what_ctypes_refused(stub):
    N = sp._native
    table, q, out, lens = T(1 << 20, 6, 11), T(2 << 20, 40, 8, 128), T(3 << 20, 40, 8, 128), T(4 << 20, 6)
    class Value:  # an enumeration's member, say
        value = 5

    for bad in (5.0, "5", None, [1], Value(), ctypes.c_int64(5), ctypes.c_float(5), AsParameter(5.0), AsParameter(Value())):
        with pytest.raises(ctypes.ArgumentError):
            N.attn_decode(Cache, q, out, lens, table, bad, 0.1, None, 0)
    for bad_table in (T(1, 6), T(1, 6, 11, 2)):
        with pytest.raises(ValueError):
            N.attn_decode(Cache, q, out, lens, bad_table, 5, 0.1, None, 0)
    with pytest.raises(IndexError):
        N.attn_decode(Cache, T(1, 40), out, lens, table, 5, 0.1, None, 0)
    with pytest.raises(AttributeError):
        N.attn_decode(Cache, q, object(), lens, table, 5, 0.1, None, 0)
    with pytest.raises(AttributeError):
        N.attn_decode(object(), q, out, lens, table, 5, 0.1, None, 0)
    for desc in (bytes(32), bytearray(32), np.zeros(4), (ctypes.c_int64 * 4)(), None):  # of the descriptor's size, but none
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            N.attn_decode(type("Cache", (), {"desc": desc}), q, out, lens, table, 5, 0.1, None, 0)
    with pytest.raises((TypeError, ValueError)):
        N.attn_decode(Cache, q, out, lens, table, 5, "x", None, 0)
    with pytest.raises((TypeError, ValueError)):
        N.attn_decode(Cache, q, out, lens, table, 5, 0.1, None, "stream")


def test_a_forked_child_asks_torch_for_the_stream_again(stub):
    """torch's public accessor refuses to work in a child of a process that has used the device; the raw ones do not."""
    N = sp._native
    asked = []
    L, _ = stub
    table, q, out, lens = T(1 << 20, 6, 11), T(2 << 20, 40, 8, 128), T(3 << 20, 40, 8, 128), T(4 << 20, 6)
    names = ("sp_kv_append", "sp_attn_prefill", "sp_chunk_step", "sp_attn_decode", "sp_attn_decode_static", "sp_decode_step")
    N.bind({n: ctypes.cast(getattr(L, n), ctypes.c_void_p).value for n in names}, ctypes.ArgumentError, ctypes.c_int32, sp.sp_cache_desc, lambda: 0, lambda dev: 0x1234, lambda: asked.append(1) or Stream())
    try:
        call = lambda: N.attn_decode(Cache, q, out, lens, table, 5, 0.1, None, None)
        call()
        first = len(asked)
        call()
        assert len(asked) == first  # the raw accessors from then on
        r, w = os.pipe()
        pid = os.fork()
        if pid == 0:
            try:
                call()
                os.write(w, bytes([len(asked) - first]))
            finally:
                os._exit(0)
        os.close(w)
        seen = os.read(r, 1)
        os.close(r)
        os.waitpid(pid, 0)
        assert seen == b"\x01"
    finally:
        sp._bind(L)

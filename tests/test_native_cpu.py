"""The native caller of the entry points (csrc/sw_python.cpp): every argument arrives in its place,
converted as the ctypes prototypes convert it; what is no address or integer is refused."""
import ctypes

import pytest

from paper_2311_18677_amd import binding as sw


def recorder(name):
    """(native function, list of the calls it made) for one entry point of the library."""
    from paper_2311_18677_amd import sw_native
    types = getattr(sw.load(), name).argtypes
    calls = []

    def record(*args):
        calls.append(args)
        return -7
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *types)(record)
    at = ctypes.cast(fn, ctypes.c_void_p).value
    lib = sw_native.Library({n: at for n in sw_native.NAMES})
    lib_call = getattr(lib, name)
    return (lambda *a, keep=fn: lib_call(*a)), calls, types


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Stream:
    cuda_stream = 0x7700000012345678


NAMES = ("sw_decode_attn", "sw_decode_attn_static", "sw_decode_attn_paged", "sw_decode_attn_append", "sw_decode_attn_paged_append",
         "sw_advance_lens", "sw_prefill_attn", "sw_prefill_attn_paged", "sw_mixed_attn", "sw_mixed_attn_paged", "sw_kv_store",
         "sw_kv_store_paged", "sw_kv_pack", "sw_kv_unpack", "sw_kv_span_plan")


def test_the_module_is_this_interpreters_and_has_every_entry_point():
    import sysconfig
    from paper_2311_18677_amd import build, sw_native
    assert sw_native.__file__.endswith("sw_native" + sysconfig.get_config_var("EXT_SUFFIX")) and sw_native.__file__ == build.NATIVE
    assert sw_native.NAMES == NAMES


@pytest.mark.parametrize("name", NAMES)
def test_every_argument_in_its_place(name):
    call, calls, types = recorder(name)
    args, want = [], []
    for i, t in enumerate(types):
        last = i == len(types) - 1
        if t is ctypes.c_void_p:
            at = 0x7f0000000000 + 4096 * (i + 1)
            args.append(Stream() if last else (Tensor(at), at, None)[i % 3])
            want.append(Stream.cuda_stream if last else (at, at, None)[i % 3])
        else:
            v = 2 ** 31 + 5 if t is ctypes.c_longlong else 1000 + i
            args.append(v)
            want.append(v)
    assert call(*args) == -7
    assert list(calls[0]) == want
    with pytest.raises(TypeError):
        call(*args[:-1])


def test_conversions_and_refusals():
    import numpy as np
    call, calls, _ = recorder("sw_prefill_attn")
    tail = (8, 1, 128, 64, None)
    assert call(1, 2, np.int64(3), True, None, Tensor(6), 7.9, ctypes.c_int(4), *tail) == -7
    assert calls[-1] == (1, 2, 3, 1, None, 6, 7, 4, 8, 1, 128, 64, None)
    call(2 ** 64 - 1, 0, 0, 0, 0, 0, -1, 2 ** 32 + 3, -8, *tail[1:])         # modulo the C types' ranges
    assert calls[-1][0] == 2 ** 64 - 1 and calls[-1][6:9] == (-1, 3, -8)
    n = len(calls)
    for bad in (("x", 1), (object(), 1), (1, 2.5), (1, "4"), (1, None), (Tensor("at"), 1)):
        with pytest.raises((TypeError, ValueError)):
            call(bad[0], 0, 0, 0, 0, 0, 0, bad[1], *tail)

    class Broken:
        def data_ptr(self):
            raise RuntimeError("no storage")
    with pytest.raises(RuntimeError, match="no storage"):
        call(Broken(), 0, 0, 0, 0, 0, 0, 1, *tail)
    assert len(calls) == n


def test_the_error_of_an_address_is_its_own():
    call, calls, _ = recorder("sw_advance_lens")

    class Raises:
        def data_ptr(self):
            raise AttributeError("freed")

    class Delegates:
        def __getattr__(self, name):
            if name == "data_ptr":
                return Raises().data_ptr
            raise AttributeError(name)
    for x in (Raises(), Delegates()):
        with pytest.raises(AttributeError, match="freed"):
            call(x, 1, 4, None)

    class Number:                       # no address of its own: what int() makes of it
        def __int__(self):
            return 4096
    call(Number(), 1, 4, Number())
    assert calls == [(4096, 1, 4, 4096)]


def test_addresses_that_ctypes_takes():
    call, calls, _ = recorder("sw_advance_lens")
    lens = (ctypes.c_int32 * 4)()
    at = ctypes.addressof(lens)

    class Wrapped:
        _as_parameter_ = at
    for given, want in ((None, None), (ctypes.c_void_p(at), at), (ctypes.c_void_p(), None), (lens, at), (ctypes.byref(lens), at),
                        (ctypes.pointer(lens), at), (Wrapped(), at)):
        stream = Stream()
        stream.cuda_stream = given
        call(Tensor(given), 1, 4, stream)
        assert calls.pop() == (want, 1, 4, want)
    for bad in (2.5, object(), [1], b"4096", "4096"):
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            call(Tensor(bad), 1, 4, None)
    assert calls == []


def test_integers_are_those_that_ctypes_takes():
    """Each value through the native caller and through a ctypes prototype of the same shape."""
    import enum
    call, calls, types = recorder("sw_advance_lens")
    by_ctypes = ctypes.CFUNCTYPE(ctypes.c_int, *types)(lambda *args: calls.append(args) or -7)

    class Parameter:
        def __init__(self, x):
            self._as_parameter_ = x

    class Index:
        def __init__(self, x):
            self.x = x

        def __index__(self):
            if self.x is None:
                raise OverflowError("no index")
            return self.x

    class Valued:
        value = 3
    Member = enum.Enum("Member", {"ONE": 1})
    taken = [3, True, -1, 2 ** 32 + 3, -2 ** 70 - 1, ctypes.c_int(4), ctypes.c_int(-4), Index(5), Parameter(6),
             Parameter(ctypes.c_int(7)), Parameter(Parameter(Index(8))), enum.IntEnum("Number", {"NINE": 9}).NINE]
    refused = [2.5, "4", b"4", None, object(), Member.ONE, Valued(), ctypes.c_longlong(2 ** 32 + 3), ctypes.c_short(2),
               ctypes.c_uint(2), Parameter(2.5), Parameter(Member.ONE), Index(None), [1], 3 + 0j]
    for x in taken:
        assert call(4096, x, 4, None) == by_ctypes(4096, x, 4, None) == -7
        native, other = calls
        assert native == other
        calls.clear()
    for x in refused:
        with pytest.raises(ctypes.ArgumentError):
            by_ctypes(4096, x, 4, None)
        with pytest.raises(ctypes.ArgumentError, match="argument 2: ") as refusal:
            call(4096, x, 4, None)
        assert isinstance(refusal.value, TypeError)
    for x in ("4096", 2.5, object()):
        with pytest.raises(ctypes.ArgumentError, match="argument 1: "):
            call(Tensor(x), 1, 4, None)
    endless = Parameter(None)
    endless._as_parameter_ = endless
    with pytest.raises((RecursionError, ctypes.ArgumentError)):
        call(4096, endless, 4, None)
    assert calls == []


def test_references_are_given_back():
    import sys
    call, calls, _ = recorder("sw_decode_attn")
    t, s = Tensor(10 ** 12), Stream()
    before = sys.getrefcount(t), sys.getrefcount(s)
    for _ in range(100):
        call(t, t, t, t, t, 1, 8, 1, 128, 64, s)
        calls.clear()
    assert (sys.getrefcount(t), sys.getrefcount(s)) == before


def test_a_library_needs_every_address():
    from paper_2311_18677_amd import sw_native
    with pytest.raises(KeyError):
        sw_native.Library({})
    with pytest.raises(ValueError):
        sw_native.Library({n: 0 for n in sw_native.NAMES})

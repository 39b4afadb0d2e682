"""How the binding takes its arguments (the same as through ctypes); nothing is launched: a call is refused, or ends in a function of the test."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2503_01873_amd as P

A = 1 << 20      # an address that is never followed


class Buffer:
    def data_ptr(self):
        return A


class Stream:
    cuda_stream = 0


class Index:
    def __index__(self):
        return 64


class Parameter:
    _as_parameter_ = 64


class Address:
    def data_ptr(self):
        return ctypes.c_void_p(A)


def chunk(**kw):
    a = dict(q=A, o=2 * A, B=1, Hq=2, Hkv=1, Nq=4, row0=0, N=64, d=64, causal=True, scale=0.125, workspace=A, workspace_bytes=1, check=False)
    a.update(kw)
    return P.pasa_attn_fwd_chunk(**a)


@pytest.mark.parametrize("kw,status", [
    ({}, 4), ({"q": None}, 1), ({"q": 2 * A}, 1), ({"q": Buffer()}, 4), ({"stream": Stream()}, 4), ({"stream": 0}, 4), ({"d": 96}, 2),
    ({"N": (1 << 32) + 64}, 4), ({"N": 0}, 1), ({"Nq": -1}, 1), ({"workspace_bytes": 1.0}, 4), ({"scale": 1}, 4), ({"causal": 2}, 1),
    ({"variant": 9}, 1), ({"beta": 1.0}, 1), ({"shift_tile": 64}, 2), ({"io_dtype": 2}, 1), ({"workspace": None, "workspace_bytes": 1 << 30}, 4),
])
def test_arguments_reach_the_library(kw, status):
    assert chunk(**kw) == status


@pytest.mark.parametrize("size", [np.int64(64), np.uint8(64), torch.tensor(64), Index(), ctypes.c_int(64), Parameter()])
def test_sizes_are_whatever_ctypes_takes_for_an_integer(size):
    assert chunk(N=size) == 4 and chunk(Nq=size, row0=0) == 4
    kw = dict(workspace=A, workspace_bytes=1, check=False)
    assert P.pasa_attn_fwd(A, A, A, 2 * A, 1, size, size, 64, 96, False, 0.125, check=False) == 2
    assert P.pasa_attn_fwd_ex(A, A, A, 2 * A, 1, size, size, size, size, False, 0.125, **kw) == 4
    assert P.pasa_attn_fwd_adaptive(A, A, A, 2 * A, size, 1, 1, size, size, False, 0.125, overflow_s=A, **kw) == 4
    assert P.pasa_prepare_kv(A, A, size, size, size, size, 0.125, **kw) == 4


def test_addresses_are_whatever_ctypes_takes_for_one():
    assert chunk(q=Address()) == 4 and chunk(q=Address(), o=A) == 1 and chunk(workspace=Address()) == 4


@pytest.mark.parametrize("kw,error", [
    ({"N": 64.0}, ctypes.ArgumentError), ({"B": "1"}, ctypes.ArgumentError), ({"q": 1.5}, AttributeError), ({"q": "x"}, AttributeError),
    ({"scale": "x"}, ValueError), ({"causal": None}, TypeError), ({"stream": "x"}, AttributeError), ({"variant": "x"}, ValueError),
])
def test_what_is_no_argument_is_refused(kw, error):
    with pytest.raises(error):
        chunk(**kw)


def test_every_route_raises_with_the_entry_points_name():
    for name, call in (
        ("pasa_attn_fwd:", lambda: P.pasa_attn_fwd(None, A, A, A, 1, 1, 1, 64, 64, False, 0.125)),
        ("pasa_attn_fwd_ex:", lambda: P.pasa_attn_fwd_ex(None, A, A, A, 1, 1, 1, 64, 64, False, 0.125, A, 1)),
        ("pasa_attn_fwd_adaptive:", lambda: P.pasa_attn_fwd_adaptive(None, A, A, A, 1, 1, 1, 64, 64, False, 0.125, A, 1)),
        ("pasa_prepare_kv:", lambda: P.pasa_prepare_kv(None, A, 1, 1, 64, 64, 0.125, A, 1)),
        ("pasa_attn_fwd_chunk:", lambda: chunk(q=None, check=True)),
    ):
        with pytest.raises(P.PasaError, match=name) as e:
            call()
        assert e.value.status == 1


VP, CI, CF, SZ = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
# entry point: its marshaller, C arguments (O: options) and the names of what comes in each place
ENTRIES = {
    "pasa_attn_fwd": ("plain", "q k v o B Hq Hkv N d causal scale stream", [VP] * 4 + [CI] * 6 + [CF, VP]),
    "pasa_attn_fwd_ex": ("whole", "q k v o B Hq Hkv N d causal scale O workspace workspace_bytes stream", [VP] * 4 + [CI] * 6 + [CF, VP, VP, SZ, VP]),
    "pasa_attn_fwd_adaptive": ("whole", "q k v o B Hq Hkv N d causal scale O workspace workspace_bytes stream", [VP] * 4 + [CI] * 6 + [CF, VP, VP, SZ, VP]),
    "pasa_prepare_kv": ("prepare", "k v B Hkv N d scale O workspace workspace_bytes stream", [VP] * 2 + [CI] * 4 + [CF, VP, VP, SZ, VP]),
    "pasa_attn_fwd_chunk": ("chunk", "q o B Hq Hkv Nq row0 N d causal scale O workspace workspace_bytes stream",
                            [VP] * 2 + [CI] * 8 + [CF, VP, VP, SZ, VP]),
}


class At:
    def __init__(self, address):
        self.address = self.cuda_stream = address

    def data_ptr(self):
        return self.address


@pytest.mark.parametrize("route", ["C", "ctypes"])
@pytest.mark.parametrize("entry", ENTRIES)
def test_every_argument_arrives_in_its_place(entry, route, monkeypatch):
    """A function of the test stands in for the entry point and keeps what it was called with."""
    import functools
    from paper_2503_01873_amd import _calls, binding
    marshaller, names, types = ENTRIES[entry]
    names = names.split()
    came = {}

    def stand_in(*args):
        came.update(zip(names, args))
        if came.get("O"):
            o = binding.pasa_opts.from_address(came["O"])
            came["O"] = {f: getattr(o, f) for f, _ in binding.pasa_opts._fields_}
        return 7

    f = ctypes.CFUNCTYPE(CI, *types)(stand_in)
    call = functools.partial(getattr(binding, "_" + marshaller), f)
    if route == "C":
        def refused(*args):
            raise AssertionError("ordinary arguments went through ctypes")
        call = functools.partial(getattr(_calls, marshaller), ctypes.cast(f, VP).value, refused)
    monkeypatch.setattr(P.lib(), "call_" + entry, call)
    given = {n: 100 + i for i, n in enumerate(names) if n != "O"}
    given.update(causal=True, scale=0.375)
    given.update({n: At((i + 1) << 40 | 0x10) for i, n in enumerate(names) if n in ("q", "v", "o", "workspace", "stream")})
    given["k"] = 3 << 44                                                  # an address as it is
    if "workspace_bytes" in names:
        given["workspace_bytes"] = (5 << 32) + 3
    given = {n: x for n, x in given.items() if n in names}
    options = dict(beta=0.25, variant=P.DIRECT, shift_tile=17, overflow_s=At(7 << 41), nonfinite_o=9 << 41, shift_mode=P.SHIFT_MATRIX, io_dtype=P.IO_BF16)
    if marshaller == "prepare":
        options["overflow_s"] = options["nonfinite_o"] = None             # it counts nothing: not among its arguments
    passed = {n: x for n, x in options.items() if x is not None} if "O" in names else {}
    assert getattr(P, entry)(**given, **passed, check=False) == 7
    plain = lambda x: x.address if isinstance(x, At) else x
    for n, x in given.items():
        assert came[n] == plain(x), n
    if "O" in names:
        assert came["O"] == {n: plain(x) for n, x in options.items()}
    if marshaller == "whole":
        assert getattr(P, entry)(**given, **passed, opts_null=True, check=False) == 7 and came["O"] is None


def test_counters_of_a_chunk_reach_the_library():
    """A chunk with a counter passes every check and is refused by its workspace; the counter's address is looked at on the way."""
    class Counter:
        asked = 0

        def data_ptr(self):
            Counter.asked += 1
            return A

    c = Counter()
    assert chunk(overflow_s=c, nonfinite_o=c) == 4 and Counter.asked == 2


def test_without_the_extension_calls_go_through_ctypes(monkeypatch):
    """An interpreter that the extension was not built for, or a machine without Python's headers."""
    import sys
    from paper_2503_01873_amd import binding
    monkeypatch.setitem(sys.modules, "paper_2503_01873_amd._calls", None)
    monkeypatch.setattr(binding, "_lib", None)
    assert binding.lib().call_pasa_attn_fwd_chunk.func is binding._chunk
    test_every_route_raises_with_the_entry_points_name()
    assert chunk() == 4 and chunk(N=np.int64(64)) == 4
    with pytest.raises(ctypes.ArgumentError):
        chunk(N=64.0)


def test_the_extension_is_for_one_interpreter_and_needs_its_headers(monkeypatch, tmp_path):
    import sysconfig
    from paper_2503_01873_amd import build
    assert build.CALLS.endswith("_calls" + sysconfig.get_config_var("EXT_SUFFIX")) and build.CALLS != "_calls.so"
    monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_calls() is None

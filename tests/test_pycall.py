"""The extension that marshals the per-token calls fills the same C structs as ctypes does, raises what ctypes raises, and can be absent."""
import ctypes as C
import os
import subprocess
import sys

import pytest

from tests import gpu_util as U

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
P = C.c_void_p


class _Tensor:                       # an address is all that a call takes from a tensor
    def __init__(self, at, n=0):
        self.at, self.n = at, n

    def data_ptr(self):
        return self.at

    def numel(self):
        return self.n

    def element_size(self):
        return 4


def _cache(kk, cls=None):
    c = (cls or kk.Cache).__new__(cls or kk.Cache)
    for i, f in enumerate(kk.Cache.FIELDS):
        setattr(c, f, _Tensor((1 << 40) + 256 * i))
    c.capacity, c.len_hint, c.plan_slots_per_split, c.plan_wavefronts = 884, True, "96", 8.0
    return c


def _recorders(kk, log):
    """C functions that note their arguments, in the order of kk._HOT."""
    def noting(*types):
        def f(lay, cache, *rest):
            log.append((C.string_at(lay, C.sizeof(kk._Layout)), C.string_at(cache, C.sizeof(kk._Cache)), *rest))
            return len(log)
        return C.CFUNCTYPE(C.c_int, P, P, *types)(f)
    return [noting(P, P, P, P, P, C.c_float, P, P, C.c_size_t, P), noting(P, P, P, P, P, C.c_float, P, P),
            noting(P, P, P, P, P, C.c_size_t, P), noting(P, C.c_float, P)]


def _bind(kk, functions, stream=77):
    from paper_2504_09936_amd import _pycall
    return dict(zip(kk._HOT, _pycall.bind(lambda device: stream + device, lambda: 2, C.ArgumentError,
                                          *(C.cast(f, P).value for f in functions))))


def _arguments(kk, cache):
    t = [_Tensor(4096 * (i + 1), 100) for i in range(7)]
    lay = kk.Layout(3, 32, 8, 128, kk.BF16, 0.0883883)
    return {"decode_step": (lay, cache, t[0], t[1], t[2], t[3], None, 0.9, t[4], t[5]), "score": (lay, cache, t[0], 1),
            "decode_step_static": (lay, cache, t[0], t[1], t[2], t[3], t[6], 0.25, None),
            "decode_attn": (lay, cache, t[0], t[1], None, t[2], None)}


def test_same_structs_and_arguments_as_ctypes(monkeypatch):
    kk = U.kk()
    a, b = [], []
    fast, slow = _bind(kk, keep := _recorders(kk, a)), _recorders(kk, b)
    monkeypatch.setattr(kk, "_stream", lambda: 79)
    for name, f in zip(kk._HOT, slow):
        monkeypatch.setattr(kk._lib, "keepkv_" + name, f)
    monkeypatch.setattr(kk, "_check", lambda st, where: None)
    monkeypatch.setattr(kk, "_fast", dict.fromkeys(kk._HOT))
    for i, (name, args) in enumerate(_arguments(kk, _cache(kk)).items()):
        assert fast[name](*args) == i + 1
        getattr(kk, name)(*args)
    assert a == b and len(a) == 4 and keep


def test_each_library_has_functions_of_its_own():
    kk = U.kk()
    a, b = [], []
    fa, fb = _recorders(kk, a), _recorders(kk, b)
    one, two = _bind(kk, fa), _bind(kk, fb, stream=5)
    one["score"](*_arguments(kk, _cache(kk))["score"])
    two["score"](*_arguments(kk, _cache(kk))["score"])
    assert len(a) == len(b) == 1 and a[0][-1] == 79 and b[0][-1] == 7


class _Raising:
    def data_ptr(self):
        raise KeyError("no storage")


WRONG = [("layout", "batch", 2.0), ("layout", "scale", "x"), ("layout", "dtype", None), ("cache", "capacity", 884.0), ("cache", "len_hint", "many"),
         ("cache", "plan_wavefronts", None), ("cache", "k", object()), ("cache", "votes", _Raising()), ("cache", "len", _Tensor("x")),
         ("argument", 2, object()), ("argument", 2, _Raising()), ("argument", 5, _Tensor(1.5)), ("argument", 7, "0.9"), ("argument", 7, None),
         ("argument", 9, object()), ("missing", "layout", "head_dim"), ("missing", "cache", "born"), ("missing", "cache", "capacity")]


@pytest.mark.parametrize("where,what,value", WRONG)
def test_wrong_arguments_raise_what_ctypes_raises(monkeypatch, where, what, value):
    kk = U.kk()
    log = []
    functions = _recorders(kk, log)
    monkeypatch.setattr(kk, "_stream", lambda: 79)

    def raised(fast):
        monkeypatch.setattr(kk, "_fast", fast)
        args = list(_arguments(kk, _cache(kk))["decode_step"])
        if where == "argument":
            args[what] = value
        elif where == "missing":
            delattr(args[0 if what == "layout" else 1], value)
        else:
            setattr(args[0 if where == "layout" else 1], what, value)
        with pytest.raises(Exception) as e:
            kk.decode_step(*args)
        return e.type

    assert raised(_bind(kk, functions)) is raised(dict.fromkeys(kk._HOT)) and not log


def test_other_classes_are_asked_for_their_own_structs(monkeypatch):
    kk = U.kk()

    class Window(kk.Cache):
        def c(self):
            s = super().c()
            s.capacity = 7
            return s

    log = []
    functions = _recorders(kk, log)
    monkeypatch.setattr(kk, "_stream", lambda: 79)
    monkeypatch.setattr(kk, "_check", lambda st, where: None)
    monkeypatch.setattr(kk, "_fast", _bind(kk, functions))
    monkeypatch.setattr(kk._lib, "keepkv_score", functions[3])
    for cls, capacity in ((kk.Cache, 884), (Window, 7)):
        kk.score(*_arguments(kk, _cache(kk, cls))["score"])
        assert kk._Cache.from_buffer_copy(log[-1][1]).capacity == capacity


def test_binding_without_the_extension():
    code = ("import sys; sys.modules['paper_2504_09936_amd._pycall'] = None\n"
            "from paper_2504_09936_amd import binding as kk\n"
            "assert not any(kk._fast.values()) and kk.version() >= 100\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

"""The calls that go through the CPython module take the arguments that a ctypes function of the same prototype takes, with the
same results: both call one recording function, for every parameter and many kinds of values. No GPU, no launch."""
import ctypes

import numpy as np
import pytest

import paper_2509_15235_amd as vs
from paper_2509_15235_amd import binding

VP, I32, I64, SZ, F32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_size_t, ctypes.c_float


class Stands:
    def __init__(self, x):
        self._as_parameter_ = x


class Index:
    def __init__(self, x):
        self.x = x

    def __index__(self):
        if isinstance(self.x, Exception):
            raise self.x
        return self.x


class Number:
    def __float__(self):
        return 2.25


class Tensor:
    def __init__(self, x):
        self.x = x

    def data_ptr(self):
        if isinstance(self.x, Exception):
            raise self.x
        return self.x


BUF = (ctypes.c_int32 * 4)()
ARRAY = np.arange(6)


class SubDesc(vs.AttnDesc):
    pass


DESC, KV, SUB = vs.AttnDesc(B=3), vs.KVDesc(B=4), SubDesc(B=5)
VALUES = [None, 0, 7, -1, 2 ** 31, 2 ** 40 + 5, 2 ** 70 + 3, True, 1.5, "text", b"bytes", [], DESC, KV, SUB, ctypes.byref(DESC), ctypes.pointer(DESC),
          I32(6), I32(-6), I64(2 ** 40 + 6), SZ(2 ** 63), F32(1.25), ctypes.c_double(1.25), ctypes.c_bool(True), ctypes.c_int8(3),
          VP(4096), VP(None), BUF, ctypes.byref(BUF), ctypes.cast(BUF, ctypes.POINTER(I32)), np.int32(-4), np.int64(4), np.float32(1.5),
          np.array(3), ARRAY, Index(11), Index(ValueError("no")), Number(), Tensor(4096), Tensor(None), Tensor(VP(64)), Tensor(np.int64(64)),
          Tensor(1.5), Tensor(2 ** 70 + 64), Tensor(RuntimeError("no")), Stands(8), Stands(I32(9)), Stands(I64(9)), Stands(F32(0.5)), Stands(Stands(12)),
          Stands(None), Stands(VP(128))]

# the calls as ctypes functions: structures by reference, pointers through binding._ptr
STRUCTS = {"vs_tree_verify_attention": vs.AttnDesc, "vs_compress_attention": vs.AttnDesc, "vs_tree_kv_commit": vs.KVDesc}


@pytest.fixture
def record():
    """Every call's address replaced by a function that keeps its arguments."""
    seen, keep, ctypes_of = [], [], {}
    for name in binding._NATIVE:
        types = getattr(vs.lib(), name).argtypes
        plain = [VP if i == 0 and name in STRUCTS else t for i, t in enumerate(types)]

        def body(*a, name=name):
            seen.append((name, a))
            return 41
        cb = ctypes.CFUNCTYPE(I32, *plain)(body)
        address = ctypes.cast(cb, VP).value
        keep.append(cb)
        ctypes_of[name] = address, ctypes.CFUNCTYPE(I32, *types)(address)
    binding._native.bind({name: a for name, (a, _) in ctypes_of.items()})
    yield seen, {name: f for name, (_, f) in ctypes_of.items()}
    binding._load_native()


def _outcome(seen, call):
    del seen[:]
    try:
        assert call() == 41
    except Exception as e:
        assert not seen
        return type(e)
    (name, args), = seen
    return [0 if a is None else a for a in args]


@pytest.mark.parametrize("name", binding._NATIVE)
def test_same_arguments_as_ctypes(record, name):
    seen, functions = record
    types = getattr(vs.lib(), name).argtypes
    struct = STRUCTS.get(name)
    good = [struct(B=2) if i == 0 and struct else 1.0 if t is F32 else 16 * i for i, t in enumerate(types)]

    def through_ctypes(args):
        return functions[name](*[ctypes.byref(a) if i == 0 and struct else binding._ptr(a) if t is VP else a for i, (t, a) in enumerate(zip(types, args))])
    for i in range(len(types)):
        for v in VALUES:
            if isinstance(v, str) and types[i] is VP:
                continue                                          # the address of a temporary
            args = good[:i] + [v] + good[i + 1:]
            want = _outcome(seen, lambda: through_ctypes(args))
            got = _outcome(seen, lambda: getattr(vs, name)(*args))
            assert got == want, (i, types[i].__name__, v)


def test_names_defaults_and_counts(record):
    seen, _ = record
    assert vs.vs_tree_mask_build(16, 1, 2, mask=32, depth=48) == 41
    assert [0 if a is None else a for a in seen[-1][1]] == [16, 1, 2, 32, 48, 0, 0]
    for args, kw in (((16, 1, 2, 32), {}), ((1,) * 8, {}), ((16, 1, 2, 32, 48), {"mask": 5}), ((16, 1, 2, 32, 48), {"other": 5})):
        with pytest.raises(TypeError):
            vs.vs_tree_mask_build(*args, **kw)

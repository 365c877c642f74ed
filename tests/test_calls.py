"""The callables of csrc/calls.c against ctypes: results, arguments that are refused, integers of more bits than the parameter."""
import ctypes as C
import importlib.machinery
import os

import numpy as np
import pytest
import torch

from paper_2406_02629_amd import binding

LIB = binding.load_library(binding.P61)


def bound(name):
    fn = getattr(LIB, name)
    pointers = sum(1 << i for i, kind in enumerate(fn.argtypes) if kind not in (C.c_int, C.c_size_t, C.c_uint64))
    return fn, binding._calls.bind(C.cast(fn, C.c_void_p).value, len(fn.argtypes), pointers)


@pytest.mark.parametrize("args", [(28, 2, 2, 0), (7, 3, 2, 1), (2, 3, 1, 0), (28 + (1 << 32), 2, 2, 0), (-1, 2, 2, 0), (True, 1, 1, 0)])
def test_integers(args):
    fn, call = bound("ssnet_pool_out_size")
    assert call(*args) == fn(*args)


class Index:
    def __index__(self):
        return 28


class Parameter:
    _as_parameter_ = 28


@pytest.mark.parametrize("value", [np.int64(28), np.uint8(28), np.int64(28 - (1 << 32)), torch.tensor(28), torch.tensor([28]), C.c_int(28), Index(), Parameter()])
def test_other_integers_as_by_ctypes(value):
    fn, _ = bound("ssnet_pool_out_size")
    call = binding._calls.bind(C.cast(fn, C.c_void_p).value, 4, 0, fn)
    assert call(value, 2, 2, 0) == fn(value, 2, 2, 0) == 14


@pytest.mark.parametrize("value", [28.0, np.float64(28), "28", b"28", None, torch.tensor(28.0), torch.tensor([28, 28]), C.c_long(28), C.c_void_p(28), [28]])
def test_refused_by_both(value):
    fn, _ = bound("ssnet_pool_out_size")
    for call in (fn, binding._calls.bind(C.cast(fn, C.c_void_p).value, 4, 0, fn)):
        with pytest.raises(C.ArgumentError):
            call(value, 2, 2, 0)


@pytest.mark.parametrize("name", binding._Entries.NAMES)
def test_entries_take_what_ctypes_takes(name):
    """null pointers in ctypes' forms and integers of numpy at every place: no launch"""
    fn = getattr(LIB, "ssnet_" + name)
    args = [kind(1) if kind in (C.c_int, C.c_size_t, C.c_uint64) else kind() for kind in fn.argtypes]
    assert getattr(LIB.entries, name)(*args) == fn(*args) == binding.EINVAL
    args = [np.int64(1) if kind in (C.c_int, C.c_size_t, C.c_uint64) else None for kind in fn.argtypes]
    assert getattr(LIB.entries, name)(*args) == fn(*args) == binding.EINVAL
    with pytest.raises(TypeError):
        getattr(LIB.entries, name)(*args[:-1])


@pytest.mark.parametrize("args", [(28, 2, 2, 0.0), ("28", 2, 2, 0), (28, None, 2, 0), (28, 2, 2, b"0")])
def test_refused_as_by_ctypes(args):
    for call in bound("ssnet_pool_out_size"):
        with pytest.raises(C.ArgumentError):
            call(*args)


def test_count_of_arguments():
    for call in bound("ssnet_pool_out_size"):
        with pytest.raises(TypeError):
            call(28, 2, 2)
    with pytest.raises(TypeError):
        bound("ssnet_pool_out_size")[1](28, 2, 2, pad=0)


@pytest.mark.parametrize("name", binding._Entries.NAMES)
def test_null_pointers_come_back_as_an_error(name):
    """every argument's place, from the first to the sixteenth, is the one that ctypes gives it: no pointer, no launch"""
    fn, call = bound("ssnet_" + name)
    args = [1 if kind in (C.c_int, C.c_size_t, C.c_uint64) else None for kind in fn.argtypes]
    assert call(*args) == fn(*args) == getattr(LIB.entries, name)(*args) == binding.EINVAL


@pytest.mark.parametrize("count", [0, 1, 5, 6, 7, 10, 11, 12, 15, 16])
def test_places_of_arguments(count):
    """a callback that weighs its arguments by their place, at the edges of the calling forms"""
    kind = C.CFUNCTYPE(C.c_int, *[C.c_int] * count)
    seen = []
    entry = kind(lambda *a: seen.append(a) or -3)
    call = binding._calls.bind(C.cast(entry, C.c_void_p).value, count, 0)
    args = tuple((-1) ** i * (1000 + i) for i in range(count))
    assert call(*args) == -3 and seen == [args]


def test_more_arguments_than_there_are_places_for():
    with pytest.raises(ValueError):
        binding._calls.bind(1, 17, 0)


def test_module_is_named_after_its_interpreter():
    """an interpreter of another version finds no module of this one"""
    name = os.path.basename(binding._calls.__file__)
    assert name == "_calls" + importlib.machinery.EXTENSION_SUFFIXES[0] and name != "_calls.so"

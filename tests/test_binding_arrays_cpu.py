"""The binding's id lists and masks: every form that a caller may pass (lists,
tuples, ranges, arrays of any integer type, stride and writability) reaches the
library as the same numbers. And the current stream, which does not depend on a
private name of torch."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

rf = pytest.importorskip("paper_2606_06309_amd.binding")

WANT = [0, 2, 3, 7]


def _read(addr, ctype, n):
    return list((ctype * n).from_address(addr))


def _frozen(a):
    a.setflags(write=False)
    return a


IDS = {
    "list": lambda: list(WANT), "tuple": lambda: tuple(WANT), "iterator": lambda: iter(WANT),
    "int32": lambda: np.array(WANT, np.int32), "int64": lambda: np.array(WANT, np.int64),
    "uint8": lambda: np.array(WANT, np.uint8), "big_endian": lambda: np.array(WANT, ">i4"),
    "strided": lambda: np.repeat(np.array(WANT, np.int32), 2)[::2],
    "reversed": lambda: np.array(WANT[::-1], np.int32)[::-1],
    "read_only": lambda: _frozen(np.array(WANT, np.int32)),
    "unaligned": lambda: np.frombuffer(b"\0" + np.array(WANT, np.int32).tobytes(), np.int32, offset=1),
}


@pytest.mark.parametrize("form", sorted(IDS))
def test_ids(form):
    a, addr = rf._ids(IDS[form]())
    assert a.dtype == np.int32 and a.size == len(WANT) and addr % 4 == 0
    assert _read(addr, ctypes.c_int32, len(WANT)) == WANT


def test_ids_that_are_no_list():
    with pytest.raises(TypeError):
        rf._ids(np.array(3, np.int32))
    with pytest.raises(TypeError):
        rf._ids(3)
    assert rf._ids([])[0].size == 0 and rf._ids(range(2, 5))[0].tolist() == [2, 3, 4]


@pytest.mark.parametrize("mask", [[1, 0, 1], (True, False, True), np.array([1, 0, 1], np.uint8),
                                  np.array([True, False, True]), np.array([1, 9, 0, 9, 1, 9], np.uint8)[::2],
                                  np.array([1, 0, 1], np.int64)], ids=str)
def test_masks(mask):
    a = rf._array(mask, rf._U8)
    assert _read(rf._addr(a), ctypes.c_uint8, 3) == [1, 0, 1]


def test_an_array_that_fits_is_passed_without_a_copy():
    ids, mask = np.array(WANT, np.int32), np.array([1, 0], np.uint8)
    assert rf._ids(ids)[0] is ids and rf._array(mask, rf._U8) is mask


def test_the_current_stream_without_torchs_private_name():
    code = """
import torch
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream
torch.cuda.current_stream = lambda: type("Stream", (), {"cuda_stream": 1234})()
from paper_2606_06309_amd import binding
assert binding._stream(None) == 1234 and binding._stream(7) == 7
print("ok")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-2000:]

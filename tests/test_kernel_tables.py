"""Every shape that the bf16 recurrence of persist_rows_bf16.hip is compiled in is the plan of some width and batch (no GPU needed)."""
import ctypes
import os
import re

from paper_1901_10997_amd import binding as B
from paper_1901_10997_amd import build


class RowsPlan(ctypes.Structure):
    _fields_ = [("shape", ctypes.c_int), ("us", ctypes.c_double), ("rows", ctypes.c_int), ("groups", ctypes.c_int), ("gn", ctypes.c_int),
                ("xcd_local", ctypes.c_int), ("layers", ctypes.c_int), ("lds", ctypes.c_size_t)]


def _table(name):
    text = open(os.path.join(build.CSRC, "persist_rows_bf16.hip")).read()
    body = re.search(rf"const RowsShape {name}\[\] = \{{(.*?)\}};", text, re.S).group(1)
    return [tuple(int(v) for v in e.split(",")) for e in re.findall(r"R_[SK]\(([^)]*)\)", body)]


def _plan(symbol):
    f = getattr(B.load(), symbol)
    f.restype, f.argtypes = RowsPlan, [ctypes.c_int] * 3
    return f


BATCHES = list(range(2, 34)) + list(range(34, 130, 4)) + [160, 192, 224, 256, 384, 512]


def test_every_shape_of_one_layer_is_taken():
    plan, table = _plan("_ZN4l35522persist_rows_bf16_planEiii"), _table("kRowsShapes")
    seen = {plan(b, h, n).shape for h in range(5, 2049, 12) for b in BATCHES for n in (1, 2)} - {-1}
    assert seen == set(range(len(table))), [table[i] for i in set(range(len(table))) - seen]


def test_every_shape_of_a_stack_is_taken():
    plan, table = _plan("_ZN4l35528persist_rows_bf16_stack_planEiii"), _table("kStackShapes")
    seen = {plan(b, h, n).shape for h in range(5, 2049, 6) for b in BATCHES for n in range(2, 7)} - {-1}
    assert seen == set(range(len(table))), [table[i] for i in set(range(len(table))) - seen]

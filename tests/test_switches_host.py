"""The environment switches that include/ddg.h lists: the library knows each, and the workgroup count of the wide weight gradients
moves the plan, within its range only (host code, no GPU)."""
import ctypes as C
import itertools
import os
import re

import pytest

from paper_1804_10574_amd.ddg import load_library

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def listed():
    text = open(os.path.join(ROOT, "include", "ddg.h")).read()
    text = text[text.index("Environment"):text.index("None of them changes a result")]
    names = set()
    for word in re.findall(r"DDG_[A-Z0-9_]+(?:(?:/_[A-Z0-9]+)+|\[[A-Z0-9_/]+\])?", text):
        m = re.fullmatch(r"(DDG_[A-Z0-9_]+)\[(.*)\]", word)
        if m:
            names |= {m[1]} | {m[1] + s for s in m[2].split("/")}
        else:
            first, *more = word.split("/")
            names |= {first} | {first[:first.rindex("_")] + s for s in more}
    return names - {"DDG_ERR_STATE"}


def test_every_listed_switch_is_read():
    names = listed()
    assert {"DDG_NO_WGRAD_XCD", "DDG_TUNE_WGRAD_WIDE_WGS", "DDG_TUNE_CONV_GRID_C64", "DDG_TUNE_WGRAD_ROWS_C16"} <= names
    csrc = os.path.join(ROOT, "paper_1804_10574_amd", "csrc")
    read = set(re.findall(r'"(DDG_(?:NO|TUNE|CHECK)_[A-Z0-9_]+)"', "".join(open(os.path.join(csrc, f)).read() for f in os.listdir(csrc))))
    assert read == names


class Plan(C.Structure):       # WgradWidePlan
    _fields_ = [("M", C.c_int), ("Cin", C.c_int), ("Cout", C.c_int), ("R", C.c_int), ("splits", C.c_int), ("launch", C.c_bool)]


class Vector(C.Structure):     # std::vector of them: begin, end, end of storage
    _fields_ = [(n, C.c_void_p) for n in ("begin", "end", "cap")]


def plan(layers):
    a = (Plan * len(layers))(*(Plan(*l, 0, False) for l in layers))
    at = C.addressof(a)
    v = Vector(at, at + C.sizeof(a), at + C.sizeof(a))
    load_library()._ZN3ddg15wgrad_wide_planERSt6vectorINS_13WgradWidePlanESaIS1_EE(C.byref(v))
    assert (v.begin, v.end) == (at, at + C.sizeof(a))
    return [(p.splits, p.launch) for p in a]


LAYERS = [(6272, 256, 1024, 1), (6272, 256, 256, 3), (6272, 1024, 256, 1)] * 7      # (pixels, input channels, output channels, kernel)


def launches(layers, got):
    """Workgroups of each launch."""
    out = [0]
    for (_, ci, co, r), (splits, last) in zip(layers, got):
        out[-1] += ci // 128 * (co // 128) * r * r * splits
        if last:
            out.append(0)
    assert out[-1] == 0
    return out[:-1]


@pytest.mark.parametrize("wgs,limit", [(None, 512), ("64", 64), ("2048", 2048), ("63", 512), ("2049", 512), ("many", 512)])
def test_workgroups_of_a_wide_weight_gradient_launch(wgs, limit, monkeypatch):
    monkeypatch.delenv("DDG_TUNE_WGRAD_WIDE_WGS", raising=False)
    usual = plan(LAYERS)
    if wgs is not None:
        monkeypatch.setenv("DDG_TUNE_WGRAD_WIDE_WGS", wgs)
    got = plan(LAYERS)
    w = launches(LAYERS, got)
    alone = max(ci // 128 * (co // 128) * r * r * 2 for _, ci, co, r in LAYERS)      # (98 steps in slices of 49: two at least)
    assert max(w) <= max(limit, alone)
    assert (got == usual) == (limit == 512)
    if limit == 64:
        assert len(w) > len(launches(LAYERS, usual))
    if limit == 2048:
        assert max(w) > 512 and len(w) < len(launches(LAYERS, usual))


@pytest.mark.parametrize("pixels,channels", itertools.product([1, 64, 65, 6272, 50176], [128, 512, 2048]))
def test_every_slice_has_a_step(pixels, channels, monkeypatch):
    for wgs in ("64", "2048"):
        monkeypatch.setenv("DDG_TUNE_WGRAD_WIDE_WGS", wgs)
        (splits, last), = plan([(pixels, channels, channels, 1)])
        assert last and 1 <= splits <= (pixels + 63) // 64

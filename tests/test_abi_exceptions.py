"""No C++ exception crosses the C ABI (stated in include/wfst.h): every entry
point of the HIP library that returns a code is a function try block that ends
in the guard which turns exceptions into codes, and the guard covers all of
them.  (Host allocations that fail cannot be forced in a running library, so
the source is checked.)"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _read(*p):
    with open(os.path.join(ROOT, *p)) as f:
        return f.read()


def test_every_entry_point_is_guarded():
    declared = set(re.findall(r"^int (wfst_\w+)\(", _read("include", "wfst.h"), re.M))
    src = _read("paper_1701_03038_amd", "csrc", "wfst_api.hip")
    src = src[src.index('extern "C" {'):]
    defined = {m.group(1): m.end() for m in re.finditer(r"^int (wfst_\w+)\(", src, re.M)}
    assert declared - set(defined) == {"wfst_att_parse"}  # host code of its own (att.cpp)
    assert "wfst_viterbi" in defined
    for name, at in defined.items():
        start = src.index("\ntry {\n", at)
        assert "\n}" not in src[at:start], f"{name} is no function try block"
        assert src[src.index("\n}\n", start):].startswith("\n}\nC_GUARD\n"), f"{name} does not end in the guard"


def test_the_guard_catches_everything():
    src = _read("paper_1701_03038_amd", "csrc", "wfst_api.hip")
    guard = src[src.index("#define C_GUARD"):]
    guard = guard[:guard.index("\n\n")]
    assert "catch (const std::bad_alloc &)" in guard and "catch (...)" in guard
    att = _read("paper_1701_03038_amd", "csrc", "att.cpp")
    assert "catch (const std::bad_alloc &)" in att or "catch (...)" in att

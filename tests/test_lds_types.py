"""How the kernels' sources read and write LDS arrays (no GPU needed): one that is accessed several values at a time says
so in its alignment, and none is read as another type than it was written as (the compiler may take two such
accesses for unrelated ones).  (Dynamic LDS, declared as 16-byte words, is raw storage and left out.)"""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_09244_amd", "csrc")
VECTOR = re.compile(r"(float|double|int|uint)([24])$")
WORD = {"uint32_t": "uint", "int32_t": "int", "unsigned": "uint"}


def lds_arrays(src):
    """{name: (element type, stated alignment)} of the static LDS arrays of a source."""
    found = {}
    for m in re.finditer(r"^\s*__shared__ (?:alignas\((\d+)\) )?(\w+) ([^;]*);", src, re.M):
        for name in re.findall(r"(\w+)\s*\[", re.sub(r"\[[^\]]*\]", "[]", m.group(3))):
            found[name] = (m.group(2), int(m.group(1) or 0))
    return found


def lds_casts(src):
    """(array name, type that it is accessed as) of every cast of one."""
    return re.findall(r"reinterpret_cast<(?:const )?(\w+)\s*\*>\(&?(\w+)", src)


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))), ids=os.path.basename)
def test_wide_accesses_are_aligned(path):
    src = open(path).read()
    arrays = lds_arrays(src)
    for as_type, name in lds_casts(src):
        wide = VECTOR.match(as_type)
        if name in arrays and wide:
            element, aligned = arrays[name]
            assert WORD.get(element, element) == wide.group(1), (name, element, as_type)
            assert aligned >= int(wide.group(2)) * (8 if element == "double" else 4), (name, as_type)


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))), ids=os.path.basename)
def test_no_array_is_accessed_as_another_type(path):
    src = open(path).read()
    arrays = lds_arrays(src)
    for as_type, name in lds_casts(src):
        if name in arrays and as_type not in ("uint8_t", "char"):
            assert VECTOR.match(as_type) or as_type == arrays[name][0], (name, arrays[name][0], as_type)

"""Kernels address no LDS array through a pointer of another type, unless that
type may alias it: under strict aliasing the compiler may move accesses of one
type past accesses of another, for instance counters' loads up past the loop
that clears them.  (Arenas are arrays of bytes, which any type may alias.)"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_02752_amd", "csrc")
MAY_ALIAS = {"lds_word", "unsigned char", "char"}


def punned(source):
    """(array, its type, the type it is addressed as) of each such use."""
    arrays = {}
    for kind, names in re.findall(r"__shared__\s+(?:__align__\(\d+\)\s+)?([\w ]+?)\s+(\w+\s*\[[^;]*);", source):
        for name in re.findall(r"(\w+)\s*\[", names):
            arrays[name] = kind
    found = []
    for kind, name in re.findall(r"reinterpret_cast<\s*(?:const\s+)?([\w ]+?)\s*(?:\*|\(\*\)[^>]*)>\(\s*&?(\w+)", source):
        own = arrays.get(name)
        # (signed and unsigned of one width may alias)
        if own and own not in MAY_ALIAS and kind.lstrip("u") != own.lstrip("u") and kind not in MAY_ALIAS:
            found.append((name, own, kind))
    return found


def test_the_check_sees_a_punned_clear():
    src = "__shared__ uint16_t s_cnt[4][8];\n reinterpret_cast<uint32_t*>(s_cnt[w])[i] = 0u;"
    assert punned(src) == [("s_cnt", "uint16_t", "uint32_t")]
    assert punned(src.replace("uint32_t*", "lds_word*")) == []


@pytest.mark.parametrize("name", sorted(n for n in os.listdir(CSRC) if n.endswith((".hip", ".h"))))
def test_lds_arrays_keep_their_type(name):
    with open(os.path.join(CSRC, name)) as f:
        assert punned(f.read()) == []

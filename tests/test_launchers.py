"""Kernel launchers of the native library: every one declared is called by another function (no GPU)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1306_3159_amd", "csrc")


def test_every_launcher_has_a_caller():
    def text(name):
        return re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())

    declared = set(re.findall(r"\b(launchb?_\w+)\s*\(", text("launch.hpp")))
    assert len(declared) > 50
    code = "".join(text(f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip"))
    code = re.sub(r"#define BRD_\w+_INST.*?#undef BRD_\w+_INST", "", code, flags=re.S)
    # definitions and explicit instantiations start with their return type
    code = re.sub(r"\b(?:void|unsigned|bool|int)\s+launchb?_\w+", "", code)
    called = set(re.findall(r"\b(launchb?_\w+)\s*(?:<[^;(]*>)?\s*\(", code))
    assert declared - called == set()

"""Pinned host memory that a running kernel writes while the host reads it (or
the reverse) must be asked for as coherent by name: with other flags alone the
runtime decides by its environment, and neither the time at which a value
becomes visible nor the order of two of them is then given.  The library
holds no other pinned memory."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_06744_amd", "csrc")


def test_pinned_memory_is_asked_for_as_coherent():
    found = 0
    for name in sorted(os.listdir(CSRC)):
        src = open(os.path.join(CSRC, name)).read()
        for m in re.finditer(r"hipHostMalloc\(([^;]*?)\)\s*(?:;|!=|==)", src):
            found += 1
            flags = m.group(1).split(",")[-1]
            assert "hipHostMallocCoherent" in flags or "kPinnedFlags" in flags, f"{name}: {m.group(0)}"
        for m in re.finditer(r"kPinnedFlags\s*=\s*([^;]*);", src):
            assert "hipHostMallocCoherent" in m.group(1) and "NonCoherent" not in m.group(1), name
        assert "hipHostRegister" not in src, name
    assert found >= 3

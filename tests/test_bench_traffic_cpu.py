"""The M2L's HBM traffic in bench.py is tied to the sources it was measured on:
every header with device code that the M2L kernel file includes counts."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_2508_02626_amd", "csrc")


def _headers(name, seen):
    for h in re.findall(r'#include "([^"]+)"', open(os.path.join(CSRC, name)).read()):
        if h not in seen and os.path.exists(os.path.join(CSRC, h)):
            seen.add(h)
            _headers(h, seen)
    return seen


def test_traffic_sources_cover_the_device_code():
    sources = {os.path.basename(f) for f in bench.M2L_SOURCES}
    assert {"m2l.hip", "m2l_tiles.hip"} <= sources
    for h in _headers("m2l.hip", set()):
        # (launch declarations and host rules carry no device code of the kernel)
        if re.search(r"^(template.*)?\s*__device__", open(os.path.join(CSRC, h)).read(), re.M):
            assert h in sources, h


def test_traffic_figures_share_the_fingerprint():
    assert len({e["fingerprint"] for e in bench.M2L_TRAFFIC.values()}) == 1
    assert all(e["bytes"] > 0 for e in bench.M2L_TRAFFIC.values())

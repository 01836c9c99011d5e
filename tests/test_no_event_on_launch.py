"""dawn_sssp_noalloc creates nothing at run time, so nothing that a launch passes
through may create an event: the device's gate event is made with the other
per-device objects (dev_info).  The rest of the host code creates events for the
kernel timer and for captures only."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2306_07872_amd", "csrc")


def _creators(name):
    """Names of the functions of a source file that create events."""
    text = open(os.path.join(CSRC, name)).read()
    text = re.sub(r"//[^\n]*", "", text)
    heads = [(m.start(), m.group(1)) for m in
             re.finditer(r"^[A-Za-z_][^\n;{}=]*?([\w:~]+)\([^;{}]*\)[^;{}]*\{", text, re.M)]
    out = set()
    for m in re.finditer(r"hipEventCreate\w*\s*\(", text):
        out.add([n for p, n in heads if p < m.start()][-1])
    return out


def test_events_are_created_off_the_launch_path():
    assert _creators("govm_sssp.hip") == set() and _creators("govm_tile.hip") == set()
    found = _creators("dawn_api.hip")
    assert "dev_info" in found
    assert found <= {"dev_info", "ktimer_begin", "ktimer_end", "dawn_kernel_timer", "dawn_batch_capture",
                     "dawn_tile_capture"}, found

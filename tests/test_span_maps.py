"""The map of a launch in spans (csrc/pgcm_spans.h, map_spans), driven natively under sanitizers: where the
workgroups' packets lie and whose key they use, for 1 to 256 keys and lists on either side of what fits."""
import os

from test_sanitized_host_code import NATIVE, ROOT, _build_and_run


def test_maps_of_batches():
    out = _build_and_run("g++", [os.path.join(NATIVE, "span_map_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    words = out.replace(",", "").split()
    total, placed, mapped = int(words[1]), int(words[4]), int(words[7])
    assert total == 126 and 0 < placed < total and mapped == 42, out

"""The steps by which the workgroups of a chunk add up its tag and agree on a verdict (csrc/pgcm_arrive.h), run on
the CPU in every order for two and three workgroups and in thousands of random ones for up to 256: on the
GPU one workgroup mostly completes all four words, and that different ones do is a matter of timing."""
import os

from test_sanitized_host_code import NATIVE, ROOT, _build_and_run


def test_every_order_of_arrival():
    out = _build_and_run("g++", [os.path.join(NATIVE, "arrive_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    ends = [int(v.rstrip(",:")) for v in out.split() if v.rstrip(",:").isdigit()]
    assert ends[0] > 400000 and all(n > 100 for n in ends[1:]), out    # each way of ending was met

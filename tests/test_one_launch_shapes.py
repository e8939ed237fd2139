"""How batches of few chunks are cut for one launch (csrc/pgcm_one_launch.h), driven natively under
AddressSanitizer and UndefinedBehaviorSanitizer over thousands of random batches: the number of passes
of a workgroup and what its chunk's first has to spare are the first that fit of all there are, tried in
turn with plain divisions; and they are found by going over the chunks seven times at most, since a call's
host time is part of it (31 times once, 30 us of it for 256 chunks)."""
import os

from test_sanitized_host_code import NATIVE, ROOT, _build_and_run


def test_shapes_of_random_batches():
    out = _build_and_run("g++", [os.path.join(NATIVE, "shape_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    assert out.startswith("batches 20000:"), out
    assert int(out.split("chunks gone over ")[1].split()[0]) <= 7, out

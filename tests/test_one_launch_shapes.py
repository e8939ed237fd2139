"""How batches of few chunks are cut for one launch (csrc/pgcm_one_launch.h), driven natively under
AddressSanitizer and UndefinedBehaviorSanitizer over thousands of random batches: the number of passes
of a workgroup and what its chunk's first has to spare are the first that fit of all there are, tried in
turn with plain divisions; and they are found by going over the chunks seven times at most, since a call's
host time is part of it (31 times once, 30 us of it for 256 chunks)."""
import os
import subprocess

from test_sanitized_host_code import NATIVE, ROOT, _build_and_run


def test_shapes_of_random_batches():
    out = _build_and_run("g++", [os.path.join(NATIVE, "shape_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    assert out.startswith("batches 20000:"), out
    assert int(out.split("chunks gone over ")[1].split()[0]) <= 7, out


def test_which_sweeps_are_written_through():
    """the last of those that every workgroup makes: the others' stores are ahead of the next one's payload, which would
    wait for them to reach host memory; and none where only the chunks' first workgroups make more than one"""
    code = """
#include "pgcm_types.h"
constexpr bool only_the_last(uint32_t passes) {
    const uint32_t sweeps = (passes + pgcm::kFoldPasses - 1) / pgcm::kFoldPasses;
    for (uint32_t s = 0; s < sweeps; ++s)
        if (pgcm::sweep_through(passes, s, sweeps) != (s + 1 == sweeps)) return false;
    return true;
}
static_assert(only_the_last(5) && only_the_last(8) && only_the_last(9) && only_the_last(pgcm::kSweptPasses));
static_assert(!pgcm::sweep_through(4, 0, 2) && !pgcm::sweep_through(4, 1, 2) && !pgcm::sweep_through(4, 0, 1));
"""
    out = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-x", "c++", "-",
                          "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")], input=code,
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout

"""The cutter of batches into spans (csrc/pgcm_spans.h), driven natively under AddressSanitizer and
UndefinedBehaviorSanitizer with arrays of exactly the sizes the host side allots, over thousands of
random batches: of one key and of several, on whole devices and on partitions of one to 304 compute
units.  Checked is what the kernel assumes of its descriptors: every row belongs to one wavefront of
one workgroup of its chunk's key, no workgroup is without a wavefront and no wavefront without a
row, a chunk's parts and slots are consecutive and name their wavefronts, the part a wavefront
starts with is found by its row, and every distance to a chunk's end has a power of H."""
import os

from test_sanitized_host_code import NATIVE, ROOT, _build_and_run


def test_spans_of_random_batches():
    out = _build_and_run("g++", [os.path.join(NATIVE, "span_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    assert out.startswith("batches 6121,"), out

"""The map of a launch in spans (csrc/pgcm_spans.h, map_spans), driven natively under sanitizers: where the
workgroups' packets lie and whose key they use, for 1 to 256 keys and lists on either side of what fits."""
import os
import subprocess

import numpy as np

import test_gpu_span_maps
from test_sanitized_host_code import ENV, NATIVE, ROOT, SAN, _build_and_run


def test_maps_of_the_gpu_tests(tmp_path):
    """the longest list, and whether packets have their places in the map and keys their tables"""
    exe = str(tmp_path / "driver")
    subprocess.run(["g++"] + SAN + ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc"),
                                    os.path.join(NATIVE, "span_map_driver.cpp"), "-o", exe], check=True)
    lines = []
    for shape in test_gpu_span_maps.SHAPES.values():
        lens, keys, cycle, _ = shape(np.random.default_rng(1))
        lines.append("%d " % len(keys) + " ".join("%d 69 %d" % (n, min(i % cycle, len(keys) - 1))
                                                  for i, n in enumerate(lens)))
    out = subprocess.run([exe, "batches"], input="\n".join(lines) + "\n", stdout=subprocess.PIPE, check=True,
                         text=True, env=ENV).stdout.split("\n")[:-1]
    got = dict(zip(test_gpu_span_maps.SHAPES, out))
    assert got.pop("keys_16").split()[1:] == ["placed", "keys"] and got.pop("keys_17").split()[1:] == ["placed"]
    assert got == {"list_31": "31 placed", "list_32": "32", "keys_list_31": "31 placed keys", "keys_list_36": "36 keys"}


def test_maps_of_batches():
    out = _build_and_run("g++", [os.path.join(NATIVE, "span_map_driver.cpp")],
                         ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")])
    words = out.replace(",", "").split()
    total, placed, mapped = int(words[1]), int(words[4]), int(words[7])
    assert total == 126 and 0 < placed < total and mapped == 42, out

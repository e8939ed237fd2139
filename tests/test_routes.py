"""The batches of the GPU tests go to the kernels that those tests name: the library's own rules
(csrc/pgcm_routes.h), built for the CPU, say so for a device of 256 compute units.  Of burst_kernel the kind and
the passes of a chunk's first workgroup are told apart, of swap_kernel the bytes of a unit."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

import test_gpu_bursts
import test_gpu_graphs
import test_gpu_long_aad
import test_gpu_parity
import test_gpu_pipeline
import test_gpu_ragged_ends
import test_gpu_random_batches
import test_gpu_reservations
import test_gpu_short_calls
import test_gpu_units_in_one_launch
import test_zz_no_alloc
import workloads
from test_sanitized_host_code import ENV, NATIVE, ROOT, SAN


@pytest.fixture(scope="module")
def kernels_of(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "driver")
    build = subprocess.run(["g++"] + SAN + ["-std=c++17", "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc"),
                                            os.path.join(NATIVE, "route_driver.cpp"), "-o", exe],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout

    def run(batches, direction=None):
        """batches: (lengths, AAD lengths, forced unit bytes, one launch[, 1: fixed buffers, 2: captured, 3: on a
        stream that has no slots for short chunks, and whose context was captured]); direction "enc" or "dec": of what
        burst_kernel takes, its instance and the wavefronts of a workgroup that have blocks"""
        lines = []
        for lens, alens, unit_bytes, one_launch, *fixed in batches:
            lines.append("256 %d 0 %d %d " % (one_launch, unit_bytes, fixed[0] if fixed else 0) +
                         " ".join("%d %d" % (n, a) for n, a in zip(lens, alens)))
        out = subprocess.run([exe] + ([direction] if direction else []), input="\n".join(lines) + "\n", stdout=subprocess.PIPE,
                             stderr=subprocess.PIPE, text=True, env=ENV)
        assert out.returncode == 0, out.stderr
        return out.stdout.split("\n")[:-1]
    return run


def _of_workload(w, unit_bytes=0, one_launch=1):
    return w.lens, [len(w.aad_of(i)) for i in range(w.n)], unit_bytes, one_launch


def test_ragged_ends(kernels_of):
    expected = {"one launch, a pass": "words", "one launch, a row a wavefront": "fold 1",
                "one launch, sweeps": "sweep 5", "one launch, units": "swap 2048",
                "one launch, units as they go": "swap 8192", "a wavefront a chunk": "small",
                "spans": "span", "units": "bulk"}
    got = {}
    for path in test_gpu_ragged_ends.PATHS:
        w, unit_bytes, one_launch = test_gpu_ragged_ends.batch_of(path)
        got[path], = kernels_of([_of_workload(w, unit_bytes, one_launch)])
    assert got == expected


def test_bursts(kernels_of):
    shapes = test_gpu_bursts.SHAPES
    got = dict(zip(shapes, kernels_of([(lens, np.resize(alens, len(lens)), 0, 1)
                                       for lens, alens in shapes.values()])))
    # the most passes of a workgroup, a chunk's first
    most = {"passes_2": 3, "passes_3": 3, "passes_4": 3, "even_2": 2, "even_4": 4, "even_4_some": 4,
            "spare_1": 2, "spare_1_payload": 2, "spare_1_long_aad": 2, "spare_2": 3, "spare_3": 4,
            "spare_of_some": 3, "whole": 4, "whole_aad": 4, "whole_long_aad": 4,
            "one_4096": 4, "one_aad_2048": 4, "one_aad_4080": 4,
            **{n: 1 for n in shapes if n.startswith("fold_1")}}
    words = {"short", "short_aad", "long_aad", "aad_before", "aad_with_last", "two", "passes_1", "many_mixed"}
    sweeps = {"sweeps_2": 2, "sweeps_2_whole": 2, "sweeps_2_spare": 3, "sweeps_2_missing": 2,
              "sweeps_2_missing_2": 2, "sweeps_3": 3, "sweeps_4": 4, "sweeps_of_each": 4}
    for name, kernel in got.items():
        kind, passes = (kernel.split() + ["0"])[:2]
        if name in most:
            assert kernel == "fold %d" % most[name], (name, kernel)
        elif name in sweeps:
            assert kind == "sweep" and -(-int(passes) // 4) == sweeps[name], (name, kernel)
        elif name in words or name.startswith(("one_", "apart_", "spread_")):
            assert kernel == "words", (name, kernel)
        else:
            assert kind == "shared", (name, kernel)
    # short chunks have one workgroup each, as ever, where they are captured, in fixed buffers or go in units
    short = [shapes["spread_64_most"][0], [0] * 32]
    assert kernels_of([(*short, 0, 1, 3), (*short, 0, 1, 2), (*short, 0, 1, 1), (*short, 0, 0)]) == ["fold 4"] * 4
    aad = [0, 5, 1024, 4096, 4097, 8192], [1008, 1024, 1025, 16, 3000, 1008]
    assert kernels_of([(*aad, 0, 1, 2), (*aad, 0, 1, 1)]) == ["fold 4"] * 2
    # ... and more than 256 of them where their slots would be cleared by a launch of its own
    apart = [shapes["many_apart_512"][0], [0] * 406]
    assert kernels_of([(*apart, 0, 1, 2), (*apart, 0, 1, 3), (*apart, 0, 1, 1)]) == ["shared apart"] + ["shared"] * 2
    assert {got[n] for n in ("many_even", "many_long")} == {"shared"}
    assert {got[n] for n in ("many_apart", "many_apart_512")} == {"shared apart"} and got["many_apart_513"] == "shared"


def test_burst_instances(kernels_of):
    """which instance of burst_kernel takes a batch, where that goes by the workgroups of a compute unit or by the direction"""
    for n, shape in ((n, s) for n in (1, 64, 65, 255, 256, 257, 512) for s in test_gpu_bursts.MORE):
        lens, alens, waves = test_gpu_bursts.more(n, shape)
        for direction in ("enc", "dec"):
            got, = kernels_of([(lens, alens, 0, 1)], direction)
            assert got == "%s %d" % ("words" if n <= 256 else "words_shared", waves), (n, shape, got)
    for name, (lens, alens) in test_gpu_bursts.APART.items():
        batch = [(lens, np.resize(alens, len(lens)), 0, 1)]
        assert kernels_of(batch, "dec") == ["fold_apart 16"] and kernels_of(batch, "enc") == ["fold 16"], name
        spare = "spare" in name
        assert kernels_of(batch) == ["fold %d" % (3 if spare else 2)], name
    passes = {name: kernels_of([(*test_gpu_bursts.SHAPES[name], 0, 1)], "dec") for name in ("fold_1_most", "passes_3")}
    assert passes == {"fold_1_most": ["fold 16"], "passes_3": ["fold 16"]}
    # what goes through the pipe and its receiver with the IV in the arguments: one chunk of each kind that there is
    sizes = [([n], [0], 0, 1) for n in test_gpu_pipeline.IN_ARGUMENTS]
    assert kernels_of(sizes, "enc") == ["words 4", "words 8", "fold 16", "fold 16", "sweep 16"]
    assert kernels_of(sizes, "dec") == ["words 4", "words 8", "fold 16", "fold_apart 16", "sweep 16"]


def test_units_in_one_launch(kernels_of):
    for name, (lens, alens, unit_bytes, _, _) in test_gpu_units_in_one_launch.SHAPES.items():
        got, = kernels_of([(lens, np.resize(alens, len(lens)), unit_bytes, 1)])
        assert got == "swap %d" % (unit_bytes or (16384 if name.startswith("whole") else 8192)), name


def test_units_or_spans(kernels_of):
    """sixteen rows a unit for a batch of 7.5 rows a wavefront and more, if eight wavefronts a workgroup do"""
    kib = 1024
    got = kernels_of([([128 * kib] * n, [0] * n, 0, 1) for n in (256, 241, 228, 140)] +
                     [([2048 * kib] * 16, [0] * 16, 0, 1), ([2048 * kib] * 16, [16] * 16, 0, 1),
                      ([33 << 20], [0], 0, 1)])
    assert got == ["swap 16384", "swap 16384", "span", "span", "swap 16384", "span", "span"], got


def test_random_batches(kernels_of):
    ways = test_gpu_random_batches.WAYS
    for way, (seeds, unit_bytes, one_launch, kinds) in ways.items():
        batches = [_of_workload(test_gpu_random_batches._random_workload(s)[0], unit_bytes, one_launch)
                   for s in seeds]
        assert {k.split()[0] for k in kernels_of(batches)} == set(kinds.split()), way


def test_captured_and_reserved_batches(kernels_of):
    expected = {"alone": "fold", "one_launch": "fold", "one_launch_staged": "shared", "spans": "span",
                "spans_uploaded": "span", "one_row": "small", "units": "bulk", "one_launch_units": "swap"}
    for name, (lens, unit_bytes) in test_gpu_graphs.SHAPES.items():
        lens = lens(np.random.default_rng([workloads.BASE_SEED, 5040, len(name)]))
        got, = kernels_of([(lens, [20] * len(lens), unit_bytes, 1, 2)])
        assert got.split()[0] == expected[name], (name, got)
    expected = {"one_launch": "sweep", "spans_few": "span", "spans_host": "span", "spans_uploaded": "span",
                "one_row": "small"}
    for name, lens in test_gpu_reservations.SHAPES.items():
        lens = lens(np.random.default_rng([workloads.BASE_SEED, 8128, len(name)]))
        got, = kernels_of([(lens, [20] * len(lens), 0, 1)])
        assert got.split()[0] == expected[name], (name, got)


def test_short_calls(kernels_of):
    got = [kernels_of([(lens, [20] * len(lens), 0, 1, where)
                       for lens in test_gpu_short_calls.SHORT + [test_gpu_short_calls.MANY]]) for where in range(4)]
    whole = ["fold 4"] * 4 + ["shared"]
    assert got == [["words"] * 4 + ["shared apart"], whole, ["fold 4"] * 4 + ["shared apart"], whole], got


def test_batches_in_fixed_buffers(kernels_of):
    got = kernels_of([_of_workload(w) + (True,) for w in test_zz_no_alloc._batches()])
    assert got == ["bulk", "swap 8192", "words", "fold 4"], got


def test_long_aad(kernels_of):
    for lens, unit_bytes, one_launch, kernel in test_gpu_parity.LONG_AAD:
        got, = kernels_of([(lens, test_gpu_parity._long_aad_lens(len(lens)), unit_bytes, one_launch)])
        assert got.split()[0] == kernel, (lens[:4], got)


def test_long_aad_in_every_place(kernels_of):
    shapes = test_gpu_long_aad.SHAPES
    got = kernels_of([(lens, np.resize(test_gpu_long_aad.AADS, len(lens)), unit_bytes, one_launch)
                      for lens, unit_bytes, one_launch, _ in shapes.values()])
    assert dict(zip(shapes, got)) == {name: s[3] for name, s in shapes.items()}


def test_what_a_launch_says_of_itself():
    """every field of the word is what was put in, whatever the others are: above all, only a launch that has its IV in
    place says so, and none whose descriptors are staged, which has no chunks in its arguments either"""
    code = """
#include <initializer_list>
#include "pgcm_types.h"
using namespace pgcm;
bool all() {
    for (uint32_t chunks : {0u, 1u, 64u})
        for (uint32_t power : {1u, 16u})
            for (uint32_t waves : {2u, 4u})
                for (uint32_t groups : {1u, 512u})
                    for (uint32_t rounds : {10u, 12u, 14u})
                        for (uint32_t bits = 0; bits < 8; ++bits) {
                            const bool each = bits & 1, order = bits & 2, iv = bits & 4;
                            const SwapMeta m = swap_meta(chunks, power, waves, each, order, groups, rounds, iv);
                            if (m.nchunks() != chunks || m.unit_power() != power || m.wave_power() != waves ||
                                m.groups() != groups || m.rounds() != rounds || m.one_group_each() != each ||
                                m.in_order() != order || m.iv_in_place() != iv)
                                return false;
                        }
    return true;
}
int main() { return all() && !swap_meta(0, 1, 2, true, true, 65, 14).iv_in_place() ? 0 : 1; }
"""
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "meta")
        out = subprocess.run(["g++"] + SAN + ["-std=c++17", "-x", "c++", "-", "-o", exe,
                                              "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc")], input=code,
                             stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert out.returncode == 0, out.stdout
        assert subprocess.run([exe], env=ENV).returncode == 0

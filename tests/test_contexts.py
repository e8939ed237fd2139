"""Which of a key's contexts a batch runs with (csrc/pgcm_contexts.h), driven natively by several host threads
under ThreadSanitizer: a call in progress shares nothing with the threads that choose meanwhile, no context
is taken from a call, and none is re-bound whose last batch nothing marks the end of."""
import os
import shutil
import subprocess

import pytest

from test_sanitized_host_code import NATIVE, ROOT


def test_threads_choose_contexts(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "driver")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread",
                            "-I" + os.path.join(ROOT, "paper_2411_03357_amd", "csrc"),
                            os.path.join(NATIVE, "context_driver.cpp"), "-o", exe],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if build.returncode != 0 and "tsan" in build.stdout.lower():
        pytest.skip("sanitizer runtime not available: " + build.stdout[-200:])
    assert build.returncode == 0, build.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True,
                         env=dict(os.environ, LD_PRELOAD=""), timeout=120)
    if "unexpected memory mapping" in run.stderr:
        pytest.skip("the sanitizer cannot lay out its memory on this kernel")
    assert run.returncode == 0, (run.returncode, run.stdout, run.stderr[-3000:])
    assert run.stdout.startswith("contexts "), run.stdout

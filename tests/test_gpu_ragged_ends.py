"""Last blocks of every length from 1 to 16 bytes, of the payload and, at every alignment, of the AAD,
on every kernel that reads and writes them in pieces: against the CPU oracle, bit for bit, the bytes
around a chunk untouched."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu

# chunks, bytes of their whole blocks, forced unit size, one launch; which kernel each takes:
# tests/test_routes.py
PATHS = {
    "one launch, a pass": (48, 16 * 20, 0, True),
    "one launch, a row a wavefront": (64, 16 * 900, 0, True),
    "one launch, sweeps": (64, 16 * 5000, 0, True),
    "one launch, units": (48, 16 * 700, 2048, True),
    "one launch, units as they go": (240, 16 * 7700, 0, True),
    "a wavefront a chunk": (528, 16 * 7, 0, True),
    "spans": (560, 16 * 700, 0, True),
    "units": (48, 16 * 700, 2048, False),
}


def batch_of(path):
    n, whole, unit_bytes, one_launch = PATHS[path]
    rng = np.random.default_rng([workloads.BASE_SEED, 1414, n])
    k = np.arange(n)
    lens = (whole + 1 + k % 16).astype(np.uint64)
    alens = 1 + (5 * k + k // 16) % 47
    offsets, total = workloads._layout(lens)
    aad_off = np.zeros(n + 1, np.uint64)
    aad_off[1:] = np.cumsum(alens)
    return workloads.Workload(path, 950, rng.integers(0, 256, 32, dtype=np.uint8),
                              workloads.iv_sequence(1 << 61, n), lens, offsets, total, "u8",
                              rng.integers(0, 256, int(alens.sum()), dtype=np.uint8),
                              aad_off), unit_bytes, one_launch


@pytest.mark.parametrize("path", PATHS)
def test_every_length_of_a_last_block(path):
    w, unit_bytes, one_launch = batch_of(path)
    # rejected by the last bit of a last block of 1, 7 and 15 bytes
    flips = [(i, int(w.lens[i]) - 1, 7, "ct") for i in (0, 6, 14)]
    _full_parity(w, flip=flips, unit_bytes=unit_bytes, one_launch=one_launch)

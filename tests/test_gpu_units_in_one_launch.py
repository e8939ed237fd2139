"""Batches that go to swap_kernel, as they go and with units of a forced size: every key length, IVs of one block
and of many, empty and ragged chunks, AAD of every kind, workgroups of four, eight and sixteen wavefronts,
descriptors as arguments and in pinned memory — against the CPU oracle, bit for bit.  (That they do go
there: tests/test_routes.py.)"""
import pytest

from test_gpu_bursts import _workload
from test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu

KIB, MIB = 1024, 1 << 20

# chunk lengths, AAD lengths in turn, bytes of a forced unit, of the key, of an IV
SHAPES = {
    "one": ([28 * 10**6 + 5], [40], 0, 32, 12),
    "a_layer": ([2 * MIB] * 14, [0], 0, 24, 40),
    "staged": ([123 * 1000 + 33 * (i % 16) for i in range(240)], [16, 0, 1024], 0, 16, 12),
    # units of sixteen rows, eight wavefronts: chunks without AAD that they cover to the block
    "whole": ([32 * MIB], [0], 0, 32, 12),
    "whole_staged": ([128 * KIB] * 255 + [128 * KIB - 15], [0], 0, 16, 40),
    "sixteen_wavefronts": ([7 * MIB + 100, 0, 50 * KIB], [0, 5, 33], 2048, 16, 60),
    "eight_wavefronts": ([3 * MIB - 11, 0, 50 * KIB, 9 * KIB - 1], [16, 0, 3000, 7], 2048, 24, 16),
    "four_wavefronts": ([70 * KIB + i for i in range(12)], [1008, 20, 0], 2048, 32, 1040),
    "four_rows": ([300 * KIB, 8193, 1, 0, 64 * KIB], [17, 0], 4096, 16, 8),
    "sixteen_rows": ([MIB + 16 * i + i % 3 for i in range(20)] + [9000], [0, 64], 16384, 16, 17),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_shapes(shape):
    lens, alens, unit_bytes, key_bytes, iv_bytes = SHAPES[shape]
    w = _workload(shape, lens, alens, key_bytes, iv_bytes)
    _full_parity(w, flip=[(i, 3, 1, "tag") for i in {0, w.n // 2}] if w.n > 1 else [], unit_bytes=unit_bytes)

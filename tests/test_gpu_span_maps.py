"""Launches in spans whose map names the tables of up to sixteen keys, and of more, which it does not; and lists of
chunks as long as a packet holds, and longer: bit for bit against the CPU oracle."""
import pytest

import test_gpu_spans

pytestmark = pytest.mark.gpu
KIB = 1024

SHAPES = {
    "keys_16": lambda r: (test_gpu_spans._even(r, 160, 40 * KIB, 400 * KIB), (32, 16, 24, 32) * 4, 16, 16),
    "keys_17": lambda r: (test_gpu_spans._even(r, 170, 40 * KIB, 400 * KIB), (32,) * 16 + (24,), 17, 12),
    # shares of some 300 rows, with neighbours of a row among them: lists of up to and of more than 31
    "list_24": lambda r: ([256 * KIB + 3] * 150 + [900] * 24 + [256 * KIB] * 150, (32,), 1, 12),
    "list_90": lambda r: ([256 * KIB + 3] * 150 + [900] * 90 + [256 * KIB] * 150, (24,), 1, 12),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_span_maps(shape, monkeypatch):
    monkeypatch.setitem(test_gpu_spans.SHAPES, shape, SHAPES[shape])
    test_gpu_spans.test_spans(shape)

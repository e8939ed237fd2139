"""Launches in spans whose map names the tables of up to sixteen keys, and of more, which it does not; and lists of
chunks as long as a packet holds, and longer, of one key and of two: bit for bit against the CPU oracle.  (What is
filled in of a shape's map: tests/test_span_maps.py.)"""
import pytest

import test_gpu_spans

pytestmark = pytest.mark.gpu
KIB = 1024


def _two_keys(run):
    """chunks of two keys in turn, the first one's with a run of short ones among them"""
    first = [256 * KIB + 3] * 100 + [900] * run + [256 * KIB] * 60
    return [v for pair in zip(first, [256 * KIB + 5] * len(first)) for v in pair]


SHAPES = {
    "keys_16": lambda r: (test_gpu_spans._even(r, 160, 40 * KIB, 400 * KIB), (32, 16, 24, 32) * 4, 16, 16),
    "keys_17": lambda r: (test_gpu_spans._even(r, 170, 40 * KIB, 400 * KIB), (32,) * 16 + (24,), 17, 12),
    # shares of some 300 rows, with neighbours of a row among them: lists of 31 at most and of more
    "list_31": lambda r: ([256 * KIB + 3] * 150 + [900] * 60 + [256 * KIB] * 150, (32,), 1, 12),
    "list_32": lambda r: ([256 * KIB + 3] * 150 + [900] * 62 + [256 * KIB] * 150, (24,), 1, 12),
    "keys_list_31": lambda r: (_two_keys(29), (32, 16), 2, 12),
    "keys_list_36": lambda r: (_two_keys(34), (16, 24), 2, 16),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_span_maps(shape, monkeypatch):
    monkeypatch.setitem(test_gpu_spans.SHAPES, shape, SHAPES[shape])
    test_gpu_spans.test_spans(shape)

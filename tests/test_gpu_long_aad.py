"""AAD of more blocks than go in lanes (64): its blocks but the last are hashed in rows of 64, by the wavefront
that has the block before the chunk's first, wherever in its pass or its sweep that is.  AAD lengths at the
edges of the rows, chunk lengths at the edges of rows and passes, on every kernel (tests/test_routes.py),
against the CPU oracle, bit for bit."""
import pytest

from test_gpu_bursts import _workload
from test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu

# 65 blocks: 64 whole ones and a byte, and whole; 66 and 67: the last but one begins a row, or is in it; two rows and three
AADS = [1025, 1040, 1041, 1056, 1057, 2049, 2080, 2081, 3000, 3105, 0, 5001]
# what a chunk's first pass may have, in blocks: "block -1" in every row of it, at both ends of each
FIRST = [0, 1, 62, 63, 64, 65, 127, 128, 191, 192, 254, 255]


def _lens(passes, n):
    return [16 * (256 * (passes - 1) + FIRST[i % len(FIRST)]) - 7 * (i % 2) for i in range(1, n + 1)]


# chunk lengths, forced unit size, one launch, and the kernel with the most passes of a workgroup
SHAPES = {
    "words": ([1, 16, 40, 1000, 2031, 0, 2032, 300, 17, 5, 64, 100], 0, True, "words"),
    "one": (_lens(3, 12), 0, True, "words"),
    "one of sixteen": (_lens(19, 12), 0, True, "fold 1"),
    "whole": (_lens(2, 72), 0, True, "fold 4"),
    "two": (_lens(3, 150), 0, True, "fold 3"),
    "four": (_lens(16, 48), 0, True, "fold 4"),
    "sweeps": (_lens(9, 130) + _lens(6, 100), 0, True, "sweep 9"),
    "shared": ([4000 + 16 * FIRST[i % 12] for i in range(400)], 0, True, "shared"),
    "units": (_lens(20, 24), 2048, True, "swap 2048"),
    "spans": (_lens(4, 300), 0, True, "span"),
    "as units": (_lens(4, 40), 1024, False, "bulk"),
    "a wavefront each": ([i % 1008 for i in range(0, 12000, 23)], 0, True, "small"),
}


@pytest.mark.parametrize("key_bytes,iv_bytes", [(32, 12), (16, 40)])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_and_places(shape, key_bytes, iv_bytes):
    lens, unit_bytes, one_launch, _ = SHAPES[shape]
    w = _workload(shape, lens, AADS, key_bytes, iv_bytes)
    _full_parity(w, flip=[(1, 3, 1, "tag")], unit_bytes=unit_bytes, one_launch=one_launch)

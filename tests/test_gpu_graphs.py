"""Batches captured into a graph after pgcm_reserve, whichever way they go, replayed between eager
batches of the same key and stream that go other ways and are of other sizes: what comes before the
first replay, every replay and what comes after it equal the CPU oracle's results, bit for bit."""
import numpy as np
import pytest
import torch

import workloads
from device_batch import DeviceBatch
from test_gpu_reservations import KIB, MIB, _encrypt_keys, _keys_batch, expected, workload

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

# chunk lengths of the captured batch; the size its units are forced to, or 0
SHAPES = {
    "alone": (lambda r: [4 * KIB, 0, 17, 1000], 0),
    "one_launch": (lambda r: [2 * MIB, 300 * KIB + 1], 0),
    "one_launch_staged": (lambda r: [int(v) for v in r.integers(1, 8 * KIB, 300)], 0),
    "spans": (lambda r: [int(v) for v in r.integers(200 * KIB, 450 * KIB, 60)], 0),
    "spans_uploaded": (lambda r: [int(v) for v in r.integers(1, 3 * KIB, 9000)], 0),
    "one_row": (lambda r: [int(v) for v in r.integers(0, 1009, 2000)], 0),
    "units": (lambda r: [int(v) for v in r.integers(KIB, 150 * KIB, 300)], 16 * KIB),
    "one_launch_units": (lambda r: [int(v) for v in r.integers(KIB, 900 * KIB, 40)], 16 * KIB),
}


class _Checked:
    def __init__(self, name, rng, lens, raw_key):
        ivs = rng.integers(0, 256, (len(lens), 12), dtype=np.uint8)
        self.w = workload(name, rng, lens, raw_key, ivs)
        host = self.w.payload_host()
        self.cipher, self.tags = expected(self.w, host)
        self.b = DeviceBatch(self.w, torch.from_numpy(host).cuda())

    def clear(self):
        for t in (self.b.cipher, self.b.tags, self.b.back, self.b.ok):
            t.zero_()

    def check(self, what):
        torch.cuda.synchronize()
        assert np.array_equal(self.b.cipher.cpu().numpy(), self.cipher), what
        assert np.array_equal(self.b.tags.cpu().numpy().reshape(-1, 16), self.tags), what
        assert bool((self.b.ok == 1).all()) and torch.equal(self.b.back, self.b.plain), what


@pytest.mark.parametrize("shape", SHAPES)
def test_captured_between_eager_batches(shape):
    rng = np.random.default_rng([workloads.BASE_SEED, 5040, len(shape)])
    raw_key = rng.integers(0, 256, 32, dtype=np.uint8)
    lens, unit = SHAPES[shape]
    graphed = _Checked("captured_" + shape, rng, lens(rng), raw_key)
    others = [_Checked("eager_spans", rng, [int(v) for v in rng.integers(1, 200 * KIB, 400)], raw_key),
              _Checked("eager_one_launch", rng, [MIB + 3] * 3, raw_key)]
    key = pgcm.expand_key(raw_key)
    stream = torch.cuda.Stream()

    def eager(k):
        # the first of them cut into units every other time
        pgcm.set_unit_bytes(key, 16 * KIB if k % 4 == 0 else 0)
        other = others[k % 2]
        other.b.encrypt(key, stream=stream)
        other.b.decrypt(key, stream=stream)
        pgcm.set_unit_bytes(key, 0)
        return other

    torch.cuda.synchronize()
    for k in range(4):                 # every staging buffer has been used
        eager(k)
    pgcm.set_unit_bytes(key, unit)
    pgcm.reserve(key, max(graphed.w.n, 400), graphed.w.payload_bytes, stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        graphed.b.encrypt(key)
        graphed.b.decrypt(key)
    pgcm.set_unit_bytes(key, 0)
    for k in range(4):
        others[k % 2].clear()
        torch.cuda.synchronize()
        eager(k).check("before the first replay, %d" % k)
    for r in range(4):
        graphed.clear()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        graphed.check("replay %d" % r)
        for k in range(3):
            others[(r + k) % 2].clear()
            torch.cuda.synchronize()
            eager(r + k).check("after replay %d, %d" % (r, k))
    torch.cuda.synchronize()
    key.free()


def test_several_keys_captured():
    """two keys' chunks in one launch, with buffers of the first; eager batches of that key between the
    replays"""
    rng = np.random.default_rng([workloads.BASE_SEED, 5042])
    b, keys, index, cipher, tags = _keys_batch(rng, [int(v) for v in rng.integers(1, 900 * KIB, 40)],
                                               (32, 24))
    other = _Checked("eager_first_key", rng, [MIB + 3] * 9, b.w.key)
    stream = torch.cuda.Stream()
    for q, key in enumerate(keys):
        mine = np.flatnonzero(index == q)
        pgcm.reserve(key, max(mine.size, 9), max(int(b.lens[mine].sum()), 10 * MIB), stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        _encrypt_keys(b, keys, index)
    for r in range(3):
        other.clear()
        b.cipher.zero_()
        b.tags.zero_()
        torch.cuda.synchronize()
        other.b.encrypt(keys[0], stream=stream)
        other.b.decrypt(keys[0], stream=stream)
        with torch.cuda.stream(stream):
            graph.replay()
        other.check("eager %d" % r)
        assert np.array_equal(b.cipher.cpu().numpy(), cipher), r
        assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags), r
    for key in keys:
        key.free()


def test_static_calls_captured_until_the_staging_is_used_up():
    rng = np.random.default_rng([workloads.BASE_SEED, 5041])
    raw_key = rng.integers(0, 256, 32, dtype=np.uint8)
    batches = [_Checked("static_%d" % i, rng, [int(v) for v in rng.integers(1, 40 * KIB, 100 + i)],
                        raw_key) for i in range(4)]
    key = pgcm.expand_key(raw_key)
    stream = torch.cuda.Stream()

    def encrypt(c):
        pgcm.encrypt_batch_static(key, c.b.ivs, c.b.aad_ptrs, c.b.aad_lens, c.b.ptrs(c.b.plain),
                                  c.b.lens, c.b.ptrs(c.b.cipher), c.b.tags, stream)

    torch.cuda.synchronize()
    for c in batches[:3]:
        encrypt(c)
    torch.cuda.synchronize()
    for _ in range(2):                 # a second graph may have the buffers again
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for c in batches:
                encrypt(c)
            with pytest.raises(pgcm.PgcmError) as e:
                encrypt(batches[0])
            assert e.value.status == -7
        for _ in range(3):
            for c in batches:
                c.clear()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            for c in batches:
                assert np.array_equal(c.b.cipher.cpu().numpy(), c.cipher)
                assert np.array_equal(c.b.tags.cpu().numpy().reshape(-1, 16), c.tags)
    key.free()

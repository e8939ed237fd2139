"""pgcm_reserve: after it, batches within the reserved sizes get no memory of any kind, whichever way
they go (one launch, spans read from host memory or uploaded, a wavefront per chunk), and their
results are the CPU oracle's, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from device_batch import DeviceBatch

import paper_2411_03357_amd as pgcm

pytestmark = pytest.mark.gpu

KIB, MIB = 1024, 1 << 20

# chunk lengths
SHAPES = {
    "one_launch": lambda r: [2 * MIB] * 3,
    "spans_few": lambda r: [int(v) for v in r.integers(200 * KIB, 450 * KIB, 60)],
    "spans_host": lambda r: [int(v) for v in r.integers(30 * KIB, 90 * KIB, 700)],
    "spans_uploaded": lambda r: [int(v) for v in r.integers(1, 3 * KIB, 9000)],
    "one_row": lambda r: [int(v) for v in r.integers(0, 1009, 2000)],
}


def workload(name, rng, lens, key, ivs):
    lens = np.array(lens, np.uint64)
    alens = rng.integers(0, 40, lens.size)
    aad_off = np.zeros(lens.size + 1, np.uint64)
    aad_off[1:] = np.cumsum(alens)
    offsets, total = workloads._layout(lens)
    return workloads.Workload(name, 950, key, ivs, lens, offsets, total, "u8",
                              rng.integers(0, 256, int(alens.sum()), dtype=np.uint8), aad_off)


def expected(w, host):
    """whole ciphertext buffer (zero between chunks) and tags by the oracle"""
    cts, tags, _ = oracle.encrypt_batch(w.key, w.ivs,
                                        [np.frombuffer(w.aad_of(i), np.uint8) for i in range(w.n)],
                                        [w.chunk(host, i) for i in range(w.n)], nthreads=16)
    out = np.zeros(w.total_bytes, np.uint8)
    for i, ct in enumerate(cts):
        out[int(w.offsets[i]):int(w.offsets[i]) + ct.size] = ct
    return out, tags


@pytest.mark.parametrize("shape", SHAPES)
def test_reserved_batches_allocate_nothing(shape):
    rng = np.random.default_rng([workloads.BASE_SEED, 8128, len(shape)])
    lens = SHAPES[shape](rng)
    w = workload("reserved_" + shape, rng, lens, rng.integers(0, 256, 32, dtype=np.uint8),
                 rng.integers(0, 256, (len(lens), 12), dtype=np.uint8))
    host = w.payload_host()
    cipher, tags = expected(w, host)
    key = pgcm.expand_key(w.key)
    b = DeviceBatch(w, torch.from_numpy(host).cuda())
    stream = torch.cuda.Stream()
    with pytest.raises(pgcm.PgcmError):
        pgcm.describe_context(key, stream)             # nothing has used the stream
    pgcm.reserve(key, w.n, w.payload_bytes, stream)
    reserved = pgcm.describe_context(key, stream)
    torch.cuda.synchronize()
    for _ in range(6):                                 # more than there are staging buffers
        b.encrypt(key, stream=stream)
        b.decrypt(key, stream=stream)
    after = pgcm.describe_context(key, stream)
    torch.cuda.synchronize()
    for field in ("allocations", "workspace_bytes", "stage_bytes"):
        assert after[field] == reserved[field], field
    assert np.array_equal(b.cipher.cpu().numpy(), cipher)
    assert np.array_equal(b.tags.cpu().numpy().reshape(-1, 16), tags)
    assert bool((b.ok == 1).all()) and torch.equal(b.back, b.plain)
    key.free()
